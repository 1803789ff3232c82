"""The bound on the walk's binary32 roundings that the count of an escaping
packet's last crossings rests on (red_eps), against the largest sum the
roundings of such a walk can come to, added up face by face: two of x at its
own size, one of the jump's difference of projections, one of the segment's
length. Weak and strong flows, thresholds at both ends of a binade.
"""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "red_bound.hpp"
extern "C" int red(double kmax, double delta, double x_eff, const double *u, double udev, double damp, float far,
                   float near, float *out)
{
    const mclya::RedBox r = mclya::red_constants(kmax, delta, x_eff, u, udev, true, damp);
    out[0] = mclya::red_eps(r, far, near);
    out[1] = r.udev;
    return r.mode;
}
"""


@pytest.fixture(scope="module")
def red(tmp_path_factory):
    d = tmp_path_factory.mktemp("red")
    (d / "red.cpp").write_text(SRC)
    lib = d / "red.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2312_11448_amd", "csrc"), "-o", str(lib), str(d / "red.cpp")], check=True)
    f = C.CDLL(str(lib)).red
    f.argtypes = [C.c_double] * 3 + [C.c_void_p] + [C.c_double] * 2 + [C.c_float] * 2 + [C.c_void_p]

    def call(delta, x_eff, u, udev, far=0.0, near=0.0):
        out, uu = (C.c_float * 2)(), (C.c_double * 3)(*u)
        mode = f(1.0, delta, x_eff, uu, udev, 0.0, far, near, out)
        return mode, out[0], out[1]
    return call


def half_ulp(v):
    return float(np.spacing(np.float32(abs(v)))) / 2.0


def worst_sum(delta, x_eff, udev, xc):
    """Largest sum of the roundings from mean-flow frequency xc on to the last
    cell that can stop the packet."""
    length = (xc + udev + x_eff) / delta
    faces = int(np.floor(np.sqrt(3.0) * length)) + 3
    at = np.minimum(np.arange(1, faces + 1) * (length / faces), length)
    x = np.minimum(np.abs(xc - delta * at) + udev, x_eff)
    hx = np.spacing(x.astype(np.float32)).astype(float) / 2.0
    return float(2.0 * hx.sum() + faces * (half_ulp(2.0 * udev) + 1.75 * delta * 2.0 ** -24))


@pytest.mark.parametrize("udev", [0.05, 0.3, 1.0, 1.9, 4.0])
@pytest.mark.parametrize("x_esc", [4.0, 6.0, 7.9])
def test_bound_holds_face_by_face(red, x_esc, udev):
    x_eff = float(np.float32(x_esc + 2.0 * udev))
    used = 0
    for delta in (0.02, 0.05, 0.2, 0.6):
        binade = 2.0 ** np.floor(np.log2(x_eff))
        for xc in np.linspace(-1.2 - udev, -x_eff + udev + 0.05, 9):
            if xc > -1.0 - udev:
                continue
            mode, _, ud = red(delta, x_eff, (0.0, 0.0, 0.0), udev)
            if mode != 2:
                continue
            far = np.float32(max((xc + ud + x_eff) / delta, 0.0))
            near = np.float32(max((xc - ud + binade) / delta, 0.0))
            _, eps, _ = red(delta, x_eff, (0.0, 0.0, 0.0), udev, far, near)
            # (and the count's own: a cast and a difference at |x| <= x_eff)
            assert eps >= worst_sum(delta, x_eff, udev, xc) + 2.0 * half_ulp(x_eff), (delta, xc)
            used += 1
    assert used


@pytest.mark.parametrize("u", [(0.0, 0.0, 0.0), (20.0, -30.0, 10.0), (60.0, 0.0, -80.0), (300.0, 200.0, -100.0),
                               (3e3, -1e3, 2e3)])
def test_bound_holds_in_a_moving_frame(red, u):
    """With a mean flow the comoving frequency X = x + k.U is as large as the
    flow: its cast to binary32, the difference X - k.U and the mean flow's own
    projection round at that size, not at x's."""
    udev, x_esc = 0.3, 6.0
    x_eff = float(np.float32(x_esc + 2.0 * udev))
    size = float(np.linalg.norm(u)) + udev + x_eff
    proj = sum(abs(a) for a in u)
    # the projection: three roundings of the sum, one of each component
    proj_err = (3.0 * half_ulp(proj) + sum(half_ulp(a) for a in u)) if proj else 0.0
    used = 0
    for delta in (0.02, 0.2, 0.6):
        for xc in np.linspace(-2.0, -x_eff + udev + 0.05, 5):
            far = np.float32((xc + udev + 1e-4 + x_eff) / delta)
            near = np.float32(max((xc - udev - 1e-4 + 4.0) / delta, 0.0))
            mode, eps, ud = red(delta, x_eff, u, udev, far, near)
            if mode != 2:
                continue
            walk = worst_sum(delta, x_eff, udev, xc)
            assert eps >= walk + half_ulp(size) + half_ulp(x_eff + 2.0 * udev), (delta, xc)
            # the cells passed over: 2 eps and udev's margin hold the projection's error too
            assert 2.0 * eps + ud - udev >= walk + proj_err, (delta, xc)
            used += 1
    assert used or proj > 1e3


def test_end_margin_holds_in_a_moving_frame(red):
    """The frequency that decides whether a packet is past its last deposit is
    formed in binary32 at the flow's size: udev's margin holds its rounding."""
    for u in ((0.0, 0.0, 0.0), (60.0, 0.0, -80.0), (3e3, -1e3, 2e3)):
        proj = sum(abs(a) for a in u)
        err = 2.0 * half_ulp(proj + 10.0) + 3.0 * half_ulp(proj) + sum(half_ulp(a) for a in u)
        _, _, ud = red(0.2, 6.6, u, 0.3)
        assert ud - 0.3 >= err
