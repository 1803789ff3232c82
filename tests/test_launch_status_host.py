"""A kernel launch that fails is reported, and nothing is launched after it
that would read what it did not write. Run on the CPU against a stand-in for
the HIP runtime's launch calls in which the first launch fails and the next
succeeds (with the status of the last call only, as hipGetLastError may give
it): the gradient's partial sums are then an earlier call's, and summing them
would return old values as new ones.
"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <cstddef>
struct Dim { unsigned x, y, z; };
static int g_launches = 0, g_last = 0;
extern "C" {
int stand_in_launches() { return g_launches; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *) { static char room[64]; *p = room; return 0; }
int __hipPushCallConfiguration(Dim, Dim, size_t, void *) { return 0; }
int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *n, void **s)
{
    *g = *b = Dim{1, 1, 1};
    *n = 0;
    *s = nullptr;
    return 0;
}
int hipLaunchKernel(const void *, Dim, Dim, void **, size_t, void *)
{
    g_last = g_launches++ == 0 ? 701 : 0;      // hipErrorLaunchOutOfResources, then success
    return g_last;
}
int hipGetLastError() { return g_last; }
}
"""

CHILD = r"""
import ctypes as C, subprocess, sys
from paper_2312_11448_amd import _abi as A
L = A.load()
buf = C.cast((C.c_double * 64)(), C.c_void_p)
def inner(name):                                # a C++ function of the library, by its unmangled name
    syms = subprocess.run(["nm", A.LIB_PATH], capture_output=True, text=True, check=True).stdout.split()
    return L[next(s for s in syms if s.startswith("_ZN5mclya%d%s" % (len(name), name)))]
what = sys.argv[2]
if what == "gradient":
    st = L.mc_lya_mlp_gradient_static(buf, buf, buf, buf, 32, buf, None)
elif what == "feed":
    st = inner("launch_feed_sums")(buf, 1, 1, buf, buf, buf, buf, buf, None)
else:
    st = inner("launch_red_list")(buf, 1, C.c_bool(True), C.c_bool(what == "ends_voigt"), None)
print(st, C.CDLL(sys.argv[1]).stand_in_launches(), flush=True)
"""


@pytest.mark.parametrize("what", ["gradient", "feed", "ends", "ends_voigt"])
def test_failed_launch_is_reported(what, tmp_path):
    import paper_2312_11448_amd as M
    if not os.path.exists(M.LIB_PATH):
        from paper_2312_11448_amd import build
        build.build()
    src, lib = tmp_path / "stand_in.cpp", tmp_path / "stand_in.so"
    src.write_text(STAND_IN)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-o", str(lib), str(src)], check=True)
    env = dict(os.environ, LD_PRELOAD=str(lib), PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", CHILD, str(lib), what], env=env, cwd=ROOT, capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stderr
    status, launches = map(int, r.stdout.split())
    assert status == (M.MC_LYA_EDEVICE if what == "gradient" else 701)
    assert launches == 1
