"""Boxes whose axes the tile edge does not divide are cut into equal tiles, the
last of an axis a little smaller: packets that cross from a tile to its
neighbours, the box's ends included, arrive in the right cells (the integers
of the walk without tiles).
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2312_11448_amd as M  # noqa: E402


@pytest.mark.parametrize("profile,flow", [("doppler", None), ("voigt", 0.08)])
@pytest.mark.parametrize("n", [(17, 18, 19), (33, 31, 47), (65, 16, 34), (225, 17, 15), (241, 3, 18)])
def test_tiles_of_an_uneven_box(n, profile, flow):
    rng = np.random.default_rng(sum(n))
    od = rng.lognormal(0.0, 0.7, size=n[::-1]).astype(np.float32)
    vel = rng.normal(0.0, flow, size=(3,) + n[::-1]).astype(np.float32) if flow else None
    spec = W.BoxSpec(n=n, overdensity=od, velocity=vel, n_packets=60_000, seed=5, profile=profile)
    out = []
    with M.Simulation(spec) as sim:
        for kernel, share, tail in ((1, 100, 0), (2, 1_000_000, 0), (2, 1_000_000, 4_000)):
            sim.set_option(M.MC_LYA_OPT_KERNEL, kernel)
            sim.set_option(M.MC_LYA_OPT_TILE_SHARE, share)
            sim.set_option(M.MC_LYA_OPT_TAIL, tail)
            sim.emit()
            sim.transport()
            t = sim.tally()
            s = t["stats"][0]
            out.append((t["absorbed"].cpu().numpy(), (s.escaped, s.crossings, s.wing, s.conserved)))
            assert s.tiled == (kernel == 2)
    for got in out[1:]:
        assert np.array_equal(got[0], out[0][0]) and got[1] == out[0][1]
