"""A box alone in its context: the walks chosen for it by size and packets
(tiles shared by several workgroups, the persistent walk with the records,
and the tallies of the smallest boxes, in LDS) give the integers of the walk
that steps every packet on its own, in one call, in ranges, in a second
emission and replayed from a graph.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2312_11448_amd as M  # noqa: E402

ALL_TILED = 1_000_000


def _box(n, flow, packets, profile="doppler", seed=3):
    rng = np.random.default_rng(sum(n) + seed)
    od = rng.lognormal(0.0, 0.7, size=n[::-1]).astype(np.float32)
    vel = rng.normal(0.0, flow, size=(3,) + n[::-1]).astype(np.float32) if flow else None
    return W.BoxSpec(n=n, overdensity=od, velocity=vel, n_packets=packets, seed=seed, profile=profile)


def _totals(sim):
    t = sim.tally()
    s = t["stats"][0]
    return t["absorbed"].cpu().numpy(), (s.escaped, s.crossings, s.wing, s.conserved), s.tiled


def _same(a, b, what):
    assert np.array_equal(a[0], b[0]) and a[1] == b[1], what


# (box, flow, packets, profile): whether the default takes tiles
CASES = [
    ((8, 8, 8), None, 3_000, "doppler", 0),          # records and tallies in LDS
    ((8, 8, 8), 0.1, 3_000, "voigt", 0),
    ((23, 23, 23), None, 4_000, "doppler", 0),       # tallies would fit, too few packets
    ((32, 32, 32), None, 20_000, "voigt", 0),        # records fit, tallies do not
    ((34, 34, 34), None, 5_000, "doppler", 0),       # records just fit (39 304 cells of 39 936)
    ((35, 34, 34), None, 5_000, "doppler", 0),       # ... just do not
    ((21, 21, 21), 0.1, 5_000, "doppler", 0),        # with a flow: 9 261 cells of 9 984
    ((22, 22, 21), 0.1, 5_000, "doppler", 0),
    ((16, 16, 16), 0.06, 500_000, "doppler", 1),     # one tile, wrapping onto itself, shared
    ((17, 40, 33), 0.06, 500_000, "doppler", 1),
    ((40, 33, 17), None, 500_000, "voigt", 1),
    ((1, 40, 40), None, 400_000, "doppler", 1),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_lone_box_walks_agree(case):
    n, flow, packets, profile, tiled = CASES[case]
    print(f"case {case}: {CASES[case]}", flush=True)
    spec = _box(n, flow, packets, profile)
    with M.Simulation(spec) as sim:
        sim.set_option(M.MC_LYA_OPT_KERNEL, 1)
        sim.emit()
        sim.transport()
        ref = _totals(sim)
        sim.set_option(M.MC_LYA_OPT_KERNEL, 2)
        for rep in range(2):
            sim.emit()
            sim.transport()
            got = _totals(sim)
            _same(got, ref, f"default, emission {rep}")
            assert got[2] == tiled
        sim.emit()
        for a, b in ((0, 1), (1, packets // 3), (packets // 3, packets)):
            sim.transport(a, b - a)
        _same(_totals(sim), ref, "ranges")
        sim.set_option(M.MC_LYA_OPT_TILE_SHARE, ALL_TILED)
        sim.set_option(M.MC_LYA_OPT_TAIL, 0)
        sim.emit()
        sim.transport()
        _same(_totals(sim), ref, "all tiled")
        sim.set_option(M.MC_LYA_OPT_GRAPH, 1)
        for rep in range(3):
            sim.emit()
            sim.transport()
            _same(_totals(sim), ref, f"graph {rep}")
            torch.zeros(1000, device="cuda").sum().item()
        sim.set_option(M.MC_LYA_OPT_TILE_SHARE, 100)
        for rep in range(2):
            sim.emit()
            sim.transport()
            _same(_totals(sim), ref, f"graph, default {rep}")
