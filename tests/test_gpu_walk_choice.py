"""Which walk a box gets, where the default decides and where an option does,
and that its integers do not depend on it.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2312_11448_amd as M  # noqa: E402


def _box(n, flow, packets, profile="doppler", rms=0.5, seed=3):
    rng = np.random.default_rng(sum(n) + seed)
    od = rng.lognormal(0.0, rms, size=n[::-1]).astype(np.float32)
    vel = rng.normal(0.0, flow, size=(3,) + n[::-1]).astype(np.float32) if flow else None
    return W.BoxSpec(n=n, overdensity=od, velocity=vel, n_packets=packets, seed=seed, profile=profile)


def _walk(sim, cuts=None):
    """The emission, walked in the given ranges: (integers, tiled per box after the last)."""
    sim.emit()
    if cuts:
        for a, b in zip(cuts, cuts[1:]):
            sim.transport(a, b - a)
    else:
        sim.transport()
    t = sim.tally()
    return (t["absorbed"].cpu().numpy(), [(s.escaped, s.crossings, s.wing, s.conserved) for s in t["stats"]],
            [s.tiled for s in t["stats"]])


def _same(a, b):
    return np.array_equal(a[0], b[0]) and a[1] == b[1]


@pytest.mark.parametrize("boxes", [[((32, 32, 32), None, 100_000)], [((16, 16, 16), 0.08, 500_000)],
                                   [((12, 12, 12), None, 30_000)] * 4])
def test_a_short_range_is_a_small_call(boxes):
    """A large emission walked whole goes to tiles; in ranges of a few hundred
    packets it is walked as a small call is, by the persistent walk."""
    specs = [_box(n, flow, packets, seed=3 + i) for i, (n, flow, packets) in enumerate(boxes)]
    total = sum(s.n_packets for s in specs)
    with M.Simulation(specs) as sim:
        whole = _walk(sim)
        assert all(whole[2])
        short = _walk(sim, [0, total - 1000, total - 500, total])
        assert not short[2][-1]
        assert _same(whole, short)


# (box, flow, profile, packets, rms of ln Delta, tiled): in a flow, boxes of
# more than 8 tiles, not cut along every axis or strongly clumped take tiles
# from 1e5 packets, others earlier
LINES = [
    ((37, 37, 37), 0.08, "voigt", 9_057, 0.5, 0), ((37, 37, 37), 0.08, "voigt", 100_000, 0.5, 1),
    ((21, 60, 13), 0.08, "voigt", 46_713, 0.5, 0), ((21, 60, 13), 0.08, "voigt", 100_000, 0.5, 1),
    ((25, 25, 25), 0.08, "doppler", 20_000, 1.5, 0), ((25, 25, 25), 0.08, "doppler", 20_000, 0.5, 1),
    ((25, 25, 25), 0.08, "doppler", 100_000, 1.5, 1), ((50, 50, 50), 0.08, "doppler", 99_999, 0.5, 0),
    ((50, 50, 50), None, "voigt", 45_000, 0.5, 1), ((7, 9, 58), 0.08, "voigt", 7_099, 0.5, 0),
]


@pytest.mark.parametrize("case", range(len(LINES)))
def test_lone_box_lines(case):
    n, flow, profile, packets, rms, tiled = LINES[case]
    with M.Simulation(_box(n, flow, packets, profile, rms)) as sim:
        got = _walk(sim)
        assert got[2] == [tiled]
        sim.set_option(M.MC_LYA_OPT_KERNEL, 1)
        assert _same(got, _walk(sim))


@pytest.mark.parametrize("flow,profile", [(0.08, "doppler"), (None, "voigt")])
@pytest.mark.parametrize("packets,tiled", [(5_000, 0), (20_000, 1)])
def test_batch_line_of_single_tiles(packets, tiled, flow, profile):
    specs = [_box((9 + i, 11, 14), flow, packets, profile, seed=1 + i) for i in range(3)]
    with M.Simulation(specs) as sim:
        got = _walk(sim)
        assert got[2] == [tiled] * 3
        sim.set_option(M.MC_LYA_OPT_KERNEL, 1)
        assert _same(got, _walk(sim))


@pytest.mark.parametrize("packets,tiled", [(150_000, 0), (200_000, 1)])
def test_batch_line_with_voigt_in_a_flow(packets, tiled):
    specs = [_box((30, 9, 20), 0.08, packets, "voigt", seed=1), _box((20, 21, 17), 0.08, packets, "voigt", seed=2)]
    with M.Simulation(specs) as sim:
        got = _walk(sim)
        assert got[2] == [tiled] * len(specs)
        sim.set_option(M.MC_LYA_OPT_KERNEL, 1)
        assert _same(got, _walk(sim))


@pytest.mark.parametrize("boxes", [[((32, 32, 32), None, 300_000)], [((16, 16, 16), 0.08, 500_000)],
                                   [((12, 12, 12), None, 30_000)] * 4])
def test_tile_share_decides_where_it_is_set(boxes):
    """A lower share than the default leaves boxes whose tiles have more than
    that much work to the persistent walk, whatever the packets."""
    specs = [_box(n, flow, packets, seed=3 + i) for i, (n, flow, packets) in enumerate(boxes)]
    with M.Simulation(specs) as sim:
        ref = _walk(sim)
        assert all(ref[2])
        for share, tiled in ((99, 0), (1, 0), (0, 0), (1_000_000, 1), (100, 1)):
            sim.set_option(M.MC_LYA_OPT_TILE_SHARE, share)
            got = _walk(sim)
            assert all(t == tiled for t in got[2]), share
            assert _same(ref, got)


@pytest.mark.parametrize("flow,profile", [(None, "doppler"), (0.08, "voigt")])
@pytest.mark.parametrize("kinds", ["one tile each", "several tiles each"])
def test_shared_tiles_beside_a_box_left_out(kinds, flow, profile):
    """A small batch by shared tiles, but for one box whose walks are so long
    that it is left to the persistent walk beside them (or after them): ranges,
    repeated emissions and replays from a graph included."""
    n, packets = ((12, 13, 14), 8_000) if kinds == "one tile each" else ((20, 21, 22), 300_000)
    specs = [_box(n, flow, packets, profile, seed=3 + i) for i in range(6)]
    long = _box(n, flow, packets, profile, seed=9)
    long.cell_cm = 5.0 * W.KPC_CM / 1e3
    specs.insert(2, long)
    total = sum(s.n_packets for s in specs)
    with M.Simulation(specs) as sim:
        sim.set_option(M.MC_LYA_OPT_KERNEL, 1)
        ref = _walk(sim)
        sim.set_option(M.MC_LYA_OPT_KERNEL, 2)
        for beside, graph, cuts in ((4, 0, None), (0, 0, None), (4, 0, [0, total // 7, total]), (4, 1, None), (4, 1, None)):
            sim.set_option(M.MC_LYA_OPT_BESIDE, beside)
            sim.set_option(M.MC_LYA_OPT_GRAPH, graph)
            got = _walk(sim, cuts)
            # (a range holds fewer packets than the line asks for)
            assert cuts or got[2] == [1, 1, 0, 1, 1, 1, 1], (beside, graph)
            assert _same(ref, got), (beside, graph, cuts)
