"""The deposit-free end of an escaping packet's walk, counted instead of
stepped (tiles, tail walk, persistent walk), against the walk that steps
through every cell (one thread per packet): every integer is the same.

Cases where the count can go wrong: no flow, a uniform flow (every jump zero)
and strong ones, boxes one cell thick, cells so small that the roundings of a
long walk reach a cell's drift (the count is then not used) and just above
that, cells so large that a packet escapes within a few, a crossing cap inside
the counted part, both profiles, weights of one unit, several boxes.
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
PC = W.KPC_CM / 1e3


def _box(n, flow, cell_pc=93.75, profile="doppler", packets=30_000, w0=1 << 31, seed=3):
    rng = np.random.default_rng(sum(n) + seed)
    od = rng.lognormal(0.0, 0.7, size=n[::-1]).astype(np.float32)
    vel = None
    if flow == "uniform":
        vel = np.broadcast_to(np.array([0.3, -0.2, 0.1], np.float32)[:, None, None, None], (3,) + n[::-1]).copy()
    elif flow:
        vel = rng.normal(0.0, flow, size=(3,) + n[::-1]).astype(np.float32)
    return W.BoxSpec(n=n, overdensity=od, velocity=vel, n_packets=packets, seed=seed, cell_cm=cell_pc * PC,
                     profile=profile, w0=w0)


def _run(boxes, opts):
    with M.Simulation(boxes) as sim:
        for k, v in opts.items():
            sim.set_option(k, v)
        sim.emit()
        sim.transport()
        t = sim.tally(check=False)
    return t["absorbed"].cpu().numpy(), [(s.escaped, s.crossings, s.capped_weight, s.capped_packets, s.wing,
                                          s.conserved) for s in t["stats"]]


CASES = [
    (dict(n=(20, 33, 17), flow=None), {}),
    (dict(n=(20, 33, 17), flow=0.06), {}),
    (dict(n=(17, 40, 19), flow=0.3), {}),
    (dict(n=(24, 24, 24), flow="uniform"), {}),
    (dict(n=(1, 33, 40), flow=0.1), {}),
    (dict(n=(16, 16, 16), flow=0.1, cell_pc=25.0, packets=8_000), {}),      # roundings above a quarter of the drift
    (dict(n=(16, 16, 16), flow=0.1, cell_pc=50.0, packets=8_000), {}),      # ... below it
    (dict(n=(9, 9, 9), flow=None, cell_pc=5.0, packets=4_000), {}),
    (dict(n=(12, 20, 16), flow=0.1, cell_pc=2000.0), {}),
    (dict(n=(20, 33, 17), flow=0.06), {M.MC_LYA_OPT_MAX_CROSSINGS: 300}),
    (dict(n=(20, 33, 17), flow=None), {M.MC_LYA_OPT_MAX_CROSSINGS: 300}),
    (dict(n=(33, 20, 17), flow=0.06, profile="voigt"), {}),
    (dict(n=(33, 20, 17), flow=None, profile="voigt"), {}),
    (dict(n=(20, 20, 20), flow=0.06, w0=1), {}),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_counted_end_equals_stepping(case):
    kw, opts = CASES[case]
    print(f"case {case}: {kw} {opts}", flush=True)
    spec = _box(**kw)
    tiled = {**opts, M.MC_LYA_OPT_TILE_SHARE: ALL_TILED}
    ref = _run(spec, {**opts, M.MC_LYA_OPT_KERNEL: 1})
    for o in ({**tiled, M.MC_LYA_OPT_TAIL: 0}, {**tiled, M.MC_LYA_OPT_TAIL: 1_000_000}, tiled,
              {**opts, M.MC_LYA_OPT_KERNEL: 0}):
        A, totals = _run(spec, o)
        assert np.array_equal(A, ref[0]), o
        assert totals == ref[1], o


def test_counted_end_in_a_batch():
    boxes = [_box((20, 33, 17), 0.06, seed=1), _box((16, 18, 40), None, seed=2),
             _box((24, 24, 24), 0.2, cell_pc=25.0, seed=4), _box((33, 16, 16), 0.1, profile="voigt", seed=5)]
    ref = _run(boxes, {M.MC_LYA_OPT_KERNEL: 1})
    for opts in ({M.MC_LYA_OPT_TILE_SHARE: ALL_TILED}, {M.MC_LYA_OPT_KERNEL: 0}):
        A, totals = _run(boxes, opts)
        assert np.array_equal(A, ref[0]) and totals == ref[1], opts
