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
