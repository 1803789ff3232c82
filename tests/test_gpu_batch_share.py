"""A batch of boxes with fewer tiles than the chip has compute units: from a
number of packets a tile its boxes are walked by tiles that several workgroups
share, one with far longer walks left to the persistent walk; on both sides of
the line the integers are those of the walk without tiles.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2312_11448_amd as M  # noqa: E402


def _boxes(dims, packets, flow, profile):
    out = []
    for i, n in enumerate(dims):
        rng = np.random.default_rng(i + sum(n))
        od = rng.lognormal(0.0, 0.5, size=n[::-1]).astype(np.float32)
        vel = rng.normal(0.0, flow, size=(3,) + n[::-1]).astype(np.float32) if flow else None
        out.append(W.BoxSpec(n=n, overdensity=od, velocity=vel, n_packets=packets, seed=3 + i, profile=profile))
    return out


# (boxes, flow, profile, packets a box below the line, at or above it)
CASES = [
    ([(9, 10, 11), (16, 16, 16), (5, 7, 3)], None, "doppler", 2_000, 2_600),
    ([(12, 9, 10)] * 5, 0.08, "voigt", 2_400, 2_500),
    ([(17, 18, 19), (30, 9, 20)], 0.08, "doppler", 100_000, 190_000),       # 8 + 4 tiles
    ([(16, 33, 8), (12, 12, 12)], None, "voigt", 30_000, 60_000),           # 3 + 1
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_batch_by_shared_tiles(case):
    dims, flow, profile, below, above = CASES[case]
    for packets, tiled in ((below, False), (above, True)):
        specs = _boxes(dims, packets, flow, profile)
        out = []
        with M.Simulation(specs) as sim:
            for kernel, graph in ((1, 0), (2, 0), (2, 0), (2, 1), (2, 1)):
                sim.set_option(M.MC_LYA_OPT_KERNEL, kernel)
                sim.set_option(M.MC_LYA_OPT_GRAPH, graph)
                sim.emit()
                sim.transport()
                t = sim.tally()
                out.append((t["absorbed"].cpu().numpy(),
                            [(s.escaped, s.crossings, s.wing, s.conserved) for s in t["stats"]]))
                if kernel == 2:
                    assert any(s.tiled for s in t["stats"]) == tiled
                    assert not tiled or all(s.tiled for s in t["stats"])
        for got in out[1:]:
            assert np.array_equal(got[0], out[0][0]) and got[1] == out[0][1]
