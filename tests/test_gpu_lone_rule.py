"""Where a lone box goes from the persistent walk to shared tiles (by its
packets, flow, profile and size), and where the tail walk takes over unset:
on both sides of each line, the integers of the walk without tiles.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2312_11448_amd as M  # noqa: E402

# (box, flow, profile, packets from which it is tiled)
LINES = [
    ((24, 25, 26), 0.08, "doppler", 10_000),
    ((24, 25, 26), 0.08, "voigt", 5_000),
    ((18, 20, 22), 0.08, "doppler", 80_000),          # records in LDS
    ((40, 41, 42), None, "doppler", 45_000),
    ((30, 31, 33), None, "voigt", 80_000),            # records in LDS
    ((9, 10, 11), 0.08, "voigt", 40_000),             # one tile
]


@pytest.mark.parametrize("case", range(len(LINES)))
def test_both_sides_of_the_line(case):
    n, flow, profile, line = LINES[case]
    rng = np.random.default_rng(sum(n))
    od = rng.lognormal(0.0, 0.6, size=n[::-1]).astype(np.float32)
    vel = rng.normal(0.0, flow, size=(3,) + n[::-1]).astype(np.float32) if flow else None
    for packets in (line - 1, line):
        spec = W.BoxSpec(n=n, overdensity=od, velocity=vel, n_packets=packets, seed=9, profile=profile)
        out = []
        with M.Simulation(spec) as sim:
            for kernel in (1, 2):
                sim.set_option(M.MC_LYA_OPT_KERNEL, kernel)
                sim.emit()
                sim.transport()
                t = sim.tally()
                s = t["stats"][0]
                out.append((t["absorbed"].cpu().numpy(), (s.escaped, s.crossings, s.wing, s.conserved)))
            assert s.tiled == (packets >= line)
        assert np.array_equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]
