"""The counted end of a walk in boxes that move as a whole, and in flows whose
deviation is several Doppler widths: every integer is that of the walk that
steps through each cell, in tiles, in the tail walk and in the persistent walk.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2312_11448_amd as M  # noqa: E402

PC = W.KPC_CM / 1e3
ALL_TILED = 1_000_000

# (mean flow, rms of the deviation, cell in pc, profile)
CASES = [((40.0, -30.0, 0.0), 0.1, 93.75, "doppler"), ((60.0, 20.0, -80.0), 0.05, 93.75, "doppler"),
         ((0.0, 0.0, 100.0), 0.1, 400.0, "voigt"), ((900.0, -500.0, 300.0), 0.1, 2000.0, "doppler"),
         ((0.0, 0.0, 0.0), 1.0, 2000.0, "doppler"), ((0.0, 0.0, 0.0), 1.0, 2000.0, "voigt"),
         ((2e4, 0.0, 0.0), 0.1, 93.75, "doppler")]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_counted_end_in_a_moving_box(case):
    mean, rms, cell, profile = CASES[case]
    n = (20, 33, 17)
    rng = np.random.default_rng(case)
    od = rng.lognormal(0.0, 0.7, size=n[::-1]).astype(np.float32)
    vel = rng.normal(0.0, rms, size=(3,) + n[::-1]).astype(np.float32)
    vel += np.array(mean, np.float32)[:, None, None, None]
    spec = W.BoxSpec(n=n, overdensity=od, velocity=vel, n_packets=30_000, seed=4, cell_cm=cell * PC, profile=profile)
    out = []
    for opts in ({M.MC_LYA_OPT_KERNEL: 1}, {M.MC_LYA_OPT_TILE_SHARE: ALL_TILED, M.MC_LYA_OPT_TAIL: 0},
                 {M.MC_LYA_OPT_TILE_SHARE: ALL_TILED, M.MC_LYA_OPT_TAIL: 1_000_000}, {M.MC_LYA_OPT_KERNEL: 0}, {}):
        with M.Simulation(spec) as sim:
            for k, v in opts.items():
                sim.set_option(k, v)
            sim.emit()
            sim.transport()
            t = sim.tally()
            s = t["stats"][0]
            out.append((t["absorbed"].cpu().numpy(), (s.escaped, s.crossings, s.wing, s.conserved)))
    for got in out[1:]:
        assert np.array_equal(got[0], out[0][0]) and got[1] == out[0][1]
