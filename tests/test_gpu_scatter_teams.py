"""The scattering Monte Carlo follows a photon by one lane, by a team of lanes
or by a whole wave, as many photons as a wave has left: a photon's history and
record do not depend on which. Ranges of a call so small that every wave holds
one photon, a few, or many, give the records of the whole range bit for bit.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2312_11448_amd as M  # noqa: E402


def _run(specs, cuts, **kw):
    with M.Simulation(specs) as sim:
        sim.emit()
        recs = [sim.scatter(a, b - a, records=True, **kw) for a, b in zip(cuts, cuts[1:])]
        if "max_events" in kw:                      # (tally() refuses a run with capped photons)
            return np.concatenate(recs), None, None
        t = sim.tally()
        stats = [(s.escaped, s.crossings, s.wing, s.scatterings, s.conserved) for s in t["stats"]]
        return np.concatenate(recs), t["absorbed"].cpu().numpy(), stats


CASES = [
    ("doppler", 0, dict(p_destroy=2e-3)),
    ("voigt", 0, dict(p_destroy=2e-3)),
    ("voigt", 1, dict(p_destroy=2e-3)),                                   # a flow
    ("voigt", 2, dict(p_destroy=2e-3)),                                   # two boxes
    ("voigt", 0, dict(p_destroy=1e-3, max_events=45)),                    # capped inside a draw of 16 events
    ("voigt", 0, dict(p_destroy=0.0, x_inert=60.0, x0=-20.0, x_return=3.0)),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_records_do_not_depend_on_the_split(case):
    profile, kind, kw = CASES[case]
    n = 24_000
    if kind:
        specs = [W.make_box("c2", n=10, n_packets=n, profile=profile, zeta=1e3, field_seed=4, seed=6)]
        if kind == 2:
            specs += [W.BoxSpec(n=(5, 6, 7), overdensity=np.ones((7, 6, 5), np.float32), zeta=1e5, n_packets=3000,
                                seed=8, profile="doppler")]
    else:
        specs = [W.BoxSpec(n=(4, 4, 4), overdensity=W.uniform_box(4), zeta=1e4, n_packets=n, seed=7, profile=profile)]
    n = sum(s.n_packets for s in specs)
    ref = _run(specs, [0, n], **kw)                          # 12 photons a wave: lanes, then teams, then waves
    got = _run(specs, [0, 1, 2, 700, 5700, 14_000, n], **kw)     # 1, 1, 1, 3, 5, 5
    for name in ref[0].dtype.names:
        assert np.array_equal(ref[0][name], got[0][name]), name
    if ref[2] is None:
        assert (ref[0]["fate"] == 2).any()
        return
    assert np.array_equal(ref[1], got[1]) and ref[2] == got[2]
    assert all(s[4] == 1 for s in ref[2])
