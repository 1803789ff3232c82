"""What this framework is timed on: the calls its users make, over the sizes they make them at.

Three kinds of program use it. One computes the recombination feed of given
boxes: new fields, emit, transport, tally, feed (``step``), or a whole
recombination history of such steps (``evolve``), or the paper's own
scattering Monte Carlo (``scatter``). One evaluates the surrogate of the mixing
correction on new fields (``surrogate``, ``correction``). One trains it
(``gradient``, ``train``). Grids are periodic, arrays are [z][y][x]; fields are
the synthetic families of ``workloads`` made on the GPU from the seed.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2312_11448_amd as M

KPC_CM = 3.0856775814913673e21
CELL_CM = 24.0 * KPC_CM / 256.0
DEV = "cuda"


def listed():
    return [
        # one small box: a quick look, a point of a parameter scan, one box of the surrogate's training set
        {"name": "step_32_lognormal", "do": "step", "nx": 32, "ny": 32, "nz": 32, "field": "lognormal", "rms": 0.3,
         "vel": "none", "xe": "uniform", "profile": "doppler", "z": 1100.0, "packets": 100_000, "boxes": 1,
         "emitted": True, "targets": False},
        # a box cut out of a larger one: no edge a multiple of anything, every output asked for
        {"name": "step_ragged", "do": "step", "nx": 90, "ny": 75, "nz": 61, "field": "grf", "rms": 1.0,
         "vel": "f32", "xe": "uniform", "profile": "doppler", "z": 1100.0, "packets": 1_500_000, "boxes": 1,
         "emitted": True, "targets": True},
        # the ordinary box with its flow
        {"name": "step_128_k2", "do": "step", "nx": 128, "ny": 128, "nz": 128, "field": "grf", "rms": 0.5,
         "vel": "f32", "xe": "uniform", "profile": "doppler", "z": 1100.0, "packets": 10_000_000, "boxes": 1,
         "emitted": False, "targets": False},
        # the same with the damping wing, half-precision flow and a given x_e field
        {"name": "step_128_voigt", "do": "step", "nx": 128, "ny": 128, "nz": 128, "field": "grf", "rms": 0.5,
         "vel": "f16", "xe": "field", "profile": "voigt", "z": 1100.0, "packets": 10_000_000, "boxes": 1,
         "emitted": False, "targets": False},
        # the largest single box, high contrast, 16 packets a cell: the benchmark's workload
        {"name": "step_256_contrast", "do": "step", "nx": 256, "ny": 256, "nz": 256, "field": "grf", "rms": 2.0,
         "vel": "f32", "xe": "uniform", "profile": "doppler", "z": 1100.0, "packets": 1 << 28, "boxes": 1,
         "emitted": False, "targets": False},
        # many uneven boxes over the redshifts of Fig. MCtravel in one context
        {"name": "step_batch", "do": "step", "nx": 80, "ny": 80, "nz": 80, "field": "grf", "rms": 2.0,
         "vel": "f32", "xe": "uniform", "profile": "doppler", "z": 1400.0, "packets": 500_000, "boxes": 24,
         "emitted": False, "targets": False},
        # a stretch of a recombination history of a small box: many small dependent transports
        {"name": "evolve_8", "do": "evolve", "n": 8, "packets": 20_000, "steps": 5, "cell_pc": 10.0, "z": 1300.0},
        # the scattering Monte Carlo with its records (Voigt, the paper's scaled expansion, raised destruction)
        {"name": "scatter_32_voigt", "do": "scatter", "n": 32, "photons": 131_072, "profile": "voigt",
         "zeta": 1.0e4, "p_destroy": 1.0e-4},
        # the surrogate over the largest box: features and inference of every cell
        {"name": "surrogate_256", "do": "surrogate", "nx": 256, "ny": 256, "nz": 256, "rms": 2.0, "vel": "f16",
         "xe": "uniform"},
        # the correction of a ragged box, with the envelope test and the Monte Carlo's values as fallback
        {"name": "correction_ragged", "do": "correction", "nx": 61, "ny": 50, "nz": 37, "rms": 1.0, "vel": "f32",
         "xe": "field"},
        # the loss gradient over one large odd batch (an outer optimiser's call)
        {"name": "gradient_300k", "do": "gradient", "cells": 300_007},
        # a chunk of training steps on index-picked batches of the stated size
        {"name": "train_65536", "do": "train", "cells": 2_000_003, "batch": 65_536, "steps": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["step", "step", "step", "step", "evolve", "scatter", "surrogate", "correction", "gradient",
                     "train"])
    if do == "step":
        boxes = rng.choice([1, 1, 1, _log_int(rng, 2, 24)])
        top = 200 if boxes == 1 else 72
        n = _log_int(rng, 16, top)
        edge = lambda: max(9, min(top, int(n * rng.uniform(0.7, 1.4))))   # noqa: E731
        nx, ny, nz = (n, n, n) if rng.random() < 0.3 else (edge(), edge(), edge())
        lo, hi = (1, 24) if boxes == 1 else (0.5, 8)
        return {"do": do, "nx": nx, "ny": ny, "nz": nz, "field": rng.choice(["grf", "grf", "lognormal"]),
                "rms": round(rng.uniform(0.2, 2.0), 3), "vel": rng.choice(["none", "f32", "f32", "f16"]),
                "xe": rng.choice(["uniform", "field"]), "profile": rng.choice(["doppler", "doppler", "voigt"]),
                "z": round(rng.uniform(950.0, 1400.0), 1),
                "packets": max(1000, int(nx * ny * nz * math.exp(rng.uniform(math.log(lo), math.log(hi))))),
                "boxes": boxes, "emitted": rng.random() < 0.5, "targets": rng.random() < 0.3}
    if do == "evolve":
        return {"do": do, "n": rng.choice([5, 8, 12, 16, 24]), "packets": _log_int(rng, 5_000, 200_000),
                "steps": rng.randint(2, 5), "cell_pc": round(_log_int(rng, 10, 10_000), 1),
                "z": round(rng.uniform(1150.0, 1350.0), 1)}
    if do == "scatter":
        return {"do": do, "n": rng.choice([4, 13, 24, 32]), "photons": _log_int(rng, 3_000, 131_072),
                "profile": rng.choice(["voigt", "voigt", "doppler"]), "zeta": float(rng.choice([1.0e3, 1.0e4])),
                "p_destroy": rng.choice([1.0e-3, 5.0e-4, 2.0e-4])}
    if do in ("surrogate", "correction"):
        n = _log_int(rng, 16, 256 if do == "surrogate" else 160)
        nx, ny, nz = (n, n, n) if rng.random() < 0.4 else (max(3, int(n * rng.uniform(0.7, 1.2))) for _ in range(3))
        return {"do": do, "nx": nx, "ny": ny, "nz": nz, "rms": round(rng.uniform(0.2, 2.0), 3),
                "vel": rng.choice(["none", "f32", "f16"]), "xe": rng.choice(["uniform", "field"])}
    if do == "gradient":
        return {"do": do, "cells": _log_int(rng, 1_000, 2_000_000)}
    return {"do": do, "cells": _log_int(rng, 100_000, 4_000_000), "batch": _log_int(rng, 1_024, 131_072),
            "steps": rng.randint(4, 10)}


# ---- inputs ---------------------------------------------------------------------

def _gen(seed, k=0):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + 7919 * k + 17) & 0x7FFFFFFFFFFF)
    return g


def _grf(nx, ny, nz, rms, g):
    """1 + delta of a k^2 field clipped to [1e-2, 1e2] and scaled to mean 1, with its curl-free flow (rms 0.1)."""
    wk = torch.fft.rfftn(torch.randn((nz, ny, nx), generator=g, device=DEV, dtype=torch.float32))
    f = lambda n: torch.fft.fftfreq(n, device=DEV)                        # noqa: E731
    kz, ky, kx = f(nz)[:, None, None], f(ny)[None, :, None], torch.fft.rfftfreq(nx, device=DEV)[None, None, :]
    k2 = kx * kx + ky * ky + kz * kz
    dk = wk * torch.where(k2 <= 0.0625, k2.sqrt(), torch.zeros_like(k2))
    delta = torch.fft.irfftn(dk, s=(nz, ny, nx))
    scale = rms / delta.square().mean().sqrt().clamp_min(1e-20)
    od = torch.clamp(1.0 + delta * scale, 1e-2, 1e2)
    safe = torch.where(k2 > 0, k2, torch.ones_like(k2))
    v = torch.stack([torch.fft.irfftn(1j * kc * dk / safe, s=(nz, ny, nx)) for kc in (kx, ky, kz)])
    v = v * (0.1 / v.square().sum(0).mean().sqrt().clamp_min(1e-20))
    return (od / od.mean()).contiguous(), v.contiguous()


def _lognormal(nx, ny, nz, sigma, g):
    return torch.exp(sigma * torch.randn((nz, ny, nx), generator=g, device=DEV) - 0.5 * sigma * sigma)


def _cosmo():
    return SimpleNamespace(h=0.67, omega_b_h2=0.0224, omega_c_h2=0.12, y_p=0.24, t_cmb0=2.7255, n_eff=3.046)


def _box(nx, ny, nz, od, vel=None, xe=None, **more):
    d = dict(n=(nx, ny, nz), ncells=nx * ny * nz, overdensity=od, velocity=vel, x_e=xe, x_e_uniform=0.1, source=None,
             temp_K=3000.0, profile="doppler", z=1100.0, zeta=1.0, x_esc=6.0, cell_cm=CELL_CM, w0=1 << 31,
             cosmo=_cosmo(), n_packets=0, seed=1)
    d.update(more)
    return SimpleNamespace(**d)


def _field_box(case, field_seed, k, nx, ny, nz, rms, **more):
    g = _gen(field_seed, k)
    if case.get("field", "grf") == "lognormal":
        od, vel = _lognormal(nx, ny, nz, 0.3, g), None
        if case["vel"] != "none":
            vel = _grf(nx, ny, nz, 0.5, g)[1]
    else:
        od, vel = _grf(nx, ny, nz, rms, g)
    vel = None if case["vel"] == "none" else vel.to(torch.float16 if case["vel"] == "f16" else torch.float32)
    xe = None
    if case["xe"] == "field":
        xe = 0.1 * torch.exp(0.2 * torch.randn((nz, ny, nx), generator=g, device=DEV))
    return _box(nx, ny, nz, od, vel, xe, **more)


def _step_boxes(case, seed):
    if case["boxes"] == 1:
        return [_field_box(case, seed, 0, case["nx"], case["ny"], case["nz"], case["rms"], profile=case["profile"],
                           z=case["z"], n_packets=case["packets"], seed=seed)]
    # uneven boxes: edges down to a fifth of the largest, redshift z down to z - 600, contrast up to rms
    r = np.random.Generator(np.random.Philox(1000 + case["boxes"]))    # the set of boxes belongs to the case
    out = []
    for b in range(case["boxes"]):
        n = [max(8, int(round(e * r.uniform(0.2, 1.0)))) for e in (case["nx"], case["ny"], case["nz"])]
        z = float(r.uniform(max(800.0, case["z"] - 600.0), case["z"]))
        out.append(_field_box(case, seed, b, *n, float(r.uniform(0.1, 1.0)) * case["rms"], profile=case["profile"],
                              z=z, temp_K=2.7255 * (1.0 + z), n_packets=case["packets"], seed=seed + b))
    return out


def _params(seed):
    """A network's parameters: weights uniform in +-1/sqrt(fan-in), biases small."""
    u = np.random.Generator(np.random.Philox(int(seed))).random(4801) * 2.0 - 1.0
    u[:512] /= math.sqrt(8)
    u[512:576] *= 0.05
    u[576:4672] /= 8.0
    u[4672:4736] *= 0.05
    u[4736:4800] /= 8.0
    u[4800] *= 0.05
    return u.astype(np.float32)


def _samples(seed, n):
    """Features, ln M and weights of n cells, as the Monte Carlo leaves them."""
    g = _gen(seed, 5)
    r = lambda: torch.randn(n, generator=g, device=DEV)                   # noqa: E731
    ln_d = 0.5 * r() - 0.12
    mean = torch.exp(0.6 * ln_d + 0.2 * r())
    var = (0.4 * mean * torch.exp(0.5 * r())).square()
    box = torch.randint(0, 3, (n,), generator=g, device=DEV)
    clump = torch.tensor([0.09, 0.2, 0.9], device=DEV)[box]
    x = torch.stack([ln_d, mean, var, 0.02 * r(), torch.zeros_like(mean), torch.full_like(mean, 0.1),
                     torch.zeros_like(mean), clump], dim=1).contiguous()
    y = 0.55 * ln_d - 0.2 * torch.log(mean) - 0.4 * clump + 0.05 * r()
    w = torch.exp(2.0 * ln_d)
    return x, y.contiguous(), (w / w.sum()).contiguous()


def _envelope():
    """Bounds that a few per cent of a new box's cells leave."""
    lo = np.array([-1.6, 0.2, -0.05, -0.1, -1.0, -0.1, -1.0, -0.1], dtype=np.float32)
    return lo, np.array([1.1, 2.4, 1.5, 0.1, 1.0, 1.1, 1.0, 2.0], dtype=np.float32)


def prepare(case, seed):
    do = case["do"]
    if do == "step":
        boxes = _step_boxes(case, seed)
        sim = M.Simulation(boxes, device=DEV)
        return SimpleNamespace(do=do, sim=sim, emitted=case["emitted"], targets=case["targets"])
    if do == "evolve":
        n = case["n"]
        g = _gen(seed)
        # two zones in slabs, as in the tests of the history, with some scatter
        slab = torch.where(torch.arange(n, device=DEV) % 2 == 0, 1.5, 0.5).expand(n, n, n)
        od = slab * torch.exp(0.05 * torch.randn((n, n, n), generator=g, device=DEV))
        od = (od / od.mean()).contiguous()
        x0 = torch.clamp(0.55 - 0.1 * (od - 1.0), 0.05, 0.95).contiguous()
        box = _box(n, n, n, od, None, x0.clone(), z=case["z"], temp_K=2.7255 * (1.0 + case["z"]),
                   cell_cm=case["cell_pc"] * KPC_CM / 1e3, n_packets=case["packets"], seed=seed)
        sim = M.Simulation(box, device=DEV, evolve=True)
        return SimpleNamespace(do=do, sim=sim, x0=x0, z=case["z"], steps=case["steps"], packets=case["packets"],
                               seed=seed)
    if do == "scatter":
        n = case["n"]
        box = _box(n, n, n, _lognormal(n, n, n, 0.3, _gen(seed)), profile=case["profile"], zeta=case["zeta"],
                   n_packets=case["photons"], seed=seed)
        return SimpleNamespace(do=do, sim=M.Simulation(box, device=DEV), p=case["p_destroy"])
    if do in ("surrogate", "correction"):
        box = _field_box(case, seed, 0, case["nx"], case["ny"], case["nz"], case["rms"], n_packets=1, seed=seed)
        sim = M.Simulation(box, device=DEV, max_packets=1)
        mlp = M.Mlp(_params(seed), device=DEV)
        s = SimpleNamespace(do=do, sim=sim, mlp=mlp, fallback=None)
        if do == "correction":
            mlp.set_envelope(*_envelope())
            s.fallback = torch.exp(0.3 * torch.randn(box.ncells, generator=_gen(seed, 9), device=DEV))
        return s
    x, y, w = _samples(seed, case["cells"])
    s = SimpleNamespace(do=do, mlp=M.Mlp(_params(seed), device=DEV), x=x, y=y, w=w)
    if do == "train":
        s.idx = torch.randint(0, case["cells"], (case["steps"], case["batch"]), generator=_gen(seed, 6), device=DEV)
        s.lrs = _rates(case["steps"])
    return s


def _rates(steps):
    return [3e-3 * 0.1 ** (k / 3000.0) for k in range(steps)]


# ---- one pass -------------------------------------------------------------------

def run(s):
    if s.do == "step":
        s.sim.refresh()
        s.sim.emit()
        s.sim.transport()
        t = s.sim.tally(want_emitted=s.emitted)
        f = s.sim.feed()
        out = {"absorbed": t["absorbed"], "ndot_e": f["ndot_e"], "mix_corr": f["mix_corr"],
               "totals": np.array([[b.absorbed, b.escaped, b.capped_weight, b.crossings, b.packets, b.wing]
                                   for b in t["stats"]], dtype=np.int64),
               "rates": np.array([[b.c_mc, b.c_mix, b.f_escape, b.x_e_global, b.ndot_e_mean, b.f_wing]
                                  for b in f["stats"]])}
        if s.emitted:
            out["emitted"] = t["emitted"]
        if s.targets:
            out["ln_m"], out["share"] = s.sim.targets()
        return out
    if s.do == "evolve":
        xe = s.sim.x_e_field(0)
        xe.copy_(s.x0)
        X = s.sim.evolve(s.z, s.z - 0.5 * s.steps, s.steps, [s.packets], s.seed)
        return {"X": X, "x_e": xe}
    if s.do == "scatter":
        s.sim.emit()
        rec = s.sim.scatter(p_destroy=s.p, records=True)
        t = s.sim.tally(want_emitted=False)
        f = s.sim.feed()
        st = t["stats"][0]
        out = {k: np.ascontiguousarray(rec[k]).astype(np.int64) for k in ("cell_end", "scatterings", "crossings",
                                                                          "fate", "escaped", "absorbed", "wing")}
        out.update({k: np.ascontiguousarray(rec[k]) for k in ("x_end", "dx", "dy", "dz")})
        out.update(tally=t["absorbed"], mix_corr=f["mix_corr"],
                   totals=np.array([st.absorbed, st.escaped, st.crossings, st.scatterings, st.wing], dtype=np.int64))
        return out
    if s.do == "surrogate":
        f = s.sim.features()
        return {"features": f, "y": s.mlp.forward(f)}
    if s.do == "correction":
        m, y, flags, count = s.mlp.correction(s.sim.features(), fallback=s.fallback)
        return {"M": m, "y": y, "outside": flags, "count": int(count)}
    if s.do == "gradient":
        g, loss = s.mlp.gradient(s.x, s.y, s.w)
        return {"gradient": np.array(g, dtype=np.float32), "loss": float(loss)}
    losses = s.mlp.train_steps(s.x, s.y, s.w, s.idx, s.lrs, want_losses=True)
    return {"losses": np.array(losses, dtype=np.float32), "params": np.array(s.mlp.params(), dtype=np.float32)}


# ---- what a pass cannot do without ----------------------------------------------

_CROSSINGS = 85          # (packet, cell) segments a packet walks, about, at the paper's cell size
_SEGMENT_FLOPS = 60      # of one segment: face choice, drift, swept profile, deposit


def work(case):
    do = case["do"]
    net = 2 * (8 * 64 + 64 * 64 + 64)
    if do == "step":
        if case["boxes"] == 1:
            cells = case["nx"] * case["ny"] * case["nz"]
        else:
            cells = int(case["boxes"] * case["nx"] * case["ny"] * case["nz"] * 0.6 ** 3)
        packets = case["packets"] * case["boxes"]
        per = 4 + {"none": 0, "f16": 6, "f32": 12}[case["vel"]] + (4 if case["xe"] == "field" else 0)
        per += 8 + 8 + 4 + (8 if case["emitted"] else 0) + (8 if case["targets"] else 0)
        return {"bytes": cells * per, "flops": packets * _CROSSINGS * _SEGMENT_FLOPS}
    if do == "evolve":
        cells = case["n"] ** 3
        return {"bytes": cells * 12, "flops": 4 * case["steps"] * case["packets"] * _CROSSINGS * _SEGMENT_FLOPS}
    if do == "scatter":
        # about 1/p scatterings a photon, some 400 operations each (random words, velocity draw, new flight)
        events = case["photons"] / case["p_destroy"]
        return {"bytes": case["n"] ** 3 * 16 + case["photons"] * 72, "flops": 400.0 * events}
    if do in ("surrogate", "correction"):
        cells = case["nx"] * case["ny"] * case["nz"]
        per = 4 + {"none": 0, "f16": 6, "f32": 12}[case["vel"]] + (4 if case["xe"] == "field" else 0)
        per += (32 + 4) if do == "surrogate" else (4 + 4 + 4 + 1)
        return {"bytes": cells * per, "flops": cells * (net + 27 * 4)}
    if do == "gradient":
        return {"bytes": case["cells"] * 40 + 4801 * 8, "flops": 3 * net * case["cells"]}
    return {"bytes": case["steps"] * (case["batch"] * 48 + 4801 * 24), "flops": 3 * net * case["batch"] * case["steps"]}


# ---- the same in 64 bits ----------------------------------------------------------

def _features64(case, seed):
    b = _field_box(case, seed, 0, case["nx"], case["ny"], case["nz"], case["rms"])
    d = b.overdensity.double()
    around = [torch.roll(d, (i, j, k), (0, 1, 2)) for i in (-1, 0, 1) for j in (-1, 0, 1) for k in (-1, 0, 1)]
    mean = sum(around) / 27.0
    var = sum((a - mean).square() for a in around) / 27.0
    div = torch.zeros_like(d)
    if b.velocity is not None:
        for c, axis in ((0, 2), (1, 1), (2, 0)):
            v = b.velocity[c].double()
            div = div + 0.5 * (torch.roll(v, -1, axis) - torch.roll(v, 1, axis))
    xe = torch.full_like(d, float(np.float32(b.x_e_uniform))) if b.x_e is None else b.x_e.double()
    clump = torch.log(d.square().mean() / d.mean().square())
    f = [torch.log(d), mean, var, div, torch.full_like(d, math.log(b.temp_K / 3000.0)), xe,
         torch.full_like(d, b.z / 1000.0 - 1.1), torch.full_like(d, float(clump))]
    return torch.stack([t.reshape(-1) for t in f], dim=1)


def _net64(p, x):
    w1, b1, w2, b2 = p[:512].view(64, 8), p[512:576], p[576:4672].view(64, 64), p[4672:4736]
    return torch.relu(torch.relu(x @ w1.t() + b1) @ w2.t() + b2) @ p[4736:4800] + p[4800]


def exact(case, seed):
    do = case["do"]
    if do in ("step", "evolve", "scatter"):
        # random walks of integer weights: whole numbers that have to be the same
        return None
    p = torch.from_numpy(_params(seed)).to(DEV).double()
    if do in ("surrogate", "correction"):
        f = _features64(case, seed)
        y = torch.cat([_net64(p, part) for part in f.split(1 << 20)])
        if do == "surrogate":
            return {"features": f, "y": y}
        lo, hi = (torch.from_numpy(v).to(DEV).double() for v in _envelope())
        out = ((f < lo) | (f > hi)).any(1)
        back = torch.exp(0.3 * torch.randn(f.shape[0], generator=_gen(seed, 9), device=DEV)).double()
        return {"M": torch.where(out, back, torch.exp(y)), "y": y, "outside": None, "count": None}
    x, t, w = (a.double() for a in _samples(seed, case["cells"]))
    p.requires_grad_(True)

    def grad(x, t, w):
        loss = (w * (_net64(p, x) - t).square()).sum() / w.sum()
        return torch.autograd.grad(loss, p)[0], float(loss.detach())

    if do == "gradient":
        g, loss = grad(x, t, w)
        return {"gradient": g, "loss": loss}
    idx = torch.randint(0, case["cells"], (case["steps"], case["batch"]), generator=_gen(seed, 6), device=DEV)
    m, v, losses = torch.zeros_like(p), torch.zeros_like(p), []
    for k, lr in enumerate(_rates(case["steps"])):
        i = idx[k]
        g, loss = grad(x[i], t[i], w[i])
        losses.append(loss)
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        with torch.no_grad():
            p -= lr * (m / (1 - 0.9 ** (k + 1))) / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    return {"losses": np.array(losses), "params": p.detach()}
