"""What is timed of this library: the calls a program makes, through the
public binding, over the range of sizes it makes them at.

A case names its kind of work and its sizes.  The kinds:

  chain     mc_sweep on one chain, then the results a program reads after a
            stretch of sweeps: positions, running energy, the decision counts
            and, where g(r) is sampled on the way, the pair counts
  ensemble  the same on a batch of uneven chains in one launch
  energy    the double-precision total-energy audit of a chain
  rdf       one g(r) sample and its read-out
  da        sweeps with the two-stage (surrogate) test
  grad      one gradient of the surrogate network
  train     one training call on a chain's move log

Starts are synthetic: random sites of a cubic lattice inside the wall, each
ion displaced at random within its cell as far as the hard cores allow, so
that a start is free of overlaps by construction at any density used here;
species are placed at random, ions ordered by species.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1602_05716_amd import mc, surrogate

# The system of the 3:-1 production runs, in ion diameters: Bjerrum length
# 7.117 A and bare Debye length 28.53 A at a diameter of 7.5 A.
LB_31 = 7.117 / 7.5
KAPPA_31 = 7.5 / 28.53
PHI_31 = 4.0 * KAPPA_31 ** 2 / (4.0 * math.pi * LB_31 * 12.0) * math.pi / 6.0


def listed():
    return [
        # the smallest calls: a few hundred ions, one sweep a call, as a
        # program does that looks at the state after every sweep
        dict(name="chain_f32_n300", kind="chain", precision="fp32", n=300, system="1:1", phi=0.02, lB=0.7,
             max_disp=0.5, sweeps=1, resum=100),
        # the double-precision workload (N = 1000), a block of ten sweeps
        dict(name="chain_f64_n1000", kind="chain", precision="fp64", n=1000, system="1:1", phi=0.01, lB=0.7,
             max_disp=0.5, sweeps=10, resum=100),
        # a mid-sized chain with an odd ion count (one neutral ion)
        dict(name="chain_f32_n4001", kind="chain", precision="fp32", n=4001, system="1:1", phi=0.03, lB=1.1,
             max_disp=2.0, sweeps=10, resum=10),
        # the headline workload: N = 32768, move size at about 40 %
        # acceptance, a hundred sweeps with the default re-sum at their end
        dict(name="chain_f32_n32768", kind="chain", precision="fp32", n=32768, system="1:1", phi=0.05, lB=0.7,
             max_disp=5.23, sweeps=100, resum=100),
        # a chain bound by its pair terms (N = 131072)
        dict(name="chain_f32_n131072", kind="chain", precision="fp32", n=131072, system="1:1", phi=0.05, lB=0.7,
             max_disp=4.44, sweeps=4, resum=0),
        # the charge- and size-asymmetric workload, g(r) every 10 sweeps
        dict(name="chain_2to1_n98304", kind="chain", precision="fp32", n=98304, system="2:1", phi=0.1, lB=0.7,
             max_disp=0.5, sweeps=10, resum=0, rdf_every=10, rmax=10.0, margin=0.0),
        # 256 uneven chains (N log-uniform in [500, 8000]) in one launch
        dict(name="ensemble_256", kind="ensemble", chains=256, n_min=500, n_max=8000, sweeps=20),
        # the energy audit after a stretch of sweeps
        dict(name="energy_f32_n65536", kind="energy", precision="fp32", n=65536, system="1:1", phi=0.05, lB=0.7),
        # one g(r) sample of the 3:-1 production system: range 10.5 bare
        # Debye lengths, centres ten more inside the wall
        dict(name="rdf_3to1_n131072", kind="rdf", precision="fp32", n=131072, system="3:1", phi=PHI_31, lB=LB_31,
             rmax=10.5 / KAPPA_31, margin=10.0 / KAPPA_31, bins=800),
        # one drift-monitor window of the two-stage chain
        dict(name="da_f32_n32768", kind="da", precision="fp32", n=32768, system="1:1", phi=0.05, lB=0.7,
             max_disp=5.23, sweeps=10),
        # one gradient of the network, at the batch the allocation-free
        # entry point is sized for
        dict(name="grad_b256", kind="grad", batch=256, noalloc=False),
        # training on a move log, one pass over it
        dict(name="train_n32768", kind="train", n=32768, sweeps=4, batch=4096, epochs=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["chain", "chain", "chain", "chain", "chain64", "2:1", "ensemble", "energy", "rdf", "da",
                       "grad", "train"])
    phi, lB = round(rng.uniform(0.005, 0.1), 4), round(rng.uniform(0.5, 2.0), 3)
    if kind == "chain":
        n = _log_int(rng, 200, 131072)
        sweeps = max(1, min(40, int(2.5e10 / (float(n) * n + 1.5e5 * n))))
        return dict(kind="chain", precision="fp32", n=n, system="1:1", phi=phi, lB=lB,
                    max_disp=round(math.exp(rng.uniform(math.log(0.3), math.log(6.0))), 3), sweeps=sweeps,
                    resum=rng.choice([0, sweeps]))
    if kind == "chain64":
        n = _log_int(rng, 64, 8192)
        return dict(kind="chain", precision="fp64", n=n, system=rng.choice(["1:1", "2:1"]), phi=phi, lB=lB,
                    max_disp=round(rng.uniform(0.3, 2.0), 3), sweeps=rng.randint(1, 20), resum=0)
    if kind == "2:1":
        n = _log_int(rng, 600, 98304)
        sweeps = max(1, min(20, int(2.5e10 / (float(n) * n + 1.5e5 * n))))
        return dict(kind="chain", precision="fp32", n=n, system="2:1", phi=phi, lB=lB, max_disp=0.5, sweeps=sweeps,
                    resum=0, rdf_every=rng.choice([1, sweeps]), margin=0.0,
                    rmax=round(min(10.0, rng.uniform(0.2, 0.6) * _radius("2:1", n, phi)), 2))
    if kind == "ensemble":
        return dict(kind="ensemble", chains=rng.randint(3, 256), n_min=300, n_max=rng.randint(2000, 8000),
                    sweeps=rng.randint(2, 20))
    if kind == "energy":
        return dict(kind="energy", precision=rng.choice(["fp32", "fp32", "fp64"]), n=_log_int(rng, 500, 65536),
                    system=rng.choice(["1:1", "2:1"]), phi=phi, lB=lB)
    if kind == "rdf":
        system = rng.choice(["1:1", "2:1", "3:1"])
        n = _log_int(rng, 1000, 131072)
        phi = PHI_31 if system == "3:1" else phi
        R = _radius(system, n, phi)
        return dict(kind="rdf", precision=rng.choice(["fp32", "fp32", "fp64"]), n=n, system=system, phi=phi, lB=lB,
                    rmax=round(min(40.0, rng.uniform(0.1, 0.5) * R), 2), margin=round(rng.choice([0.0, 0.2]) * R, 2),
                    bins=rng.choice([100, 200, 333]))
    if kind == "da":
        return dict(kind="da", precision="fp32", n=_log_int(rng, 2048, 32768), system="1:1", phi=phi, lB=lB,
                    max_disp=round(rng.uniform(0.5, 5.5), 3), sweeps=10)
    if kind == "grad":
        noalloc = rng.random() < 0.25
        return dict(kind="grad", batch=32 * rng.randint(1, 8 if noalloc else 128), noalloc=noalloc)
    return dict(kind="train", n=2 * rng.randint(6000, 16384), sweeps=4, batch=32 * rng.randint(2, 64), epochs=1)


# --------------------------------------------------------------------------- #
# Inputs                                                                      #
# --------------------------------------------------------------------------- #

def _radius(system, n, phi):
    """Wall radius of n ions at volume fraction phi, to rounding of the species counts."""
    return (n * (1.0 if system != "2:1" else (1.0 + 2.0 * 0.8 ** 3) / 3.0) / (8.0 * phi)) ** (1.0 / 3.0)


def _system(case_system, n, phi, rng):
    """(xyz, q, sigma, R) of a start with n ions at volume fraction phi."""
    if case_system == "2:1":
        n_a, qs, ss = n // 3, (2.0, -1.0), (1.0, 0.8)
        n_b = 2 * n_a
    elif case_system == "3:1":
        n_a, qs, ss = n // 4, (3.0, -1.0), (1.0, 1.0)
        n_b = 3 * n_a
    else:
        n_a, qs, ss = n // 2, (1.0, -1.0), (1.0, 1.0)
        n_b = n_a
    n_0 = n - n_a - n_b  # neutral ions make up an odd count
    q = np.concatenate([np.full(n_a, qs[0]), np.full(n_b, qs[1]), np.zeros(n_0)])
    sigma = np.concatenate([np.full(n_a, ss[0]), np.full(n_b, ss[1]), np.full(n_0, ss[1])])
    R = float((np.sum(sigma ** 3) / (8.0 * phi)) ** (1.0 / 3.0))
    a = R - 0.5
    cell = a * (4.0 * math.pi / 3.0 / (1.6 * n)) ** (1.0 / 3.0)  # about 1.6 sites an ion
    while True:  # narrower where fewer sites than ions fit inside the wall
        m = int(a / cell) + 1
        g = np.arange(-m, m + 1) * cell
        x = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
        half = 0.5 * (cell - 1.0)  # cores of diameter <= 1 stay apart
        room = a - math.sqrt(3.0) * max(half, 0.0) * 0.999
        x = x[np.einsum("ij,ij->i", x, x) <= room * room]
        if half >= 0.0 and len(x) >= n:
            break
        cell *= 0.97
        if cell < 1.0:
            raise ValueError("too dense for a lattice start")
    xyz = x[rng.permutation(len(x))[:n]] + rng.uniform(-half, half, (n, 3)) * 0.999
    return xyz, q, sigma, R


def _inputs(case, seed):
    rng = np.random.default_rng([seed, 1602])
    xyz, q, sigma, R = _system(case["system"], case["n"], case["phi"], rng)
    return xyz, q, sigma, R, int(rng.integers(1 << 62))


def _ensemble_inputs(case, seed):
    sizes = np.random.default_rng([case["chains"], case["n_min"], case["n_max"]])  # the case's own
    rng = np.random.default_rng([seed, 5716])
    out = []
    for _ in range(case["chains"]):
        n = int(2 * round(0.5 * math.exp(sizes.uniform(math.log(case["n_min"]), math.log(case["n_max"])))))
        phi, lB = float(rng.uniform(0.005, 0.1)), float(rng.uniform(0.5, 2.0))
        xyz, q, sigma, R = _system("1:1", n, phi, rng)
        # about the move size that gives 40 % acceptance at this density
        out.append((xyz, q, sigma, R, lB, min(R, 1.8 / phi ** (1.0 / 3.0))))
    return out, int(rng.integers(1 << 62))


def _grad_inputs(case, seed):
    """Neighbour histograms, targets and bfloat16 weights of a network."""
    rng = np.random.default_rng([seed, 33153])
    b = case["batch"]
    feats = rng.poisson(0.6, (b, 256)).astype(np.uint8)
    target = rng.normal(0.0, 0.5, b)
    params = rng.normal(0.0, 0.08, mc.DA_NPARAM).astype(np.float32)
    params = (torch.from_numpy(params).to(torch.bfloat16)).double().numpy()
    return feats, target, params


def _stream():
    """torch's default-priority side stream, as bench.py hands it over."""
    return torch.cuda.Stream()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "grad":
        feats, target, params = _grad_inputs(case, seed)
        return {"case": case, "feats": feats, "target": target, "params": params}
    stream = _stream()
    st = {"case": case, "stream": stream}
    if kind == "ensemble":
        systems, st["seed"] = _ensemble_inputs(case, seed)
        h = mc.Batch([s[:5] for s in systems], max_disp=[s[5] for s in systems], precision="fp32", resum_every=100,
                     hip_stream=stream.cuda_stream)
        h.autotune(2, st["seed"])  # the schedule a program keeps
        st["h"] = h
        return st
    if kind == "train":
        rng = np.random.default_rng([seed, 77])
        xyz, q, sigma, R = _system("1:1", case["n"], 0.05, rng)
        st["moves"] = case["sweeps"] * case["n"]
        h = mc.Chain(xyz, q, sigma, R, 0.7, precision="fp32", max_disp=1.5, resum_every=0, waves=4,
                     log_moves=st["moves"], hip_stream=stream.cuda_stream)
        h.sweep(case["sweeps"], int(rng.integers(1 << 62)))
        st["h"] = h
        return st
    xyz, q, sigma, R, st["seed"] = _inputs(case, seed)
    opts = dict(precision=case["precision"], max_disp=min(case.get("max_disp", 0.5), R),
                resum_every=case.get("resum", 0), hip_stream=stream.cuda_stream)
    if case.get("rdf_every") or kind == "rdf":
        opts.update(rdf_every=case.get("rdf_every", 0), rdf_bins=case.get("bins", 200), rdf_rmax=case["rmax"],
                    rdf_margin=case["margin"])
    if kind == "da":
        opts.update(waves=4, resum_every=100)
    h = mc.Chain(xyz, q, sigma, R, case["lB"], **opts)
    if kind == "da":
        h.set_surrogate(surrogate.truncated_coulomb_params(4.0), 0.9, True)
    st["h"] = h
    return st


# --------------------------------------------------------------------------- #
# One pass                                                                    #
# --------------------------------------------------------------------------- #

def _counts(stats):
    return np.array([stats["moves"], stats["accepted"], stats["rejected_wall"], stats["rejected_overlap"],
                     stats["rejected_metropolis"]], np.int64)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "grad":
        f = mc.mlp_grad_noalloc if case["noalloc"] else mc.mlp_grad
        loss, grad = f(state["feats"], state["target"], state["params"])
        # the library computes the gradient in float and hands it out in
        # doubles: the caller's float optimizer takes it back exactly
        return {"loss": loss, "grad": grad.astype(np.float32)}
    h = state["h"]
    if kind == "chain":
        h.sweep(case["sweeps"], state["seed"])
        out = {"xyz": h.positions(), "energy": h.energy(), "counts": _counts(h.stats())}
        if case.get("rdf_every"):
            r = h.rdf()
            out.update(g=r["g"], pairs=r["counts"].astype(np.int64), centres=r["centres"].astype(np.int64))
        return out
    if kind == "ensemble":
        h.sweep(case["sweeps"], state["seed"])
        m = h.count
        return {"xyz": np.concatenate([h.positions(k) for k in range(m)]),
                "energy": np.array([h.energy(k) for k in range(m)])}
    if kind == "energy":
        running, exact_ = h.energy(exact=True)
        return {"running": running, "exact": exact_}
    if kind == "rdf":
        h.rdf_reset()
        h.rdf_sample()
        r = h.rdf()
        return {"g": r["g"], "pairs": r["counts"].astype(np.int64), "centres": r["centres"].astype(np.int64)}
    if kind == "da":
        h.sweep(case["sweeps"], state["seed"])
        s = h.stats()
        return {"xyz": h.positions(), "energy": h.energy(), "counts": _counts(s),
                "stages": np.array([s["da_moves"], s["da_conflicts"], s["da_stage1_rejected"],
                                    s["da_stage1_passed"], s["da_stage2_rejected"]], np.int64)}
    t = h.train_surrogate(state["moves"], epochs=case["epochs"], batch=case["batch"], lr=2e-3, seed=7)
    # parameters are bfloat16 values handed out in doubles
    return {"params": t["params"].astype(np.float32), "loss": t["loss"], "val_loss": t["val_loss"]}


# --------------------------------------------------------------------------- #
# What a pass cannot do without                                               #
# --------------------------------------------------------------------------- #

def _ions(case):
    if case["kind"] == "ensemble":  # expected values of the log-uniform sizes
        a, b, m = float(case["n_min"]), float(case["n_max"]), case["chains"]
        l = math.log(b / a)
        return m * (b - a) / l, m * (b * b - a * a) / (2.0 * l)
    n = float(case["n"])
    return n, n * n


def work(case):
    kind = case["kind"]
    if kind == "grad":
        rows, layer = 2.0 * case["batch"], 2.0 * 128 * 128
        # two layers forward, the two weight gradients and one input gradient
        return {"bytes": 264.0 * case["batch"] + 2 * 8.0 * mc.DA_NPARAM, "flops": 5.0 * rows * layer}
    if kind == "train":
        moves = float(case["n"]) * case["sweeps"]
        return {"bytes": 273.0 * moves, "flops": case["epochs"] * 5.0 * 2.0 * moves * 2.0 * 128 * 128}
    n, n2 = _ions(case)
    rec = 16.0 if case.get("precision", "fp32") == "fp32" else 32.0
    if kind == "energy":  # 9 operations and an inverse square root a pair
        return {"bytes": 1.25 * rec * n, "flops": 0.5 * n2 * 10.0}
    rdf = 0.0
    if kind == "rdf" or case.get("rdf_every"):
        # the ordered pairs within rmax of the centres, 8 operations each
        R = _radius(case["system"], n, case["phi"])
        c = max(0.0, 1.0 - (case["rmax"] + case["margin"]) / R) ** 3
        rdf = 8.0 * n * c * n * min(1.0, (case["rmax"] / R) ** 3)
        if kind == "rdf":
            return {"bytes": 1.25 * rec * n, "flops": max(rdf, 8.0 * n)}
    s = float(case["sweeps"])
    if case.get("rdf_every"):
        rdf *= s // case["rdf_every"]
    # a pair term: two squared distances (8 each), two inverse square
    # roots, their difference, its weighted sum and the contact test; the
    # state is read once and written once a call
    return {"bytes": 2.25 * rec * n, "flops": s * n2 * 21.0 + rdf}


# --------------------------------------------------------------------------- #
# The same in 64 bits                                                         #
# --------------------------------------------------------------------------- #

def _philox_words(seed, sweep, n, chain=0):
    """Philox4x32-10 of counters (i, sweep, chain, 0), i < n: uint32 [n, 4]."""
    m = np.uint64(0xFFFFFFFF)
    c = [np.arange(n, dtype=np.uint64), np.full(n, sweep, np.uint64), np.full(n, chain, np.uint64),
         np.zeros(n, np.uint64)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & m, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1),
             p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return np.stack(c, -1)


def _energy64(x, q, lB):
    x = torch.as_tensor(x, dtype=torch.float64)
    q = torch.as_tensor(q, dtype=torch.float64)
    if torch.cuda.is_available():
        x, q = x.cuda(), q.cuda()
    n, e = len(q), 0.0
    step = max(1, int(3e7 // n))
    for a in range(0, n, step):
        d = torch.zeros((min(step, n - a), n), dtype=torch.float64, device=x.device)
        for k in range(3):
            d += (x[a:a + step, k, None] - x[None, :, k]) ** 2
        d.sqrt_()
        i = torch.arange(d.shape[0], device=x.device)
        d[i, a + i] = math.inf
        e += float((q[a:a + step, None] * q[None, :] / d).sum())
    return 0.5 * lB * e


def _rdf64(x, q, sigma, R, rmax, margin, bins):
    """(g, counts, centre counts), species by decreasing charge, then diameter."""
    keys = sorted({(float(a), float(b)) for a, b in zip(q, sigma)}, key=lambda t: (-t[0], t[1]))
    lut = {k: i for i, k in enumerate(keys)}
    t = np.array([lut[(float(a), float(b))] for a, b in zip(q, sigma)])
    nt, dr = len(keys), rmax / bins
    rc = R - rmax - margin
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    X = torch.as_tensor(x, dtype=torch.float64, device=dev)
    T = torch.as_tensor(t, device=dev)
    r2 = X[:, 0] * X[:, 0] + X[:, 1] * X[:, 1] + X[:, 2] * X[:, 2]
    idx = torch.nonzero(r2 <= rc * rc).reshape(-1) if rc >= 0 else torch.zeros(0, dtype=torch.int64, device=dev)
    cnt = torch.zeros(nt * nt * bins, dtype=torch.int64, device=dev)
    step = max(1, int(3e7 // len(x)))
    for a in range(0, len(idx), step):
        i = idx[a:a + step]
        d = [X[i, k, None] - X[None, :, k] for k in range(3)]
        d2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        d2[torch.arange(len(i), device=dev), i] = math.inf
        ii, jj = torch.nonzero(d2 < rmax * rmax * (1 + 1e-12), as_tuple=True)
        r = d2[ii, jj].sqrt()
        k = torch.floor(r / dr).long()
        ok = (r < rmax) & (k < bins)
        key = (T[i[ii]] * nt + T[jj]) * bins + k
        cnt += torch.bincount(key[ok], minlength=nt * nt * bins)
    counts = cnt.cpu().numpy().reshape(nt, nt, bins)
    cen = np.bincount(t[idx.cpu().numpy()], minlength=nt)
    edges = np.arange(bins + 1) * dr
    vol = 4.0 / 3.0 * math.pi * (edges[1:] ** 3 - edges[:-1] ** 3)
    g = np.zeros((nt, nt, bins))
    of = np.bincount(t, minlength=nt)
    for a in range(nt):
        for b in range(nt):
            rb = R - 0.5 * keys[b][1]
            dens = (of[b] - (a == b)) / (4.0 / 3.0 * math.pi * rb ** 3)
            den = cen[a] * dens * vol
            g[a, b] = np.where(den > 0, counts[a, b] / np.where(den > 0, den, 1.0), 0.0)
    return g, counts, cen


def _chain64(case, seed):
    """The sequential chain with every dE and contact test in double.  The
    float chain stores its positions and forms its trials in float: that is
    its state, and the exact chain has the same."""
    xyz, q, sigma, R, key = _inputs(case, seed)
    n, lB = case["n"], case["lB"]
    f = np.float32 if case["precision"] == "fp32" else np.float64
    D = f(2.0 * min(case["max_disp"], R))
    x = xyz.astype(f)
    X = [x[:, k].astype(np.float64) for k in range(3)]
    half = (0.5 * sigma).astype(f).astype(np.float64)
    qf = q.astype(f).astype(np.float64)
    e = _energy64(x.astype(np.float64), q, lB)
    acc = wall = over = 0
    for s in range(case["sweeps"]):
        w = _philox_words(key, s, n)
        if f is np.float32:
            u = (w[:, :3] >> np.uint64(8)).astype(f) * f(2.0 ** -24)
        else:
            u = w[:, :3].astype(f) * f(2.0 ** -32)
        step = D * (u - f(0.5))
        with np.errstate(divide="ignore"):
            thr = -np.log(w[:, 3].astype(np.float64) * 2.0 ** -32)
        for i in range(n):
            new = x[i] + step[i]
            nx, ny, nz = (float(v) for v in new)
            if nx * nx + ny * ny + nz * nz > (R - 0.5 * sigma[i]) ** 2:
                wall += 1
                continue
            d2 = (X[0] - nx) ** 2 + (X[1] - ny) ** 2 + (X[2] - nz) ** 2
            d2[i] = math.inf
            if np.any(d2 < (half + half[i]) ** 2):
                over += 1
                continue
            o2 = (X[0] - X[0][i]) ** 2 + (X[1] - X[1][i]) ** 2 + (X[2] - X[2][i]) ** 2
            o2[i] = math.inf
            de = lB * qf[i] * float(np.dot(qf, 1.0 / np.sqrt(d2) - 1.0 / np.sqrt(o2)))
            if de <= 0.0 or de < thr[i]:
                acc += 1
                e += de
                x[i] = new
                X[0][i], X[1][i], X[2][i] = nx, ny, nz
    moves = case["sweeps"] * n
    out = {"xyz": x.astype(np.float64), "energy": e,
           "counts": np.array([moves, acc, wall, over, moves - acc - wall - over], np.int64)}
    if case.get("rdf_every"):
        out.update(g=None, pairs=None, centres=None)
        if case["rdf_every"] == case["sweeps"]:
            g, pairs, cen = _rdf64(out["xyz"], q, sigma, R, case["rmax"], case["margin"], 200)
            out.update(g=g, pairs=pairs, centres=cen)
    return out


def _grad64(case, seed):
    """Backpropagation in double through the network's definition: hidden
    activations rounded to bfloat16, the rounding's derivative taken as 1."""
    f, y, p = _grad_inputs(case, seed)

    def t(a):
        return torch.as_tensor(a, dtype=torch.float64)

    H = 128
    W1, b1, p = t(p[:H * H]).reshape(H, H), t(p[H * H:H * H + H]), p[H * H + H:]
    W2, b2, w3 = t(p[:H * H]).reshape(H, H), t(p[H * H:H * H + H]), t(p[H * H + H:H * H + 2 * H])
    x = t(np.concatenate([f[:, :H], f[:, H:]]).astype(np.float64))
    B = len(y)
    z1 = x @ W1 + b1
    h1 = torch.relu(z1).float().to(torch.bfloat16).double()
    z2 = h1 @ W2 + b2
    h2 = torch.relu(z2).float().to(torch.bfloat16).double()
    o = h2 @ w3
    r = o[B:] - o[:B] - t(y)
    loss = float((r * r).mean())
    do = torch.cat([-2.0 * r / B, 2.0 * r / B])
    d2 = do[:, None] * w3[None, :] * (z2 > 0)
    d1 = (d2 @ W2.T) * (z1 > 0)
    g = torch.cat([(x.T @ d1).reshape(-1), d1.sum(0), (h1.T @ d2).reshape(-1), d2.sum(0), h2.T @ do, do.sum()[None]])
    return {"loss": loss, "grad": g.numpy()}


def exact(case, seed):
    kind = case["kind"]
    if kind == "grad":
        return _grad64(case, seed)
    if kind == "chain" and case["sweeps"] * float(case["n"]) * (2.5e4 + case["n"]) < 2.2e9:
        return _chain64(case, seed)
    if kind == "energy":
        xyz, q, _, _, _ = _inputs(case, seed)
        x = xyz.astype(np.float32) if case["precision"] == "fp32" else xyz
        e = _energy64(x.astype(np.float64), q, case["lB"])
        return {"running": e, "exact": e}
    if kind == "rdf":
        xyz, q, sigma, R, _ = _inputs(case, seed)
        x = (xyz.astype(np.float32) if case["precision"] == "fp32" else xyz).astype(np.float64)
        g, pairs, cen = _rdf64(x, q, sigma, R, case["rmax"], case["margin"], case["bins"])
        return {"g": g, "pairs": pairs, "centres": cen}
    return None
