"""The cases the framework's speed is measured on: what programs do with it,
through its public Python API, over the sizes they do it at.

Every case is a chain of sweeps (or many of them) with its per-sweep records;
the kinds differ in the update, the lattice, who owns the buffers and how the
work reaches the library.  `listed()` are fixed representatives, `draw()` gives
others of the same kinds and ranges, lattice sizes that are not multiples of a
power of two among them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1101_0876_amd as potts

OPS_PER_SITE = 20  # 32-bit operations of the two Philox4x32-10 words of a site update


def beta_c(q):
    return math.log1p(math.sqrt(q))


def listed():
    return [
        # a program that looks at the lattice after every sweep: latency of one call
        dict(name="step_L64", kind="step", L=64, q=9, beta=1.02 * math.log(4.0), n=1),
        # the plain method: one small lattice, many sweeps, every record kept
        dict(name="plain_L64", kind="chain", L=64, q=9, beta=1.02 * math.log(4.0), n=1000),
        # finite-size scaling: a small lattice at the transition
        dict(name="chain_L256", kind="chain", L=256, q=6, beta=beta_c(6), n=400),
        # a decimal lattice size: not a multiple of 16
        dict(name="chain_L1000", kind="chain", L=1000, q=6, beta=beta_c(6), n=200),
        # the paper's end-to-end protocol, shortened: points of a heating ramp at L = 1024
        dict(name="ramp_L1024", kind="ramp", L=1024, q=9, points=3, equil=50, n=200),
        # one mid-size lattice on the caller's buffers and stream
        dict(name="device_L4096", kind="device", L=4096, q=6, beta=beta_c(6), n=128),
        # the benchmark's single large lattice
        dict(name="device_L32768", kind="device", L=32768, q=6, beta=beta_c(6), n=40),
        # heat-bath updates at the benchmark's size
        dict(name="heatbath_L8192", kind="heatbath", L=8192, q=9, beta=beta_c(9), n=50),
        # the simple-cubic lattice
        dict(name="cube_L256", kind="cube", L=256, q=3, beta=0.5505, n=400),
        # first and second neighbours (L a multiple of 12)
        dict(name="nnn_L2040", kind="nnn", L=2040, q=9, beta=0.8, j2=0.5, n=200),
        # replicas of mixed sizes in one batch
        dict(name="batch_96", kind="batch", jobs=96, lmin=7, lmax=11, n=100),
        # a burst of ramps through the serving loop
        dict(name="serve_16", kind="serve", jobs=16, lmin=7, lmax=10, points=4, n=160),
    ]


def _log(rng, lo, hi, step):
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(x / step)) * step))


def draw(rng):
    kind = rng.choice(["step", "chain", "chain", "chain", "ramp", "device", "device", "heatbath", "cube", "nnn",
                       "batch", "serve"])
    # q: the paper's values mostly, now and then another comparison class
    q = rng.choice([2, 3, 4, 6, 9, 12, 15, 16, 24, 96, 200])
    step = rng.choice([4, 4, 8, 16, 32])
    c = dict(kind=kind, q=q, beta=beta_c(q) * rng.uniform(0.97, 1.03))
    if kind == "step":
        c.update(L=_log(rng, 32, 2048, step), n=1)
    elif kind == "chain":
        L = _log(rng, 32, 3072, step)
        c.update(L=L, n=min(1000, max(40, 200_000_000 // (L * L))))
    elif kind == "ramp":
        L = _log(rng, 64, 2048, step)
        c.update(L=L, points=rng.randint(2, 5), equil=rng.randint(10, 60), n=min(300, max(40, 200_000_000 // (L * L))))
    elif kind == "device":
        L = _log(rng, 2048, 24576, step)
        c.update(L=L, n=max(20, min(128, 20_000_000_000 // (L * L))))
    elif kind == "heatbath":
        L = _log(rng, 64, 8192, step)
        c.update(L=L, n=max(40, min(500, 3_000_000_000 // (L * L))))
    elif kind == "cube":
        L = _log(rng, 16, 320, step)
        c.update(L=L, beta=0.5505, n=max(40, min(500, 6_000_000_000 // L**3)))
    elif kind == "nnn":
        L = _log(rng, 60, 4092, 12)
        c.update(L=L, beta=0.8, j2=rng.choice([0.25, 0.5, 1.0]), n=max(40, min(400, 1_000_000_000 // (L * L))))
    elif kind == "batch":
        c = dict(kind=kind, jobs=rng.randint(24, 128), lmin=6, lmax=rng.choice([8, 9, 10, 11]), n=rng.randint(40, 100))
    else:
        c = dict(kind=kind, jobs=rng.randint(4, 24), lmin=7, lmax=rng.choice([8, 9, 10]), points=rng.randint(2, 6),
                 n=rng.randint(60, 160))
    return c


def _jobs(case, seed):
    rng = np.random.default_rng(seed)
    Ls = 2 ** rng.integers(case["lmin"], case["lmax"] + 1, size=case["jobs"])
    qs = rng.integers(3, 13, size=case["jobs"])
    f = rng.uniform(0.98, 1.02, size=case["jobs"])
    return [dict(L=int(L), q=int(q), seed=int(seed) * 1000 + i + 1, start=potts.RANDOM,
                 beta=beta_c(int(q)) * float(x), nsweeps=case["n"]) for i, (L, q, x) in enumerate(zip(Ls, qs, f))]


def prepare(case, seed):
    kind, s = case["kind"], dict(case=case, seed=seed)
    if kind in ("step", "chain", "ramp") or (kind == "heatbath" and case["L"] < 2048):
        s["lat"] = potts.Lattice(case["L"], case["q"], seed + 1, potts.RANDOM)
    elif kind in ("device", "heatbath"):
        s["lat"] = potts.Lattice.from_torch(case["L"], case["q"], seed + 1, potts.RANDOM)
        # the program's own tensor: the first of the two buffers holds the lattice between calls
        s["spins"] = s["lat"]._keep[0].view(case["L"], case["L"])
    elif kind == "cube":
        s["lat"] = potts.Cube(case["L"], case["q"], seed + 1, potts.RANDOM)
    elif kind == "nnn":
        s["lat"] = potts.NnnLattice(case["L"], case["q"], seed + 1, potts.RANDOM)
    elif kind == "batch":
        s["batch"] = potts.Batch(_jobs(case, seed), tune=False)
    else:
        s["server"] = potts.Server()
        s["jobs"] = _jobs(case, seed)
    if kind == "ramp":
        b = beta_c(case["q"])
        s["betas"] = [b * (1.02 - 0.04 * k / max(case["points"] - 1, 1)) for k in range(case["points"])]
    return s


def _points(points):
    return np.array([[p["e"], p["C"], p["V_L"], p["m"], p["chi"]] for p in points])


def run(s):
    case = s["case"]
    kind, n = case["kind"], case["n"]
    if kind == "batch":
        s["batch"].run()
        r = s["batch"].results()
        # one replica is looked at more closely, the others by their statistics
        return {"e_sat": np.array([x["e_sat"] for x in r]), "nmax": np.array([x["nmax"] for x in r]),
                "stats": _points(r), "spins": s["batch"].spins(0),
                "records": s["batch"].records(0, r[0]["t"] - n, n)}
    if kind == "serve":
        srv, b = s["server"], s["jobs"]
        tickets = [srv.submit(j["L"], j["q"], j["seed"], j["start"],
                              [j["beta"] * (1.0 + 0.01 * k) for k in range(case["points"])], [n] * case["points"])
                   for j in b]
        srv.drain()
        srv.wait(len(b), 0)
        got = [srv.collect(t) for t in tickets]
        return {"e_sat": np.array([g["e_sat"] for g in got]), "nmax": np.array([g["nmax"] for g in got]),
                "stats": np.concatenate([_points(g["points"]) for g in got])}
    lat = s["lat"]
    t0 = lat.t
    if kind == "ramp":
        pts = lat.ramp(s["betas"], case["equil"], n)
        return {"stats": _points(pts), "records": lat.records(lat.t - n, n), "spins": lat.spins()}
    if kind == "heatbath":
        lat.sweep_heatbath(case["beta"], n)
    elif kind == "nnn":
        lat.sweep(case["beta"], case["j2"], n)
    else:
        lat.sweep(case["beta"], n)
    if kind == "step":
        o = lat.observables()
        return {"e_sat": o["e_sat"], "nmax": o["nmax"], "hist": o["hist"]}
    rec = lat.records(t0, n)
    # a large lattice stays on the GPU
    return {"records": rec, "spins": s["spins"] if "spins" in s else lat.spins()}


def _sites(case):
    """(sites summed over the case's lattices, site updates of a pass, bytes of records)"""
    kind, n = case["kind"], case["n"]
    if kind in ("batch", "serve"):
        # the mean of L^2 over the sizes drawn
        m = float(np.mean([4.0**k for k in range(case["lmin"], case["lmax"] + 1)]))
        sites = case["jobs"] * m
        n *= case.get("points", 1)
        return sites, sites * n, case["jobs"] * n * 8.0 * 9
    sites = float(case["L"]) ** (3 if kind == "cube" else 2)
    if kind == "ramp":
        n = case["points"] * (case["equil"] + n)
    return sites, sites * n, n * 8.0 * (case["q"] + (2 if kind == "nnn" else 1))


def work(case):
    """The lattice read once and written once, the records written; the random
    words of every site update (32-bit integer operations)."""
    sites, updates, rec = _sites(case)
    return {"bytes": 2.0 * sites + rec, "flops": OPS_PER_SITE * updates}


# ---- the chain in plain numpy, for the cases small enough -------------------

M0, M1, W0, W1 = 0xD2511F53, 0xCD9E8D57, 0x9E3779B9, 0xBB67AE85
LOW = np.uint64(0xFFFFFFFF)


def _philox(c0, c1, c2, c3, key):
    x = [np.uint64(c0), c1.astype(np.uint64), np.uint64(c2), np.uint64(c3)]
    k0, k1, sh = key & 0xFFFFFFFF, key >> 32, np.uint64(32)
    for r in range(10):
        a, b = np.uint64((k0 + r * W0) & 0xFFFFFFFF), np.uint64((k1 + r * W1) & 0xFFFFFFFF)
        p0, p1 = np.uint64(M0) * x[0], np.uint64(M1) * x[2]
        x = [(p1 >> sh) ^ x[1] ^ a, p1 & LOW, (p0 >> sh) ^ x[3] ^ b, p0 & LOW]
    return [np.broadcast_to(v, c1.shape) for v in x]


def _chain(L, q, key, beta, n):
    """Spins and records of n Metropolis sweeps from the random start."""
    chunk = np.arange(L * L // 4, dtype=np.uint64)
    sh = np.uint64(32)
    w = _philox(0, chunk, 0, 2, key)
    s = np.stack([(v * np.uint64(q)) >> sh for v in w], 1).reshape(L, L).astype(np.int64)
    thr = [1 << 32] + [min(int(math.exp(-beta * d) * 2.0**32), 2**32 - 1) for d in range(1, 5)]
    thr = np.array(thr, dtype=np.uint64)
    colour = np.add.outer(np.arange(L), np.arange(L)) & 1
    rec = np.zeros((n, 1 + q), dtype=np.int64)
    for t in range(n):
        for c in (0, 1):
            w = _philox(t & 0xFFFFFFFF, chunk, t >> 32, c, key)
            k = np.repeat(np.stack([w[0], w[2]], 1).reshape(L, L // 2), 2, 1)
            a = np.repeat(np.stack([w[1], w[3]], 1).reshape(L, L // 2), 2, 1)
            k = ((k * np.uint64(q)) >> sh).astype(np.int64)
            near = [np.roll(s, 1, 0), np.roll(s, -1, 0), np.roll(s, 1, 1), np.roll(s, -1, 1)]
            d = sum((v == s).astype(np.int64) - (v == k) for v in near)
            s = np.where((colour == c) & (a < thr[np.maximum(d, 0)]), k, s)
        rec[t, 0] = np.sum(s == np.roll(s, -1, 0)) + np.sum(s == np.roll(s, -1, 1))
        rec[t, 1:] = np.bincount(s.ravel(), minlength=q)
    return s.astype(np.uint8), rec


def exact(case, seed):
    if case["kind"] not in ("step", "chain") or case["L"] ** 2 * case["n"] > 20_000_000:
        return None  # minutes in numpy; the outputs are whole numbers and have to stay equal anyway
    spins, rec = _chain(case["L"], case["q"], seed + 1, case["beta"], case["n"])
    if case["kind"] == "step":
        return {"e_sat": int(rec[-1, 0]), "nmax": int(rec[-1, 1:].max()), "hist": rec[-1, 1:]}
    return {"records": rec, "spins": spins}
