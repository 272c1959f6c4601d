"""Performance cases of the engine: what its users run, from the smallest call to the largest.

Each case is one call (or one forward and backward, or a scoring and its spectrum) through
``paper_2501_19221_amd.qpa`` on instances of the families the repository generates, made
here with torch on the GPU from the seed alone so that fresh ones are quick to make.

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  instance in device memory, engine, parameters
  run(state)           one pass
  work(case)           bytes and operations that a pass cannot do without
  exact(case, seed)    outputs in 64 bits, for the cases that have such a value
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2501_19221_amd import qpa

DEV = "cuda"


def listed():
    return [
        # A small all-to-all QUBO with integer entries, brute-forceable size (the dense20
        # workload): all steps in one launch, latency and the call's fixed costs.
        {"name": "dense20", "family": "dense_int", "n": 20, "replicas": 256, "steps": 2000},
        # The size of the small benchmark sets (n = 40..200, 150 internal states).
        {"name": "dense100", "family": "dense_int", "n": 100, "replicas": 150, "steps": 1000},
        # A Wishart-planted instance as the optimality-gap tables solve it (FP32 couplings).
        {"name": "wishart512", "family": "dense_f32", "n": 512, "replicas": 256, "steps": 2000},
        # A dense Gaussian instance of ordinary, odd size on the BF16 matrix-core path.
        {"name": "sk1001", "family": "dense_bf16", "n": 1001, "replicas": 200, "steps": 1000},
        # The headline workload: dense SK, 4096 variables, 1024 replicas, 2000 steps, BF16.
        {"name": "sk4096", "family": "dense_bf16", "n": 4096, "replicas": 1024, "steps": 2000},
        # A Chimera C16 graph with +-1 couplings, the state on chip for all steps.
        {"name": "chimera16", "family": "chimera", "m": 16, "weights": "pm1", "solver": "pa",
         "replicas": 1024, "steps": 5000},
        # A tile-planted lattice of 90000 spins as the gap tables solve it, streamed sparse
        # step (fewer steps: each costs the same).
        {"name": "tile300", "family": "tile", "L": 300, "replicas": 256, "steps": 200},
        # A very large planted 3-regular graph with few replicas, two-pass binned step.
        {"name": "planted3r", "family": "planted3r", "n": 24_000_000, "replicas": 4, "steps": 100},
        # Many uneven Erdos-Renyi QUBOs in one call (the er512 workload).
        {"name": "er512", "family": "er_batch", "count": 512, "nmin": 100, "nmax": 2000,
         "replicas": 64, "steps": 500},
        # A step of schedule tuning: relaxed energy of a batch, forward and backward.
        {"name": "er_grad", "family": "er_grad", "count": 96, "nmin": 100, "nmax": 2000,
         "replicas": 64, "steps": 150, "ckpt": 50},
        # Simulated bifurcation steps on a dense SK instance, resumed through sbm_steps.
        {"name": "sbm_sk4096", "family": "sbm_dense", "n": 4096, "replicas": 1024, "steps": 40},
        # Scoring a caller's sample set and listing its low-energy spectrum.
        {"name": "samples", "family": "samples", "n": 1500, "replicas": 1024, "keep": 64},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    f = rng.choice(["dense_int", "dense_f32", "dense_bf16", "chimera", "tile", "planted3r",
                    "er_batch", "er_grad", "sbm_dense", "samples"])
    if f == "dense_int":
        return {"family": f, "n": _log(rng, 12, 200), "replicas": _log(rng, 16, 512),
                "steps": rng.randint(500, 2000)}
    if f == "dense_f32":
        return {"family": f, "n": _log(rng, 128, 2048), "replicas": _log(rng, 32, 512),
                "steps": rng.randint(100, 400)}
    if f == "dense_bf16":
        return {"family": f, "n": _log(rng, 256, 4096), "replicas": _log(rng, 64, 1024),
                "steps": rng.randint(100, 500)}
    if f == "chimera":
        return {"family": f, "m": rng.randint(4, 16), "weights": rng.choice(["pm1", "uniform"]),
                "solver": rng.choice(["pa", "sbm"]), "replicas": _log(rng, 64, 1024),
                "steps": rng.randint(500, 2000)}
    if f == "tile":
        return {"family": f, "L": 2 * rng.randint(48, 150), "replicas": _log(rng, 32, 256),
                "steps": rng.randint(50, 200)}
    if f == "planted3r":
        return {"family": f, "n": 2 * _log(rng, 1_000_000, 12_000_000),
                "replicas": rng.randint(1, 8), "steps": rng.randint(20, 60)}
    if f == "er_batch":
        lo = rng.randint(50, 400)
        return {"family": f, "count": _log(rng, 8, 256), "nmin": lo,
                "nmax": lo + rng.randint(50, 1200), "replicas": rng.choice([32, 64, 100, 128]),
                "steps": rng.randint(50, 200)}
    if f == "er_grad":
        lo = rng.randint(50, 400)
        return {"family": f, "count": _log(rng, 1, 48), "nmin": lo,
                "nmax": lo + rng.randint(50, 1200), "replicas": rng.choice([16, 64, 100]),
                "steps": rng.randint(50, 120), "ckpt": 50}
    if f == "sbm_dense":
        return {"family": f, "n": _log(rng, 256, 4096), "replicas": _log(rng, 32, 1024),
                "steps": rng.randint(10, 40)}
    return {"family": "samples", "n": _log(rng, 64, 3000), "replicas": _log(rng, 100, 2048),
            "keep": rng.randint(8, 100)}


# ---- instances (torch, on the GPU) ------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 13)


def _dense_int(n, g):
    """Symmetric int32 entries and linear terms, uniform in [-10, 10]."""
    u = torch.randint(-10, 11, (n, n), generator=g, device=DEV, dtype=torch.int32)
    q = torch.triu(u)
    q = q + torch.triu(q, 1).T
    c = torch.randint(-10, 11, (n,), generator=g, device=DEV, dtype=torch.int32)
    return qpa.Problem(qpa.QPA_KIND_QUBO, n, dense=q.contiguous(), linear=c)


def _sk(n, g):
    """J_ij ~ N(0, 1/n), fields ~ N(0, 0.1)."""
    j = torch.triu(torch.randn(n, n, generator=g, device=DEV) / math.sqrt(n), 1)
    b = torch.randn(n, generator=g, device=DEV) * math.sqrt(0.1)
    return qpa.Problem(qpa.QPA_KIND_ISING, n, dense=(j + j.T).contiguous(), linear=b)


def _wishart(n, g):
    """Wishart planting at alpha = 1: (1/n) W W^T without its diagonal, randomly gauged."""
    z = torch.randn(n, n, generator=g, device=DEV, dtype=torch.float64)
    w = math.sqrt(n / (n - 1.0)) * (z - z.mean(0, keepdim=True))
    s = 2.0 * torch.randint(0, 2, (n,), generator=g, device=DEV).double() - 1.0
    j = (w @ w.T) / n * torch.outer(s, s)
    j = ((j + j.T) / 2).fill_diagonal_(0.0)
    return qpa.Problem(qpa.QPA_KIND_ISING, n, dense=j.float().contiguous(),
                       linear=torch.zeros(n, device=DEV))


def _csr(kind, n, u, v, w, lin, index=torch.int32):
    """Both directions of the edges (u, v, w), rows in order, columns ascending."""
    key, order = torch.sort(torch.cat([u * n + v, v * n + u]))
    rows = torch.div(key, n, rounding_mode="floor")
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return qpa.Problem(kind, n, row_ptr=rp.int(), col=(key - rows * n).to(index),
                       weights=torch.cat([w, w])[order].contiguous(), linear=lin)


def _chimera(m, weights, g):
    """m x m cells of K4,4; couplings +-1 (int8) or uniform in [-1, 1] (float)."""
    cell = torch.arange(m * m, device=DEV).reshape(m, m, 1, 1)
    a = torch.arange(4, device=DEV)
    u = [(cell * 8 + a.reshape(4, 1)).expand(m, m, 4, 4).reshape(-1)]
    v = [(cell * 8 + 4 + a.reshape(1, 4)).expand(m, m, 4, 4).reshape(-1)]
    cell = cell.reshape(m, m, 1)
    u += [(cell[:-1] * 8 + a).reshape(-1), (cell[:, :-1] * 8 + 4 + a).reshape(-1)]
    v += [(cell[1:] * 8 + a).reshape(-1), (cell[:, 1:] * 8 + 4 + a).reshape(-1)]
    u, v, n = torch.cat(u), torch.cat(v), 8 * m * m
    if weights == "pm1":
        w = (2 * torch.randint(0, 2, u.shape, generator=g, device=DEV) - 1).to(torch.int8)
        lin = torch.zeros(n, dtype=torch.int8, device=DEV)
    else:
        w = 2.0 * torch.rand(u.shape, generator=g, device=DEV) - 1.0
        lin = 2.0 * torch.rand(n, generator=g, device=DEV) - 1.0
    return _csr(qpa.QPA_KIND_ISING, n, u, v, w, lin)


def _tile(L, g):
    """Periodic L x L lattice, edge magnitudes 1 or 2, randomly gauged, some frustrated."""
    i = torch.arange(L * L, device=DEV)
    x, y = i % L, torch.div(i, L, rounding_mode="floor")
    u = torch.cat([i, i])
    v = torch.cat([y * L + (x + 1) % L, ((y + 1) % L) * L + x])
    s = 2 * torch.randint(0, 2, (L * L,), generator=g, device=DEV) - 1
    mag = torch.randint(1, 3, u.shape, generator=g, device=DEV)
    neg = torch.rand(u.shape, generator=g, device=DEV) < 0.25
    w = torch.where(neg, 1, -mag) * s[u] * s[v]
    return _csr(qpa.QPA_KIND_ISING, L * L, u, v, w.to(torch.int8),
                torch.zeros(L * L, dtype=torch.int8, device=DEV))


def _planted3r(n, g):
    """A Hamiltonian cycle through a random order plus a random perfect matching without
    any of its edges; |w| in 1..7 gauged by a random planted state."""
    p = torch.randperm(n, generator=g, device=DEV)
    pos = torch.empty_like(p)
    pos[p] = torch.arange(n, device=DEV)
    q = torch.randperm(n, generator=g, device=DEV)
    mu, mv = q[0::2].clone(), q[1::2].clone()
    del q
    while True:
        d = (pos[mu] - pos[mv]) % n
        bad = torch.nonzero((d == 1) | (d == n - 1)).reshape(-1).tolist()
        if not bad:
            break
        for k in bad:
            j = (k + n // 5) % (n // 2)
            a, b = mv[k].item(), mv[j].item()
            mv[k], mv[j] = b, a
    nxt, prv = torch.empty_like(p), torch.empty_like(p)
    nxt[p], prv[p] = torch.roll(p, -1), torch.roll(p, 1)
    nb = torch.empty((n, 3), dtype=torch.int64, device=DEV)
    nb[:, 0], nb[:, 1] = nxt, prv
    nb[mu, 2], nb[mv, 2] = mv, mu
    del nxt, prv, p, pos
    nb = torch.sort(nb, 1).values
    rows = torch.arange(n, device=DEV).reshape(n, 1)
    s = (2 * torch.randint(0, 2, (n,), generator=g, device=DEV) - 1).to(torch.int8)
    # a magnitude that both ends agree on, from the pair
    mag = ((rows + nb) * 2654435761 % 2147483647 % 7 + 1).to(torch.int8)
    w = -mag * s.reshape(n, 1) * s[nb]
    return qpa.Problem(qpa.QPA_KIND_ISING, n,
                       row_ptr=(torch.arange(n + 1, device=DEV) * 3).int(),
                       col=nb.int().reshape(-1), weights=w.reshape(-1).contiguous(),
                       linear=torch.zeros(n, dtype=torch.int8, device=DEV))


def _er(n, g):
    """Erdos-Renyi QUBO: pairs with probability 0.1, int16 entries in [-100, 100]."""
    keep = torch.triu(torch.rand(n, n, generator=g, device=DEV) < 0.1, 1)
    q = torch.triu(torch.randint(-100, 101, (n, n), generator=g, device=DEV, dtype=torch.int16), 1)
    keep, q = keep | keep.T, q + q.T
    rc = torch.nonzero(keep)
    rp = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.cumsum(keep.sum(1), 0)
    c = torch.randint(-100, 101, (n,), generator=g, device=DEV, dtype=torch.int16)
    return qpa.Problem(qpa.QPA_KIND_QUBO, n, row_ptr=rp, col=rc[:, 1].to(torch.int16),
                       weights=q[keep], linear=c)


def _sizes(case):
    """Instance sizes of a batch, spread evenly over its range."""
    c, lo, hi = case["count"], case["nmin"], case["nmax"]
    return [lo + ((2 * k + 1) * 40503 % (2 * c)) * (hi - lo) // (2 * c) for k in range(c)]


# ---- one pass ---------------------------------------------------------------------------

def prepare(case, seed):
    f, g = case["family"], _gen(seed)
    R, T = case["replicas"], case.get("steps", 0)
    st = {"family": f, "engine": qpa.Engine(0)}
    s = int(seed) + 1
    if f == "dense_int":
        st["problem"] = _dense_int(case["n"], g)
        st["params"] = qpa.make_params(R, T, 0.002, 0.9, 30.0, 0.1, s)
    elif f == "dense_f32":
        st["problem"] = _wishart(case["n"], g)
        st["params"] = qpa.make_params(R, T, 0.125, 0.8, 8.0, 0.1, s)
    elif f == "dense_bf16":
        st["problem"] = _sk(case["n"], g)
        st["params"] = qpa.make_params(R, T, 0.2, 0.8, 4.0, 0.1, s, qpa.QPA_PREC_BF16)
    elif f == "chimera":
        st["problem"] = _chimera(case["m"], case["weights"], g)
        st["sbm"] = case["solver"] == "sbm"
        st["params"] = (qpa.make_sbm_params(R, T, 0.5, sigma0=0.1, seed=s) if st["sbm"] else
                        qpa.make_params(R, T, 0.2, 0.8, 10.0, 0.1, s))
    elif f == "tile":
        st["problem"] = _tile(case["L"], g)
        st["params"] = qpa.make_params(R, T, 0.1, 0.8, 10.0, 0.1, s)
    elif f == "planted3r":
        st["problem"] = _planted3r(case["n"], g)
        st["params"] = qpa.make_params(R, T, 0.1, 0.8, 10.0, 0.1, s)
    elif f == "er_batch":
        st["problems"] = [_er(n, g) for n in _sizes(case)]
        st["params"] = qpa.make_params(R, T, 0.0002, 0.8, 200.0, 0.1, s)
    elif f == "er_grad":
        st["problems"] = [_er(n, g) for n in _sizes(case)]
        st["args"] = (R, 0.1, s, case["ckpt"])
        st["eta"], st["alpha"], st["lam"] = (
            t.requires_grad_() for t in _schedule(T))
    elif f == "sbm_dense":
        st["problem"] = _sk(case["n"], g)
        st["params"] = qpa.make_sbm_params(R, 1000, 0.5, c0=0.5, seed=s)
        st["t1"] = T
        st["q0"] = 0.2 * torch.rand(R, case["n"], generator=g, device=DEV) - 0.1
        st["p0"] = torch.zeros_like(st["q0"])
    else:
        st["problem"], st["spins"] = _sample_set(case, g)
        st["params"] = qpa.make_params(R, 0, 0.1, 0.8, 1.0)
        st["keep"] = case["keep"]
    return st


def _schedule(T):
    return (torch.tensor(2e-4, dtype=torch.float64), torch.tensor(0.8, dtype=torch.float64),
            200.0 * (1.0 - torch.arange(T, dtype=torch.float64) / T))


def _sample_set(case, g):
    """A dense integer instance and samples with repeats: each a planted state with a few
    spins flipped, drawn from a quarter as many states."""
    n, R = case["n"], case["replicas"]
    prob = _dense_int(n, g)
    base = 2 * torch.randint(0, 2, (n,), generator=g, device=DEV) - 1
    k = max(1, R // 4)
    flip = torch.rand(k, n, generator=g, device=DEV) < 0.05
    states = torch.where(flip, -base, base).to(torch.int8)
    pick = torch.randint(0, k, (R,), generator=g, device=DEV)
    return prob, states[pick].contiguous()


def _solved(out, integer):
    keys = ("spins", "energy", "energy_i64", "best") if integer else ("spins", "energy", "best")
    return {k: out[k] for k in keys}


def run(st):
    f, eng = st["family"], st["engine"]
    if f == "er_batch":
        # one array per output over the whole batch, instances one after the other
        outs = [_solved(o, True) for o in eng.solve_batch(st["problems"], st["params"])]
        return {k: torch.cat([o[k].reshape(-1) for o in outs]) for k in outs[0]}
    if f == "er_grad":
        loss = qpa.RelaxedEnergy.apply(st["eta"], st["alpha"], st["lam"], eng, st["problems"],
                                       *st["args"])
        return (loss.detach(),) + torch.autograd.grad(loss, (st["eta"], st["alpha"], st["lam"]))
    if f == "sbm_dense":
        q, p = st["q0"].clone(), st["p0"].clone()
        g = eng.sbm_steps(st["problem"], st["params"], 0, st["t1"], q, p, want_g=True)
        return {"q": q, "p": p, "g": g}
    if f == "samples":
        e, ei, best = eng.energy(st["problem"], st["params"], st["spins"])
        low = eng.spectrum(st["spins"], e, st["keep"])
        return {"energy": e, "energy_i64": ei, "best": best, "low": low}
    if st.get("sbm"):
        return _solved(eng.sbm_solve(st["problem"], st["params"]),
                       not st["problem"].weights.is_floating_point())
    p = st["problem"]
    c = p.dense if p.dense is not None else p.weights
    return _solved(eng.solve(p, st["params"]), not c.is_floating_point())


def work(case):
    """Couplings and outputs moved once, plus x and m read and written every step where they
    (8 bytes per variable and replica) are far more than the chip's caches hold; one multiply
    and add per coupling, replica and step plus about 8 operations of each update."""
    f, R, T = case["family"], case["replicas"], case.get("steps", 0)
    if f in ("dense_int", "dense_f32", "dense_bf16", "sbm_dense"):
        n = case["n"]
        out = 12.0 * R * n if f == "sbm_dense" else 1.0 * R * n
        state = 8.0 * R * n if f == "sbm_dense" else 0.0
        return {"bytes": 4.0 * n * n + out + state, "flops": T * R * (2.0 * n * n + 8.0 * n)}
    if f == "chimera":
        n, nnz = 8 * case["m"] ** 2, 2 * (16 * case["m"] ** 2 + 8 * case["m"] * (case["m"] - 1))
        return {"bytes": 8.0 * nnz + n * R, "flops": T * R * (2.0 * nnz + 8.0 * n)}
    if f in ("tile", "planted3r"):
        n, d = (case["L"] ** 2, 4) if f == "tile" else (case["n"], 3)
        step = 5.0 * d * n + (16.0 * n * R if 8.0 * n * R > 2.0 ** 28 else 0.0)
        return {"bytes": T * step + 1.0 * n * R, "flops": T * R * (2.0 * d * n + 8.0 * n)}
    if f in ("er_batch", "er_grad"):
        n = float(sum(_sizes(case)))
        nnz = 0.1 * sum(k * (k - 1.0) for k in _sizes(case))
        big = 8.0 * n * R > 2.0 ** 28
        passes = 3.0 if f == "er_grad" else 1.0     # forward, recomputation, reverse
        step = 4.0 * nnz + (16.0 * n * R if big else 0.0)
        return {"bytes": passes * T * (step if big else 0.0) + 4.0 * nnz + n * R,
                "flops": passes * T * R * (2.0 * nnz + 8.0 * n)}
    n = case["n"]
    return {"bytes": 4.0 * n * n + 2.0 * n * R, "flops": 2.0 * R * n * n}


# ---- outputs in 64 bits -----------------------------------------------------------------

def exact(case, seed):
    f, g = case["family"], _gen(seed)
    if f == "sbm_dense":
        prob = _sk(case["n"], g)
        R, T = case["replicas"], case["steps"]
        q = (0.2 * torch.rand(R, case["n"], generator=g, device=DEV) - 0.1).double()
        j, b, p = prob.dense.double(), prob.linear.double(), torch.zeros_like(q)
        for t in range(T):
            h = q @ j + b
            p = p - 0.5 * ((q * q + 1.0 - t / 1000.0) * q + 0.5 * h)
            q = q + 0.5 * p
        return {"q": q, "p": p, "g": h}
    if f == "samples":
        prob, s = _sample_set(case, g)
        x = (1.0 + s.double()) / 2.0
        e = ((x @ prob.dense.double()) * x).sum(1) + x @ prob.linear.double()
        return {"energy": e, "energy_i64": None, "best": None, "low": None}
    if f == "er_grad" and case["count"] * case["steps"] <= 20000:
        return _exact_grad(case, seed, g)
    # whole annealing runs: the signs of the state steer it, so that a run in 64 bits is
    # another run
    return None


def _exact_grad(case, seed, g):
    R, T, m64 = case["replicas"], case["steps"], (1 << 64) - 1
    total, grads = 0.0, None
    for k, n in enumerate(_sizes(case)):
        prob = _er(n, g)
        rp = prob.row_ptr.long()
        rows = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
        j = torch.zeros(n, n, dtype=torch.float64, device=DEV)
        j[rows, prob.col.long()] = prob.weights.double()
        b = j.sum(1) + prob.linear.double()
        # initial state: SplitMix64 outputs 1 .. R n of the instance's seed
        with np.errstate(over="ignore"):
            z = (np.arange(1, R * n + 1, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
                 + np.uint64((int(seed) + 1 + k) & m64))
            z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
            z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        u = ((z ^ (z >> np.uint64(31))) >> np.uint64(40)).astype(np.float64) * 2.0 ** -24
        x = np.float32(0.1) * (2.0 * u - 1.0).astype(np.float32)
        x = torch.from_numpy(x.astype(np.float64)).to(DEV).reshape(R, n)
        m = torch.zeros_like(x)
        eta, alpha, lam = _schedule(T)
        eta, alpha, lam = (float(np.float32(eta)), float(np.float32(alpha)),
                           lam.float().double().to(DEV))
        xs, ms, hs, inside = [], [], [], []
        for t in range(T):
            h = x @ j + b
            xs.append(x), ms.append(m), hs.append(h)
            m = alpha * m - eta * (lam[t] * x + h)
            y = x + m
            inside.append((y.abs() <= 1.0))
            x = y.clamp(-1.0, 1.0)
        total = total + (0.5 * (x * (x @ j)).sum() + (x @ b).sum())
        xb, mb = x @ j + b, torch.zeros_like(x)
        de, da, dl = 0.0, 0.0, [None] * T
        for t in range(T - 1, -1, -1):
            yb = xb * inside[t]
            mu = mb + yb
            de = de - (mu * (lam[t] * xs[t] + hs[t])).sum()
            da = da + (mu * ms[t]).sum()
            dl[t] = -eta * (mu * xs[t]).sum()
            xb = yb - eta * (lam[t] * mu + mu @ j)
            mb = alpha * mu
        one = [de, da, torch.stack(dl)]
        grads = one if grads is None else [a + c for a, c in zip(grads, one)]
        del j, xs, ms, hs, inside
    scale = 1.0 / (R * case["count"])
    return tuple((scale * v).cpu() for v in [total] + grads)
