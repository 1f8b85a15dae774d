"""The work that programs have this library do, as cases to be timed.

Every case is the whole call that a program with a new matrix makes: the
decomposition is set up, iterated and its results are fetched, through the
public entry points of paper_1309_0302_amd.binding.  The inputs are made on
the GPU from the seed, after the recipes of paper_1309_0302_amd.workloads
(X = low rank + sparse + noise at the sizes used there, in the tests and in
the benchmark).

In FP32 the spikes of the sparse part have magnitudes in [amp / 2, amp] with
random signs and k is their number (the planted form), so that the selected
support is a property of the input and not of the last bit of a residual: with
magnitudes down to zero the k-th largest residual lies among the noise, and
any two correct FP32 programs keep a few different entries there.  In FP64
that does not happen, and the spikes are uniform in [-amp, amp].  For the same
reason the multi-label matrices carry about as many labels per sample as their
subspaces can be told apart.
"""

import math
import random

import numpy as np
import torch

from paper_1309_0302_amd import binding as gd

DEV = "cuda"


# ---- the cases --------------------------------------------------------------

def _solve(name, m, n, r, q, T, dtype="f32", prec="native", rho=0.05, lstep=0):
    return {"name": name, "kind": "solve", "m": m, "n": n, "r": r, "q": q, "T": T,
            "dtype": dtype, "prec": prec, "rho": rho, "lstep": lstep}


def _video(name, frames, T, scene):
    # scene: the seed of the paths of the moving blocks (they decide k)
    return {"name": name, "kind": "video", "frames": frames, "r": 2, "q": 1, "T": T,
            "prec": "native", "scene": scene}


def listed():
    return [
        # a small matrix, a few iterations: launches and latency are all of it
        _solve("small_400x300_f32", 400, 300, 5, 2, 3),
        # the double-precision problem of the synthetic experiments (Table 1's first size)
        _solve("w1_500x500_f64", 500, 500, 5, 2, 20, dtype="f64"),
        # odd sizes on both sides, mixed precision, high rank
        _solve("ragged_2001x1503_r20_bf16", 2001, 1503, 20, 2, 10, prec="bf16"),
        # a surveillance sequence: pixels x frames, background of rank 2
        _video("video_25344x200_f32", 200, 50, 1002),
        # the large dense matrix, in the mixed-precision form and in plain FP32
        _solve("w3_10000x10000_r20_bf16", 10000, 10000, 20, 2, 30, prec="bf16", rho=0.02),
        _solve("w3_10000x10000_r20_f32", 10000, 10000, 20, 2, 10, rho=0.02),
        # a matrix with a tenth of its entries unobserved, completed
        {"name": "completion_10000x10000_r20", "kind": "completion", "m": 10000, "n": 10000,
         "r": 20, "q": 2, "T": 10, "frac": 0.1, "prec": "native"},
        # many problems of different sizes advanced together
        {"name": "batch_32_problems", "kind": "batch", "count": 32, "shapes": 1004, "mlo": 2000,
         "mhi": 20000, "nlo": 100, "nhi": 400, "q": 1, "T": 20},
        # the unrolled layer in a training step: forward, loss, backward
        {"name": "layer_16x4096x256_r4", "kind": "layer", "b": 16, "m": 4096, "n": 256, "r": 4,
         "q": 1, "T": 10, "dtype": "f32"},
        # the same in double precision on one small problem (gradient checks, small models)
        {"name": "layer_1x520x96_r3_f64", "kind": "layer", "b": 1, "m": 520, "n": 96, "r": 3,
         "q": 1, "T": 5, "dtype": "f64"},
        # greedy bilateral smoothing of a video-sized matrix
        {"name": "grebsmo_25344x500_r4", "kind": "grebsmo", "m": 25344, "n": 500, "r": 4, "dr": 1,
         "K": 10, "power": 2, "lam": 0.125, "dtype": "f32"},
        # multi-label training: label subspaces fitted one after another (labels: the seed of the
        # labels' row sets and ranks)
        {"name": "mse_65536x512_k16", "kind": "mse", "n": 65536, "p": 512, "k": 16, "rmax": 8,
         "prob": 0.05, "labels": 1011, "T": 10, "dtype": "f32"},
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["solve", "solve", "solve", "solve64", "video", "completion", "batch",
                       "layer", "grebsmo", "mse"])
    if kind == "solve":
        m, n = _logint(rng, 300, 10000), _logint(rng, 300, 10000)
        r = rng.randint(1, min(32, min(m, n) // 40))
        T = rng.randint(2, 12)
        # without power passes a sketch of many columns need not converge
        c = _solve("", m, n, r, rng.randint(0 if r <= 8 else 1, 2), T, prec=rng.choice(["native", "bf16"]),
                   rho=round(rng.uniform(0.01, 0.05), 3), lstep=rng.choice([0, 0, 0, 1]))
    elif kind == "solve64":
        m, n = _logint(rng, 100, 1500), _logint(rng, 100, 1500)
        r = rng.randint(1, min(20, max(1, min(m, n) // 40)))
        c = _solve("", m, n, r, rng.randint(0, 2), rng.randint(3, 20), dtype="f64")
    elif kind == "video":
        c = _video("", rng.randint(100, 500), rng.randint(10, 50), rng.randint(0, 1 << 30))
    elif kind == "completion":
        m, n = _logint(rng, 300, 8000), _logint(rng, 300, 8000)
        r = rng.randint(1, min(20, min(m, n) // 40))
        c = {"kind": "completion", "m": m, "n": n, "r": r, "q": rng.randint(0 if r <= 8 else 1, 2), "T": rng.randint(2, 10),
             "frac": round(rng.uniform(0.05, 0.3), 3), "prec": rng.choice(["native", "bf16"])}
    elif kind == "batch":
        c = {"kind": "batch", "count": rng.randint(2, 24), "shapes": rng.randint(0, 1 << 30),
             "mlo": 500, "mhi": 20000, "nlo": 100, "nhi": 512, "q": rng.randint(0, 2),
             "T": rng.randint(2, 20)}
    elif kind == "layer":
        f64 = rng.random() < 0.3
        c = {"kind": "layer", "b": 1 if f64 else rng.randint(1, 16),
             "m": _logint(rng, 200, 600 if f64 else 4096), "n": _logint(rng, 64, 160 if f64 else 512),
             "r": rng.randint(1, 4), "q": rng.randint(0, 2), "T": rng.randint(2, 10),
             "dtype": "f64" if f64 else "f32"}
    elif kind == "grebsmo":
        r = rng.randint(2, 8)
        c = {"kind": "grebsmo", "m": _logint(rng, 500, 25344), "n": _logint(rng, 200, 500), "r": r,
             "dr": rng.randint(1, 2), "K": rng.randint(4, 12), "power": rng.randint(1, 2),
             "lam": 0.125, "dtype": rng.choice(["f32", "f32", "f64"])}
    else:
        f64, k = rng.random() < 0.5, rng.randint(3, 16)
        c = {"kind": "mse", "n": _logint(rng, 4096, 32768 if not f64 else 8192),
             "p": rng.randint(100, 512 if not f64 else 256), "k": k, "rmax": rng.randint(3, 8),
             "prob": round(rng.uniform(0.2, 1.0) / k, 4), "labels": rng.randint(0, 1 << 30), "T": rng.randint(2, 10),
             "dtype": "f64" if f64 else "f32"}
    c.pop("name", None)
    return c


# ---- inputs -----------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _dt(case):
    return torch.float64 if case.get("dtype") == "f64" else torch.float32


def _spike(X, k, amp, dtype, g):
    """Add k spikes at uniformly drawn entries of X (in place)."""
    idx = torch.randperm(X.numel(), generator=g, device=DEV)[:k]
    u = torch.rand(k, generator=g, device=DEV, dtype=X.dtype) * 2.0 - 1.0
    if dtype == torch.float32:      # |v| in [amp / 2, amp]
        u = torch.sign(u) * (0.5 + 0.5 * u.abs())
    X.view(-1)[idx] += amp * u


def _lowrank_part(m, n, r, g):
    """U V^T with entries of unit variance."""
    std = (1.0 / math.sqrt(r)) ** 0.5
    U = torch.randn((m, r), generator=g, device=DEV, dtype=torch.float64) * std
    V = torch.randn((n, r), generator=g, device=DEV, dtype=torch.float64) * std
    return U @ V.t()


def _planted(m, n, r, k, amp, noise, dtype, g):
    """Low rank + k spikes + noise, built in FP64, cast once."""
    X = _lowrank_part(m, n, r, g)
    if k > 0:
        _spike(X, k, amp, dtype, g)
    X += torch.randn((m, n), generator=g, device=DEV, dtype=torch.float64) * noise
    return X.to(dtype)


def _scene(case, height=144, width=176, blocks=8, block=16):
    """Offsets of the moving blocks, pixels x frames."""
    rng = np.random.default_rng(case["scene"])
    frames = case["frames"]
    add = np.zeros((frames, height, width))
    lim = np.array([height - block, width - block])
    pos = np.stack([rng.integers(0, lim[0] + 1, blocks), rng.integers(0, lim[1] + 1, blocks)], 1)
    vel = rng.integers(1, 4, size=(blocks, 2)) * rng.choice([-1, 1], size=(blocks, 2))
    offs = rng.uniform(0.3, 0.7, size=blocks)
    for f in range(frames):
        for b in range(blocks):
            y, x = pos[b]
            add[f, y:y + block, x:x + block] += offs[b]
        pos += vel
        low, high = pos < 0, pos > lim
        vel[low | high] *= -1
        pos = np.where(low, -pos, np.where(high, 2 * lim - pos, pos))
    return add.reshape(frames, -1).T


def _batch_shapes(case):
    rng = random.Random(case["shapes"])
    out = []
    for _ in range(case["count"]):
        m, n = rng.randint(case["mlo"], case["mhi"]), rng.randint(case["nlo"], case["nhi"])
        out.append((m, n, rng.randint(1, 8), int(rng.uniform(0.03, 0.10) * m * n)))
    return out


def _labels(case):
    """Row sets of the labels and their ranks."""
    rng = np.random.default_rng(case["labels"])
    n, k = case["n"], case["k"]
    Y = rng.random((n, k)) < case["prob"]
    none = np.flatnonzero(~Y.any(axis=1))
    Y[none, rng.integers(0, k, size=none.size)] = True
    ranks = [int(v) for v in rng.integers(2, case["rmax"] + 1, size=k)]
    return [np.flatnonzero(Y[:, i]).astype(np.int64) for i in range(k)], ranks


def prepare(case, seed):
    g, kind, dt = _gen(seed), case["kind"], _dt(case)
    s = {"case": case, "seed": int(seed)}
    if kind == "video":
        A = _scene(case)
        s["k"] = int(np.count_nonzero(A))
        U = torch.rand((A.shape[0], 2), generator=g, device=DEV, dtype=torch.float64)
        V = torch.rand((A.shape[1], 2), generator=g, device=DEV, dtype=torch.float64)
        X = U @ V.t()
        X = X / X.max() + torch.from_numpy(A).to(DEV)
        X += torch.randn(X.shape, generator=g, device=DEV, dtype=torch.float64) * 0.02
        s["X"] = X.to(dt).contiguous()
    elif kind == "solve":
        m, n = case["m"], case["n"]
        s["k"] = int(case["rho"] * m * n)
        noise, amp = (math.sqrt(1e-3), 10.0) if dt == torch.float64 else (0.01, 5.0)
        s["X"] = _planted(m, n, case["r"], s["k"], amp, noise, dt, g)
    elif kind == "completion":
        m, n = case["m"], case["n"]
        s["X"] = _planted(m, n, case["r"], 0, 0.0, 0.01, dt, g)
        s["k"] = int(case["frac"] * m * n)
        hidden = torch.randperm(m * n, generator=g, device=DEV)[:s["k"]]
        s["support"] = torch.sort(hidden).values
        s["X"].view(-1)[hidden] = 0.0
    elif kind == "batch":
        s["specs"] = [(_planted(m, n, r, k, 5.0, math.sqrt(1e-3), dt, g), r, k, int(seed) + 17 * i)
                      for i, (m, n, r, k) in enumerate(_batch_shapes(case))]
    elif kind == "layer":
        b, m, n = case["b"], case["m"], case["n"]
        s["k"] = int(0.05 * m * n)
        s["X"] = torch.stack([_planted(m, n, case["r"], s["k"], 5.0, math.sqrt(1e-3), dt, g)
                              for _ in range(b)])
        s["Lt"] = torch.randn((b, m, n), generator=g, device=DEV, dtype=dt)
        s["St"] = torch.randn((b, m, n), generator=g, device=DEV, dtype=dt)
    elif kind == "grebsmo":
        m, n = case["m"], case["n"]
        s["X"] = _planted(m, n, case["r"], int(0.05 * m * n), 5.0, 0.02, dt, g)
    elif kind == "mse":
        n, p = case["n"], case["p"]
        labels, ranks = _labels(case)
        X = torch.zeros((n, p), device=DEV, dtype=torch.float64)
        for rows, r in zip(labels, ranks):
            X[torch.from_numpy(rows).to(DEV)] += _lowrank_part(rows.size, p, r, g)
        K = int(0.02 * n * p)
        _spike(X, K, 5.0, dt, g)
        X += torch.randn((n, p), generator=g, device=DEV, dtype=torch.float64) * math.sqrt(1e-3)
        s.update(X=X.to(dt), labels=labels, ranks=ranks, K=K)
    return s


# ---- one pass ---------------------------------------------------------------

def _named(UL, VL, idx, val, info):
    return {"UL": UL, "VL": VL, "S_idx": idx, "S_val": val, "info": info}


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind in ("solve", "video", "completion"):
        prec = gd.GODEC_PREC_BF16_REFINE if case["prec"] == "bf16" else gd.GODEC_PREC_NATIVE
        opts, _ = gd.make_opts(prec=prec, support=s.get("support"), lstep=case.get("lstep", 0))
        return _named(*gd.godec_solve(s["X"], case["r"], s["k"], case["q"], s["seed"], case["T"],
                                      opts))
    if kind == "batch":
        b = gd.GoDecBatch(s["specs"], case["q"])
        b.step(case["T"])
        f = [b.factors(i) for i in range(len(s["specs"]))]
        S = [b.S(i) for i in range(len(s["specs"]))]
        err = np.array([b.info(i)["rel_err_sq"] for i in range(len(s["specs"]))])
        b.close()
        # one tensor of each kind for all problems
        return {"UL": torch.cat([u.reshape(-1) for u, _ in f]),
                "VL": torch.cat([v.reshape(-1) for _, v in f]),
                "S_idx": torch.cat([i for i, _ in S]), "S_val": torch.cat([v for _, v in S]),
                "rel_err_sq": err}
    if kind == "layer":
        X = s["X"].detach().requires_grad_(True)
        L, S = gd.godec_layer_fn(X, case["r"], s["k"], case["q"], case["T"], s["seed"])
        loss = ((S - s["St"]) ** 2).sum() + ((L - s["Lt"]) ** 2).sum()
        (dX,) = torch.autograd.grad(loss, X)
        return {"L": L.detach(), "S": S.detach(), "dX": dX}
    if kind == "grebsmo":
        h = gd.GreBsmo(s["X"], case["r"], case["dr"], case["power"], case["lam"], s["seed"])
        info = h.solve(case["K"])
        U, Vt = h.factors()
        S = h.S()
        h.close()
        return {"U": U, "Vt": Vt, "S": S, "rank": info.rank, "rel_err_sq": info.rel_err_sq,
                "l1": info.l1}
    h = gd.GoDecMSE(s["X"], s["labels"], s["ranks"], s["K"], s["seed"])
    h.step(case["T"])
    f = [h.factors(i) for i in range(case["k"])]
    idx, val = h.S()
    info = h.info()
    h.close()
    return {"U": torch.cat([u.reshape(-1) for u, _ in f]),
            "V": torch.cat([v.reshape(-1) for _, v in f]), "S_idx": idx, "S_val": val,
            "rel_err_sq": info["rel_err_sq"]}


# ---- what a pass cannot do without ------------------------------------------

def _solve_work(m, n, r, k, q, T, e, lstep=0):
    """X in; the factors and S out; the products of Algorithm 1's chains and the residual."""
    passes = 2 * (2 * q + 1) + (1 if lstep else 2 * q + 1)
    return {"bytes": m * n * e + (m + n) * r * e + k * (8 + e),
            "flops": T * 2.0 * m * n * r * (passes + 1)}


def work(case):
    kind, e = case["kind"], 8 if case.get("dtype") == "f64" else 4
    if kind == "video":         # the blocks cover 8 x 256 of 25 344 pixels, less what overlaps
        n = case["frames"]
        return _solve_work(25344, n, case["r"], 0.078 * 25344 * n, case["q"], case["T"], e)
    if kind == "solve":
        k = case["rho"] * case["m"] * case["n"]
        return _solve_work(case["m"], case["n"], case["r"], k, case["q"], case["T"], e,
                           case["lstep"])
    if kind == "completion":
        m, n = case["m"], case["n"]
        w = _solve_work(m, n, case["r"], case["frac"] * m * n, case["q"], case["T"], e)
        w["bytes"] += 8 * case["frac"] * m * n      # the support
        return w
    if kind == "batch":
        ws = [_solve_work(m, n, r, k, case["q"], case["T"], e)
              for m, n, r, k in _batch_shapes(case)]
        return {"bytes": sum(w["bytes"] for w in ws), "flops": sum(w["flops"] for w in ws)}
    if kind == "layer":
        mn, r, q = case["b"] * case["m"] * case["n"], case["r"], case["q"]
        p = 2 * q + 1
        fwd = 2 * p + p + 1                          # products with D, and the residual
        bwd = fwd + 2 * (p + q + 2) + (p + q + 1)    # the panels again, their adjoints, X's update
        return {"bytes": 6 * mn * e, "flops": case["T"] * 2.0 * mn * r * (fwd + bwd)}
    if kind == "grebsmo":
        mn, r = case["m"] * case["n"], case["r"]
        ranks = list(range(case["dr"], r, case["dr"])) + [r]
        flops = sum(2.0 * mn * (2 * case["power"] * case["dr"] + 3 * case["K"] * x) for x in ranks)
        return {"bytes": 2 * mn * e, "flops": flops}
    # label rows: the labels drawn, and one for each sample that got none
    rows = case["n"] * (case["k"] * case["prob"] + (1 - case["prob"]) ** case["k"])
    r = (2 + case["rmax"]) / 2
    np_ = case["n"] * case["p"]
    return {"bytes": 2 * np_ * e + rows * r * e + case["k"] * case["p"] * r * e + 0.02 * np_ * 12,
            "flops": case["T"] * rows * case["p"] * r * 8.0}


# ---- the same in 64 bits ----------------------------------------------------

def _a1(seed, n, r):
    """The library's documented draw: SplitMix64 outputs as 53-bit uniforms, Box-Muller pairs."""
    npair = (n * r + 1) // 2
    i = np.arange(2 * npair, dtype=np.uint64)
    with np.errstate(over="ignore"):
        z = np.uint64(int(seed) & ((1 << 64) - 1)) + (i + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    u = ((z >> np.uint64(11)).astype(np.float64) + 0.5) * 2.0 ** -53
    rad, ang = np.sqrt(-2.0 * np.log(u[0::2])), 2.0 * math.pi * u[1::2]
    out = np.stack([rad * np.cos(ang), rad * np.sin(ang)], 1).reshape(-1)[: n * r]
    return torch.from_numpy(out.reshape(n, r)).to(DEV)


def _orth(Y):
    """The orthonormal factor of Y's QR with a positive diagonal (through Cholesky, twice;
    the r x r side on the CPU)."""
    for _ in range(2):
        Y = Y / Y.detach().abs().amax(dim=(-2, -1), keepdim=True)
        C = torch.linalg.cholesky((Y.transpose(-1, -2).contiguous() @ Y).cpu())
        inv = torch.linalg.solve_triangular(C, torch.eye(C.shape[-1], dtype=C.dtype).expand(C.shape),
                                            upper=False)
        Y = Y @ inv.transpose(-1, -2).to(Y.device)
    return Y


def _lowrank(D, A1, q, lstep=0):
    """The power-scheme update of Algorithm 1: factors of L (the last two dimensions are D's)."""
    Dt = D.transpose(-1, -2).contiguous()
    Z = A1
    for _ in range(2 * q + 1):
        Z = _orth(Dt @ (D @ Z))
    if lstep:
        return D @ Z, Z
    B = D @ Z
    for _ in range(q):
        B = D @ (Dt @ B)
    p = 2 * q + 1
    lam, V = torch.linalg.eigh((B.transpose(-1, -2).contiguous() @ B).cpu())
    K = (V * (lam ** ((1.0 - p) / (2.0 * p))).unsqueeze(-2)) @ V.transpose(-1, -2)
    return B @ K.to(D.device), Z


def _keeps_rank(D, A1, q):
    """The rank check of Algorithm 1 on the sketch Y2 = (D^T D)^(2q+1) A1."""
    Y, Dt = A1, D.t().contiguous()
    for _ in range(2 * q + 1):
        Y = Dt @ (D @ Y)
        Y = Y / Y.abs().max()
    sv = torch.linalg.svdvals(Y.cpu())
    return bool(sv[-1] ** 2 > 4 * A1.shape[1] * 2.0 ** -52 * sv[0] ** 2)


def _top(R, k):
    """Indices (ascending) of the k entries of largest magnitude."""
    idx = torch.topk(R.reshape(-1).abs(), k, sorted=False).indices
    return torch.sort(idx).values


def _godec64(X, r, k, q, seed, T, lstep=0, support=None):
    A1 = _a1(seed, X.shape[1], r)
    D = X.clone()
    for _ in range(T):
        if not lstep and not _keeps_rank(D, A1, q):
            return None     # the rank goes down on the way: no value of its own here
        UL, VL = _lowrank(D, A1, q, lstep)
        R = X - UL @ VL.t()
        idx = _top(R, k) if support is None else support
        val = R.view(-1)[idx]
        D.copy_(X)
        D.view(-1)[idx] -= val
    e2 = float((R ** 2).sum())
    off = R.clone()
    off.view(-1)[idx] = 0.0
    nx2 = float((X ** 2).sum())
    info = {"rel_err_sq": float((off ** 2).sum()) / nx2, "sum_r2": e2, "norm_x2": nx2,
            "threshold": float(val.abs().min()) if support is None and k else None}
    return _named(UL, VL, idx, val, info)


def exact(case, seed):
    s, kind = prepare(case, seed), case["kind"]
    if kind in ("solve", "video", "completion"):
        return _godec64(s["X"].double(), case["r"], s["k"], case["q"], s["seed"], case["T"],
                        case.get("lstep", 0), s.get("support"))
    if kind == "batch":
        got = [_godec64(X.double(), r, k, case["q"], sd, case["T"]) for X, r, k, sd in s["specs"]]
        if any(o is None for o in got):
            return None
        return {"UL": torch.cat([o["UL"].reshape(-1) for o in got]),
                "VL": torch.cat([o["VL"].reshape(-1) for o in got]),
                "S_idx": torch.cat([o["S_idx"] for o in got]),
                "S_val": torch.cat([o["S_val"] for o in got]),
                "rel_err_sq": np.array([o["info"]["rel_err_sq"] for o in got])}
    if kind == "layer":
        return _layer64(case, s)
    if kind == "grebsmo":
        return _grebsmo64(case, s)
    return _mse64(case, s)


def _layer64(case, s):
    """T unrolled iterations, the supports held fixed, differentiated by autograd."""
    X = s["X"].double().requires_grad_(True)
    b, m, n = X.shape
    A1 = torch.stack([_a1(s["seed"] + i, n, case["r"]) for i in range(b)])
    S = torch.zeros_like(X)
    for _ in range(case["T"]):
        UL, VL = _lowrank(X - S, A1, case["q"])
        R = X - UL @ VL.transpose(-1, -2).contiguous()
        M = torch.zeros((b, m * n), device=DEV, dtype=torch.float64)
        for i in range(b):
            M[i, _top(R[i].detach(), s["k"])] = 1.0
        S = M.view(b, m, n) * R
    L = X - R
    loss = ((S - s["St"]) ** 2).sum() + ((L - s["Lt"]) ** 2).sum()
    (dX,) = torch.autograd.grad(loss, X)
    return {"L": L.detach(), "S": S.detach(), "dX": dX}


def _grebsmo64(case, s):
    X, r, dr, lam = s["X"].double(), case["r"], case["dr"], case["lam"]
    m, n = X.shape
    Om = _a1(s["seed"], n, r)
    S, U = torch.zeros_like(X), torch.zeros((m, 0), device=DEV, dtype=torch.float64)
    V = torch.zeros((0, n), device=DEV, dtype=torch.float64)
    c = 0
    while c < r:
        R = X - U @ V - S
        Z = Om[:, c:min(c + dr, r)].contiguous()
        for _ in range(case["power"]):
            Z = _orth(R.t() @ (R @ Z))
        V = torch.cat([V, Z.t()])
        c = V.shape[0]
        for _ in range(case["K"]):
            D = X - S
            U = _orth(D @ V.t().contiguous())
            V = U.t().contiguous() @ D
            E = X - U @ V
            S = torch.sign(E) * torch.clamp(E.abs() - lam, min=0.0)
    err = float(((X - U @ V - S) ** 2).sum()) / float((X ** 2).sum())
    return {"U": U, "Vt": V.t().contiguous(), "S": S, "rank": None, "rel_err_sq": err,
            "l1": float(S.abs().sum())}


def _mse64(case, s):
    X, k, K = s["X"].double(), case["k"], s["K"]
    n, p = X.shape
    rows = [torch.from_numpy(v).to(DEV) for v in s["labels"]]
    cnt = torch.zeros(n, device=DEV, dtype=torch.float64)
    for v in rows:
        cnt[v] += 1.0
    Ls = [X[v] / cnt[v, None] for v in rows]
    E = X.clone()
    for v, L in zip(rows, Ls):
        E[v] -= L
    fU, fV = [None] * k, [None] * k
    for t in range(case["T"]):
        for i, v in enumerate(rows):
            N = E[v] + Ls[i]
            Q = _orth(N.t() @ (N @ _a1(s["seed"] + t * k + i, p, s["ranks"][i])))
            fU[i], fV[i] = N @ Q, Q
            Ls[i] = fU[i] @ Q.t()
            E[v] = N - Ls[i]
        if t > 0:
            E.view(-1)[idx] += val
        idx = _top(E, K)
        val = E.view(-1)[idx]
        E.view(-1)[idx] = 0.0
    return {"U": torch.cat([u.reshape(-1) for u in fU]),
            "V": torch.cat([v.reshape(-1) for v in fV]), "S_idx": idx, "S_val": val,
            "rel_err_sq": float((E ** 2).sum()) / float((X ** 2).sum())}
