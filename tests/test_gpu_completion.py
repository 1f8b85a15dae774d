"""GPU parity of GoDec matrix completion (Sec. 2: the S update on a fixed
support set) against the FP64 oracle, through the C ABI.

Per step: the GPU's own S_{t-1} is fed to the oracle's L update with the
oracle's A1, and L_t must match within 1e-10 (FP64) / 1e-5 (FP32), the
relative Frobenius bars of the BRP path (BF16 panels: 2e-3, then 1e-5 in the
refinement iteration).  The S list must be the given
support, bit for bit, and its values the GPU's own residual at those
entries, bit for bit.  Trajectories: a rank-3 matrix with 30 % of its entries
missing is completed to 1e-10 by both the GPU and the oracle.
"""
import numpy as np
import pytest
from conftest import oracle_a1

from oracle import completion_ref as cr
from oracle import godec_ref as g

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(X):
    return torch.from_numpy(np.ascontiguousarray(X)).cuda()


def case(m, n, r, frac, seed, dtype=np.float64, noise=0.0):
    rng = np.random.default_rng(seed)
    X0 = rng.standard_normal((m, r)) @ rng.standard_normal((r, n))
    X0 += noise * rng.standard_normal((m, n))
    miss = np.sort(rng.choice(m * n, size=int(round(frac * m * n)), replace=False))
    X = X0.copy()
    X.flat[miss] = 0.0
    return X0.astype(dtype), X.astype(dtype), miss


def make(X, r, q, miss, seed, prec=0):
    from paper_1309_0302_amd.binding import GoDec
    sup = torch.from_numpy(miss.astype(np.int64)).cuda()
    return GoDec(dev(X), r, int(miss.size), q, seed=seed, support=sup, prec=prec)


def per_step(X, r, q, miss, iters, tol, seed=3, prec=0, tols=None):
    print(f"\n[completion] shape={X.shape} dtype={X.dtype} r={r} q={q} missing={miss.size} "
          f"iters={iters} prec={prec}", flush=True)
    gd = make(X, r, q, miss, seed, prec)
    A1 = oracle_a1(gd)
    X64 = X.astype(np.float64)
    S = np.zeros_like(X64)
    errs = []
    for t in range(iters):
        r_eff = gd.info()["rank_eff"]
        gd.step(1, iters)
        torch.cuda.synchronize()
        ref = g.brp_power(X64 - S, A1[:, :r_eff], q)
        L = gd.L_dense().cpu().numpy().astype(np.float64)
        errs.append(g.rel_fro(L, ref.L))
        idx, val = gd.S()
        idx = idx.cpu().numpy()
        val = val.cpu().numpy()
        assert np.array_equal(idx, miss), t
        R = gd.residual().cpu().numpy()
        assert np.array_equal(val.view(np.uint8), R.flat[miss].view(np.uint8)), t
        S = np.zeros_like(X64)
        S.flat[idx] = val.astype(np.float64)
    print(f"  per-step L errors: {[f'{e:.2e}' for e in errs]}", flush=True)
    for t, e in enumerate(errs):
        assert e <= (tols[t] if tols is not None else tol), (t, e)
    gd.close()


@pytest.mark.parametrize("m,n,r,q", [(120, 100, 3, 1), (333, 257, 5, 2), (150, 400, 4, 0)])
def test_f64_per_step(m, n, r, q):
    _, X, miss = case(m, n, r, 0.3, seed=m + n)
    per_step(X, r, q, miss, 4, 1e-10)


@pytest.mark.parametrize("m,n,r,q", [(1000, 700, 8, 1), (2001, 1503, 20, 2), (30, 20, 2, 1)])
def test_f32_per_step(m, n, r, q):
    _, X, miss = case(m, n, r, 0.2, seed=m + n, dtype=np.float32, noise=1e-3)
    per_step(X, r, q, miss, 3, 1e-5)


def test_f64_completes_like_the_oracle():
    X0, X, miss = case(120, 100, 3, 0.3, seed=3)
    gd = make(X, 3, 1, miss, 9)
    gd.step(100)
    L = gd.L_dense().cpu().numpy()
    info = gd.info()
    ref = cr.godec_completion(X, 3, 1, oracle_a1(gd), miss, 100)
    eL = np.linalg.norm(L - X0) / np.linalg.norm(X0)
    print(f"\n[completion] 100 iterations: L vs truth {eL:.2e}, vs oracle "
          f"{np.linalg.norm(L - ref.L) / np.linalg.norm(ref.L):.2e}, rel err "
          f"{info['rel_err_sq']:.2e} (oracle {ref.rel_err_sq[-1]:.2e})", flush=True)
    assert eL <= 1e-10
    assert np.linalg.norm(L - ref.L) <= 1e-10 * np.linalg.norm(ref.L)
    assert info["rel_err_sq"] <= 1e-20 and info["nnz"] == miss.size
    gd.close()


def g_a1(seed, n, r):
    from oracle.rng_ref import a1_gaussian
    return a1_gaussian(seed, n, r)


def test_solve_tol_stops_like_the_oracle():
    from paper_1309_0302_amd.binding import godec_solve_tol, make_opts
    X0, X, miss = case(120, 100, 3, 0.3, seed=4)
    sup = torch.from_numpy(miss).cuda()
    opts, _ = make_opts(support=sup)
    out = godec_solve_tol(dev(X), 3, int(miss.size), 1, 11, 200, 1e-12, opts)
    info = out[-1]
    ref = cr.godec_completion(X, 3, 1, g_a1(11, 100, 3), miss, 200, eps=1e-12)
    assert info["iters"] == len(ref.rel_err_sq)
    assert info["rel_err_sq"] <= 1e-12


@pytest.mark.parametrize("bad", ["unsorted", "duplicate", "range", "k"])
def test_bad_support_rejected(bad):
    from paper_1309_0302_amd.binding import GoDec, GodecError
    _, X, miss = case(60, 50, 2, 0.2, seed=5)
    k = miss.size
    if bad == "unsorted":
        miss = miss[::-1].copy()
    elif bad == "duplicate":
        miss = np.concatenate([miss[:1], miss[:-1]])
    elif bad == "range":
        miss = miss.copy()
        miss[-1] = 60 * 50
    else:
        k = k - 1
    sup = torch.from_numpy(miss.astype(np.int64)).cuda()
    with pytest.raises(GodecError) as ei:
        GoDec(dev(X), 2, k, 1, support=sup)
    assert ei.value.status == 1


@pytest.mark.parametrize("m,n,r,q", [(1000, 700, 8, 1), (2001, 1503, 20, 2)])
def test_bf16_refine_per_step(m, n, r, q):
    """BF16 panels on the fixed support: 2e-3 per step before the refinement
    iteration, 1e-5 in it (the bars of the BRP path's BF16 form)."""
    _, X, miss = case(m, n, r, 0.2, seed=m + n + 1, dtype=np.float32, noise=1e-3)
    per_step(X, r, q, miss, 4, None, prec=1, tols=[2e-3, 2e-3, 2e-3, 1e-5])


@pytest.mark.parametrize("lstep,warm", [(1, 0), (0, 1), (1, 1)])
def test_completion_with_other_l_updates(lstep, warm):
    """The fixed-support S update combines with the projection form and the
    warm-started chains: the rank-3 matrix is still completed."""
    from paper_1309_0302_amd.binding import GoDec
    X0, X, miss = case(120, 100, 3, 0.3, seed=3)
    sup = torch.from_numpy(miss).cuda()
    gd = GoDec(dev(X), 3, int(miss.size), 1, seed=9, support=sup, lstep=lstep, warm_start=warm)
    gd.step(100)
    L = gd.L_dense().cpu().numpy()
    eL = np.linalg.norm(L - X0) / np.linalg.norm(X0)
    print(f"\n[completion] lstep={lstep} warm={warm}: L vs truth {eL:.2e}", flush=True)
    assert eL <= 1e-10
    gd.close()


@pytest.mark.parametrize("kind", ["equal", "last twice", "descending", "negative", "past the end"])
def test_bad_supports_are_refused_at_once(kind):
    """A list that is not strictly ascending within the matrix is GODEC_E_INVAL,
    whatever it holds, in the time a good one takes (a list of equal entries is
    one long run of the first word; the good list here is set up in
    milliseconds)."""
    import time
    from paper_1309_0302_amd.binding import GoDec, GodecError
    m, n, k = 5000, 4000, 10000000
    X = torch.randn((m, n), device="cuda:0")
    good = torch.arange(0, 2 * k, 2, device="cuda:0")
    GoDec(X, 2, k, 1, support=good).close()
    bad = good.clone()
    if kind == "equal":
        bad.zero_()
    elif kind == "last twice":
        bad[-1] = bad[-2]
    elif kind == "descending":
        bad = good.flip(0).contiguous()
    elif kind == "negative":
        bad[0] = -1
    else:
        bad[-1] = m * n
    torch.cuda.synchronize()
    t = time.perf_counter()
    with pytest.raises(GodecError) as ei:
        GoDec(X, 2, k, 1, support=bad)
    assert ei.value.status == 1 and time.perf_counter() - t < 1.0
