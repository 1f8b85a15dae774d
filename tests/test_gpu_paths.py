"""GPU checks of single branches of the launch code and of kernels at the
sizes where they can go wrong (tile edges, remainders, ends of the ranges)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1309_0302_amd import workloads as wl

pytestmark = pytest.mark.gpu


def topk_indices(R, k):
    """Ascending indices of the k largest |R| (ties by index, zeros never)."""
    a = np.abs(R).ravel()
    order = np.lexsort((np.arange(a.size), -a))[:k]
    return np.sort(order[a[order] > 0])


# 32 entries per bitmap word, 1024 words per scan block: one word, one entry
# past a word, one block, one block and one word, several blocks
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (4, 8, 32), (3, 11, 5), (64, 512, 0),
                                   (64, 512, 32768), (65, 505, 1700), (2100, 129, 20000)])
def test_batch_list_in_index_order(m, n, k):
    """godec_batch_get_S returns the list sorted by linear index, with the
    values of the residual the selection used."""
    from paper_1309_0302_amd.binding import GoDecBatch
    rng = np.random.default_rng(m + n)
    X = torch.from_numpy(rng.standard_normal((m, n)).astype(np.float32)).to("cuda:0")
    Y = torch.from_numpy(rng.standard_normal((70, 40)).astype(np.float32)).to("cuda:0")
    b = GoDecBatch([(X, 1, k, 3), (Y, 2, 140, 4)], 1)
    b.step(2)
    for i, kk in ((0, k), (1, 140)):
        idx, val = b.S(i)
        R = b.residual(i).cpu().numpy()
        ref = topk_indices(R, kk)
        assert np.array_equal(idx.cpu().numpy(), ref)
        assert np.array_equal(val.cpu().numpy(), R.ravel()[ref])
    b.step(1)   # the getter leaves the state of the iterations alone
    c = GoDecBatch([(X, 1, k, 3), (Y, 2, 140, 4)], 1)
    c.step(3)
    for i in (0, 1):
        for u, v in zip(b.S(i), c.S(i)):
            assert torch.equal(u, v)
    b.close()
    c.close()


# pieces of 16 rows x 64 columns, column blocks of 256: inside, at and past the
# edges; empty, partial and full supports; D, D and its bf16 copy, FP64
@pytest.mark.parametrize("prec", ["f32", "bf16", "f64"])
@pytest.mark.parametrize("m,n,frac", [(1, 1, 1.0), (16, 64, 0.5), (17, 65, 0.3), (33, 321, 0.0),
                                      (5, 300, 1.0), (70, 257, 0.05)])
def test_fixed_support_pass(m, n, frac, prec):
    """The list is the support with the residual the getter reports, and the
    working copy the pass leaves is X - S: the next L update on it agrees
    with the same update on X - S formed on the host (test bar: the FP32 or
    FP64 rounding of one rank-1 update, 1e-5 or 1e-11; bf16 panels 2e-3)."""
    from oracle.godec_ref import brp_power, rel_fro
    from oracle.rng_ref import a1_gaussian
    from paper_1309_0302_amd.binding import GoDec
    rng = np.random.default_rng(m * 1000 + n)
    dt = np.float64 if prec == "f64" else np.float32
    X = (np.outer(rng.uniform(1, 2, m), rng.uniform(1, 2, n))
         + 0.01 * rng.standard_normal((m, n))).astype(dt)
    sup = np.sort(rng.permutation(m * n)[:int(round(frac * m * n))]).astype(np.int64)
    sd = torch.from_numpy(sup).to("cuda:0")
    gd = GoDec(torch.from_numpy(X).to("cuda:0"), 1, sup.size, 1, seed=3, support=sd,
               prec=1 if prec == "bf16" else 0, refine_iters=1)
    gd.step(1, 3)
    idx, val = (t.cpu().numpy() for t in gd.S())
    assert np.array_equal(idx, sup)
    assert np.array_equal(val, gd.residual().cpu().numpy().ravel()[sup])
    info = gd.info()
    R = X.astype(np.float64) - gd.L_dense().cpu().numpy().astype(np.float64)
    on = np.zeros(m * n, bool)
    on[sup] = True
    obs = np.sum(R.ravel()[~on] ** 2) / np.sum(X.astype(np.float64) ** 2)
    assert abs(info["rel_err_sq"] - obs) <= 1e-6 * obs + 1e-13
    D = X.astype(np.float64).ravel()
    D[idx] -= val
    A1 = a1_gaussian(3, n, 1)
    for step, tol in ((2, {"f32": 1e-5, "bf16": 2e-3, "f64": 1e-11}[prec]),
                      (3, {"f32": 1e-5, "bf16": 1e-5, "f64": 1e-11}[prec])):
        gd.step(1, 3)
        ref = brp_power(D.reshape(m, n), A1, 1).L
        assert rel_fro(gd.L_dense().cpu().numpy().astype(np.float64), ref) <= tol
        idx, val = (t.cpu().numpy() for t in gd.S())
        D = X.astype(np.float64).ravel()
        D[idx] -= val
    gd.close()


# the L update through A = D^T D: panel widths, 16- and 32-column edges of its
# passes, the widest matrix and panel it takes and the first ones it leaves to
# the general path, few and many rows, q = 0, 1, 2, both forms of the update
@pytest.mark.parametrize("m,n,r,q,lstep", [
    (40, 31, 1, 0, 0), (64, 32, 2, 1, 0), (65, 33, 3, 2, 0), (700, 200, 8, 1, 1),
    (513, 256, 12, 2, 0), (400, 320, 16, 1, 0), (400, 321, 16, 1, 0), (90, 512, 8, 2, 0),
    (90, 513, 8, 2, 0), (6000, 100, 5, 1, 0), (20, 300, 4, 1, 0), (33, 17, 2, 0, 1)])
@pytest.mark.parametrize("dt,tol", [(np.float64, 1e-10), (np.float32, 1e-5)])
def test_l_update_of_narrow_matrices(m, n, r, q, lstep, dt, tol):
    """Two steps against the oracle's update on the library's own S (the bars
    of the per-step parity tests)."""
    from oracle import godec_ref as g
    from oracle.rng_ref import a1_gaussian
    from paper_1309_0302_amd.binding import GoDec
    w = wl.tiny(m, n, r, seed=m + n, dtype=dt)
    gd = GoDec(torch.from_numpy(w.X).to("cuda:0"), r, w.k, q, seed=9, lstep=lstep)
    A1 = a1_gaussian(9, n, r)
    X = w.X.astype(np.float64)
    D = X.copy()
    for _ in range(2):
        gd.step(1)
        ref = g.brp_projection(D, A1, q) if lstep else g.brp_power(D, A1, q)
        assert g.rel_fro(gd.L_dense().cpu().numpy().astype(np.float64), ref.L) <= tol
        UL, VL = (t.cpu().numpy().astype(np.float64) for t in gd.factors())
        assert np.abs(VL.T @ VL - np.eye(r)).max() <= 10 * tol
        idx, val = (t.cpu().numpy() for t in gd.S())
        D = X.copy()
        D.ravel()[idx] -= val
    assert gd.info()["rank_eff"] == r
    gd.close()


# the r x r eigen-solver: every padded width (one or several waves of items,
# one or two items per thread), full and padded, cold and warm starts
@pytest.mark.parametrize("m,n,r,q", [
    (60, 600, 2, 1), (70, 530, 7, 1), (600, 540, 11, 1), (540, 600, 16, 1), (530, 600, 17, 1),
    (600, 530, 20, 2), (530, 540, 23, 1), (540, 530, 32, 1), (530, 560, 29, 0)])
@pytest.mark.parametrize("dt,tol", [(np.float64, 1e-10), (np.float32, 1e-5)])
def test_core_of_every_width(m, n, r, q, dt, tol):
    """Three steps against the oracle's update on the library's own S (the
    bars of the per-step parity tests)."""
    from oracle import godec_ref as g
    from oracle.rng_ref import a1_gaussian
    from paper_1309_0302_amd.binding import GoDec
    w = wl.tiny(m, n, r, seed=m + n, dtype=dt)
    gd = GoDec(torch.from_numpy(w.X).to("cuda:0"), r, w.k, q, seed=9)
    A1 = a1_gaussian(9, n, r)
    X = w.X.astype(np.float64)
    D = X.copy()
    for _ in range(3):
        gd.step(1)
        ref = g.brp_power(D, A1, q)
        assert g.rel_fro(gd.L_dense().cpu().numpy().astype(np.float64), ref.L) <= tol
        idx, val = (t.cpu().numpy() for t in gd.S())
        D = X.copy()
        D.ravel()[idx] -= val
    assert gd.info()["rank_eff"] == r
    gd.close()


# partial Grams: rows at the edges of a step and past 128 steps (several steps
# per block), panels narrower than a tile, with and without chunk partials
@pytest.mark.parametrize("m,n,r,q", [
    (1, 600, 1, 1), (127, 640, 2, 1), (129, 16600, 3, 1), (16500, 520, 1, 1), (16385, 513, 2, 0),
    (2000, 16384, 5, 1)])
@pytest.mark.parametrize("dt,tol", [(np.float64, 1e-10), (np.float32, 1e-5)])
def test_panel_row_edges(m, n, r, q, dt, tol):
    """One step against the oracle's update (the bars of the per-step parity
    tests) and the orthonormality of V_L."""
    from oracle import godec_ref as g
    from oracle.rng_ref import a1_gaussian
    from paper_1309_0302_amd.binding import GoDec
    w = wl.tiny(m, n, r, seed=m + n, dtype=dt)
    gd = GoDec(torch.from_numpy(w.X).to("cuda:0"), r, w.k, q, seed=9)
    gd.step(1)
    ref = g.brp_power(w.X.astype(np.float64), a1_gaussian(9, n, r), q)
    assert g.rel_fro(gd.L_dense().cpu().numpy().astype(np.float64), ref.L) <= tol
    VL = gd.factors()[1].cpu().numpy().astype(np.float64)
    assert np.abs(VL.T @ VL - np.eye(r)).max() <= 10 * tol
    gd.close()


def _mse_identity(X, K, steps):
    """MSE training with one empty label: the sparse step selects from X
    itself, so the input sets the ties.  Yields S after each step."""
    from paper_1309_0302_amd.binding import GoDecMSE
    tr = GoDecMSE(torch.from_numpy(X).to("cuda:0"), [np.zeros(0, np.int64)], [1], K, seed=1)
    for _ in range(steps):
        tr.step(1)
        idx, val = tr.S()
        yield idx.cpu().numpy(), val.cpu().numpy(), tr.info()
    E = tr.residual().cpu().numpy()
    ref = X.copy()
    ref.ravel()[idx.cpu().numpy()] = 0
    assert np.array_equal(E, ref)
    tr.close()


# the last histogram bin: a few entries, over 1024 (radix select of its list),
# ties that fit and that do not (taken by index), more ties than the candidate
# buffer holds (index-ordered scan), nothing, everything, more than the nonzeros
@pytest.mark.parametrize("dt,n,p,K,values", [
    (np.float32, 300, 512, 50000, "ints"), (np.float64, 300, 256, 30000, "ints"),
    (np.float32, 2048, 512, 400000, "grid"), (np.float64, 3000, 200, 200001, "grid"),
    (np.float32, 1025, 77, 3000, "normal"), (np.float64, 1025, 77, 3000, "normal"),
    (np.float32, 4096, 512, 1000, "signs"), (np.float64, 5000, 256, 70, "signs"),
    (np.float32, 65, 33, 0, "normal"), (np.float32, 65, 33, 65 * 33, "normal"),
    (np.float64, 500, 100, 40000, "few"), (np.float32, 1, 1, 1, "normal"),
    (np.float64, 700, 256, 5000, "wide")])
def test_selection_lists(dt, n, p, K, values):
    """S against a sort of the input by (magnitude, index), in the first step
    (full histogram) and in later ones (carried window); the objective's
    sums to FP64 rounding of sums of n p terms."""
    rng = np.random.default_rng(n + p + K)
    x = rng.standard_normal((n, p))
    if values == "ints":
        x = np.round(3 * x)
    elif values == "grid":
        x = np.round(x * 512) / 512
    elif values == "signs":
        x = np.sign(x)
    elif values == "few":
        x = np.where(rng.random((n, p)) < 0.3, x, 0.0)
    elif values == "wide":
        x = x * 10.0 ** rng.integers(-30, 30, size=(n, p))
    X = x.astype(dt)
    ref = topk_indices(X, K)
    seen = []
    for idx, val, info in _mse_identity(X, K, 3):
        assert np.array_equal(idx, ref)
        assert np.array_equal(val, X.ravel()[ref])
        X64 = X.astype(np.float64)
        thr = np.abs(val).min() if ref.size == K and K > 0 else 0.0
        assert info["threshold"] == thr
        rest = np.delete(X64.ravel(), ref)
        # the objective is the difference of two sums of up to n p squares
        tol = 1e-15 * np.sqrt(n * p) * 4
        assert abs(info["rel_err_sq"] - np.sum(rest ** 2) / np.sum(X64 ** 2)) <= tol
        seen.append(info["rel_err_sq"])
    for idx, val, info in _mse_identity(X, K, 1):
        assert info["rel_err_sq"] == seen[0]


def _close_values(n, p, values, dt, rng):
    x = rng.standard_normal((n, p))
    if values == "ints":            # ties
        return np.round(3 * x).astype(dt)
    # many different values within 1e-5 of each other, less than a histogram bin
    return (np.round(8 * x) / 8 * (1 + 1e-5 * rng.random((n, p)))).astype(dt)


# a last bin of more than 2048 candidates, narrowed by key or by index: by the
# two passes there are when the candidates hold every entry, or by more; ties
# that are cut by the index, and ones that all fit
@pytest.mark.parametrize("dt,n,p,K,values", [
    (np.float32, 2048, 512, 400000, "clusters"), (np.float32, 8192, 512, 300000, "clusters"),
    (np.float64, 3000, 256, 200000, "clusters"), (np.float64, 9000, 256, 150000, "clusters"),
    (np.float32, 2048, 512, 400000, "ints"), (np.float32, 8192, 512, 300000, "ints"),
    (np.float64, 3000, 256, 200000, "ints"), (np.float64, 9000, 256, 150000, "ints"),
    (np.float32, 8192, 512, 0, "ints")])
def test_long_last_bins(dt, n, p, K, values):
    """S against a sort by (magnitude, index), its threshold, and the same
    objective on every run (K = 0: every entry of magnitude 3 or more)."""
    rng = np.random.default_rng(n + p + K)
    X = _close_values(n, p, values, dt, rng)
    K = K or int((np.abs(X) >= 3).sum())
    ref = topk_indices(X, K)
    runs = [[info["rel_err_sq"] for idx, val, info in _mse_identity(X, K, 3)
             if np.array_equal(idx, ref) and np.array_equal(val, X.ravel()[ref])
             and info["threshold"] == np.abs(val).min()] for _ in range(2)]
    assert len(runs[0]) == 3 and runs[0] == runs[1]


def test_close_values_are_not_slow():
    """A selection step on values that lie close together stays within five
    times one on spread values (narrowed on all CUs it is within twice; a list
    of them in one block was 30 times and more)."""
    from paper_1309_0302_amd.binding import GoDecMSE
    n, p, K = 40000, 512, 6000000
    ms = {}
    for values in ("normal", "clusters"):
        g = torch.Generator(device="cuda:0")
        g.manual_seed(5)
        x = torch.randn((n, p), generator=g, device="cuda:0")
        if values == "clusters":
            x = (x * 2).round() / 2 * (1 + 1e-5 * torch.rand((n, p), generator=g, device="cuda:0"))
        tr = GoDecMSE(x, [np.zeros(0, np.int64)], [1], K, seed=1)
        tr.step(2)
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        times = []
        for _ in range(5):
            torch.cuda.synchronize()
            a.record()
            tr.step(1)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        ms[values] = min(times)
        tr.close()
    assert ms["clusters"] <= 5 * ms["normal"], ms


# one and two columns, widths up to the widest panel
@pytest.mark.parametrize("m,n,r", [(500, 500, 1), (500, 200, 1), (120, 100, 1), (300, 400, 2)])
def test_narrow_panel_norms(m, n, r):
    """V_L of a narrow FP64 matrix is orthonormal to the rounding of its entries
    and of a sum in short chains: |v|^2 - 1 is below 4 u on average (r.m.s. over
    12 inputs; entries alone give about u)."""
    from paper_1309_0302_amd.binding import GoDec
    dev = []
    for seed in range(12):
        rng = np.random.default_rng(seed)
        X = rng.standard_normal((m, r)) @ rng.standard_normal((n, r)).T
        gd = GoDec(torch.from_numpy(X).to("cuda:0"), r, 0, 1, seed=seed + 1)
        gd.step(1)
        V = gd.factors()[1].cpu().numpy().astype(np.longdouble)
        dev.append((V.T @ V - np.eye(r)).astype(np.float64))
        gd.close()
    assert np.sqrt(np.mean(np.square(dev))) <= 4 * 2.0 ** -53


# sizes the A = D^T D form takes in the root form; projection form, the rank
# check off, warm starts (three steps)
@pytest.mark.parametrize("m,n,r", [(500, 200, 4), (300, 300, 2), (400, 256, 8)])
@pytest.mark.parametrize("lstep,q,warm,rank_tol,ratio,bar", [
    (1, 1, 0, 0.0, 1e-3, 16), (1, 2, 0, 0.0, 1e-3, 16), (1, 0, 1, 0.0, 1e-3, 16),
    (0, 1, 0, 1e-40, 1e-3, 16), (0, 1, 0, 0.0, 0.1, 16)])
def test_graded_spectrum_fp64(m, n, r, lstep, q, warm, rank_tol, ratio, bar):
    """L of a matrix of exact rank r whose singular values fall to `ratio` of the
    largest is the matrix itself.  D and D^T applied to an orthonormal panel
    keep that to a few roundings (bar: 16 u, u = 2^-53), r.m.s. over six
    inputs."""
    from paper_1309_0302_amd.binding import GoDec
    err = []
    for seed in range(6):
        rng = np.random.default_rng(seed)
        U, V = (np.linalg.qr(rng.standard_normal((k, r)))[0].astype(np.longdouble) for k in (m, n))
        X = ((U * np.logspace(0, np.log10(ratio), r)) @ V.T).astype(np.float64)
        gd = GoDec(torch.from_numpy(X).to("cuda:0"), r, 0, q, seed=seed + 1, lstep=lstep,
                   warm_start=warm, rank_tol=rank_tol)
        gd.step(3 if warm else 1)
        UL, VL = (t.cpu().numpy().astype(np.longdouble) for t in gd.factors())
        # (with the default check an A1 that sees s_r weakly drops it: not L's rounding)
        if rank_tol > 0 or lstep or gd.info()["rank_eff"] == r:
            err.append(np.linalg.norm((UL @ VL.T - X).astype(np.float64)) / np.linalg.norm(X))
        gd.close()
    assert len(err) >= 2 and np.sqrt(np.mean(np.square(err))) <= bar * 2.0 ** -53


# the narrow form's buffers in the sparse step's scratch: beside a fixed
# support's words, no selection (its counts lie behind them), the shortest
# matrices that hold them and the first ones that do not, the widest
@pytest.mark.parametrize("m,n,r,kind", [
    (120, 400, 4, "sparse"), (160, 400, 4, "sparse"), (130, 512, 8, "sparse"),
    (320, 512, 8, "sparse"), (300, 400, 4, "none"), (300, 400, 4, "support"),
    (180, 400, 4, "support"), (2000, 64, 16, "support")])
@pytest.mark.parametrize("dt,tol", [(np.float64, 1e-10), (np.float32, 1e-5)])
def test_narrow_buffers_share_the_scratch(m, n, r, kind, dt, tol):
    """Three steps against the oracle's update on the library's own S (the bars
    of the per-step parity tests)."""
    from oracle import godec_ref as g
    from oracle.rng_ref import a1_gaussian
    from paper_1309_0302_amd.binding import GoDec
    w = wl.tiny(m, n, r, seed=m + n, dtype=dt)
    k, sup = (0 if kind == "none" else w.k), None
    if kind == "support":
        sup = np.sort(np.random.default_rng(m).permutation(m * n)[:k]).astype(np.int64)
    gd = GoDec(torch.from_numpy(w.X).to("cuda:0"), r, k, 1, seed=9,
               support=None if sup is None else torch.from_numpy(sup).to("cuda:0"))
    A1 = a1_gaussian(9, n, r)
    X = w.X.astype(np.float64)
    D = X.copy()
    for _ in range(3):
        gd.step(1)
        assert g.rel_fro(gd.L_dense().cpu().numpy().astype(np.float64),
                         g.brp_power(D, A1, 1).L) <= tol
        idx, val = (t.cpu().numpy() for t in gd.S())
        R = gd.residual().cpu().numpy()
        assert np.array_equal(idx, topk_indices(R, k) if sup is None else sup)
        assert np.array_equal(val, R.ravel()[idx])
        D = X.copy()
        D.ravel()[idx] -= val
    gd.close()


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("m,n,lstep,support,names", [
    (900, 200, 0, False, {"gram(D^T*D)": 1, "mm_a(D*Z)": 1, "select_pass(hist)": 1}),
    (900, 200, 0, True, {"gram(D^T*D)": 1, "mm_a(D*Z)": 1, "fixed_support_pass": 1}),
    (300, 600, 0, False, {"mm_a(D*Z)": 5, "mm_b(W^T*D)": 4, "select_pass(hist)": 1}),
    (300, 600, 1, True, {"mm_a(D*Z)": 4, "mm_b(W^T*D)": 3, "fixed_support_pass": 1})])
def test_timing_covers_the_streaming_kernels(m, n, lstep, support, names, dt):
    """godec_profile reports every kernel that streams D or X, with its launches
    (per iteration at q = 1: the passes of the general chain; one Gram and U_L
    in the narrow form), a time and the operand's bytes."""
    from paper_1309_0302_amd.binding import GoDec
    w = wl.tiny(m, n, 4, seed=3, dtype=dt)
    sup = torch.arange(0, m * n, 7, device="cuda:0") if support else None
    gd = GoDec(torch.from_numpy(w.X).to("cuda:0"), 4, sup.numel() if support else w.k, 1, seed=9,
               lstep=lstep, support=sup)
    gd.step(1)
    gd.profile(True)
    gd.step(3)
    stats = {s["name"]: s for s in gd.profile_read()}
    gd.profile(False)
    assert {k: s["launches"] for k, s in stats.items()} == {k: 3 * v for k, v in names.items()}
    for s in stats.values():
        assert 0 < s["total_ms"] < 1000 and s["bytes_per_launch"] == m * n * np.dtype(dt).itemsize
    gd.close()


# exactly rank-deficient X on the panel path (n > 512): inactive columns in the
# Cholesky QR launches, r_eff below the padded width in later cores
@pytest.mark.parametrize("r,true", [(6, 3), (20, 7), (24, 1)])
@pytest.mark.parametrize("lstep,warm,q", [(0, 0, 1), (0, 1, 1), (1, 0, 1), (1, 1, 0), (0, 0, 2)])
@pytest.mark.parametrize("dt,tol", [(np.float64, 1e-10), (np.float32, 1e-5)])
def test_rank_drop_on_the_panel_path(r, true, lstep, warm, q, dt, tol):
    """L is X and the oracle's L after each of three steps; the root form's check
    leaves the true rank; V_L has that many orthonormal columns and zeros (the
    bars of the per-step parity tests).  In the projection form at q = 0 one
    Cholesky QR step decides, on a Gram as ill-conditioned as A1's part in X's
    row space: a direction of rounding noise may stay, orthonormal to the rest."""
    from oracle import godec_ref as g
    from oracle.rng_ref import a1_gaussian
    from paper_1309_0302_amd.binding import GoDec
    m, n = 650, 600
    rng = np.random.default_rng(100 * r + true)
    X = (rng.standard_normal((m, true)) @ rng.standard_normal((true, n))).astype(dt)
    X64 = X.astype(np.float64)
    gd = GoDec(torch.from_numpy(X).to("cuda:0"), r, 0, q, seed=9, lstep=lstep, warm_start=warm)
    A1 = a1_gaussian(9, n, r)
    for _ in range(3):
        gd.step(1)
        ref = g.brp_projection(X64, A1, q) if lstep else g.brp_power(X64, A1[:, :r], q)
        L = gd.L_dense().cpu().numpy().astype(np.float64)
        assert g.rel_fro(L, ref.L) <= tol and g.rel_fro(L, X64) <= tol
        V = gd.factors()[1].cpu().numpy().astype(np.float64)
        on = np.abs(V).max(axis=0) > 0
        assert on.sum() == true if q > 0 else true <= on.sum() <= r
        assert np.abs(V[:, on].T @ V[:, on] - np.eye(on.sum())).max() <= 10 * tol
    info = gd.info()
    assert info["rank_eff"] == (r if lstep else true) and bool(info["flags"] & 2) == (not lstep)
    gd.close()


def test_batch_lists_from_two_threads():
    """The same problem's S fetched by two threads at once: each gets the whole
    sorted list (the index sort has one scratch per problem)."""
    import threading
    from paper_1309_0302_amd.binding import GoDecBatch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(3)
    X = torch.randn((4000, 300), generator=g, device="cuda:0")
    b = GoDecBatch([(X, 2, 100000, 3), (X * 2, 2, 60000, 4)], 1)
    b.step(2)
    ref = [tuple(t.clone() for t in b.S(i)) for i in (0, 1)]
    wrong = []

    def fetch(i):
        for _ in range(200):
            idx, val = b.S(i)
            if not (torch.equal(idx, ref[i][0]) and torch.equal(val, ref[i][1])):
                wrong.append(i)

    th = [threading.Thread(target=fetch, args=(i,)) for i in (0, 0, 1, 0)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not wrong
    b.close()


def test_fp64_layer_with_a_smaller_rank_tol():
    """The rank check's tolerance may choose the form of an FP64 layer's L update;
    L, S and dX agree with the default's to the oracle bars (1e-10)."""
    from paper_1309_0302_amd.binding import GoDecLayer
    w = wl.tiny(520, 96, 3, seed=4, dtype=np.float64)
    X = torch.from_numpy(w.X[None]).to("cuda:0")
    G = torch.randn(X.shape, generator=torch.Generator("cuda:0").manual_seed(1), device="cuda:0",
                    dtype=torch.float64)
    out = []
    for tol in (0.0, 1e-40):
        layer = GoDecLayer(3, w.k, 1, 3, seed=5, rank_tol=tol)
        L, S = layer.forward(X)
        out.append((L.clone(), S.clone(), layer.backward(G, G).clone()))
    for a, c in zip(*out):
        assert (a - c).norm() <= 1e-10 * a.norm()
