"""Kernel variants chosen by size, at the sizes where they can go wrong.

Every case is checked bit for bit against the CPU FP64 oracle, so no
tolerance is involved.
"""
import numpy as np
import pytest

import oracle as orc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _rm():
    import paper_2504_13445_amd as rm
    return rm


def _g(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(_dev())


def _say(*a):
    print("[case]", *a, flush=True)


# FP32 screening: FP32 steps below 32 dimensions, split FP16 rows from there
# on (a row is padded to 16 values, a half row is 1 to 16 chunk pairs); rows
# whose values span 12 decades lose the small ones' low parts to the bound
@pytest.mark.parametrize("d", [31, 32, 33, 48, 49, 100, 127, 128, 129, 200, 224, 225, 255, 256])
@pytest.mark.parametrize("wide", [False, True])
def test_split_rows(d, wide):
    _say("split rows", d, wide)
    rng = np.random.default_rng(d)
    n, m, k = 259, 193, 9
    U = synth.isotropic(rng, n, d, 0.3)
    P = synth.isotropic(rng, m, d, 0.6)
    if wide:
        U = (U * 10.0 ** rng.uniform(-9, 3, (n, d))).astype(np.float32)
        P = (P * 10.0 ** rng.uniform(-9, 3, (m, d))).astype(np.float32)
    rm = _rm()
    t, j, tk = orc.kmips_c(U, P, k)
    tau, tid, topk = rm.thresholds(_g(U), _g(P), k, with_topk=True)
    assert np.array_equal(tau.cpu().numpy().view(np.uint64), t.view(np.uint64))
    assert np.array_equal(tid.cpu().numpy(), j) and np.array_equal(topk.cpu().numpy(), tk)
    sc = orc.histogram_scores(tk, m)
    got = rm.scores(_g(U), tau, tid, _g(P), torch.arange(m, dtype=torch.int32, device=_dev()))
    assert np.array_equal(got.cpu().numpy(), sc)
    ids, s, _ = rm.topn(_g(U), _g(P), k, 20)
    ri, rs = orc.topn_from_scores(sc, 20)
    assert ids.tolist() == ri.tolist() and s.tolist() == rs.tolist()


# Step (5) of the budgeted build: d' = d for d <= 10 (its general and its full
# width), so that the Eq. (3) bound is v plus 2^-30 |u||p| and rounding far
# below that; list lengths around the multiples of 4 and user counts around
# the workgroup's 512, with one and with several workgroups per tile range
@pytest.mark.parametrize("n,m,d,kmax", [(1, 300, 10, 4), (511, 257, 10, 5), (512, 700, 7, 1),
                                        (513, 1500, 10, 32), (1025, 513, 3, 9),
                                        (700, 256, 10, 25)])
def test_budget_step5(n, m, d, kmax):
    _say("budget step 5", n, m, d, kmax)
    rng = np.random.default_rng(n + m)
    U = synth.isotropic(rng, n, d, 0.3)
    P = synth.isotropic(rng, m, d, 0.5)
    bi = _rm().BudgetIndex(_g(U), _g(P), kmax, kmax + 2, 3 * n, "exp")
    g = {k: v.cpu().numpy() for k, v in bi.state().items()}
    V = orc.inner_products_c(U, P)
    nn = np.linalg.norm(U.astype(np.float64), axis=1)[:, None] * \
        np.linalg.norm(P.astype(np.float64), axis=1)[None, :]
    hi = V + 2.0 ** -29 * nn
    posof = np.empty(m, np.int64)
    posof[g["order"]] = np.arange(1, m + 1)
    u2 = np.nonzero(g["pos"] > 0)[0]
    lo_cnt, hi_cnt = np.zeros((kmax, m), np.int64), np.zeros((kmax, m), np.int64)
    for u in u2:
        # the range ends where |u||p| falls below the kmax-th value
        rest = posof > g["pos"][u]
        inr = rest & (nn[u] >= g["Av"][u, -1] * (1 + 1e-9))
        if rest.any():
            assert g["lam"][u] <= hi[u, rest].max()
        if inr.any():
            assert g["lam"][u] >= V[u, inr].max()
        for k in range(kmax):
            a = g["Av"][u, k]
            lo_cnt[k] += inr & (V[u] >= a)
            hi_cnt[k] += rest & (hi[u] >= a - 2.0 ** -22 * abs(a))
    hist = np.stack([orc.histogram_scores(g["Aj"][:, :k + 1], m) for k in range(kmax)])
    got = g["uscore"].astype(np.int64) - hist
    assert np.all(got >= lo_cnt) and np.all(got <= hi_cnt)


# The k_max table's bounds: one pass for every k must give the counts of the
# pass per k (rmips_topn's bound_out of the same k, bound kernels of every row
# length), around the item blocks (128, 384, 512, 576) and user stages (64, 128)
@pytest.mark.parametrize("n,m,d,kmax", [(63, 130, 14, 3), (129, 513, 30, 32), (1000, 577, 33, 4),
                                        (257, 385, 62, 25), (600, 1100, 110, 7),
                                        (1025, 1153, 174, 5), (300, 700, 175, 9),
                                        (513, 800, 222, 3), (777, 1200, 256, 6)])
def test_index_bounds_all_k(n, m, d, kmax):
    _say("index bounds", n, m, d, kmax)
    rng = np.random.default_rng(n + d)
    U = synth.isotropic(rng, n, d, 0.3)
    P = synth.isotropic(rng, m, d, 0.6)
    P[m // 2:m // 2 + 40] = P[:40]  # ties
    U[0] = 0.0
    rm = _rm()
    ix = rm.Index(_g(U), _g(P), kmax)
    for k in range(1, kmax + 1):
        b = torch.empty(m, dtype=torch.int32, device=_dev())
        rm.topn(_g(U), _g(P), k, 5, bound_out=b, prepass=0)
        assert torch.equal(ix.bounds(k), b), k


# Selection and recomputation by list length: nearly equal items keep every
# candidate to the end, so that m sets the list (registers per lane, and the
# lists past 1024 and 2048 entries) and the values to recompute (the users of
# a wave joined up to 8 values, one wave per user to 64, 256, 1024 and more);
# rows of whole 16-byte vectors and not, exact ties, S_k asked for and not
@pytest.mark.parametrize("prec,m,d,k", [("fp32", 3, 20, 2), ("fp32", 9, 21, 9), ("fp32", 64, 36, 10),
                                        ("bf16", 65, 33, 32), ("bf16", 200, 20, 10),
                                        ("fp8", 257, 75, 1), ("fp8", 520, 40, 16),
                                        ("fp8", 1000, 13, 10), ("fp8", 1200, 24, 20),
                                        ("fp4", 1500, 20, 16), ("fp4", 2000, 31, 3),
                                        ("fp6", 1900, 132, 4), ("fp4", 3000, 16, 32)])
def test_selection_lengths(prec, m, d, k):
    _say("selection", prec, m, d, k)
    rng = np.random.default_rng(m)
    n = 131
    U = synth.isotropic(rng, n, d, 0.3)
    base = synth.isotropic(rng, 1, d, 0.0)
    P = (base + 1e-6 * rng.standard_normal((m, d))).astype(np.float32)
    P[m // 2:m // 2 + m // 8] = P[:m // 8]  # exact ties
    t, j, tk = orc.kmips_c(U, P, k)
    for topk in (False, True):
        r = _rm().thresholds(_g(U), _g(P), k, prec, with_topk=topk)
        assert np.array_equal(r[0].cpu().numpy().view(np.uint64), t.view(np.uint64)), topk
        assert np.array_equal(r[1].cpu().numpy(), j), topk
        if topk:
            assert np.array_equal(r[2].cpu().numpy(), tk)


# The same with an unaligned catalogue (rows of whole vectors off 16 bytes)
def test_recompute_unaligned_rows():
    _say("unaligned rows")
    rng = np.random.default_rng(5)
    n, m, d, k = 300, 700, 24, 12
    U = synth.isotropic(rng, n, d, 0.3)
    P = synth.isotropic(rng, m, d, 0.1)
    t, j, tk = orc.kmips_c(U, P, k)
    buf = torch.zeros(m * d + 1, dtype=torch.float32, device=_dev())
    Pg = buf[1:].view(m, d)
    Pg.copy_(_g(P))
    for prec in ("fp32", "fp8"):
        tau, tid, topk = _rm().thresholds(_g(U), Pg, k, prec, with_topk=True)
        assert np.array_equal(tau.cpu().numpy().view(np.uint64), t.view(np.uint64))
        assert np.array_equal(tid.cpu().numpy(), j) and np.array_equal(topk.cpu().numpy(), tk)
        tau, tid = _rm().thresholds(_g(U), Pg, k, prec)
        assert np.array_equal(tau.cpu().numpy().view(np.uint64), t.view(np.uint64))


# Screening copies and augmented rows: whole vectors and not, one part of a row
# and two (D past 128), row words in one to three rounds of 16 lanes, users off
# 16 bytes, row counts around a block's 64 and 32
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("n,m,d", [(63, 65, 4), (65, 64, 128), (129, 127, 130), (31, 33, 132),
                                   (97, 96, 256), (64, 129, 255)])
@pytest.mark.parametrize("off", [0, 1])
def test_row_copies(prec, n, m, d, off):
    _say("row copies", prec, n, m, d, off)
    rng = np.random.default_rng(n * d)
    U = synth.isotropic(rng, n, d, 0.3)
    P = synth.isotropic(rng, m, d, 0.6)
    P[-1] = 0.0
    buf = torch.zeros(n * d + off, dtype=torch.float32, device=_dev())
    Ug = buf[off:].view(n, d)
    Ug.copy_(_g(U))
    k = min(8, m)
    _, _, tk = orc.kmips_c(U, P, k)
    sc = orc.histogram_scores(tk, m)
    b = torch.empty(m, dtype=torch.int32, device=_dev())
    ids, s, _ = _rm().topn(Ug, _g(P), k, 10, prec, bound_out=b)
    ri, rs = orc.topn_from_scores(sc, 10)
    assert ids.tolist() == ri.tolist() and s.tolist() == rs.tolist()
    assert np.all(b.cpu().numpy() >= sc)


# Sorts by length: one workgroup (up to 1,024 elements per round of 1, 2, 4 or 8),
# blocks of 1,024 and 4,096 without scans, blocks of 1,024 with scans; the norm
# order (stable: equal norms stay in id order) and the users' orders show in the
# results
@pytest.mark.parametrize("n,m", [(1, 1024), (1024, 1025), (1025, 2048), (2049, 4097), (4096, 8192),
                                 (8193, 8193), (131072, 300), (131073, 64), (524288, 40),
                                 (524289, 33)])
def test_sort_lengths(n, m):
    _say("sort lengths", n, m)
    rng = np.random.default_rng(n + m)
    d, k = 8, 3
    U = synth.isotropic(rng, n, d, 0.3)
    P = synth.isotropic(rng, m, d, 0.5)
    P[1::2] = P[0:m - m % 2:2][:P[1::2].shape[0]]  # every norm twice
    _, _, tk = orc.kmips_c(U, P, k)
    sc = orc.histogram_scores(tk, m)
    N = min(m, 50)
    ri, rs = orc.topn_from_scores(sc, N)
    ids, s, _ = _rm().topn(_g(U), _g(P), k, N)
    assert ids.tolist() == ri.tolist() and s.tolist() == rs.tolist()


# Relaxed score: one and two query blocks per wave (up to 64 queries and more),
# slices of whole 64-user chunks up to the 384 slices and past them, the three
# passes (S, gradient, both) and their reductions.  Tolerance: the calls' 1e-4
# of the FP64 values, at a temperature where z stays small (|z| < 40: FP32 z
# within 40 * 2^-21, S and G within 2e-5)
@pytest.mark.parametrize("n,d,nq", [(1, 5, 1), (63, 61, 63), (64, 100, 64), (65, 128, 65),
                                    (24576, 16, 17), (24577, 33, 40), (49217, 61, 64),
                                    (50000, 20, 129)])
def test_soft_slices(n, d, nq):
    _say("soft slices", n, d, nq)
    rng = np.random.default_rng(n + nq)
    U = synth.isotropic(rng, n, d, 0.25)
    Q = (rng.standard_normal((nq, d)) / np.sqrt(d)).astype(np.float32)
    tau = rng.uniform(0.2, 0.6, n).astype(np.float32)
    T = 0.1
    dS = np.linspace(0.5, 1.5, nq).astype(np.float32)
    S64 = orc.soft_score(U, tau.astype(np.float64), Q, T)
    G64 = orc.soft_grad(U, tau.astype(np.float64), Q, T)
    rm = _rm()
    a = (_g(U), _g(tau), _g(Q), T)
    S, G = rm.soft_fwd_grad(*a)
    assert torch.equal(rm.soft_fwd(*a), S)
    dQ = rm.soft_bwd(*a, _g(dS)).cpu().numpy().astype(np.float64)
    S, G = S.cpu().numpy().astype(np.float64), G.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(S - S64) <= 1e-4 * S64)
    den = np.linalg.norm(G64, axis=1)
    assert np.all(np.linalg.norm(G - G64, axis=1) <= 1e-4 * den)
    assert np.all(np.linalg.norm(dQ - G64 * dS[:, None], axis=1) <= 1e-4 * den * dS)


# Phase-1 tiles by precision, k and catalogue: 6 up to 24 tiles of 64 items,
# then 5 + k / 2 (10 + k / 2 with the wide bands) up to a quarter of the tiles
@pytest.mark.parametrize("prec,m,k", [("fp32", 6 * 64 + 1, 32), ("fp32", 28 * 64, 32),
                                      ("bf16", 84 * 64 + 1, 32), ("bf16", 30 * 64, 1),
                                      ("fp8", 25 * 64, 1), ("fp8", 104 * 64 + 1, 32)])
def test_phase1_tiles(prec, m, k):
    _say("phase 1", prec, m, k)
    rng = np.random.default_rng(m)
    U, P = synth.isotropic(rng, 300, 40, 0.3), synth.isotropic(rng, m, 40, 0.3)
    t, j, tk = orc.kmips_c(U, P, k)
    r = _rm().thresholds(_g(U), _g(P), k, prec, with_topk=True)
    assert np.array_equal(r[0].cpu().numpy().view(np.uint64), t.view(np.uint64))
    assert np.array_equal(r[1].cpu().numpy(), j) and np.array_equal(r[2].cpu().numpy(), tk)


# Rechecks by window with the wide bands: nearly equal items leave every pair
# open (16384 per chunk: rounds of 4096), single chunks and ragged ones, items
# past one workgroup's 256, rows of whole 16-byte vectors and not, one to
# eight slices of 32 dims
@pytest.mark.parametrize("prec,n,q,d,noise", [("fp8", 1, 1, 3, 0.0), ("fp8", 63, 256, 32, 0.0),
                                              ("fp8", 65, 257, 33, 1e-6), ("fp6", 700, 300, 100, 1e-6),
                                              ("fp4", 1025, 31, 67, 1e-6), ("fp8", 5000, 260, 61, 0.3),
                                              ("fp4", 3001, 513, 128, 0.3), ("fp8", 300, 256, 256, 1e-6)])
def test_recheck_windows(prec, n, q, d, noise):
    _say("windows", prec, n, q, d, noise)
    rng = np.random.default_rng(n)
    m, k = 40, 7
    U = synth.isotropic(rng, n, d, 0.2)
    P = synth.isotropic(rng, 1, d, 0.0) + noise * rng.standard_normal((m, d))
    Q = synth.isotropic(rng, 1, d, 0.0) + noise * rng.standard_normal((q, d))
    P = P.astype(np.float32)
    Q = np.where((np.arange(q) % 3 == 0)[:, None], P[np.arange(q) % m], Q).astype(np.float32)
    t, j, _ = orc.kmips_c(U, P, k)
    rm = _rm()
    got = rm.scores(_g(U), _g(t), _g(j), _g(Q), prec=prec)
    assert np.array_equal(got.cpu().numpy(), orc.reverse_counts_c(U, t, j, Q))


# Queries by whole rounds of workgroups: one block and several, a last block of
# one query, more blocks than a round holds, few users
@pytest.mark.parametrize("prec,n,q,d", [("fp32", 40000, 257, 8), ("fp32", 40000, 129, 224),
                                        ("bf16", 3000, 3000, 5), ("bf16", 300, 70000, 3),
                                        ("fp32", 64, 2000, 33)])
def test_query_rounds(prec, n, q, d):
    _say("rounds", prec, n, q, d)
    rng = np.random.default_rng(q)
    U, P, Q = (synth.isotropic(rng, r, d, 0.3) for r in (n, 50, q))
    t, j, _ = orc.kmips_c(U, P, 5)
    got = _rm().scores(_g(U), _g(t), _g(j), _g(Q), prec=prec)
    assert np.array_equal(got.cpu().numpy(), orc.reverse_counts_c(U, t, j, Q))


# Sorts on at most eight key bits (the visit order of fewer than 256 users, the
# step (5) ranges of fewer than 255 items) of more elements than one workgroup
# takes: a pass never writes where it reads.  Blocks of 1,024 and 4,096, and
# with scans
@pytest.mark.parametrize("n,m,N", [(200, 8193, 1000), (255, 20000, 1000), (31, 140000, 200),
                                   (3, 524289, 60)])
def test_sort_few_bits_visit(n, m, N):
    _say("few bits, visit", n, m)
    rng = np.random.default_rng(m)
    U, P = synth.isotropic(rng, n, 6, 0.3), synth.isotropic(rng, m, 6, 0.3)
    k = 30
    _, _, tk = orc.kmips_c(U, P, k)
    ri, rs = orc.topn_from_scores(orc.histogram_scores(tk, m), N)
    for dprime in (None, 2):  # (loose bounds: long runs of equal keys)
        ids, s, _ = _rm().topn(_g(U), _g(P), k, N, dprime=dprime, batch=(64, 256))
        assert ids.tolist() == ri.tolist() and s.tolist() == rs.tolist()


@pytest.mark.parametrize("n,m", [(20000, 200), (150000, 120)])
def test_sort_few_bits_budget(n, m):
    _say("few bits, budget", n, m)
    rng = np.random.default_rng(n)
    U, P = synth.isotropic(rng, n, 12, 0.3), synth.isotropic(rng, m, 12, 0.2)
    kmax, N = 5, 40
    bi = _rm().BudgetIndex(_g(U), _g(P), kmax, kmax + 1, 2 * n, "uniform")
    assert bi.info["u_dprime"] > 8192
    us = bi.state()["uscore"].cpu().numpy()
    _, _, tk = orc.kmips_c(U, P, kmax)
    for k in (1, kmax):
        sc = orc.histogram_scores(tk[:, :k], m)
        assert np.all(us[k - 1] >= sc)
        ids, s, _ = bi.topn(k, N)
        ri, rs = orc.topn_from_scores(sc, N)
        assert ids.tolist() == ri.tolist() and s.tolist() == rs.tolist()


# Items far smaller than their tile's largest (whose scale they share) are
# stored as zero, but the norm-ordered scan ends where it does with zero rows
# in their place
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8", "fp6"])
@pytest.mark.parametrize("scale", [1e-6, 1e-10, 1e-16])
def test_near_zero_items_keep_scan_end(prec, scale):
    _say("near-zero items", prec, scale)
    rng = np.random.default_rng(3)
    n, m, d, k = 700, 6000, 48, 8
    U, P = synth.isotropic(rng, n, d, 0.2), synth.isotropic(rng, m, d, 0.8)
    small = [7, 3000, m - 1]
    P[small] /= np.linalg.norm(P[small], axis=1, keepdims=True)
    P0 = P.copy()
    P[small] *= np.float32(scale)
    P0[small] = 0.0
    _, _, tk = orc.kmips_c(U, P, k)
    ri, rs = orc.topn_from_scores(orc.histogram_scores(tk, m), 30)
    ids, s, st = _rm().topn(_g(U), _g(P), k, 30, prec)
    assert ids.tolist() == ri.tolist() and s.tolist() == rs.tolist()
    st0 = _rm().topn(_g(U), _g(P0), k, 30, prec)[2]
    assert st["thresh_pairs"] <= 1.02 * st0["thresh_pairs"]
    assert st0["thresh_pairs"] < 0.8 * n * m  # (the scan does end early)


# Rows of small and of very different magnitudes with FP32 screening: a power
# of two on the users or the items changes no screened pair's band, so the
# candidates stay what they are without it
@pytest.mark.parametrize("su,sp", [(-70, 0), (0, -70), (-36, -36), (30, -90), (-95, 40)])
def test_split_rows_small_magnitudes(su, sp):
    _say("small magnitudes", su, sp)
    rng = np.random.default_rng(8)
    n, m, d, k = 700, 3000, 48, 8
    U, P = synth.isotropic(rng, n, d, 0.2), synth.isotropic(rng, m, d, 0.6)
    st0 = _rm().topn(_g(U), _g(P), k, 20)[2]
    Us, Ps = U * np.float32(2.0 ** su), P * np.float32(2.0 ** sp)
    _, _, tk = orc.kmips_c(Us, Ps, k)
    ri, rs = orc.topn_from_scores(orc.histogram_scores(tk, m), 20)
    ids, s, st = _rm().topn(_g(Us), _g(Ps), k, 20)
    assert ids.tolist() == ri.tolist() and s.tolist() == rs.tolist()
    for key in ("thresh_pairs", "cand_listed", "cand_pairs"):
        assert st[key] <= 1.02 * st0[key] + 10, key


# The ends of the range: values down to 2^-126 (the products then lie below
# every band, and all pairs are decided in FP64), rows and items that differ
# by 2^150, one row of each
@pytest.mark.parametrize("d", [32, 75, 200])
def test_split_rows_extreme_magnitudes(d):
    _say("extreme magnitudes", d)
    rng = np.random.default_rng(d)
    n, m, k = 200, 260, 7
    for eu, ep in [(-60, -60), (-118, 55), (55, -118), (-118, -20), (50, 50)]:
        U = synth.isotropic(rng, n, d, 0.3) * np.float32(2.0 ** eu)
        P = synth.isotropic(rng, m, d, 0.6) * np.float32(2.0 ** ep)
        U[::7] = synth.isotropic(rng, len(U[::7]), d, 0.0)
        P[::9] = synth.isotropic(rng, len(P[::9]), d, 0.0)
        U, P = U.astype(np.float32), P.astype(np.float32)
        t, j, tk = orc.kmips_c(U, P, k)
        tau, tid, topk = _rm().thresholds(_g(U), _g(P), k, with_topk=True)
        assert np.array_equal(tau.cpu().numpy().view(np.uint64), t.view(np.uint64)), (eu, ep)
        assert np.array_equal(tid.cpu().numpy(), j) and np.array_equal(topk.cpu().numpy(), tk)
        ids_all = torch.arange(m, dtype=torch.int32, device=_dev())
        sc = _rm().scores(_g(U), tau, tid, _g(P), ids_all)
        assert np.array_equal(sc.cpu().numpy(), orc.histogram_scores(tk, m)), (eu, ep)


# Reductions of the relaxed score by 4 and by 16 waves (from 128 slices on for at
# most 256 workgroups of the gradient), around both lines, with the same sums in
# every entry point; the tolerance of test_soft_slices
@pytest.mark.parametrize("n,d,nq", [(127 * 64, 20, 5), (127 * 64 + 1, 20, 5), (20000, 70, 128),
                                    (20000, 70, 129), (9000, 64, 255), (9000, 64, 257),
                                    (100, 9, 700)])
def test_soft_reductions(n, d, nq):
    _say("soft reductions", n, d, nq)
    rng = np.random.default_rng(n + nq)
    U = synth.isotropic(rng, n, d, 0.25)
    Q = (rng.standard_normal((nq, d)) / np.sqrt(d)).astype(np.float32)
    tau = rng.uniform(0.2, 0.6, n).astype(np.float32)
    T = 0.1
    S64 = orc.soft_score(U, tau.astype(np.float64), Q, T)
    G64 = orc.soft_grad(U, tau.astype(np.float64), Q, T)
    rm = _rm()
    a = (_g(U), _g(tau), _g(Q), T)
    S, G = rm.soft_fwd_grad(*a)
    assert torch.equal(rm.soft_fwd(*a), S)
    assert torch.equal(rm.soft_bwd(*a, torch.ones(nq, device=_dev())), G)
    S, G = (x.cpu().numpy().astype(np.float64) for x in (S, G))
    assert np.all(np.abs(S - S64) <= 1e-4 * S64)
    assert np.all(np.linalg.norm(G - G64, axis=1) <= 1e-4 * np.linalg.norm(G64, axis=1))


# The selection's variants by the lists' capacity (64 k with e4m3: up to 1024,
# 1536 and 2048 entries), at the values of k on both sides of each line, with
# lists from short to nearly full
@pytest.mark.parametrize("k", [16, 17, 24, 25, 32])
@pytest.mark.parametrize("noise", [0.0, 0.02, 0.4])
def test_selection_capacities(k, noise):
    _say("selection capacities", k, noise)
    rng = np.random.default_rng(k)
    n, m, d = 1500, 64 * k - 40, 24
    U = synth.isotropic(rng, n, d, 0.3)
    P = (synth.isotropic(rng, 1, d, 0.0) + noise * rng.standard_normal((m, d))).astype(np.float32)
    t, j, tk = orc.kmips_c(U, P, k)
    for topk in (False, True):
        r = _rm().thresholds(_g(U), _g(P), k, "fp8", with_topk=topk)
        assert np.array_equal(r[0].cpu().numpy().view(np.uint64), t.view(np.uint64)), topk
        assert np.array_equal(r[1].cpu().numpy(), j), topk
        if topk:
            assert np.array_equal(r[2].cpu().numpy(), tk)


# Per-launch times carry the name of the kernel that ran: the selection in
# registers up to lists of 2,048 entries, in LDS beyond (e2m1 at k = 32: 4,096)
@pytest.mark.parametrize("prec,k,name", [("fp32", 10, "k_thresh_select"), ("fp8", 32, "k_thresh_select"),
                                         ("fp4", 32, "k_thresh_final")])
def test_selection_profile_name(prec, k, name):
    _say("selection name", prec, k)
    rng = np.random.default_rng(1)
    U, P = _g(synth.isotropic(rng, 300, 20, 0.3)), _g(synth.isotropic(rng, 600, 20, 0.5))
    rm = _rm()
    rm.set_profiling(True)
    rm.thresholds(U, P, k, prec)
    names = {x[0].split("/")[0] for x in rm.profile()}
    rm.set_profiling(False)
    assert name in names
    assert names & {"k_thresh_select", "k_thresh_final"} == {name}
