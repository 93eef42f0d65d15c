"""GPU parity of the offline compression calls (Sec. III-A, III-C, III-D)
against the fp64 oracle: the Gram matrix (centred and plain, fp32 and bf16
samples, ragged tiles), the CKA head similarity, and the two pipelines
(Algorithm 1 for keys, the calibration refinement for values)."""

import numpy as np
import pytest
import torch

from oracle import calibrate as ocal
from oracle import compress as oc

import decisions

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


def _gram_bound(A64, center, rows):
    # fp32 rounding of the centring (means, differences) and of a sum of
    # `rows` products: |dG| <= gamma * sum_t (|a_ti| + |mu_i|)(|a_tj| + |mu_j|)
    mu = np.abs(A64.mean(axis=0)) if center else np.zeros(A64.shape[1])
    M = np.abs(A64) + mu[None, :]
    gamma = 2.0 * (rows + 8) * U32
    return gamma * (M.T @ M) + 1e-30


# (rows, cols, dtype, centre): ragged sample counts (not a multiple of the
# 32-sample step), column counts that leave partial 128-column tiles, one
# sample, the smallest width; 4000 columns take the 192-column tiles (the
# last one partial)
CASES = [(200, 72, "f32", True), (1000, 264, "f32", True), (1000, 264, "f32", False),
         (37, 8, "f32", True), (513, 392, "bf16", True), (1, 16, "f32", True),
         (2048, 256, "bf16", False), (100, 4000, "f32", True), (70, 4000, "bf16", False)]


@pytest.mark.parametrize("rows, cols, dtype, center", CASES)
def test_gram_matches_oracle(rows, cols, dtype, center):
    from paper_2607_24331_amd import gram
    g = np.random.default_rng(rows * 7 + cols)
    A = (g.standard_normal((rows, cols)) + g.standard_normal(cols)[None, :]).astype(np.float32)
    At = torch.from_numpy(A).cuda()
    if dtype == "bf16":
        At = At.to(torch.bfloat16)
        A = At.float().cpu().numpy()                        # the values the GPU sees
    print(f"[gram] rows {rows} cols {cols} {dtype} center {center}", flush=True)
    G = gram(At, center=center)
    torch.cuda.synchronize()
    got = G.double().cpu().numpy()
    A64 = A.astype(np.float64)
    ref = ocal.gram(oc.centered(A64) if center else A64)
    assert np.all(np.abs(got - ref) <= _gram_bound(A64, center, rows))
    assert np.array_equal(got, got.T)                       # mirrored tiles are exact copies


# edges of the 64-, 128- and 192-column tiles and of the 32- and 64-row stages,
# one row to several stages of the three-buffer ring, and more row blocks than
# a tile adds up by itself (64 of 256 rows); both ways of taking the samples
# (bf16 as they are; fp32 or centred in three bf16 parts).  The bound is the
# one above: every product of bf16 samples is exact in fp32, and the three
# products of parts that are left out are below 2^-22 of a term, the bound's
# 2 (rows + 8) 2^-24 at one row.
EDGES = [(1, 8), (31, 56), (32, 64), (33, 72), (63, 128), (64, 136), (65, 192), (127, 200),
         (191, 384), (193, 392), (257, 1152), (16641, 24)]


@pytest.mark.parametrize("rows, cols", EDGES)
@pytest.mark.parametrize("dtype, center", [("bf16", False), ("bf16", True), ("f32", False), ("f32", True)])
def test_gram_at_tile_edges(rows, cols, dtype, center):
    from paper_2607_24331_amd import gram
    g = np.random.default_rng(rows + cols)
    A = (g.standard_normal((rows, cols)) * 3 + g.standard_normal(cols)[None, :]).astype(np.float32)
    At = torch.from_numpy(A).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16)
    A64 = At.double().cpu().numpy()
    got = gram(At, center=center).double().cpu().numpy()
    ref = ocal.gram(oc.centered(A64) if center else A64)
    assert np.all(np.abs(got - ref) <= _gram_bound(A64, center, rows))
    assert np.array_equal(got, got.T)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_gram_of_infinities_and_nans(dtype):
    # one infinity in column 3, one NaN in column 70: those rows and columns of
    # G are what sums of products give (infinite with the partner's sign, NaN
    # against a zero), every other element is unchanged
    from paper_2607_24331_amd import gram
    g = np.random.default_rng(3)
    A = g.integers(-4, 5, (40, 136)).astype(np.float32)        # exact: sums of small integers
    A[7, 3], A[9, 70] = -np.inf, np.nan
    got = gram(torch.from_numpy(A).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16),
               center=False).cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = np.stack([(A[:, i:i + 1] * A).sum(axis=0) for i in range(A.shape[1])])
    assert np.array_equal(got, ref, equal_nan=True)


# samples that are not finite over 64-, 128- and 192-column tiles and many row
# stages: a whole row of NaN, a row of infinities of both signs, and single ones
# in columns that meet zeros.  Small integers, so that every finite element is
# exact; centred, a column with such a sample has a mean that is not finite, and
# its whole row and column of G are NaN.  The call takes at most as long again
# as with finite samples, whatever they hold (a factor of 3 and 2 ms here, for
# the clock).
@pytest.mark.parametrize("cols", [136, 2816, 4096])
@pytest.mark.parametrize("dtype, center", [("f32", False), ("f32", True), ("bf16", True)])
@pytest.mark.parametrize("kind", ["nan_row", "inf_row", "single"])
def test_gram_not_finite_at_length(cols, dtype, center, kind):
    from paper_2607_24331_amd import gram
    rows = 4099
    g = np.random.default_rng(cols)
    A = g.integers(-2, 3, (rows, cols)).astype(np.float32)
    bad = np.arange(cols)
    finite = A.copy()
    if kind == "nan_row":
        A[rows - 1] = np.nan
    elif kind == "inf_row":
        A[17] = np.where(np.arange(cols) % 3 == 0, -np.inf, np.inf)
    else:
        bad = np.array([3, 70, 71, cols - 1])
        A[[5, 4000, 4000, 9], bad] = [np.inf, np.nan, -np.inf, -np.inf]
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    At, Ft = torch.from_numpy(A).cuda().to(tdt), torch.from_numpy(finite).cuda().to(tdt)

    def timed(X):
        best, G = float("inf"), gram(X, center=center)
        for _ in range(3):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            G = gram(X, center=center)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return G.cpu().numpy(), best
    got, t_bad = timed(At)
    good, t_good = timed(Ft)
    assert t_bad <= 3 * t_good + 2.0, (t_bad, t_good)
    if center:                                # the finite columns' means do not change
        ref = good
        ref[bad, :] = np.nan
        ref[:, bad] = np.nan
    else:
        with np.errstate(invalid="ignore"):
            ref = A.astype(np.float64).T @ A.astype(np.float64)
    assert np.array_equal(got, ref.astype(np.float32), equal_nan=True)


# at most 32 samples: every product of parts is summed, so G is no further off
# float64 (2-norm) than fp32 products added in sample order (for one sample the
# product rounded once: half a unit of the last place for each element, and a
# sixty-fourth more for the parts' own sum, whose roundings are that small)
@pytest.mark.parametrize("rows", [1, 2, 3, 5, 8, 31, 32])
@pytest.mark.parametrize("dtype, center", [("f32", False), ("f32", True), ("bf16", True)])
def test_gram_of_few_rows_is_no_further_off_than_fp32(rows, dtype, center):
    from paper_2607_24331_amd import gram
    g = np.random.default_rng(rows)
    A = (g.standard_normal((rows, 200)) + 0.25 * g.standard_normal(200)[None, :]).astype(np.float32)
    At = torch.from_numpy(A).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16)
    A = At.float().cpu().numpy()
    D = A - (A.sum(axis=0, dtype=np.float32) / np.float32(rows))[None, :] if center else A
    seq = np.zeros((200, 200), np.float32)
    for r in range(rows):
        seq += np.outer(D[r], D[r])
    got = gram(At, center=center).double().cpu().numpy()
    A64 = A.astype(np.float64)
    ref = ocal.gram(oc.centered(A64) if center else A64)
    assert np.linalg.norm(got - ref) <= 1.02 * np.linalg.norm(seq - ref)
    if rows == 1 and not center:
        assert np.all(np.abs(got - ref) <= (1 + 2.0 ** -6) * 2.0 ** -24 * np.abs(ref))


def test_gram_of_few_rows_not_finite():
    from paper_2607_24331_amd import gram
    A = np.random.default_rng(5).integers(-4, 5, (20, 136)).astype(np.float32)
    A[7, 3], A[9, 70] = -np.inf, np.nan
    with np.errstate(invalid="ignore"):
        ref = np.stack([(A[:, i:i + 1] * A).sum(axis=0) for i in range(A.shape[1])])
    assert np.array_equal(gram(torch.from_numpy(A).cuda(), center=False).cpu().numpy(), ref, equal_nan=True)


def test_gram_is_bitwise_reproducible():
    from paper_2607_24331_amd import gram
    A = torch.randn(777, 200, device="cuda")
    a = gram(A).clone()
    b = gram(A)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


def _acts(seed, h, d, N, groups):
    # per-head activations X W_h with heads of one planted group sharing a subspace
    g = np.random.default_rng(seed)
    m = 64
    W = np.zeros((m, h * d))
    for grp in groups:
        B = g.standard_normal((m, 6))
        for hh in grp:
            W[:, hh * d:(hh + 1) * d] = B @ g.standard_normal((6, d)) + 0.3 * g.standard_normal((m, d))
    X = g.standard_normal((N, m))
    return W, (X @ W + 0.5).astype(np.float32)


def test_head_similarity_matches_oracle():
    from paper_2607_24331_amd.offline import key_similarity
    for h, d, N in [(8, 16, 300), (12, 64, 1000), (5, 8, 77)]:
        groups = [list(range(0, h, 3)), list(range(1, h, 3)), list(range(2, h, 3))]
        _, acts = _acts(h * d, h, d, N, groups)
        print(f"[sim] h {h} d {d} N {N}", flush=True)
        S = key_similarity(torch.from_numpy(acts).cuda(), h, d)
        torch.cuda.synchronize()
        ref = oc.head_similarity(acts.astype(np.float64), h, d)
        Sh = S.double().cpu().numpy()
        assert np.max(np.abs(Sh - ref)) <= 1e-4
        assert np.array_equal(Sh, Sh.T)                     # CKA is symmetric: exactly so here


def test_head_similarity_full_size_sampled():
    # 32 heads x 128 over 2048 samples: S in full, the Gram on sampled rows
    from paper_2607_24331_amd import gram, head_similarity
    h, d, N = 32, 128, 2048
    groups = [list(range(k, h, 4)) for k in range(4)]
    _, acts = _acts(99, h, d, N, groups)
    At = torch.from_numpy(acts).cuda()
    G = gram(At, center=True)
    S = head_similarity(G, h, d)
    torch.cuda.synchronize()
    ref = oc.head_similarity(acts.astype(np.float64), h, d)
    assert np.max(np.abs(S.double().cpu().numpy() - ref)) <= 1e-4
    A64 = oc.centered(acts.astype(np.float64))
    rows = np.random.default_rng(5).choice(h * d, 48, replace=False)
    ref_rows = A64[:, rows].T @ A64
    bound = _gram_bound(acts.astype(np.float64), True, N)[rows]
    assert np.all(np.abs(G.double().cpu().numpy()[rows] - ref_rows) <= bound)


# every start of G that its 4-byte alignment allows, with head sizes that are and
# are not a multiple of 4; float64 sums of the same G, bound of d^2 fp32 additions
@pytest.mark.parametrize("h, d", [(3, 64), (5, 36), (4, 30)])
@pytest.mark.parametrize("first", [0, 1, 2, 3])
def test_head_similarity_of_any_alignment(h, d, first):
    from paper_2607_24331_amd import head_similarity
    n = h * d
    g = np.random.default_rng(n + first)
    X = g.standard_normal((2 * n, n))
    G = (X.T @ X).astype(np.float32)
    buf = torch.zeros(n * n + 4, device="cuda")
    Gt = buf[first:first + n * n].view(n, n)
    Gt.copy_(torch.from_numpy(G))
    assert Gt.data_ptr() % 16 == 4 * first
    got = head_similarity(Gt, h, d).double().cpu().numpy()
    F = (G.astype(np.float64).reshape(h, d, h, d) ** 2).sum(axis=(1, 3))
    ref = F / np.sqrt(np.outer(np.diag(F), np.diag(F)))
    assert np.all(np.abs(got - ref) <= 2 * (d * d + 8) * U32 * np.abs(ref))


def test_compress_keys_matches_oracle():
    from paper_2607_24331_amd import cluster_merges
    from paper_2607_24331_amd.offline import compress_keys, key_similarity
    h, d = 12, 8
    groups = [[0, 4, 7, 9], [1, 2, 10], [3, 5, 6, 8, 11]]
    W, acts = _acts(7, h, d, 600, groups)
    S = key_similarity(torch.from_numpy(acts).cuda(), h, d).double().cpu().numpy()
    r, cands = 40, [2, 3, 4, 6]
    got = compress_keys(W, S, r, cands, d)
    ref = oc.compress(W, S, r, cands, d)             # the same S: the same decisions
    # decisions: the library's merge path is the oracle's up to near-ties
    # (tests/decisions.py); where no near-tie alternative was taken the
    # groups, ranks and objectives are identical
    merges = cluster_merges(S)
    first_dev = decisions.check_merges(S, merges)
    for a, b in zip(got["all"], ref["all"]):
        K = a["K"]
        gid = decisions.cut(merges, h, K)
        assert a["groups"] == [[x for x in range(h) if gid[x] == k] for k in range(K)]
        Wg = oc.group_matrices(W, a["groups"], d)
        sig = [np.linalg.svd(Wi, compute_uv=False) for Wi in Wg]
        assert decisions.init_ranks_agree(a["init_ranks"], [oc.energy(Wi) for Wi in Wg], oc.energy(W),
                                          [min(Wi.shape) for Wi in Wg], r)
        reachable, exact = decisions.greedy_reachable(a["init_ranks"], sig, a["heads"], r, a["ranks"])
        assert reachable
        factors = [oc.group_decompose(Wi, ri) for Wi, ri in zip(Wg, a["ranks"])]
        assert a["objective"] == pytest.approx(oc.objective(Wg, factors, a["ranks"], r), rel=1e-9, abs=1e-9)
        for (La, Ra), (Lb, Rb) in zip(a["factors"], factors):
            assert np.allclose(La @ Ra, Lb @ Rb, atol=1e-9)
        if h - K <= first_dev and exact:
            assert a["groups"] == b["groups"] and a["ranks"] == b["ranks"]
            assert a["init_ranks"] == b["init_ranks"]
            assert a["objective"] == pytest.approx(b["objective"], rel=1e-9, abs=1e-9)
    objs = [a["objective"] for a in got["all"]]
    assert got["best"]["objective"] == min(objs)
    assert got["best"]["K"] == min(a["K"] for a in got["all"] if a["objective"] == min(objs))
    assert first_dev == h - 1 and got["best"]["K"] == ref["best"]["K"]   # continuous S: no near-ties
    assert oc.cluster_heads(S, 3) == groups


def test_refine_value_matches_oracle():
    from paper_2607_24331_amd.offline import refine_value
    g = np.random.default_rng(8)
    m, n, N, r = 64, 48, 700, 12
    W = g.standard_normal((m, n))
    X = (g.standard_normal((N, m)) * np.logspace(0, 1, m)[None, :]).astype(np.float32)
    got = refine_value(W, r, torch.from_numpy(X).cuda())
    ref = ocal.refine(X.astype(np.float64), W, r)
    # the GPU Gram is fp32: the refined product agrees to fp32-level relative error
    scale = np.max(np.abs(ref["L"] @ ref["R"]))
    assert np.max(np.abs(got["L"] @ got["R"] - ref["L"] @ ref["R"])) <= 1e-4 * scale
    assert got["eps"] <= got["eps_mid"] * (1 + 1e-6) <= got["eps_svd"] * (1 + 1e-6)
    assert got["eps"] == pytest.approx(ref["eps"], rel=1e-4)
