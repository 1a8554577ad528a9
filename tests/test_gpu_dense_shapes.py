"""The dense products at the edges of their tiles: X W with W in LDS slabs and in registers, and the weight gradient's X^T S."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, device_graph
from test_gpu_backward import check, run_backward
from workloads import dense_normal, glorot_uniform, tiny_random_csr

pytestmark = pytest.mark.gpu


def gemm(m, k, n, ldx=0, pad=0):
    import torch
    import paper_2412_08902_amd.binding as hc
    X, W = dense_normal(m, k, seed=m + k), dense_normal(k, n, seed=k + n)
    Xd = torch.full((m, max(k, ldx)), float("nan"), device="cuda")
    Xd[:, :k] = torch.from_numpy(X)
    T = torch.full((m, n + pad), -5.0, device="cuda")
    hc.hcspmm_gemm_f32(Xd[:, :k], torch.from_numpy(W).cuda(), T[:, :n])
    torch.cuda.synchronize()
    got = T.cpu().numpy().astype(np.float64)
    assert np.all(got[:, n:] == -5.0)
    rows = np.unique(np.concatenate([np.arange(0, m, 1 + m // 2000), np.arange(max(0, m - 70), m)]))
    assert_close(got[rows, :n], oracle.gemm(X[rows], W), oracle.gemm(X[rows], W, use_abs=True), 1e-5, "%d x %d x %d" % (m, k, n))


# column counts of one to eight tiles and their remainders, one group, pairs of groups, three groups; odd widths of W
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 47, 48, 68, 80, 97, 112, 127, 128, 129, 144, 250, 256, 260, 384])
@pytest.mark.parametrize("m,k", [(65, 130), (130, 31)])
def test_slab_product_widths(m, k, n):
    gemm(m, k, n, pad=n % 3)


# whole slabs, one and two units beyond them, lanes with one to three values of their own
@pytest.mark.parametrize("k", [1, 2, 3, 4, 15, 16, 17, 30, 32, 33, 47, 48, 50, 63, 64, 65, 96, 602])
@pytest.mark.parametrize("m", [1, 15, 64, 79])
def test_slab_product_depths(m, k):
    gemm(m, k, 132, ldx=k + k % 3)


# W in registers: any row count where W is tiny, long X where it is small; depths and widths off the tiles, 1, 2 and 4 column groups
@pytest.mark.parametrize("m,k,n", [(1, 4, 1), (17, 16, 16), (300, 12, 33), (2049, 4, 250), (500, 32, 32), (4097, 60, 17),
                                   (65536, 128, 64), (65537, 100, 47), (65600, 64, 128), (70003, 36, 200), (66001, 8, 1000),
                                   (65551, 116, 70), (65536, 20, 3)])
@pytest.mark.parametrize("extra", [0, 1])
def test_register_product(m, k, n, extra):
    gemm(m, k, n, ldx=k + extra, pad=extra)


# fp32 X on the bf16 units: three to eight tiles of columns and their remainders, several groups; depths around the slabs of 32; rows around
# the workgroups' 128 and on both sides of the row counts from which each width is taken
@pytest.mark.parametrize("m,k,n", [(16384, 32, 65), (16385, 40, 80), (16383, 64, 96), (16384 + 127, 63, 97), (16512, 96, 112), (17001, 65, 127),
                                   (16640, 602, 128), (16384, 31, 128), (129, 32, 129), (127, 100, 250), (1, 64, 256), (128, 47, 384),
                                   (32768, 64, 33), (32767, 64, 48), (32900, 67, 47), (32769, 90, 64), (32768, 63, 64), (70001, 70, 52),
                                   (32768, 72, 52), (49152, 96, 96), (49153, 32, 70), (49152, 64, 112), (49152, 128, 101), (65536, 32, 96), (65536, 48, 100), (65536, 64, 90),
                                   (65537, 40, 72), (4095, 70, 272), (5505, 33, 300), (12288, 32, 150), (100000, 72, 45), (99999, 72, 45)])
@pytest.mark.parametrize("extra", [0, 1])
def test_split_product(m, k, n, extra):
    gemm(m, k, n, ldx=k + extra, pad=extra)


# the same with four and eight waves to a workgroup (up to 256 workgroups of 64 rows and beyond), on both sides of the depths and row counts of 33 to 64
# columns, a last slab of one to 31 rows, and W as a column slice of a wider array
@pytest.mark.parametrize("m,k,n", [(16385, 96, 33), (16448, 64, 64), (32768, 95, 48), (32769, 96, 40), (57344, 65, 36), (200001, 129, 47), (200000, 128, 64),
                                   (64, 32, 129), (8192, 61, 200), (8193, 33, 256), (300, 97, 500), (16400, 94, 128)])
def test_split_product_of_few_rows_and_columns(m, k, n):
    import torch
    import paper_2412_08902_amd.binding as hc
    X, W = dense_normal(m, k, seed=m + k), dense_normal(k, n, seed=k + n)
    Wd = torch.full((k + 1, n + 5), float("nan"), device="cuda")
    Wd[:k, 2:n + 2] = torch.from_numpy(W)
    T = torch.full((m + 1, n), -5.0, device="cuda")
    hc.hcspmm_gemm_f32(torch.from_numpy(X).cuda(), Wd[:k, 2:n + 2], T[:m])
    got = T.cpu().numpy().astype(np.float64)
    assert np.all(got[m:] == -5.0)
    rows = np.unique(np.concatenate([np.arange(0, m, 1 + m // 2000), np.arange(max(0, m - 70), m)]))
    assert_close(got[rows], oracle.gemm(X[rows], W), oracle.gemm(X[rows], W, use_abs=True), 1e-5, "%d x %d x %d" % (m, k, n))


def test_split_product_of_values_without_a_remainder():
    """Infinities, NaN and values that round to infinity in bf16 come out as the fp32 units give them, in their own rows and
    columns alone; sums that overflow are infinite."""
    import torch
    import paper_2412_08902_amd.binding as hc
    m, k, n = 16500, 70, 100
    X, W = dense_normal(m, k, seed=1), dense_normal(k, n, seed=2)
    big = np.float32(3.4e38)
    X[5, 3], X[200, 69], X[16499, 64], X[300, 0], X[301, 1] = np.inf, -np.inf, np.nan, big, -big
    X[302, :2] = big
    W[:, 97] = 0.25
    W[10, 7], W[69, 50] = np.inf, np.nan
    W[0, 98], W[1, 98] = big, np.float32(0.0)
    T = torch.empty((m, n), device="cuda")
    hc.hcspmm_gemm_f32(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), T)
    got = T.cpu().numpy().astype(np.float64)
    with np.errstate(all="ignore"):
        ref = X.astype(np.float64) @ W.astype(np.float64)
        ref = np.where(np.abs(ref) > np.finfo(np.float32).max, np.sign(ref) * np.inf, ref)
        bound = np.abs(X.astype(np.float64)) @ np.abs(W.astype(np.float64))
    # (sums within rounding of the largest value may go either way)
    sure = ~(np.isfinite(bound) & (bound > 3.36e38) & (np.abs(ref) < 3.44e38))
    whole = np.isfinite(ref)
    assert np.array_equal(np.isnan(got)[sure], np.isnan(ref)[sure])
    assert np.array_equal(got[sure & ~whole & ~np.isnan(ref)], ref[sure & ~whole & ~np.isnan(ref)])
    ok = whole & sure & np.isfinite(bound)
    assert ok.mean() > 0.95 and np.all(np.abs(got[ok] - ref[ok]) <= 1e-5 * bound[ok])


# Small values keep all their bits, those below the normal range too, and large ones whose products come back into it: 2-norms against 64 bits of
# at most 2^-24 of the result for what each slab of 32 terms leaves out and rounds, and 2^-24 for each of the additions, which add up as a random walk.
# Values of 2^105 and more and results of 2^82 and more come from the fp32 units: half of 2^-24 for each term, as a random walk.
@pytest.mark.parametrize("m,k,n", [(16640, 128, 100), (300, 100, 160), (33000, 96, 40)])
@pytest.mark.parametrize("x_exp,w_exp", [(-105, 0), (-112, 0), (-120, 0), (-120, 100), (0, -115), (-140, 30), (20, -140), (-60, -60), (60, 0), (110, -100), (100, 20)])
def test_split_product_of_small_and_large_values(m, k, n, x_exp, w_exp):
    import torch
    import paper_2412_08902_amd.binding as hc
    X, W = np.ldexp(dense_normal(m, k, seed=1), x_exp), np.ldexp(dense_normal(k, n, seed=2), w_exp)
    assert X.dtype == np.float32 and W.dtype == np.float32
    T = torch.empty((m, n), device="cuda")
    hc.hcspmm_gemm_f32(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), T)
    rows = np.unique(np.concatenate([np.arange(0, m, 1 + m // 1000), np.arange(m - 70, m)]))
    ref = np.ldexp(X[rows].astype(np.float64), -x_exp) @ np.ldexp(W.astype(np.float64), -w_exp)
    got = np.ldexp(T.cpu().numpy()[rows].astype(np.float64), -x_exp - w_exp)
    roundings = 0.5 * np.sqrt(k) if max(x_exp, w_exp) >= 100 and x_exp >= 0 else 1 + np.sqrt(k / 32)
    assert np.linalg.norm(got - ref) <= roundings * 2.0 ** -24 * np.linalg.norm(ref)


@pytest.mark.parametrize("m,k,n", [(16640, 32, 128), (16640, 128, 100), (4000, 602, 160), (33000, 96, 40)])
@pytest.mark.parametrize("positive_x", [0, 1])
def test_split_product_has_no_one_sided_error(m, k, n, positive_x):
    """Results are rounded up as often as down: a bias would add up where rows of them are summed over neighbours.  The mean error, relative to the mean
    sum of magnitudes, is that of at most 2^-24 each over all results, by six standard deviations."""
    import torch
    import paper_2412_08902_amd.binding as hc
    X, W = dense_normal(m, k, seed=1), dense_normal(k, n, seed=2)
    if positive_x:
        X = np.maximum(X, 0)
    T = torch.empty((m, n), device="cuda")
    hc.hcspmm_gemm_f32(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), T)
    rows = slice(0, 4000)
    off = T.cpu().numpy()[rows].astype(np.float64) - X[rows].astype(np.float64) @ W.astype(np.float64)
    assert abs(off.mean()) <= 6 / np.sqrt(off.size) * 2.0 ** -24 * (np.abs(X[rows]) @ np.abs(W)).mean()


@pytest.mark.parametrize("m,k,n", [(16640, 128, 100), (300, 602, 160), (33000, 96, 40)])
def test_split_product_of_single_terms(m, k, n):
    """One non-zero to a row of X: results are rounded once.  To nearest that is 0.42 units of 2^-24 as a 2-norm (uniform by 0.58 of half a unit in the
    last place, over mantissas from 1 to 2 spread by their logarithm)."""
    import torch
    import paper_2412_08902_amd.binding as hc
    X, W = np.zeros((m, k), np.float32), dense_normal(k, n, seed=2)
    X[np.arange(m), np.random.default_rng(3).integers(0, k, m)] = dense_normal(m, 1, seed=1)[:, 0]
    T = torch.empty((m, n), device="cuda")
    hc.hcspmm_gemm_f32(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), T)
    rows = slice(0, 4000)
    ref = X[rows].astype(np.float64) @ W.astype(np.float64)
    assert np.linalg.norm(T.cpu().numpy()[rows].astype(np.float64) - ref) <= 0.45 * 2.0 ** -24 * np.linalg.norm(ref)


def test_split_product_is_no_less_exact():
    """Against 64 bits the products in three parts are no further off than a fp32 sum of as many terms: half the square root of
    the terms in units of 2^-24 (their roundings' random walk) as a 2-norm, relative to the result."""
    import torch
    import paper_2412_08902_amd.binding as hc
    for m, k, n, seed in ((16384, 32, 128, 1), (16384, 128, 128, 2), (2000, 602, 256, 3), (33000, 256, 64, 4)):
        X, W = dense_normal(m, k, seed=seed), glorot_uniform(k, n, seed=seed)
        X[:, ::3] *= np.float32(1e-3)
        T = torch.empty((m, n), device="cuda")
        hc.hcspmm_gemm_f32(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), T)
        rows = slice(0, 2000)
        ref = X[rows].astype(np.float64) @ W.astype(np.float64)
        off = np.linalg.norm(T.cpu().numpy()[rows].astype(np.float64) - ref) / np.linalg.norm(ref)
        assert off <= 0.5 * np.sqrt(k) * 2.0 ** -24, (m, k, n, off)


def test_layer_of_split_products_over_many_neighbours():
    """Y = A (X W) against 64 bits: about 300 rows of T to a row of Y, in units of 2^-24 as a 2-norm.  An addition is rounded by 0.42 and the sums grow as a random
    walk, over 300 neighbours and, for each T, 19 slabs: 5.3 at most.  An error of T of one sign, 1.7e-9 of its terms' magnitudes, comes to 10 by itself."""
    import torch
    import paper_2412_08902_amd.binding as hc
    n, k, d = 2000, 602, 160
    g = tiny_random_csr(n, n, 0.15, seed=5)
    g.vals[:] = 1
    X, W = dense_normal(n, k, seed=1), glorot_uniform(k, d, seed=2)
    plan = hc.hcspmm_prepare(n, n, *device_graph(g), route_mode=1, d_hint=d)
    ws = torch.empty(hc.hcspmm_gcn_workspace_bytes(plan, k, d), dtype=torch.uint8, device="cuda")
    Y = torch.empty((n, d), device="cuda")
    hc.hcspmm_gcn_layer(plan, torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), Y, ws, apply_relu=False)
    torch.cuda.synchronize()
    plan.destroy()
    A = np.zeros((n, n))
    A[np.repeat(np.arange(n), np.diff(g.rowptr)), g.colind] = 1
    ref = A @ (X.astype(np.float64) @ W.astype(np.float64))
    assert np.linalg.norm(Y.cpu().numpy().astype(np.float64) - ref) <= 0.42 * np.sqrt((300 + 1) / 2 + (19 + 1) / 2) * 2.0 ** -24 * np.linalg.norm(ref)


# X^T S: blocks of one to four tiles each way, widths that vectors divide and widths they do not, several row groups and
# workgroups, row counts around batches of 16 and below one
@pytest.mark.parametrize("d_in,d_out", [(1, 1), (16, 16), (15, 33), (48, 32), (64, 64), (50, 80), (96, 128), (130, 47), (257, 64), (65, 300)])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 700, 5003])
def test_weight_gradient(n, d_in, d_out):
    g = tiny_random_csr(n, n, min(1.0, 5.0 / n), seed=n + d_in)
    G, X, W = dense_normal(n, d_out, seed=1), dense_normal(n, d_in, seed=2), glorot_uniform(d_in, d_out, seed=3)
    dX, dW, S = run_backward(g, G, X, W, mode=1, pad=d_in % 2)
    check(g, G, X, W, dX, dW, S)


def test_slab_product_with_a_pitch_beyond_32_bit_offsets():
    """W as a column slice of a very wide array: 31 rows of its pitch are more than 4 GiB.  Full slabs of 32 and a rest of K;
    one column group, two in a workgroup, three."""
    import torch
    import paper_2412_08902_amd.binding as hc
    pitch, k, m = 34_700_001, 37, 70
    big = torch.empty((k, pitch), device="cuda")                  # 5.1 GB, of which the slice below is written and read
    X = dense_normal(m, k, seed=1)
    for n in (20, 130, 300):
        W = dense_normal(k, n, seed=n)
        big[:, 8:8 + n] = torch.from_numpy(W).cuda()
        T = torch.full((m, n), float("nan"), device="cuda")
        hc.hcspmm_gemm_f32(torch.from_numpy(X).cuda(), big[:, 8:8 + n], T)
        torch.cuda.synchronize()
        assert_close(T.cpu().numpy().astype(np.float64), oracle.gemm(X, W), oracle.gemm(X, W, use_abs=True), 1e-5, "n=%d" % n)
