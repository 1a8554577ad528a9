"""dX = S W^T and dW = X^T S in one kernel (widths of up to 128): row counts around its batches and turns, widths around its
tiles, pitches off the vectors, and rows past the last batch that must not be touched or read."""
import numpy as np
import pytest

from workloads import dense_normal, glorot_uniform, tiny_random_csr
from gpu_util import device_graph
from test_gpu_backward import check

pytestmark = pytest.mark.gpu


def padded(a, pad):
    """a as a view of a wider array of NaN: nothing beside it may be read into a result"""
    import torch
    t = torch.full((a.shape[0], a.shape[1] + pad), float("nan"), device="cuda")
    t[:, :a.shape[1]] = torch.from_numpy(a).cuda()
    return t[:, :a.shape[1]]


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 100, 1023, 3500, 3501, 4112, 9000])
@pytest.mark.parametrize("d_in,d,pad", [(128, 128, 0), (128, 128, 3), (112, 72, 0), (66, 96, 1), (69, 100, 0), (100, 84, 2),
                                        (120, 124, 5), (96, 68, 0), (127, 80, 0)])       # whole tiles of columns and parts of them
def test_products(n, d_in, d, pad):
    products(n, d_in, d, pad)


# Walks of three, five and nine batches of 32 rows: both buffers come round several times, and either has the last turn.
@pytest.mark.parametrize("n,d_in,d,pad", [(20481, 128, 128, 0), (20481, 100, 84, 2), (40007, 96, 96, 0), (40007, 128, 72, 1), (40007, 72, 128, 0),
                                          (65535, 96, 96, 0), (70001, 128, 128, 0), (70001, 112, 72, 3), (70001, 96, 96, 0)])
def test_products_of_many_batches(n, d_in, d, pad):
    products(n, d_in, d, pad)


def products(n, d_in, d, pad):
    import torch
    import paper_2412_08902_amd.binding as hc
    g = tiny_random_csr(n, n, min(1.0, 8.0 / n), seed=n + d)
    G, X, W = dense_normal(n, d, seed=1), dense_normal(n, d_in, seed=2), glorot_uniform(d_in, d, seed=3)
    plan = hc.hcspmm_prepare(n, n, *device_graph(g), route_mode=1, d_hint=d, update_fusion=2)
    ws = torch.empty(hc.hcspmm_layer_backward_workspace_bytes(plan, d_in, d), dtype=torch.uint8, device="cuda")
    dX = torch.full((n + 1, d_in + pad), -3.0, device="cuda")
    dW = torch.full((d_in + 1, d + pad), -3.0, device="cuda")
    hc.hcspmm_layer_backward(plan, padded(G, pad), padded(X, pad), padded(W, pad), dX[:n, :d_in], dW[:d_in, :d], ws)
    torch.cuda.synchronize()
    plan.destroy()
    S = ws[:n * d * 4].view(torch.float32).reshape(n, d).cpu().numpy().astype(np.float64)
    dX, dW = dX.cpu().numpy().astype(np.float64), dW.cpu().numpy().astype(np.float64)
    assert np.all(dX[n:] == -3.0) and np.all(dX[:, d_in:] == -3.0) and np.all(dW[d_in:] == -3.0) and np.all(dW[:, d:] == -3.0)
    check(g, G, X, W, dX[:n, :d_in], dW[:d_in, :d], S)


# X of up to 64 columns (no barriers): one and two tiles per wave, widths off the tiles and vectors, S of eight to 128 columns, row counts around
# the batches of 32, around the walk of every G-th batch (256 workgroups) and around the waves' turns
@pytest.mark.parametrize("n", [1, 31, 32, 33, 129, 5003])
@pytest.mark.parametrize("d_in,d,pad", [(1, 8, 0), (16, 16, 1), (31, 9, 0), (32, 128, 3), (33, 47, 0), (47, 100, 1), (64, 64, 0), (64, 127, 2), (50, 96, 0)])
def test_products_of_few_columns(n, d_in, d, pad):
    products(n, d_in, d, pad)


@pytest.mark.parametrize("n", [8192, 8193, 20481, 41000])
@pytest.mark.parametrize("d_in,d,pad", [(16, 24, 0), (64, 70, 1), (100, 16, 0), (65, 33, 2), (128, 127, 1)])
def test_products_of_several_turns(n, d_in, d, pad):
    products(n, d_in, d, pad)


def whole(n, d_in, d, change=None):
    """layer_backward of the identity graph: S = A G as it was formed, X, W, dX, dW"""
    import torch
    import paper_2412_08902_amd.binding as hc
    G, X, W = dense_normal(n, d, seed=1), np.maximum(dense_normal(n, d_in, seed=2), 0), glorot_uniform(d_in, d, seed=3)
    if change:
        change(G, X, W)
    rowptr = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    plan = hc.hcspmm_prepare(n, n, rowptr, rowptr[:n].clone(), torch.ones(n, device="cuda"), route_mode=1, d_hint=d, update_fusion=2)
    ws = torch.empty(hc.hcspmm_layer_backward_workspace_bytes(plan, d_in, d), dtype=torch.uint8, device="cuda")
    dX, dW = torch.empty((n, d_in), device="cuda"), torch.empty((d_in, d), device="cuda")
    hc.hcspmm_layer_backward(plan, *(torch.from_numpy(a).cuda() for a in (G, X, W)), dX, dW, ws)
    torch.cuda.synchronize()
    plan.destroy()
    S = ws[:n * d * 4].view(torch.float32).reshape(n, d).cpu().numpy()
    return S, X, W, dX.cpu().numpy().astype(np.float64), dW.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("d_in,d", [(128, 128), (48, 64)])
def test_products_are_no_less_exact(d_in, d):
    """Against 64 bits.  dX: a 32-bit sum of d terms rounds at random by half the square root of d, in units of 2^-24.  dW of 169,343
    rows: 21 sums of batches, then 16 and 16 partial sums, each rounded by up to 2^-24 of a partial result that is smaller on average than
    the last: 4.4 units (the fp32 units came to 4.3; a truncation that does not cancel over the batches to 8.5)."""
    S, X, W, dX, dW = whole(169343, d_in, d)
    ref = X.astype(np.float64).T @ S.astype(np.float64)
    assert np.linalg.norm(dW - ref) <= 4.4 * 2.0 ** -24 * np.linalg.norm(ref)
    rows = slice(0, 4000)
    ref = S[rows].astype(np.float64) @ W.astype(np.float64).T
    assert np.linalg.norm(dX[rows] - ref) <= 0.5 * np.sqrt(d) * 2.0 ** -24 * np.linalg.norm(ref)


@pytest.mark.parametrize("n,d_in,d", [(8000, 128, 100), (8000, 100, 30), (24000, 128, 128), (40007, 60, 90), (9000, 48, 64)])
def test_products_have_no_one_sided_error(n, d_in, d):
    """Results are rounded up as often as down, whatever the number of batches to a workgroup: the mean error, relative to the mean sum of
    magnitudes, is that of at most 2^-24 each over all results, by six standard deviations."""
    S, X, W, dX, dW = whole(n, d_in, d)
    for got, a, b in ((dX[:4000], S[:4000].astype(np.float64), W.astype(np.float64).T), (dW, X.astype(np.float64).T, S.astype(np.float64))):
        off = got - a @ b
        assert abs(off.mean()) <= 6 / np.sqrt(off.size) * 2.0 ** -24 * (np.abs(a) @ np.abs(b)).mean()


@pytest.mark.parametrize("n,d_in,d", [(5003, 128, 100), (5003, 60, 90), (9000, 17, 64)])
def test_products_of_single_terms(n, d_in, d):
    """One non-zero to a row of S: dX is rounded once, which is 0.42 units of 2^-24 as a 2-norm."""
    def change(G, X, W):
        keep = np.random.default_rng(3).integers(0, d, n)
        G[np.arange(d) != keep[:, None]] = 0
    S, X, W, dX, dW = whole(n, d_in, d, change)
    ref = S.astype(np.float64) @ W.astype(np.float64).T
    assert np.linalg.norm(dX - ref) <= 0.45 * 2.0 ** -24 * np.linalg.norm(ref)


# Small values keep all their bits, and large ones whose products come back into the range: 2-norms of at most 2^-24 for what a batch leaves
# out and rounds, and 2^-24 for each addition (dX: d / 32 of them; dW: a workgroup's batches, then 16 and 16 partial sums).
@pytest.mark.parametrize("n,d_in,d", [(5003, 128, 100), (20481, 70, 30), (5003, 60, 90), (9000, 17, 64)])
@pytest.mark.parametrize("g_exp,x_exp,w_exp", [(-105, 0, 0), (-112, 0, 0), (-120, 0, 0), (0, -112, -118), (-120, 100, 100), (100, -112, -105), (-140, 40, 30)])
def test_products_of_small_and_large_values(n, d_in, d, g_exp, x_exp, w_exp):
    def change(G, X, W):
        for a, e in ((G, g_exp), (X, x_exp), (W, w_exp)):
            a[...] = np.ldexp(a, e)
    S, X, W, dX, dW = whole(n, d_in, d, change)
    S, X, W = (np.ldexp(a.astype(np.float64), -e) for a, e in ((S, g_exp), (X, x_exp), (W, w_exp)))
    for got, ref, sums in ((np.ldexp(dX, -g_exp - w_exp), S @ W.T, d / 32), (np.ldexp(dW, -g_exp - x_exp), X.T @ S, 35)):
        assert np.linalg.norm(got - ref) <= (1 + np.sqrt(sums)) * 2.0 ** -24 * np.linalg.norm(ref)


@pytest.mark.parametrize("d_in,d", [(128, 100), (70, 47), (60, 90), (17, 64)])
def test_products_of_values_without_a_remainder(d_in, d):
    """Infinities, NaN and values that round to infinity in bf16 come out as the fp32 units give them, where they belong alone."""
    def change(G, X, W):
        G[5, 3], G[9000, d - 1], G[9010, 0] = np.inf, np.nan, np.float32(3.4e38)
        X[77, 2], X[9050, d_in - 1] = np.inf, np.float32(3.4e38)
        W[1, 7] = -np.inf
    S, X, W, dX, dW = whole(9051, d_in, d, change)
    for got, a, b in ((dX, S, W.T), (dW, X.T, S)):
        with np.errstate(all="ignore"):
            ref = a.astype(np.float64) @ b.astype(np.float64)
            bound = np.abs(a.astype(np.float64)) @ np.abs(b.astype(np.float64))
        ref = np.where(np.abs(ref) > np.finfo(np.float32).max, np.sign(ref) * np.inf, ref)
        sure = ~(np.isfinite(bound) & (bound > 3.36e38))            # (sums within rounding of the largest value may go either way)
        assert np.array_equal(np.isnan(got)[sure], np.isnan(ref)[sure])
        odd = sure & ~np.isfinite(ref) & ~np.isnan(ref)
        assert np.array_equal(got[odd], ref[odd])
        ok = sure & np.isfinite(ref)
        assert ok.mean() > 0.8 and np.all(np.abs(got[ok] - ref[ok]) <= 1e-5 * bound[ok])
