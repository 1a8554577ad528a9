"""The dense products at the edges of their tiles: X W with W in LDS slabs and in registers, and the weight gradient's X^T S."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close
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
