"""GPU parity of the wave-per-window matrix kernel at the edges of its column tile (128, 160 and 192 columns by form), of its
rounds of non-zeros (384, 896 and 512 more at a time), and of graphs with windows of both kinds and a list of the scalar rows."""
import numpy as np
import pytest

import oracle
from workloads import CSRGraph, dense_normal, to_bf16_bits, to_f16_bits
from gpu_util import gpu_spmm, assert_close, oracle_pair

pytestmark = pytest.mark.gpu
ALL_MFMA, PER_WINDOW = 2, 3


def windows(cols_nnz, n_cols=1000, seed=0):
    """One 16-row window per (columns, non-zeros) pair: every column at least once, duplicates where there are too many non-zeros."""
    rng = np.random.default_rng(seed)
    rows = []
    for nc, nnz in cols_nnz:
        cols = rng.choice(n_cols, nc, replace=False)
        k = np.concatenate([cols, rng.choice(cols, nnz - nc)])
        r = rng.integers(0, 16, nnz)
        rows += [np.sort(k[r == i]) for i in range(16)]
    rowptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    colind = np.concatenate(rows).astype(np.int32)
    return CSRGraph(len(rows), n_cols, rowptr, colind, rng.uniform(-1, 1, len(colind)).astype(np.float32))


EDGES = [(1, 1), (63, 383), (64, 384), (65, 385), (127, 895), (128, 896), (129, 897), (159, 1407), (160, 1408), (161, 1409),
         (191, 700), (192, 2000), (193, 193), (255, 4096), (256, 5000), (32, 4096), (130, 130)]


@pytest.mark.parametrize("x_bits,d", [(None, 16), (None, 20), (None, 50), (None, 64), (None, 100), (None, 128), (None, 256),
                                      ("bf16", 32), ("bf16", 68), ("bf16", 128), ("bf16", 256), ("f16", 200), ("f16", 72)])
def test_tile_and_round_edges(x_bits, d):
    g = windows(EDGES, seed=d)
    X = dense_normal(g.n_cols, d, seed=d)
    if x_bits is None:
        Y, info = gpu_spmm(g, X, ALL_MFMA)
        ref, bound = oracle_pair(g, X)
        tol = 1e-5
    else:
        bits, kind, code = (to_bf16_bits, oracle.DT_BF16, 1) if x_bits == "bf16" else (to_f16_bits, oracle.DT_F16, 2)
        X = bits(X)
        Y, info = gpu_spmm(g, X, ALL_MFMA, x_bits=x_bits, mfma_dtype=code)
        ref, bound = oracle_pair(g, X, x_dtype=kind)
        tol = 2e-2                                              # A is rounded to the 16-bit type on this path
    assert info["n_mfma_small"] == len(EDGES)
    assert_close(Y, ref, bound, tol, "%s d=%d" % (x_bits, d))


@pytest.mark.parametrize("matrix_windows", [0, 1, 6, 7, 50, 99, 100])
def test_scalar_rows_beside_matrix_windows(matrix_windows):
    # a sixteenth of 100 windows is between 6 and 7; windows of few non-zeros per column stay scalar
    kinds = [(40, 500)] * matrix_windows + [(120, 130)] * (100 - matrix_windows)
    np.random.default_rng(3).shuffle(kinds)
    g = windows(kinds, seed=matrix_windows)
    X = dense_normal(g.n_cols, 48, seed=1)
    Y, info = gpu_spmm(g, X, PER_WINDOW, sel_coef=[1, 0, -100])  # columns > 100: scalar
    assert info["n_mfma_windows"] == matrix_windows
    ref, bound = oracle_pair(g, X)
    assert_close(Y, ref, bound, 1e-5)
