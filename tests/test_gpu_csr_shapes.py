"""Scalar-path launch shapes against the oracle: vector widths and remainders of a lane group, column slices, row tiers."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, device_graph, gpu_spmm, oracle_pair
from workloads import tiny_random_csr, to_bf16_bits, to_f16_bits
from workloads.graphs import CSRGraph

pytestmark = pytest.mark.gpu


def rows_of(lengths, n_cols, seed):
    """CSR with the given row lengths, ascending distinct columns, normal values."""
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(n_cols, k, replace=False)) for k in lengths]
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    colind = np.concatenate(cols).astype(np.int32) if cols else np.empty(0, np.int32)
    return CSRGraph(len(lengths), n_cols, rowptr, colind, rng.standard_normal(colind.shape[0]).astype(np.float32))


# every tier and batch edge: empty, around 8 and 16, around the wave-per-row and segment thresholds, several segments
LENGTHS = [0, 1, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 127, 128, 129, 1023, 1024, 1025, 2049, 4999, 3, 0, 2]


@pytest.mark.parametrize("d", [1, 3, 4, 15, 16, 17, 18, 31, 32, 33, 47, 63, 64, 65, 127, 129, 131, 160, 255, 257])
def test_fp32_widths_and_row_lengths(d):
    g = rows_of(LENGTHS, 5000, d)
    X = np.random.default_rng(d).standard_normal((g.n_cols, d)).astype(np.float32)
    Y, _ = gpu_spmm(g, X, 1, pad_x=d % 3, pad_y=d % 2)
    ref, bound = oracle_pair(g, X)
    assert_close(Y, ref, bound, 1e-5, "fp32 d=%d" % d)


# four lanes to a row: one, two and four (16-bit: two, four, eight) columns per lane, the last vector moved left or whole
@pytest.mark.parametrize("d", [1, 2, 4, 5, 6, 7, 8, 9, 10, 13, 14, 16])
@pytest.mark.parametrize("n", [40, 20_000])
def test_narrow_rows(n, d):
    g = rows_of(np.resize(LENGTHS[:16] if n > 1000 else LENGTHS, n), 5000, d)
    X = np.random.default_rng(d).standard_normal((g.n_cols, d)).astype(np.float32)
    rows = np.unique(np.concatenate([np.arange(0, n, 1 + n // 2000), np.arange(n - 20, n)]))
    Y, _ = gpu_spmm(g, X, 1, pad_x=d % 3, pad_y=d % 4)
    ref, bound = oracle_pair(g, X, rows=rows)
    assert_close(Y[rows], ref, bound, 1e-5, "fp32 d=%d" % d)
    for kind, code, bits in (("bf16", oracle.DT_BF16, to_bf16_bits), ("f16", oracle.DT_F16, to_f16_bits)):
        X = bits(np.random.default_rng(d).standard_normal((g.n_cols, 2 * d)).astype(np.float32))
        Y, _ = gpu_spmm(g, X, 1, pad_x=2 * (d % 3), pad_y=d % 4, x_bits=kind)
        ref, bound = oracle_pair(g, X, rows=rows, x_dtype=code)
        assert_close(Y[rows], ref, bound, 1e-5, "%s d=%d" % (kind, 2 * d))


def short_rows(lengths, n_cols, seed):
    """CSR with the given row lengths (at most n_cols), distinct columns in no order, for many rows."""
    rng = np.random.default_rng(seed)
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    at = np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], lengths)
    step = 7 if n_cols % 7 else 11
    colind = ((np.repeat(rng.integers(0, n_cols, len(lengths)), lengths) + step * at) % n_cols).astype(np.int32)
    return CSRGraph(len(lengths), n_cols, rowptr, colind, rng.standard_normal(colind.shape[0]).astype(np.float32))


# eight lanes to an output row: rows of X off the 16-byte pieces, or a matrix of rows that are many for their width (100,000 of
# up to 32 bytes, 200,000 of up to 64, a million of up to 128); one, two and four columns per lane (16-bit: two, four, eight),
# the last vector moved left or whole
@pytest.mark.parametrize("n,d", [(n, d) for n in (48, 100_003) for d in (1, 4, 5, 7, 8, 9, 10, 13, 16, 17, 30, 31, 32)] +
                         [(200_003, 9), (200_003, 16), (1_000_003, 17), (1_000_003, 32)])
def test_eight_lanes_to_a_row(n, d):
    lengths = np.resize([3, 0, 7, 8, 9, 1, 16, 17, 12, 2, 20], n)
    lengths[[5, n - 1]] = [129, 64]
    if n > 1000:
        lengths[[77, 50_000, 99_999]] = [300, 1025, 2049]
    g = short_rows(lengths, 5000, d)
    rows = np.unique(np.concatenate([np.arange(0, n, 1 + n // 3000), np.flatnonzero(lengths > 20), np.arange(n - 40, n)]))
    pad = 0 if n > 1000 else 1 + (d + 1) % 4 + (d % 4 == 3)           # (the small matrix: an odd pitch)
    X = np.random.default_rng(d).standard_normal((g.n_cols, d)).astype(np.float32)
    Y, _ = gpu_spmm(g, X, 1, pad_x=pad, pad_y=d % 4)
    ref, bound = oracle_pair(g, X, rows=rows)
    assert_close(Y[rows], ref, bound, 1e-5, "fp32 d=%d" % d)
    for kind, code, bits in (("bf16", oracle.DT_BF16, to_bf16_bits), ("f16", oracle.DT_F16, to_f16_bits)):
        X = bits(np.random.default_rng(d).standard_normal((g.n_cols, 2 * d)).astype(np.float32))
        Y, _ = gpu_spmm(g, X, 1, pad_x=2 * pad, pad_y=d % 4, x_bits=kind)
        ref, bound = oracle_pair(g, X, rows=rows, x_dtype=code)
        assert_close(Y[rows], ref, bound, 1e-5, "%s d=%d" % (kind, 2 * d))


@pytest.mark.parametrize("kind", ["bf16", "f16"])
@pytest.mark.parametrize("d,pad", [(1, 0), (2, 0), (15, 0), (16, 1), (18, 0), (32, 2), (34, 0), (62, 0), (64, 0), (66, 2), (128, 0),
                                   (130, 0), (131, 0), (256, 0), (258, 0)])
def test_16bit_widths_and_row_lengths(kind, d, pad):
    g = rows_of(LENGTHS, 5000, d)
    X = np.random.default_rng(d).standard_normal((g.n_cols, d)).astype(np.float32)
    bits = to_bf16_bits(X) if kind == "bf16" else to_f16_bits(X)
    code = oracle.DT_BF16 if kind == "bf16" else oracle.DT_F16
    Y, _ = gpu_spmm(g, bits, 1, pad_x=pad, x_bits=kind)
    ref, bound = oracle_pair(g, bits, x_dtype=code)
    assert_close(Y, ref, bound, 1e-5, "%s d=%d" % (kind, d))


# rows of degree 20 and 60: slices of 256 and of 128 bytes; counts that XCDs own (2, 4, 8) and counts taken in turn
@pytest.mark.parametrize("d", [64, 96, 128, 160, 192, 256, 300, 520])
@pytest.mark.parametrize("n,degree", [(700, 20), (700, 60), (20011, 12)])
def test_column_slices(n, degree, d):
    g = tiny_random_csr(n, n, degree / n, seed=d + degree)
    X = np.random.default_rng(d).standard_normal((n, d)).astype(np.float32)
    Y, _ = gpu_spmm(g, X, 1)
    rows = np.unique(np.concatenate([np.arange(0, n, 37), np.arange(max(0, n - 40), n)]))
    ref, bound = oracle_pair(g, X, rows=rows)
    assert_close(Y[rows], ref, bound, 1e-5, "slices n=%d degree=%d d=%d" % (n, degree, d))


# rows of a sparse matrix are cut into segments from 257 non-zeros on, those of a matrix of a handful of rows from 1025 on
@pytest.mark.parametrize("n,long_rows", [(255, 1), (256, 3), (170_000, 3)])
def test_long_rows_of_sparse_matrices(n, long_rows):
    lengths = np.ones(n, np.int64)
    hubs = np.array([5, n // 2, n // 2 + 1, n - 1])
    lengths[hubs] = [256, 257, 1024, 1025]
    rng = np.random.default_rng(n)
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    g = CSRGraph(n, 2000, rowptr, rng.integers(0, 2000, rowptr[-1]).astype(np.int32),
                 rng.standard_normal(rowptr[-1]).astype(np.float32))
    X = rng.standard_normal((g.n_cols, 64)).astype(np.float32)
    Y, info = gpu_spmm(g, X, 1)
    assert info["n_long_rows"] == info["n_segments"] == long_rows
    rows = np.unique(np.concatenate([hubs, np.arange(0, n, 97)]))
    ref, bound = oracle_pair(g, X, rows=rows)
    assert_close(Y[rows], ref, bound, 1e-5, "n=%d" % n)


@pytest.mark.parametrize("kind", ["bf16", "f16"])
@pytest.mark.parametrize("d,pad", [(192, 0), (160, 32), (132, 60)])
def test_three_slices_of_16bit_rows(kind, d, pad):
    """Rows of 257 to 511 bytes that start on 128-byte lines: three slices of a line, taken in turn by lane groups (more rows
    than the small matrices' wave per row takes) and by the waves and workgroups of longer rows."""
    g = short_rows(np.concatenate([np.resize(LENGTHS, 48), np.resize([20, 0, 33, 8, 17, 1], 4001)]), 20000, d)
    X = np.random.default_rng(d).standard_normal((g.n_cols, d)).astype(np.float32)
    bits = to_bf16_bits(X) if kind == "bf16" else to_f16_bits(X)
    Y, _ = gpu_spmm(g, bits, 1, pad_x=pad, x_bits=kind)
    ref, bound = oracle_pair(g, bits, x_dtype=oracle.DT_BF16 if kind == "bf16" else oracle.DT_F16)
    assert_close(Y, ref, bound, 1e-5, "%s d=%d" % (kind, d))


@pytest.mark.parametrize("d", [256, 260, 320, 512])
def test_halves_of_16bit_rows_that_take_a_wave_each(d):
    """Rows of more non-zeros than the short tier takes, in few columns (nothing to gain from narrow slices)."""
    g = rows_of([150] * 700, 300, d)
    bits = to_bf16_bits(np.random.default_rng(d).standard_normal((300, d)).astype(np.float32))
    Y, _ = gpu_spmm(g, bits, 0, x_bits="bf16", mfma_dtype=1, sel_coef=[0, 0, 1])
    ref, bound = oracle_pair(g, bits, x_dtype=oracle.DT_BF16)
    assert_close(Y, ref, bound, 1e-5, "bf16 d=%d" % d)


# whole rows of four vectors (16-bit: two) off the 128-byte lines, on either side of the degrees from which they take three and two waves per SIMD
@pytest.mark.parametrize("kind,degree,d,pad", [(None, 14, 131, 0), (None, 16, 131, 0), (None, 16, 203, 2), (None, 16, 256, 1), (None, 45, 167, 0),
                                               (None, 45, 203, 1), ("bf16", 27, 202, 0), ("bf16", 29, 202, 0), ("bf16", 29, 250, 2),
                                               ("f16", 29, 138, 0), ("bf16", 45, 202, 0), ("f16", 45, 250, 2)])
def test_whole_rows_of_several_vectors(kind, degree, d, pad):
    n, n_cols = 5000, 110_000
    rng = np.random.default_rng(d)
    lengths = rng.integers(degree - 13, degree + 14, n)
    lengths[:4] = [0, 300, 2500, 129]                           # (0.6 on average)
    g = short_rows(lengths, n_cols, seed=d)
    X = rng.standard_normal((n_cols, d)).astype(np.float32)
    if kind is None:
        Y, _ = gpu_spmm(g, X, 1, pad_x=pad, pad_y=1)
        ref, bound = oracle_pair(g, X)
    else:
        bits, code = (to_bf16_bits, oracle.DT_BF16) if kind == "bf16" else (to_f16_bits, oracle.DT_F16)
        X = bits(X)
        Y, _ = gpu_spmm(g, X, 1, pad_x=pad, pad_y=1, x_bits=kind)
        ref, bound = oracle_pair(g, X, x_dtype=code)
    assert_close(Y, ref, bound, 1e-5, "%s d=%d degree=%d" % (kind, d, degree))


# both sides of the line up to which every row takes a wave (rows times slices), with rows of several segments, a relu and a pitched Y
@pytest.mark.parametrize("kind,n,d", [(None, 4096, 32), (None, 4097, 32), (None, 2048, 256), (None, 2049, 256), ("bf16", 6144, 64), ("bf16", 6145, 64), (None, 600, 1030)])
def test_few_rows_with_long_ones(kind, n, d):
    import torch
    import paper_2412_08902_amd.binding as hc
    lengths = np.full(n, 3, np.int64)
    lengths[[1, n // 2, n - 1]] = [5000, 300, 2049]
    rng = np.random.default_rng(n + d)
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    g = CSRGraph(n, 3000, rowptr, rng.integers(0, 3000, rowptr[-1]).astype(np.int32), rng.standard_normal(rowptr[-1]).astype(np.float32))
    X = rng.standard_normal((g.n_cols, d)).astype(np.float32)
    bits = X if kind is None else to_bf16_bits(X)
    Xd = torch.from_numpy(bits).cuda() if kind is None else torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)
    plan = hc.hcspmm_prepare(n, g.n_cols, *device_graph(g), route_mode=1, d_hint=d, mfma_dtype=0 if kind is None else 1)
    Y = torch.full((n, d + 3), -7.0, device="cuda")
    hc.hcspmm_spmm(plan, Xd, Y[:, :d])
    torch.cuda.synchronize()
    plan.destroy()
    ref, bound = oracle_pair(g, bits, **({} if kind is None else {"x_dtype": oracle.DT_BF16}))
    assert_close(Y[:, :d].cpu().numpy().astype(np.float64), ref, bound, 1e-5, "n=%d d=%d" % (n, d))
    assert bool((Y[:, d:] == -7.0).all())


# long scattered rows of one 16-byte vector per lane on 36 MB of X and more: five waves per SIMD from 40 non-zeros per row on, four from 60
# (up to 32 columns of fp32 from 70)
@pytest.mark.parametrize("kind,d", [("f32", 20), ("f32", 32), ("f32", 47), ("f32", 128), ("bf16", 64), ("bf16", 100), ("f16", 62), ("f16", 128)])
@pytest.mark.parametrize("degree", [40, 60, 70])
def test_fewer_waves_for_long_scattered_rows(kind, d, degree):
    es = 4 if kind == "f32" else 2
    n_cols = (37 << 20) // (d * es)
    lengths = np.full(5000, degree)
    lengths[[0, 1, 2, 3, 4]] = [0, 1, 300, 1100, 5000]
    g = short_rows(lengths, n_cols, d)
    assert degree <= g.nnz / g.n_rows < degree + 20
    X = np.random.default_rng(d).standard_normal((n_cols, d)).astype(np.float32)
    code, bits = {"f32": (None, None), "bf16": (oracle.DT_BF16, to_bf16_bits), "f16": (oracle.DT_F16, to_f16_bits)}[kind]
    if bits:
        X = bits(X)
    rows = np.unique(np.concatenate([np.arange(8), np.arange(8, 5000, 7), np.arange(4980, 5000)]))
    Y, _ = gpu_spmm(g, X, 1, pad_y=d % 3, x_bits=kind if bits else None)
    ref, bound = oracle_pair(g, X, rows=rows, x_dtype=code)
    assert_close(Y[rows], ref, bound, 1e-5, "%s d=%d" % (kind, d))


# the same for 16-bit X with more rows than those that all take a wave (6,144 times the slices), so that rows of up to 64 non-zeros take a lane group each
@pytest.mark.parametrize("kind,d", [("bf16", 64), ("bf16", 100), ("f16", 62), ("f16", 128)])
@pytest.mark.parametrize("degree", [40, 60])
def test_fewer_waves_for_short_rows_of_16_bit(kind, d, degree):
    n, n_cols = 14000, (37 << 20) // (2 * d)
    lengths = np.where(np.arange(n) % 2 == 0, degree, degree + 3)          # on both sides of 64 where degree is 60: 60 and 63, beside rows of a wave
    lengths[:5] = [0, 1, 300, 1100, 5000]
    lengths[5::16] = 66
    g = short_rows(lengths, n_cols, d)
    assert degree <= g.nnz / g.n_rows < degree + 20 and g.n_rows > 2 * 6144
    code, bits = (oracle.DT_BF16, to_bf16_bits) if kind == "bf16" else (oracle.DT_F16, to_f16_bits)
    X = bits(np.random.default_rng(d).standard_normal((n_cols, d)).astype(np.float32))
    rows = np.unique(np.concatenate([np.arange(40), np.arange(40, n, 13), np.arange(n - 40, n)]))
    Y, _ = gpu_spmm(g, X, 1, pad_y=d % 3, x_bits=kind)
    ref, bound = oracle_pair(g, X, rows=rows, x_dtype=code)
    assert_close(Y[rows], ref, bound, 1e-5, "%s d=%d" % (kind, d))
