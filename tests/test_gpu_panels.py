"""Column panels of the scalar path (many non-zeros per row, X far larger than an L2) against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, device_graph, gpu_spmm, oracle_pair
from test_gpu_update import update_and_check
from test_gpu_y16 import close_16, from_dev_16, torch_16, widen
from workloads import CSRGraph, to_bf16_bits

pytestmark = pytest.mark.gpu
N_COLS = 120_000                     # four panels of 128-byte slices from 150 non-zeros per row on (400 for 16-bit rows of 128 bytes)


def graph(n_rows, n_cols=N_COLS, seed=1, ascending=True, times=1):
    """Rows of about 170 non-zeros (or so many times that) that favour low columns; empty rows, hubs of one and several
    segments, rows that miss whole panels, repeated columns."""
    rng = np.random.default_rng(seed)
    length = times * rng.integers(110, 240, n_rows)
    length[rng.choice(n_rows, n_rows // 20, replace=False)] = 0
    length[rng.choice(n_rows, 6, replace=False)] = [1023, 1025, 2049, 4096, 5000, 9000]
    length[-1], length[0] = 0, 3
    row = np.repeat(np.arange(n_rows), length)
    col = (n_cols * rng.random(row.shape[0]) ** 2).astype(np.int64)
    third = row % 7 == 3
    col[third] = n_cols // 2 + col[third] // 8
    col[::50] = col[row.searchsorted(row[::50])]
    col = col[np.lexsort((col, row))]
    if not ascending:
        col[1], col[2] = n_cols - 1, 0
    rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int32)
    return CSRGraph(n_rows, n_cols, rowptr, col.astype(np.int32), rng.standard_normal(col.shape[0]).astype(np.float32))


def has_panels(g, d, mfma_dtype=0):
    """A scalar-only plan holds more memory with panels (their tables) than a plan of the same matrix that may not take any."""
    import paper_2412_08902_amd.binding as hc
    dev = device_graph(g)
    size = []
    for kernels in (hc.HCSPMM_MATRIX_AUTO, hc.HCSPMM_MATRIX_PER_WINDOW):
        plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *dev, route_mode=1, d_hint=d, mfma_dtype=mfma_dtype, matrix_kernels=kernels)
        size.append(hc.hcspmm_plan_info(plan)["device_bytes"])
        plan.destroy()
    return size[0] > size[1]


# 300: a wave per row and slice; 9001: the short tier and a ragged last block
@pytest.mark.parametrize("n_rows", [300, 9001])
@pytest.mark.parametrize("d,pad", [(32, 0), (33, 0), (64, 1), (128, 0), (130, 3), (256, 0)])
@pytest.mark.parametrize("mode", [0, 1])
def test_fp32_panels(n_rows, d, pad, mode):
    g = graph(n_rows)
    assert has_panels(g, d)
    X = np.random.default_rng(d).standard_normal((N_COLS, d)).astype(np.float32)
    Y, _ = gpu_spmm(g, X, mode, pad_x=pad, pad_y=pad)
    rows = np.unique(np.concatenate([np.arange(0, n_rows, 1 + n_rows // 300), np.flatnonzero(np.diff(g.rowptr) > 1000), [n_rows - 1]]))
    ref, bound = oracle_pair(g, X, rows=rows)
    assert_close(Y[rows], ref, bound, 1e-5, "panels n=%d d=%d mode=%d" % (n_rows, d, mode))


# an odd pitch is read element by element and takes no panels
@pytest.mark.parametrize("d,pad", [(64, 0), (66, 2), (128, 0), (64, 1), (256, 0)])
def test_16bit_panels(d, pad):
    g = graph(300, times=3)
    assert has_panels(g, d, 1)
    bits = to_bf16_bits(np.random.default_rng(d).standard_normal((N_COLS, d)).astype(np.float32))
    Y, _ = gpu_spmm(g, bits, 0, pad_x=pad, x_bits="bf16", mfma_dtype=1)
    ref, bound = oracle_pair(g, bits, x_dtype=oracle.DT_BF16)
    assert_close(Y, ref, bound, 1e-5, "bf16 panels d=%d" % d)


# on either side of the widths that are held to three and to two waves per SIMD, and two slices of more than a slice's limit
@pytest.mark.parametrize("n_rows,times", [(300, 3), (9001, 1)])
@pytest.mark.parametrize("kind", ["bf16", "f16"])
@pytest.mark.parametrize("d", [160, 168, 216, 224, 400])
def test_wide_16bit_panels(n_rows, times, kind, d):
    from workloads import to_f16_bits
    g = graph(n_rows, times=times)
    to_bits, code = (to_bf16_bits, oracle.DT_BF16) if kind == "bf16" else (to_f16_bits, oracle.DT_F16)
    assert has_panels(g, d, 1 if kind == "bf16" else 2)
    bits = to_bits(np.random.default_rng(d).standard_normal((N_COLS, d)).astype(np.float32))
    Y, _ = gpu_spmm(g, bits, 1, x_bits=kind, mfma_dtype=1 if kind == "bf16" else 2)
    rows = np.unique(np.concatenate([np.arange(0, n_rows, 1 + n_rows // 300), np.flatnonzero(np.diff(g.rowptr) > 1000), [n_rows - 1]]))
    ref, bound = oracle_pair(g, bits, rows=rows, x_dtype=code)
    assert_close(Y[rows], ref, bound, 1e-5, "%s panels n=%d d=%d" % (kind, n_rows, d))


def test_rows_that_do_not_ascend_take_no_panels():
    g = graph(300, ascending=False)
    assert not has_panels(g, 64)
    X = np.random.default_rng(3).standard_normal((N_COLS, 64)).astype(np.float32)
    Y, _ = gpu_spmm(g, X, 0)
    ref, bound = oracle_pair(g, X)
    assert_close(Y, ref, bound, 1e-5, "unsorted")


# communities in consecutive rows: their X rows meet in L2 without panels, and in the small ones without column slices
@pytest.mark.parametrize("size,panels", [(1000, False), (20_000, False), (120_000, True)])
@pytest.mark.parametrize("mode", [0, 1])
def test_communities_take_no_panels(size, panels, mode):
    n_rows, per_row = 8000, 160
    rng = np.random.default_rng(size)
    first = np.arange(n_rows) * N_COLS // n_rows // size * size
    col = np.sort(first[:, None] + rng.integers(0, size, (n_rows, per_row)), axis=1).astype(np.int32).ravel()
    g = CSRGraph(n_rows, N_COLS, (per_row * np.arange(n_rows + 1)).astype(np.int32), col, rng.standard_normal(col.shape[0]).astype(np.float32))
    assert has_panels(g, 64) == panels
    for d in (64, 130):
        X = rng.standard_normal((N_COLS, d)).astype(np.float32)
        Y, _ = gpu_spmm(g, X, mode)
        rows = np.arange(0, n_rows, 41)
        ref, bound = oracle_pair(g, X, rows=rows)
        assert_close(Y[rows], ref, bound, 1e-5, "communities of %d, d=%d" % (size, d))


@pytest.mark.parametrize("ykind", ["f32", "bf16"])
@pytest.mark.parametrize("relu", [False, True])
def test_layer_over_panels(ykind, relu):
    """X W first, then the panels: 16-bit results keep their sums in fp32 between panels and are rounded once."""
    import torch
    import paper_2412_08902_amd.binding as hc
    g = graph(700)
    rng = np.random.default_rng(4)
    X, W = rng.standard_normal((N_COLS, 20)).astype(np.float32), rng.standard_normal((20, 64)).astype(np.float32)
    plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *device_graph(g), d_hint=64)
    ws = torch.empty(hc.hcspmm_gcn_workspace_bytes(plan, 20, 64), dtype=torch.uint8, device="cuda")
    Y = torch.full((g.n_rows, 64), 3.0, dtype=torch.float32 if ykind == "f32" else torch_16(ykind), device="cuda")
    for _ in range(2):                                            # (the second call finds the row sums of the first)
        hc.hcspmm_gcn_layer_ex(plan, torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), Y, ws, apply_relu=relu)
    torch.cuda.synchronize()
    plan.destroy()
    T = X.astype(np.float64) @ W.astype(np.float64)
    ref, bound = np.zeros((g.n_rows, 64)), np.zeros((g.n_rows, 64))
    Ta = np.abs(X).astype(np.float64) @ np.abs(W).astype(np.float64)
    for r in range(g.n_rows):
        k = slice(g.rowptr[r], g.rowptr[r + 1])
        v = g.vals[k].astype(np.float64)
        ref[r], bound[r] = v @ T[g.colind[k]], np.abs(v) @ Ta[g.colind[k]]
    if relu:
        ref = np.maximum(ref, 0.0)
    if ykind == "f32":
        assert_close(Y.cpu().numpy().astype(np.float64), ref, bound, 1e-5, "layer")
    else:
        close_16(widen(from_dev_16(Y), ykind), ref, bound, 1e-5, ykind, "layer")


def test_update_of_a_plan_with_panels():
    """Edits that move rows between tiers and panels; the exported plan equals the re-derivation."""
    import paper_2412_08902_amd.binding as hc
    g = graph(300)
    plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *device_graph(g), d_hint=64)
    h = graph(300, seed=9)
    changed = np.array([0, 5, 17, 160, 299], np.int32)
    parts = [(h if r in changed else g) for r in range(300)]
    length = np.array([p.rowptr[r + 1] - p.rowptr[r] for r, p in enumerate(parts)])
    cut = lambda p, r, a: a[p.rowptr[r]:p.rowptr[r + 1]]
    g2 = CSRGraph(300, N_COLS, np.concatenate([[0], np.cumsum(length)]).astype(np.int32),
                  np.concatenate([cut(p, r, p.colind) for r, p in enumerate(parts)]).astype(np.int32),
                  np.concatenate([cut(p, r, p.vals) for r, p in enumerate(parts)]))
    update_and_check(plan, g2, changed, 0, d=64)
    plan.destroy()


@pytest.mark.parametrize("kind", ["bf16", "f16"])
@pytest.mark.parametrize("d,hint", [(128, 128), (64, 128), (256, 128)])
def test_16bit_outputs_keep_fp32_sums_between_panels(kind, d, hint):
    """16-bit X and Y: rounded once, the same bits from both entry points (the second allocates nothing), whatever ran before;
    a width beyond the plan's takes all columns at once.  The sums outlive an update."""
    import torch
    import paper_2412_08902_amd.binding as hc
    from workloads import to_f16_bits
    g = graph(300, times=3)
    x = np.random.default_rng(d).standard_normal((N_COLS, d)).astype(np.float32)
    bits, code = (to_bf16_bits(x), oracle.DT_BF16) if kind == "bf16" else (to_f16_bits(x), oracle.DT_F16)
    X = torch.from_numpy(bits.view(np.int16)).cuda().view(torch_16(kind))
    dev = device_graph(g)
    plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *dev, d_hint=hint, mfma_dtype=1 if kind == "bf16" else 2)
    ref, bound = oracle_pair(g, bits, x_dtype=code)
    for _ in range(2):
        Y, Z = (torch.full((g.n_rows, d), 3.0, dtype=torch_16(kind), device="cuda") for _ in range(2))
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        hc.hcspmm_spmm_noalloc(plan, X, Z)
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free
        hc.hcspmm_spmm(plan, X, Y)
        assert torch.equal(Y, Z)
        close_16(widen(from_dev_16(Y), kind), ref, bound, 1e-5, kind, "d=%d" % d)
        # a layer grows the sums for its own width; the products' route must not follow
        W = torch.eye(512, device="cuda")[:, :512]
        T = torch.empty((g.n_rows, 512), dtype=torch_16(kind), device="cuda")
        ws = torch.empty(hc.hcspmm_gcn_workspace_bytes(plan, 512, 512), dtype=torch.uint8, device="cuda")
        hc.hcspmm_gcn_layer_ex(plan, torch.zeros((N_COLS, 512), device="cuda"), W, T, ws, t_dtype=1 if kind == "bf16" else 2)
        hc.hcspmm_plan_update(plan, *dev, np.array([1, 2], np.int32))
    plan.destroy()
