"""Preparation at the edges of its size classes and tiles, against the CPU re-derivation, and the row tables through the product."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, device_graph
from test_gpu_plan import KEYS, check_plan
from workloads import CSRGraph

pytestmark = pytest.mark.gpu


def ragged(lengths, n_cols, seed):
    rng = np.random.default_rng(seed)
    lengths = np.asarray(lengths, np.int64)
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    col = rng.integers(0, n_cols, int(lengths.sum()))
    rows = np.repeat(np.arange(lengths.shape[0]), lengths)
    col = col[np.lexsort((col, rows))].astype(np.int32)           # ascending inside a row; duplicates stay
    return CSRGraph(lengths.shape[0], n_cols, rowptr, col, rng.standard_normal(col.shape[0]).astype(np.float32))


@pytest.mark.parametrize("per_window", [1023, 1024, 1025, 4095, 4096, 4097, 16384, 16385])
@pytest.mark.parametrize("mode", [0, 2])
def test_windows_around_the_counting_classes(per_window, mode):
    lengths = np.zeros(16 * 5, np.int64)
    for w in (0, 2, 4):
        lengths[16 * w: 16 * w + 15] = per_window // 15
        lengths[16 * w + 15] = per_window - 15 * (per_window // 15)
    check_plan(ragged(lengths, 20_000, per_window), mode, sel_coef=[1, 300, -200])


@pytest.mark.parametrize("n", [1, 15, 16, 1023, 1024, 1025, 4 * 1024, 4 * 1024 + 1, 70_001])
@pytest.mark.parametrize("mode", [0, 1, 3])
def test_tiles_of_rows_and_their_tables(n, mode):
    rng = np.random.default_rng(n)
    lengths = rng.integers(0, 6, n)
    heavy = rng.choice(n, min(n, 40), replace=False)
    lengths[heavy] = rng.choice([60, 64, 65, 128, 129, 256, 257, 1024, 1025, 2048, 2049, 5000], heavy.shape[0])
    g = ragged(lengths, 3000, n)
    import torch
    import paper_2412_08902_amd.binding as hc
    check_plan(g, mode, sel_coef=[1, 300, -280])
    X = rng.standard_normal((g.n_cols, 32)).astype(np.float32)
    W = rng.standard_normal((32, 16)).astype(np.float32)
    plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *device_graph(g), route_mode=mode, sel_coef=[1, 300, -280])
    Xd, Wd = torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda()
    Y = torch.full((n, 32), float("nan"), device="cuda")
    hc.hcspmm_spmm(plan, Xd, Y)
    ref, bound = (oracle.spmm(g.rowptr, g.colind, g.vals, X, use_abs=b) for b in (False, True))
    assert_close(Y.cpu().numpy().astype(np.float64), ref, bound, 1e-5, "spmm")
    # the fused layer walks the rest_rows table as well
    hc.hcspmm_plan_set_update_fusion(plan, hc.HCSPMM_UPDATE_FUSED)
    ws = torch.empty(max(256, hc.hcspmm_aggregate_update_workspace_bytes(plan, 32, 16)), dtype=torch.uint8, device="cuda")
    Z = torch.full((n, 16), float("nan"), device="cuda")
    hc.hcspmm_aggregate_update(plan, Xd, Wd, Z, ws)
    ref, bound = (oracle.aggregate_update(g.rowptr, g.colind, g.vals, X, W, use_abs=b) for b in (False, True))
    assert_close(Z.cpu().numpy().astype(np.float64), ref, bound, 1e-5, "aggregate-update")


@pytest.mark.parametrize("where", ["first", "middle", "last"])
@pytest.mark.parametrize("bad", [-1, 300])
def test_bad_columns_are_found_in_every_size_class(where, bad):
    import paper_2412_08902_amd.binding as hc
    for per_row in (3, 100, 500, 1100):                           # windows of 48, 1600, 8000 and 17600 non-zeros
        g = ragged(np.full(48, per_row), 300, per_row)
        col = g.colind.copy()
        col[{"first": 0, "middle": col.shape[0] // 2, "last": -1}[where]] = bad
        for mode in (0, 1):
            with pytest.raises(hc.HcspmmError) as e:
                hc.hcspmm_prepare(g.n_rows, g.n_cols, *device_graph(CSRGraph(48, 300, g.rowptr, col, g.vals)), route_mode=mode)
            assert e.value.status == hc.HCSPMM_EBADCSR


def test_update_of_more_windows_than_the_pinned_list_holds():
    """16,000 changed rows, each in a window of its own, of 2.1 M rows: equal to a preparation from scratch."""
    import torch
    import paper_2412_08902_amd.binding as hc
    n = 2_100_000
    rng = np.random.default_rng(5)
    rowptr = np.arange(n + 1, dtype=np.int32)
    col = rng.integers(0, 1000, n).astype(np.int32)
    rows = (np.arange(16_000) * 128 + 5).astype(np.int32)
    col2 = col.copy()
    col2[rows] += 1
    va = torch.ones(n, device="cuda")
    rp, c1, c2 = (torch.from_numpy(x).cuda() for x in (rowptr, col, col2))
    plan = hc.hcspmm_prepare(n, 1002, rp, c1, va)
    hc.hcspmm_plan_update(plan, rp, c2, va, rows)
    fresh = hc.hcspmm_prepare(n, 1002, rp, c2, va)
    a, b = hc.hcspmm_plan_export(plan), hc.hcspmm_plan_export(fresh)
    for k in KEYS:
        assert np.array_equal(a[k], b[k]), k


# one row behind the last matrix whose tiles of 1024 rows are added up directly, and whole and ragged groups of 256 tiles
@pytest.mark.parametrize("n", [4096 * 1024, 4096 * 1024 + 1, 4352 * 1024 + 17])
def test_more_tiles_than_are_added_up_directly(n):
    import torch
    import paper_2412_08902_amd.binding as hc
    rng = np.random.default_rng(n)
    lengths = rng.integers(0, 3, n)
    heavy = rng.choice(n, 3000, replace=False)
    lengths[heavy] = rng.choice([128, 129, 257, 1024, 1025, 2049], heavy.shape[0])
    g = ragged(lengths, 5000, n)
    coef = [1, 300, -300]                                         # both routes get about half of the windows
    check_plan(g, 3, sel_coef=coef)
    X = rng.standard_normal((g.n_cols, 4)).astype(np.float32)
    plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *device_graph(g), route_mode=3, sel_coef=coef)
    assert min(hc.hcspmm_plan_info(plan)[k] for k in ("n_mfma_small", "n_mid_rows", "n_long_rows", "n_short_rows")) > 0
    Y = torch.full((n, 4), float("nan"), device="cuda")
    hc.hcspmm_spmm(plan, torch.from_numpy(X).cuda(), Y)
    ref, bound = (oracle.spmm(g.rowptr, g.colind, g.vals, X, use_abs=b) for b in (False, True))
    assert_close(Y.cpu().numpy().astype(np.float64), ref, bound, 1e-5, "spmm")


def test_panels_of_more_tiles_than_are_added_up_directly():
    """4.2 M rows of 150 non-zeros (631 M in all) in column panels: short rows, rows that lie in one panel, rows of several
    segments; sampled rows in 64 bits."""
    import torch
    import paper_2412_08902_amd.binding as hc
    n, n_cols, d = 4097 * 1024 + 5, 120_000, 32
    length = torch.full((n,), 150, dtype=torch.int64, device="cuda")
    length[::40_000] = 3000
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(length, 0, out=rowptr[1:])
    col = torch.empty(int(rowptr[-1]), dtype=torch.int32, device="cuda")
    for r0 in range(0, n, 1 << 20):                               # (in pieces: a 64-bit row number per non-zero is 5 GB)
        r = torch.arange(r0, min(n, r0 + (1 << 20)), device="cuda")
        row = r.repeat_interleave(length[r])
        j = torch.arange(int(rowptr[r[0]]), int(rowptr[r[-1] + 1]), device="cuda") - rowptr[row]
        step = torch.where(length[row] == 3000, 40, torch.where(row % 97 == 0, 150, 800))
        col[int(rowptr[r[0]]):int(rowptr[r[-1] + 1])] = (j * step + (row * 7 + j * 13) % step).to(torch.int32)
    vals = torch.rand(col.numel(), device="cuda") - 0.5
    rp = rowptr.to(torch.int32)
    X = torch.randn((n_cols, d), device="cuda")
    Y = torch.full((n, d), float("nan"), device="cuda")
    plan = hc.hcspmm_prepare(n, n_cols, rp, col, vals, route_mode=1, d_hint=d)
    hc.hcspmm_spmm(plan, X, Y)
    sample = torch.cat([torch.arange(0, n, 40_000), torch.arange(0, n, 97 * 331), torch.arange(3, n, 9973), torch.arange(n - 40, n)]).unique().cuda()
    for r in sample.split(512):
        row = torch.arange(r.numel(), device="cuda").repeat_interleave(length[r])
        first = torch.cumsum(length[r], 0) - length[r]
        k = rowptr[r][row] + torch.arange(row.numel(), device="cuda") - first[row]
        terms = vals[k].double()[:, None] * X[col[k].long()].double()
        ref = torch.zeros((r.numel(), d), dtype=torch.float64, device="cuda").index_add_(0, row, terms)
        bound = torch.zeros_like(ref).index_add_(0, row, terms.abs())
        assert_close(Y[r].double().cpu().numpy(), ref.cpu().numpy(), bound.cpu().numpy(), 1e-5, "panels")
    assert torch.isfinite(Y).all()


# 1.2 M non-zeros: a scalar-only preparation samples the columns beside its check of them
@pytest.mark.parametrize("community", [500, 40_000])
def test_scalar_only_plans_that_sample_their_columns(community):
    import torch
    import paper_2412_08902_amd.binding as hc
    n, per_row = 40_000, 30
    rng = np.random.default_rng(community)
    first = np.arange(n) // community * community
    col = np.sort(first[:, None] + rng.integers(0, community, (n, per_row)), axis=1).astype(np.int32).ravel()
    g = CSRGraph(n, n, (per_row * np.arange(n + 1)).astype(np.int32), col, rng.standard_normal(col.shape[0]).astype(np.float32))
    check_plan(g, 1)
    X = rng.standard_normal((n, 128)).astype(np.float32)
    plan = hc.hcspmm_prepare(n, n, *device_graph(g), route_mode=1, d_hint=128)
    Y = torch.full((n, 128), float("nan"), device="cuda")
    hc.hcspmm_spmm(plan, torch.from_numpy(X).cuda(), Y)
    rows = np.arange(0, n, 53)
    ref, bound = (oracle.spmm_rows(rows, g.rowptr, g.colind, g.vals, X, None, use_abs=b) for b in (False, True))
    assert_close(Y.cpu().numpy()[rows].astype(np.float64), ref, bound, 1e-5, "spmm")
    for at in (0, col.shape[0] // 2, col.shape[0] - 1):
        for bad in (-1, n):
            c = col.copy()
            c[at] = bad
            with pytest.raises(hc.HcspmmError) as e:
                hc.hcspmm_prepare(n, n, *device_graph(CSRGraph(n, n, g.rowptr, c, g.vals)), route_mode=1)
            assert e.value.status == hc.HCSPMM_EBADCSR


def test_plan_info_tells_windows_that_the_scalar_path_has_taken_over():
    """The canonical plan keeps its routes; the launch tables say that no matrix-path kernel runs."""
    import paper_2412_08902_amd.binding as hc
    from test_gpu_runs import scattered_windows
    g = scattered_windows()
    dev = device_graph(g)
    for kernels, runs in ((hc.HCSPMM_MATRIX_AUTO, False), (hc.HCSPMM_MATRIX_PER_WINDOW, True)):
        plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *dev, d_hint=128, mfma_dtype=1, matrix_kernels=kernels)
        info = hc.hcspmm_plan_info(plan)
        assert info["n_mfma_windows"] > 900 and (info["n_mfma_small"] + info["n_mfma_big"] == info["n_mfma_windows"]) == runs
        assert runs or info["n_mfma_small"] + info["n_mfma_big"] == 0
        assert hc.hcspmm_plan_export(plan)["route"].sum() == info["n_mfma_windows"]
        plan.destroy()


def mixed_sizes(n, seed, per_class=3, n_cols=3000):
    """Mostly small windows; some around every counting class, next to each other and far apart; rows of every tier."""
    rng = np.random.default_rng(seed)
    lengths = rng.integers(0, 7, n)
    windows = rng.permutation(n // 16)
    sizes = [1024, 1025, 4096, 4097, 8192, 8193, 16384, 16385]
    for i, size in enumerate(np.repeat(sizes, per_class)[: windows.shape[0] // 2]):
        w = windows[i] if i % 2 else min(i, n // 16 - 1)
        lengths[16 * w: 16 * w + 15] = size // 15
        lengths[16 * w + 15] = size - 15 * (size // 15)
    return ragged(lengths, n_cols, seed)


# one, two and four windows to a workgroup, whole and ragged; the last matrices whose windows one launch counts and the first beyond, by rows and
# by columns (one pass of the bitmap, two, and the classes)
@pytest.mark.parametrize("n,n_cols", [(2000, 3000), (16 * 513, 3000), (16 * 1021, 3000), (2048 * 16, 3000), (2048 * 16 + 1, 3000),
                                      (3000, 1 << 19), (3000, (1 << 19) + 1), (3000, 1 << 20), (3000, (1 << 20) + 1)])
@pytest.mark.parametrize("mode", [0, 3])
def test_one_launch_counts_few_windows_of_every_size(n, n_cols, mode):
    import torch
    import paper_2412_08902_amd.binding as hc
    g = mixed_sizes(n, n, n_cols=n_cols)
    coef = [1, 300, -328]                                         # (windows of up to some 47 columns on the matrix path)
    check_plan(g, mode, sel_coef=coef)
    plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *device_graph(g), route_mode=mode, sel_coef=coef)
    X = np.random.default_rng(n).standard_normal((g.n_cols, 8)).astype(np.float32)
    Y = torch.full((n, 8), float("nan"), device="cuda")
    hc.hcspmm_spmm(plan, torch.from_numpy(X).cuda(), Y)
    ref, bound = (oracle.spmm(g.rowptr, g.colind, g.vals, X, use_abs=b) for b in (False, True))
    assert_close(Y.cpu().numpy().astype(np.float64), ref, bound, 1e-5, "spmm")


@pytest.mark.parametrize("n,every", [(30_000, 16), (70_000, 16), (70_000, 400)])
def test_updates_that_touch_every_size_class(n, every):
    """Windows of every counting class among the touched ones, counted by one launch (up to 2,048) or by class."""
    import torch
    import paper_2412_08902_amd.binding as hc
    g = mixed_sizes(n, n, 4)
    rows = np.flatnonzero((np.arange(n) % every == 0) | (np.diff(g.rowptr) > 60))
    rows = rows[np.diff(g.rowptr)[rows] > 0].astype(np.int32)
    col2 = g.colind.copy()
    last = g.rowptr[rows + 1] - 1
    col2[last] = 3000 + rows % 5                                  # (rows stay ascending)
    rp, c1, c2, va = (torch.from_numpy(a).cuda() for a in (g.rowptr, g.colind, col2, g.vals))
    plan = hc.hcspmm_prepare(n, 3005, rp, c1, va)
    hc.hcspmm_plan_update(plan, rp, c2, va, rows)
    a, b = hc.hcspmm_plan_export(plan), hc.hcspmm_plan_export(hc.hcspmm_prepare(n, 3005, rp, c2, va))
    for k in KEYS:
        assert np.array_equal(a[k], b[k]), k


# the launch for few windows: fewer of them than the workgroups for the larger ones, as many, and up to 32 to each of these; columns around one, two and
# four passes of their bitmap
@pytest.mark.parametrize("n,n_cols", [(16 * 63, 1 << 18), (16 * 64, (1 << 18) + 1), (16 * 65, 65_537), (2047 * 16 + 3, 1 << 18), (3000, 3 << 18), (3000, (3 << 18) + 1)])
def test_larger_windows_of_few(n, n_cols):
    check_plan(mixed_sizes(n, n, n_cols=n_cols), 3, sel_coef=[1, 300, -328])


@pytest.mark.parametrize("row", [0, 1, 700, 1599, 1600])
@pytest.mark.parametrize("value", [-5, 1 << 30])
def test_unsound_offsets_of_few_windows(row, value):
    """No offset leads a window's reads outside the arrays, and the error is the offsets', whatever the columns hold."""
    import torch
    import paper_2412_08902_amd.binding as hc
    g = ragged(np.full(1600, 90), 300, row)
    col = g.colind.copy()
    col[::997] = 300
    rp, ci, va = device_graph(CSRGraph(1600, 300, g.rowptr, col, g.vals))
    rp[row] = value
    with pytest.raises(hc.HcspmmError) as e:
        hc.hcspmm_prepare(1600, 300, rp, ci, va)
    assert e.value.status == hc.HCSPMM_EBADCSR and "rowptr" in str(e.value) and "column" not in str(e.value)


# more workgroups for the larger windows where a matrix has many of them: 256 from 257 non-zeros per window on, 512 from 1,025 on; fewer windows than those,
# as many, and several to a workgroup, with small and empty ones between
@pytest.mark.parametrize("per_window", [256, 257, 1024, 1025, 2500])
@pytest.mark.parametrize("windows", [63, 256, 257, 513, 1100])
def test_many_larger_windows(per_window, windows):
    rng = np.random.default_rng(windows + per_window)
    share = rng.choice([0.0, 0.3, 1.0, 1.7], windows)
    sizes = np.floor(share * per_window).astype(np.int64)
    sizes[-1] = max(0, per_window * windows - sizes[:-1].sum())   # exactly the average
    while sizes.sum() > per_window * windows:
        big = sizes.argmax()
        sizes[big] -= min(sizes[big], sizes.sum() - per_window * windows)
    lengths = np.repeat(sizes // 16, 16)
    lengths[::16] += sizes % 16
    check_plan(ragged(lengths, 5000, windows), 3, sel_coef=[1, 300, -328])
