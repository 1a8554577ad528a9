"""GPU parity of Y = act((A X) W) where the library computes act(A (X W)): widths and types on both sides of the rule, the
product with 16-bit X at its remainders, and the calls that keep the other order.  The route is read off the workspace, which
then starts with X W."""
import numpy as np
import pytest

import oracle
from workloads import CSRGraph, dense_normal, glorot_uniform, to_bf16_bits, to_f16_bits
from gpu_util import device_graph, assert_close

pytestmark = pytest.mark.gpu
KINDS = {"f32": (0, None), "bf16": (1, oracle.DT_BF16), "f16": (2, oracle.DT_F16)}


def graph(n_rows, n_cols, degree, seed):
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 2 * degree + 1, n_rows)
    lens[0] = min(n_cols, 3000)                                 # a long row of several segments, and empty rows
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colind = rng.integers(0, n_cols, rowptr[-1]).astype(np.int32)
    row = np.repeat(np.arange(n_rows), lens)
    colind = colind[np.lexsort((colind, row))]
    return CSRGraph(n_rows, n_cols, rowptr, colind, rng.uniform(-1, 1, len(colind)).astype(np.float32))


def run(g, X, W, kind, x_pad=0, x_off=0, relu=True, **options):
    """(Y, the workspace's first n_cols x d_out floats, reference, bound)"""
    import torch
    import paper_2412_08902_amd.binding as hc
    code, dt = KINDS[kind]
    bits = X if kind == "f32" else (to_bf16_bits if kind == "bf16" else to_f16_bits)(X)
    host = torch.from_numpy(bits if kind == "f32" else bits.view(np.int16))
    flat = torch.zeros(x_off + g.n_cols * (X.shape[1] + x_pad), dtype=host.dtype, device="cuda")
    Xd = torch.as_strided(flat, X.shape, (X.shape[1] + x_pad, 1), x_off)
    Xd.copy_(host)
    if kind != "f32":
        Xd = Xd.view(torch.bfloat16 if kind == "bf16" else torch.float16)
    plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *device_graph(g), d_hint=X.shape[1], mfma_dtype=code, **options)
    d_out = W.shape[1]
    ws = torch.zeros(hc.hcspmm_aggregate_update_workspace_bytes(plan, X.shape[1], d_out), dtype=torch.uint8, device="cuda")
    Y = torch.full((g.n_rows, d_out), -777.0, device="cuda")
    hc.hcspmm_aggregate_update(plan, Xd, torch.from_numpy(W).cuda(), Y, ws, apply_relu=relu)
    torch.cuda.synchronize()
    plan.destroy()
    T = ws.view(torch.float32)[: min(ws.numel() // 4, g.n_cols * d_out)].cpu().numpy()
    ref = oracle.aggregate_update(g.rowptr, g.colind, g.vals, bits, W, relu=relu, x_dtype=dt)
    bound = oracle.aggregate_update(g.rowptr, g.colind, g.vals, bits, W, relu=relu, x_dtype=dt, use_abs=True)
    XW = oracle.gemm(bits, W, x_dtype=dt)
    first = T.size == XW.size and np.allclose(T.reshape(XW.shape), XW, rtol=0, atol=1e-4 * np.abs(XW).max())
    return Y.cpu().numpy().astype(np.float64), first, ref, bound


# n_rows, degree, d_in, d_out, kind, taken
CASES = [(9000, 12, 32, 16, "f32", False),                      # one line either way
         (9000, 18, 38, 32, "f32", True), (9000, 30, 32, 32, "f32", False),         # ... and two, of narrower rows and of as wide ones
         (9000, 12, 64, 32, "f32", True), (9000, 18, 160, 128, "f32", True), (9000, 18, 144, 115, "f32", True),     # fewer loads of a row
         (9000, 18, 128, 96, "f32", False), (9000, 12, 128, 112, "f32", False), (9000, 18, 192, 160, "f32", False),    # as many
         (35_000, 5, 192, 160, "f32", True), (65000, 2, 192, 166, "f32", False),     # ... X of 24 MB; lines
         (65537, 2, 192, 146, "f32", True), (40_001, 4, 192, 146, "f32", False),     # ... of 48 MB for rows off the 16-byte pieces
         (8192, 30, 33, 7, "f32", True), (9000, 12, 160, 128, "f32", False), (9000, 5, 64, 32, "f32", False),   # too little to save
         (40001, 3, 64, 28, "f32", True), (40001, 3, 64, 33, "f32", False), (40001, 3, 144, 115, "f32", True), (40001, 3, 64, 64, "f32", False),
         (65537, 2, 128, 64, "bf16", True), (40001, 3, 128, 64, "bf16", False),      # as many lines: X of 16 MB
         (40001, 3, 128, 65, "f16", False), (90000, 2, 98, 47, "bf16", False), (40001, 3, 16, 8, "bf16", False),
         (40001, 3, 56, 11, "bf16", False), (40001, 3, 56, 12, "bf16", True),        # off the 16-byte pieces and on them
         (9000, 12, 128, 64, "bf16", False), (9000, 18, 128, 17, "bf16", True),
         # 16-bit X: K below, at and above the slabs and units of the product, ragged widths of W
         (9000, 18, 66, 3, "bf16", True), (9000, 12, 100, 1, "f16", True), (9000, 12, 131, 5, "bf16", True),
         (9000, 18, 160, 31, "f16", True), (9000, 18, 254, 62, "bf16", True), (9000, 12, 257, 47, "f16", True),
         # ... and with W in registers (from 65,536 rows on, or k n <= 1024)
         (65537, 2, 128, 64, "f16", True), (65537, 2, 100, 20, "bf16", True), (65537, 2, 84, 24, "bf16", True),
         (9000, 12, 80, 4, "bf16", True), (9000, 18, 68, 15, "f16", True),
         # bf16 X on the bf16 units, W in LDS (up to 256 of depth): from 16,384 rows on, one column tile from 49,152; K around its slabs, ends of tiles
         (16383, 18, 256, 64, "bf16", True), (16384, 18, 256, 64, "bf16", True), (16385, 18, 250, 64, "bf16", True), (16399, 18, 191, 33, "bf16", True),
         (49151, 12, 128, 16, "bf16", True), (49153, 12, 128, 15, "bf16", True), (16400, 18, 222, 80, "bf16", True), (49185, 3, 96, 1, "bf16", True),
         # ... the same from 65,536 rows on, and the last two beyond 256 of depth: K around the slabs of 32, one to four column tiles, two groups of them
         (65600, 2, 130, 47, "bf16", True), (65536, 2, 65, 16, "bf16", True),
         (65541, 2, 159, 31, "bf16", True), (65536, 2, 288, 95, "bf16", True), (65537, 2, 322, 128, "bf16", True)]


@pytest.mark.parametrize("n_rows,degree,d_in,d_out,kind,taken", CASES)
def test_both_sides_of_the_rule(n_rows, degree, d_in, d_out, kind, taken):
    g = graph(n_rows, n_rows, degree, seed=d_in + d_out)
    X, W = dense_normal(n_rows, d_in, seed=1), glorot_uniform(d_in, d_out, seed=2)
    pad = d_in % 2                                              # rows of 16-bit X on whole words
    Y, first, ref, bound = run(g, X, W, kind, x_pad=pad, relu=d_out % 2 == 0, route_mode=1)
    assert first == taken
    assert_close(Y, ref, bound, 1e-5)


@pytest.mark.parametrize("d_in,d_out,mode,taken", [
    (80, 45, 1, True), (80, 45, 2, False),                      # 45 columns value by value take two walks over the windows
    (128, 112, 1, False), (132, 128, 2, True),                  # ... and so do 132 in pieces of four
    (63, 48, 1, False), (63, 48, 2, True), (64, 48, 2, False)])  # as many walks and loads
def test_walks_over_matrix_path_windows(d_in, d_out, mode, taken):
    g = graph(9000, 9000, 18, seed=d_in)
    X, W = dense_normal(9000, d_in, seed=1), glorot_uniform(d_in, d_out, seed=2)
    Y, first, ref, bound = run(g, X, W, "f32", route_mode=mode)
    assert first == taken
    assert_close(Y, ref, bound, 1e-5)


@pytest.mark.parametrize("d_in,d_out,apart", [(80, 97, False), (96, 97, True), (96, 98, False)])
def test_odd_widths_of_w_and_the_product_in_the_windows(d_in, d_out, apart):
    """A X reaches the workspace only where the product is a launch of its own."""
    import torch
    import paper_2412_08902_amd.binding as hc
    g = graph(9000, 9000, 8, seed=d_in)
    X, W = dense_normal(9000, d_in, seed=1), glorot_uniform(d_in, d_out, seed=2)
    plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *device_graph(g), d_hint=d_in, route_mode=2)
    assert 2 * hc.hcspmm_plan_info(plan)["n_mfma_small"] > hc.hcspmm_plan_info(plan)["n_windows"]
    ws = torch.zeros(hc.hcspmm_aggregate_update_workspace_bytes(plan, d_in, d_out), dtype=torch.uint8, device="cuda")
    Y = torch.empty((9000, d_out), device="cuda")
    hc.hcspmm_aggregate_update(plan, torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(), Y, ws, apply_relu=True)
    torch.cuda.synchronize()
    plan.destroy()
    Z = ws.view(torch.float32)[:9000 * d_in].cpu().numpy().reshape(9000, d_in)
    AX = oracle.spmm(g.rowptr, g.colind, g.vals, X)
    assert np.allclose(Z, AX, rtol=0, atol=1e-4 * np.abs(AX).max()) == apart
    args = (g.rowptr, g.colind, g.vals, X, W)
    assert_close(Y.cpu().numpy().astype(np.float64), oracle.aggregate_update(*args, relu=True), oracle.aggregate_update(*args, relu=True, use_abs=True), 1e-5)


@pytest.mark.parametrize("kind,n_rows,n_cols,x_pad,x_off,options", [
    ("f32", 9000, 9001, 0, 0, {}),                              # X W would be larger than the other order's rows
    ("bf16", 9000, 9000, 1, 0, {}), ("f16", 9000, 9000, 0, 1, {}),      # X off the 4-byte words
    ("f32", 9000, 9000, 0, 0, {"update_fusion": 1}), ("f32", 9000, 9000, 0, 0, {"update_fusion": 2}),
    ("f32", 9000, 1000, 1, 1, {}), ("bf16", 9000, 1000, 2, 2, {})])
def test_calls_that_keep_their_order(kind, n_rows, n_cols, x_pad, x_off, options):
    g = graph(n_rows, n_cols, 12, seed=5)
    X, W = dense_normal(n_cols, 128, seed=1), glorot_uniform(128, 16, seed=2)
    Y, first, ref, bound = run(g, X, W, kind, x_pad=x_pad, x_off=x_off, route_mode=1, **options)
    assert first == (n_cols == 1000)                            # the last two are taken
    assert_close(Y, ref, bound, 1e-5)


def test_rows_that_would_become_wider_keep_their_order():
    """63 fp32 values off the 128-byte lines, and 64 of them on two lines: partial sums grow with the width, not with the lines."""
    g = graph(9000, 1000, 12, seed=5)
    X, W = dense_normal(1000, 63, seed=1), glorot_uniform(63, 64, seed=2)
    Y, first, ref, bound = run(g, X, W, "f32", route_mode=1)
    assert not first
    assert_close(Y, ref, bound, 1e-5)


def test_infinities_and_nan_in_bf16_products():
    """Y = I (X W): an infinity meets the zero remainders of split values nowhere, a NaN stays one.  (Sixteen entries of a
    sixteenth to a row of I: the aggregation multiplies a row's last X row with zeros where its last batch is not full.)"""
    import torch
    import paper_2412_08902_amd.binding as hc
    n, d_in, d_out = 65600, 130, 60
    dev = "cuda"
    ip = torch.arange(0, 16 * n + 1, 16, dtype=torch.int32, device=dev)
    ci, va = torch.arange(n, dtype=torch.int32, device=dev).repeat_interleave(16), torch.full((16 * n,), 1 / 16, device=dev)
    torch.manual_seed(3)
    X, W = torch.randn(n, d_in).bfloat16(), torch.randn(d_in, d_out)
    W[7, 3] = 0.5                                               # a value whose remainders are zero
    X[5, 7], X[77, 129], X[65599, 0], X[200, 64] = float("inf"), float("-inf"), float("nan"), torch.finfo(torch.bfloat16).max
    for w_at in (None, (40, 11), (129, 59)):
        if w_at:
            W[w_at] = float("inf") if w_at[0] == 40 else torch.finfo(torch.float32).max
        plan = hc.hcspmm_prepare(n, n, ip, ci, va, route_mode=1, d_hint=d_in, mfma_dtype=1)
        ws = torch.empty(hc.hcspmm_aggregate_update_workspace_bytes(plan, d_in, d_out), dtype=torch.uint8, device=dev)
        Y = torch.zeros(n, d_out, device=dev)
        hc.hcspmm_aggregate_update(plan, X.cuda(), W.cuda(), Y, ws, apply_relu=False)
        torch.cuda.synchronize()
        plan.destroy()
        got, want = Y.cpu().double(), X.double() @ W.double()
        want = want.float().double()                            # (what overflows fp32 is an infinity)
        assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf())
        assert torch.equal(got[want.isinf()], want[want.isinf()])
        fin = want.isfinite()
        bound = (X.double().abs() @ W.double().abs())[fin]
        assert torch.all((got[fin] - want[fin]).abs() <= 1e-5 * bound)


def test_bits_beside_an_infinity_do_not_depend_on_timing():
    """An infinity in one column of W takes its slab and those behind it to the fp32 units, in every wave alike: rows that are equal
    have equal results, wherever they are multiplied."""
    import torch
    import paper_2412_08902_amd.binding as hc
    n, d_in, d_out = 80000, 256, 64
    ip = torch.arange(0, 16 * n + 1, 16, dtype=torch.int32, device="cuda")
    ci, va = torch.arange(n, dtype=torch.int32, device="cuda").repeat_interleave(16), torch.full((16 * n,), 1 / 16, device="cuda")
    torch.manual_seed(5)
    X, W = torch.randn(16, d_in).bfloat16().cuda().repeat(n // 16, 1), torch.randn(d_in, d_out).cuda()
    W[100, 11] = float("inf")
    plan = hc.hcspmm_prepare(n, n, ip, ci, va, route_mode=1, d_hint=d_in, mfma_dtype=1)
    ws = torch.empty(hc.hcspmm_aggregate_update_workspace_bytes(plan, d_in, d_out), dtype=torch.uint8, device="cuda")
    Y = torch.empty(n, d_out, device="cuda")
    hc.hcspmm_aggregate_update(plan, X, W, Y, ws, apply_relu=False)
    torch.cuda.synchronize()
    plan.destroy()
    T = ws[:4 * n * d_out].view(torch.int32).view(n // 16, 16, d_out)          # X W, as bits
    finite = torch.arange(d_out, device="cuda") != 11
    assert torch.equal(T[:, :, finite], T[:1, :, finite].expand(n // 16, -1, -1))
    assert bool(T.view(torch.float32)[:, :, 11].isinf().all())
    want = X[:16].double() @ W[:, finite].double()
    assert torch.all((T[0][:, finite].view(torch.float32).double() - want).abs() <= 1e-5 * (X[:16].double().abs() @ W[:, finite].double().abs()))
