"""GPU parity of Y = act(A (X W)) where the library computes act((A X) W): widths on both sides of the rule, each place that the
update can take, and the calls that keep their order.  The route is read off the workspace, which starts with X W when that came
first."""
import numpy as np
import pytest

import oracle
from workloads import dense_normal, glorot_uniform
from gpu_util import assert_close, device_graph
from test_gpu_update_first import graph

pytestmark = pytest.mark.gpu


def run(g, d_in, d_out, x_pad=0, x_off=0, y="f32", t=0, relu=True, **options):
    import torch
    import paper_2412_08902_amd.binding as hc
    X, W = dense_normal(g.n_cols, d_in, seed=1), glorot_uniform(d_in, d_out, seed=2)
    flat = torch.zeros(x_off + g.n_cols * (d_in + x_pad), device="cuda")
    Xd = torch.as_strided(flat, X.shape, (d_in + x_pad, 1), x_off)
    Xd.copy_(torch.from_numpy(X))
    plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *device_graph(g), d_hint=d_out, **options)
    need = hc.hcspmm_gcn_workspace_bytes(plan, d_in, d_out)
    ws = torch.zeros(need + 1024, dtype=torch.uint8, device="cuda")
    ws[need:] = 77
    Y = torch.full((g.n_rows, d_out), -777.0, device="cuda").to({"f32": torch.float32, "bf16": torch.bfloat16}[y])
    hc.hcspmm_gcn_layer_ex(plan, Xd, torch.from_numpy(W).cuda(), Y, ws[:need], t_dtype=t, apply_relu=relu)
    torch.cuda.synchronize()
    plan.destroy()
    assert bool((ws[need:] == 77).all())
    ref = oracle.gcn_layer(g.rowptr, g.colind, g.vals, X, W, relu=relu)
    bound = oracle.gcn_layer(g.rowptr, g.colind, g.vals, X, W, relu=relu, use_abs=True)
    XW = oracle.gemm(X, W)
    T = ws[:4 * XW.size].view(torch.float32).cpu().numpy().reshape(XW.shape)
    return Y.float().cpu().numpy().astype(np.float64), np.allclose(T, XW, rtol=0, atol=1e-4 * np.abs(XW).max()), ref, bound


# n_rows, degree, d_in, d_out, X W first
CASES = [(300, 5, 8, 16, False), (300, 5, 32, 144, False), (300, 5, 1, 32, True), (2000, 9, 96, 173, False),     # in one pass
         (2000, 60, 32, 96, True), (6000, 60, 32, 144, False),      # ... with hubs, less and more than it costs
         (20_001, 12, 16, 32, False), (20_001, 12, 40, 188, False), (20_001, 12, 33, 70, False), (20_001, 12, 150, 300, False),
         (20_001, 12, 128, 160, False), (20_001, 12, 300, 602, False),
         # as many loads of a row, and nearly as many lines: X W of 48 MB
         (8_000, 12, 256, 300, True), (20_001, 12, 256, 300, False), (20_001, 12, 163, 200, True), (70_001, 3, 163, 200, False),
         (8_000, 12, 96, 128, True), (20_001, 12, 96, 128, False),
         # ... off the 16-byte pieces
         (20_001, 12, 11, 21, True), (20_001, 12, 9, 27, True), (20_001, 12, 9, 64, False), (20_001, 12, 11, 40, False),
         # ... on the pieces where X W is off them
         (20_001, 12, 200, 223, False), (20_001, 12, 212, 223, True),
         # ... of several lines and more than a few thousand, in no larger pieces or short
         (20_001, 12, 160, 224, False), (20_001, 12, 161, 224, True), (8_192, 12, 160, 224, True), (20_001, 12, 33, 50, False),
         # as many lines, or more
         (20_001, 12, 32, 32, True), (20_001, 12, 48, 64, True), (20_001, 12, 15, 16, True), (20_001, 12, 167, 176, True),
         (20_001, 12, 64, 32, True), (20_001, 12, 9, 16, True)]


@pytest.mark.parametrize("mode", [0, 1, 3])
@pytest.mark.parametrize("n,degree,d_in,d_out,first", CASES)
def test_both_sides_of_the_rule(n, degree, d_in, d_out, first, mode):
    options = {"sel_coef": [1, 300, -280]} if mode == 3 else {}   # (mode 3: some windows on the matrix path)
    Y, got, ref, bound = run(graph(n, n, degree, seed=d_in + d_out), d_in, d_out, relu=d_out % 2 == 0, route_mode=mode, **options)
    assert got == first
    assert_close(Y, ref, bound, 1e-5)


@pytest.mark.parametrize("d_in,d_out,mode,first", [
    (41, 80, 1, False), (41, 80, 2, True),                      # 41 columns value by value take two walks over the windows, 80 in fours one
    (51, 69, 2, False), (160, 223, 2, False),                   # ... one against two; two against four
    (112, 128, 2, True), (64, 192, 2, False)])                  # as many walks
def test_walks_over_matrix_path_windows(d_in, d_out, mode, first):
    Y, got, ref, bound = run(graph(9000, 9000, 12, seed=d_in + d_out), d_in, d_out, route_mode=mode)
    assert got == first
    assert_close(Y, ref, bound, 1e-5)


def test_narrower_rows_that_touch_more_lines_keep_their_order():
    """Rows of 63 fp32 values off the 128-byte lines touch more of them than rows of 64 (2.94 against 2); the scratch of a product grows
    with its width, so that a call whose rows would become wider keeps the order that it was made room for."""
    Y, got, ref, bound = run(graph(2000, 9000, 12, seed=3), 64, 63, route_mode=1)
    assert got
    assert_close(Y, ref, bound, 1e-5)


@pytest.mark.parametrize("n_rows,n_cols,x_pad,x_off,options,first", [
    (9000, 2000, 0, 0, {}, True),                               # A X has no room in the workspace
    (2000, 9000, 0, 0, {}, False), (9000, 9000, 1, 1, {}, False),
    (9000, 9000, 0, 0, {"update_fusion": 1}, True), (9000, 9000, 0, 0, {"update_fusion": 2}, True),
    (9000, 9000, 0, 0, {"t": 1}, True)])                        # T in bf16 is the caller's choice
def test_calls_with_a_reason_of_their_own(n_rows, n_cols, x_pad, x_off, options, first):
    if options.get("t"):
        g = graph(n_rows, n_cols, 12, seed=3)
        Y, got, _, bound = run(g, 32, 96, route_mode=1, **options)
        X, W = dense_normal(n_cols, 32, seed=1), glorot_uniform(32, 96, seed=2)
        ref = oracle.gcn_layer(g.rowptr, g.colind, g.vals, X, W, t_dtype=oracle.DT_BF16)
        assert not got                                          # (fp32 X W is not what the workspace holds)
        assert_close(Y, ref, bound, 2.0 ** -8)
        return
    Y, got, ref, bound = run(graph(n_rows, n_cols, 12, seed=3), 32, 96, x_pad=x_pad, x_off=x_off, route_mode=1, **options)
    assert got == first
    assert_close(Y, ref, bound, 1e-5)


def test_16_bit_results_round_once():
    Y, got, ref, bound = run(graph(9000, 9000, 12, seed=3), 32, 96, y="bf16", route_mode=1)
    assert not got
    assert np.all(np.abs(Y - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5 * bound)


@pytest.mark.parametrize("n", [1500, 20_001])                   # in one pass and apart, where the library has the choice
@pytest.mark.parametrize("over,first", [("X", True), ("the last value of X", True), ("W", True), ("nothing", False)])
@pytest.mark.parametrize("mode", [1, 2])
def test_results_over_the_inputs(n, over, first, mode):
    """Y in the memory of X or of W: X W is complete before anything is stored, and the bits are those of that order."""
    import torch
    import paper_2412_08902_amd.binding as hc
    d_in, d_out = 32, 96
    g = graph(n, n, 12, seed=4)
    X, W = dense_normal(n, d_in, seed=1), glorot_uniform(d_in, d_out, seed=2)
    dev, X_size = device_graph(g), n * d_in

    def run(over, fusion):
        flat = torch.full((X_size + n * d_out,), -777.0, device="cuda")
        Y = flat[X_size:].view(n, d_out)
        Xd, Wd = flat[:X_size].view(n, d_in), torch.empty((d_in, d_out), device="cuda")         # X ends where Y begins
        if over == "X":
            Xd = Y[:, :d_in]
        elif over == "the last value of X":
            Y = flat[X_size - 1:-1].view(n, d_out)
        elif over == "W":
            Wd = Y[n - d_in:]
        Xd.copy_(torch.from_numpy(X))
        Wd.copy_(torch.from_numpy(W))
        plan = hc.hcspmm_prepare(n, n, *dev, route_mode=mode, d_hint=d_out, update_fusion=fusion)
        ws = torch.zeros(hc.hcspmm_gcn_workspace_bytes(plan, d_in, d_out), dtype=torch.uint8, device="cuda")
        hc.hcspmm_gcn_layer(plan, Xd, Wd, Y, ws)
        torch.cuda.synchronize()
        plan.destroy()
        return Y.cpu().numpy(), ws[:4 * n * d_out].view(torch.float32).cpu().numpy()

    want, XW = run("nothing", 2)
    Y, T = run(over, 0)
    assert np.array_equal(T, XW) == first
    assert not first or np.array_equal(Y, want)
    ref, bound = (oracle.gcn_layer(g.rowptr, g.colind, g.vals, X, W, use_abs=b) for b in (False, True))
    assert_close(Y.astype(np.float64), ref, bound, 1e-5)
