"""Scratch of the layer calls follows from the shapes, not from where X lies: the order of the two products goes by X's base and
pitch, so a call may take one order and a later one of the same shapes the other, under capture too."""
import numpy as np
import pytest

import oracle
from workloads import CSRGraph, dense_normal, glorot_uniform
from gpu_util import assert_close, device_graph
from test_gpu_panels import N_COLS, graph as panel_graph

pytestmark = pytest.mark.gpu


def graph(n=9000, seed=5):
    """Rows of several segments, and windows of more columns than a slice of the workgroup kernel holds."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 24, n)
    lens[[0, 17, n - 1]] = [3000, 6000, 5000]
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colind = rng.integers(0, n, rowptr[-1]).astype(np.int32)
    colind = colind[np.lexsort((colind, np.repeat(np.arange(n), lens)))]
    return CSRGraph(n, n, rowptr, colind, rng.uniform(-1, 1, len(colind)).astype(np.float32))


def placed(X, offset):
    """X as a view that starts `offset` elements into its memory."""
    import torch
    flat = torch.zeros(offset + X.numel() + 64, dtype=X.dtype, device="cuda")
    view = flat[offset:offset + X.numel()].view(X.shape)
    view.copy_(X)
    return view


# widths and modes for which aligned X takes the layer's other order and X one element off the lines does not, or the other way round
@pytest.mark.parametrize("call,d_in,d_out,kind,order_changes", [
    ("layer", 64, 80, "f32", [1]), ("layer", 64, 96, "f32", [1]), ("layer", 48, 80, "f32", [2]), ("layer", 16, 160, "f32", []),
    ("layer", 128, 64, "f32", []), ("aggregate", 128, 16, "bf16", [1]), ("aggregate", 128, 64, "f32", []), ("aggregate", 64, 96, "f32", [])])
@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("first", [0, 1])
def test_same_shapes_same_scratch(call, d_in, d_out, kind, order_changes, mode, first):
    import torch
    import paper_2412_08902_amd.binding as hc
    if kind != "f32" and mode == 2:
        pytest.skip("the matrix path refuses 16-bit X off its vectors")
    g = graph()
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}[kind]
    Xh = torch.from_numpy(dense_normal(g.n_cols, d_in, seed=1)).to(dt)
    W = glorot_uniform(d_in, d_out, seed=2)
    Xs, Wd = [placed(Xh.cuda(), 0), placed(Xh.cuda(), 1)], torch.from_numpy(W).cuda()
    plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *device_graph(g), route_mode=mode, d_hint=d_in, mfma_dtype=0 if kind == "f32" else 1)
    size = hc.hcspmm_gcn_workspace_bytes if call == "layer" else hc.hcspmm_aggregate_update_workspace_bytes
    ws = torch.zeros(size(plan, d_in, d_out), dtype=torch.uint8, device="cuda")
    Y = torch.empty((g.n_rows, d_out), device="cuda")

    def run(X):
        if call == "layer":
            hc.hcspmm_gcn_layer(plan, X, Wd, Y, ws)
        else:
            hc.hcspmm_aggregate_update(plan, X, Wd, Y, ws)

    Xf = Xh.float().numpy()
    XW = oracle.gemm(Xf, W)

    def update_first():
        T = ws.view(torch.float32)[:XW.size].cpu().numpy()
        return T.size == XW.size and np.allclose(T.reshape(XW.shape), XW, rtol=0, atol=1e-4 * np.abs(XW).max())

    eager, held, orders = [None, None], [], [None, None]
    for i in (first, 1 - first):
        run(Xs[i])
        torch.cuda.synchronize()
        eager[i], orders[i] = Y.clone(), update_first()
        held.append(hc.hcspmm_plan_info(plan)["device_bytes"])
    assert (orders[0] != orders[1]) == (mode in order_changes)
    # the product that used to be the call's second half is prepared for, too
    wide = d_out if call == "layer" else d_in
    Z = torch.empty((g.n_rows, wide), device="cuda")
    hc.hcspmm_spmm(plan, torch.zeros((g.n_cols, wide), device="cuda"), Z)
    held.append(hc.hcspmm_plan_info(plan)["device_bytes"])
    assert held[0] == held[1] == held[2]

    side = torch.cuda.Stream()
    for i in (0, 1):
        side.wait_stream(torch.cuda.current_stream())
        captured = torch.cuda.CUDAGraph()
        with torch.cuda.graph(captured, stream=side):
            run(Xs[i])
        for _ in range(3):
            run(Xs[1 - i])                                      # eager work of the other order in between
            Y.fill_(-1.0)
            torch.cuda.synchronize()
            captured.replay()
            torch.cuda.synchronize()
            assert torch.equal(Y, eager[i])
        del captured
    plan.destroy()
    layer = oracle.gcn_layer if call == "layer" else oracle.aggregate_update
    ref, bound = (layer(g.rowptr, g.colind, g.vals, Xf, W, relu=True, use_abs=b) for b in (False, True))
    for got in eager:
        assert_close(got.cpu().numpy().astype(np.float64), ref, bound, 1e-5)


@pytest.mark.parametrize("first", [0, 1])
def test_sums_between_panels_follow_from_the_shapes(first):
    """A 16-bit result of a matrix in column panels: the layer's X W order keeps fp32 sums in the plan, the other order none."""
    import torch
    import paper_2412_08902_amd.binding as hc
    g = panel_graph(300)
    d_in, d_out = 32, 40                                        # a line and two; 1.97 off the lines
    X = torch.from_numpy(dense_normal(N_COLS, d_in, seed=1)).cuda()
    X = [placed(X, 0), placed(X, 1)]
    W = torch.from_numpy(glorot_uniform(d_in, d_out, seed=2)).cuda()
    plan = hc.hcspmm_prepare(g.n_rows, g.n_cols, *device_graph(g), route_mode=1, d_hint=64)
    ws = torch.zeros(hc.hcspmm_gcn_workspace_bytes(plan, d_in, d_out), dtype=torch.uint8, device="cuda")
    Y = torch.empty((g.n_rows, d_out), dtype=torch.bfloat16, device="cuda")
    held = []
    for i in (first, 1 - first):
        hc.hcspmm_gcn_layer_ex(plan, X[i], W, Y, ws)
        held.append(hc.hcspmm_plan_info(plan)["device_bytes"])
    torch.cuda.synchronize()
    plan.destroy()
    assert held[0] == held[1]


def test_order_does_not_depend_on_earlier_calls():
    """A layer call may leave sums between panels in a plan that was made without them; another call's order, and with it the
    last bits of its result, are the same before and after."""
    import torch
    import paper_2412_08902_amd.binding as hc
    n, degree, d_in, d_out = 60_000, 160, 128, 64               # two panels
    rng = np.random.default_rng(1)
    col = rng.integers(0, n // degree, (n, 1)) + n // degree * np.arange(degree)
    g = CSRGraph(n, n, np.arange(0, n * degree + 1, degree, dtype=np.int32), col.ravel().astype(np.int32),
                 rng.standard_normal(n * degree).astype(np.float32))
    X = torch.from_numpy(dense_normal(n, d_in, seed=1)).cuda()
    W = torch.from_numpy(glorot_uniform(d_in, d_out, seed=2)).cuda()
    plan = hc.hcspmm_prepare(n, n, *device_graph(g), route_mode=1, d_hint=d_in)
    ws = torch.zeros(max(hc.hcspmm_gcn_workspace_bytes(plan, d_in, d_in), hc.hcspmm_aggregate_update_workspace_bytes(plan, d_in, d_out)),
                     dtype=torch.uint8, device="cuda")
    Y = [torch.empty((n, d_out), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    hc.hcspmm_aggregate_update(plan, X, W, Y[0], ws)
    big = torch.empty((n, d_in), dtype=torch.bfloat16, device="cuda")
    hc.hcspmm_gcn_layer_ex(plan, X, torch.eye(d_in, device="cuda"), big, ws)
    hc.hcspmm_aggregate_update(plan, X, W, Y[1], ws)
    torch.cuda.synchronize()
    plan.destroy()
    assert torch.equal(Y[0], Y[1])
