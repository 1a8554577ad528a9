"""dX = S W^T and dW = X^T S in one kernel (widths of 65 to 128): row counts around its batches and spans, widths around its
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


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 100, 1023, 4112, 9000])
@pytest.mark.parametrize("d_in,d,pad", [(128, 128, 0), (128, 128, 3), (112, 72, 0), (66, 96, 1), (69, 100, 0), (100, 84, 2),
                                        (120, 124, 5), (96, 68, 0), (127, 80, 0)])       # the last three: two kernels
def test_products(n, d_in, d, pad):
    products(n, d_in, d, pad)


# Spans of 5 and 6, 9 and 10, 17 and 18 batches: both buffers of a half come round several times, and either half has the last turn.
# From 65,536 rows on widths of X up to 96 are left to the two kernels.
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
