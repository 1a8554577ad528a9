"""X W for bf16 X on the bf16 matrix units, W in three parts: values of any scale, infinities and NaN, and the shapes of both kernels (up to
256 of depth with all of W in LDS, beyond it with two slabs), read from the workspace of the aggregate-then-update call, which starts with X W."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def product(X, W, pitch=None):
    """X W as the library forms it in front of an aggregation whose rows have sixteen non-zeros"""
    import torch
    import paper_2412_08902_amd.binding as hc
    (n, d_in), d_out = X.shape, W.shape[1]
    wide = torch.full((n, pitch or d_in), float("nan"), dtype=torch.bfloat16, device="cuda")
    wide[:, :d_in] = X.cuda()
    ip = torch.arange(0, 16 * n + 1, 16, dtype=torch.int32, device="cuda")
    ci, va = torch.arange(n, dtype=torch.int32, device="cuda").repeat_interleave(16), torch.full((16 * n,), 1 / 16, device="cuda")
    plan = hc.hcspmm_prepare(n, n, ip, ci, va, route_mode=1, d_hint=d_in, mfma_dtype=1)
    ws = torch.full((hc.hcspmm_aggregate_update_workspace_bytes(plan, d_in, d_out),), 255, dtype=torch.uint8, device="cuda")
    hc.hcspmm_aggregate_update(plan, wide[:, :d_in], W.cuda(), torch.empty((n, d_out), device="cuda"), ws, apply_relu=False)
    torch.cuda.synchronize()
    plan.destroy()
    return ws[:4 * n * d_out].view(torch.float32).view(n, d_out)


def exact(X, W):
    return X.cuda().double() @ W.cuda().double()


def operands(n, k, d_out, w_bits, seed):
    """Quarters below 2 and values of w_bits bits from 1/2 on, of either sign: bits that a power of two cannot push out of a format"""
    import torch
    rng = np.random.default_rng(seed)
    X = rng.integers(-7, 8, (n, k)) / 4.0
    W = np.floor(rng.uniform(0.5, 2.0, (k, d_out)) * 2.0 ** (w_bits - 1)) * 2.0 ** (1 - w_bits) * rng.choice([-1.0, 1.0], (k, d_out))
    return torch.from_numpy(X), torch.from_numpy(W)


# (rows, depth, columns): the forms of one to four column tiles, of two workgroups and one to a CU, and the deep ones
SHAPES = [(16385, 250, 64), (16400, 222, 80), (16399, 190, 33), (49185, 128, 16), (65541, 290, 31), (65537, 322, 128)]


@pytest.mark.parametrize("n,k,d_out", SHAPES)
def test_a_power_of_two_changes_exponents_only(n, k, d_out):
    """Small W keeps all its bits, down to the last one of the format, and so does X below bf16's normal range; large values come out to the fp32
    units' precision (half of 2^-24 for each term, as a random walk), which the others' 2-norms are held to as well."""
    import torch
    for w_bits, scales in ((24, [(0, -90), (0, -112), (30, -116), (60, -120), (100, -125), (-131, 40), (-120, 100), (90, -20), (-20, 106), (-40, 120), (119, 0)]),
                           (10, [(20, -139), (100, -139)])):
        X, W = operands(n, k, d_out, w_bits, seed=n + w_bits)
        base = product(X.bfloat16(), W.float())
        ref = exact(X, W)
        fp32_units = 0.5 * np.sqrt(k) * 2.0 ** -24 * ref.norm()
        assert (base.double() - ref).norm() <= fp32_units
        for x_exp, w_exp in scales:
            Xs, Ws = X * 2.0 ** x_exp, W * 2.0 ** w_exp
            assert torch.equal(Xs.bfloat16().double(), Xs) and torch.equal(Ws.float().double(), Ws)
            got = product(Xs.bfloat16(), Ws.float()).double() * 2.0 ** (-x_exp - w_exp)
            if w_exp >= 104 or x_exp + w_exp >= 90:             # formed on the fp32 units
                assert (got - ref).norm() <= fp32_units, (x_exp, w_exp)
            else:
                assert torch.equal(got, base.double()), (x_exp, w_exp)


@pytest.mark.parametrize("n,k,d_out", [(16420, 250, 60), (49170, 222, 15), (65600, 290, 31), (65560, 291, 15), (65555, 322, 95), (65540, 602, 64)])
@pytest.mark.parametrize("w_at", [None, "middle", "last", "largest"])
def test_infinities_and_nan(n, k, d_out, w_at):
    """They reach the results that they belong to and no others, from the middle of the depth and from its last, partly filled slab."""
    import torch
    torch.manual_seed(k)
    X, W = torch.randn(n, k).bfloat16(), torch.randn(k, d_out)
    W[7, 3] = 0.5                                               # a value whose remainders are zero
    X[5, 7], X[77, k - 1], X[n - 1, 0], X[300, k - 2] = float("inf"), float("-inf"), float("nan"), float("nan")
    if w_at is None:                                            # (beside an infinity a sum that overflows on its way is another result)
        X[200, 64] = torch.finfo(torch.bfloat16).max
    X[1000:1016, 40] = 0.0                                      # (times an infinity)
    if w_at == "middle":
        W[40, d_out - 1] = float("inf")
    elif w_at == "last":
        W[k - 1, 2] = float("-inf")
    elif w_at == "largest":
        W[k - 2, 0] = torch.finfo(torch.float32).max
    got, want = product(X, W, pitch=k + k % 2 + 2).double(), exact(X, W)
    want = want.float().double()                                # (what overflows fp32 is an infinity)
    assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf())
    assert torch.equal(got[want.isinf()], want[want.isinf()])
    fin = want.isfinite()
    assert torch.all((got[fin] - want[fin]).abs() <= 1e-5 * (X.cuda().double().abs() @ W.cuda().double().abs())[fin])


@pytest.mark.parametrize("n,k,d_out", [(65536, 322, 64), (65536, 290, 31)])
def test_equal_rows_beside_an_infinity_of_a_deep_product(n, k, d_out):
    """An infinity of W in the middle of the depth: rows that are equal have equal results, whichever wave multiplies them."""
    import torch
    torch.manual_seed(5)
    X, W = torch.randn(16, k).bfloat16().repeat(n // 16, 1), torch.randn(k, d_out)
    W[100, 11] = float("inf")
    T = product(X, W).view(n // 16, 16, d_out)
    finite = torch.arange(d_out, device="cuda") != 11
    assert torch.equal(T[:, :, finite], T[:1, :, finite].expand(n // 16, -1, -1))
    assert bool(T[:, :, 11].isinf().all())


# the deep kernel's remainders: one to four column tiles and two groups of them, an odd depth, a last slab of two values and a full one
@pytest.mark.parametrize("n,k,d_out", [(65537, 291, 15), (65541, 290, 31), (65600, 258, 47), (65536, 320, 64), (65537, 321, 128), (65551, 602, 16)])
def test_deep_products(n, k, d_out):
    import torch
    torch.manual_seed(n)
    X, W = torch.randn(n, k).bfloat16(), torch.randn(k, d_out)
    got, ref = product(X, W, pitch=k + k % 2), exact(X, W)
    assert torch.all((got.double() - ref).abs() <= 1e-5 * (X.cuda().double().abs() @ W.cuda().double().abs()))
