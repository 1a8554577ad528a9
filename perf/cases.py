"""Performance cases of the library: the calls a user makes, over the range of graphs they are made on.

``listed()`` names the cases that are followed over time, ``draw(rng)`` gives further ones of the same ranges,
``prepare`` builds what a program has in hand before the call (graph, features, weights, workspace and plan),
``run`` makes one pass through the public entry points, and ``work`` / ``tolerance`` say what a pass cannot do without and
how close another correct implementation comes.

A case is a dict of plain values:

    op       "spmm"       Y = A X with a plan that is kept
             "layer"      Y = ReLU(A (X W)), the GCN layer's forward pass (``t``: storage type of X W)
             "aggregate"  Y = ReLU((A X) W), the layer in the other order (GIN)
             "backward"   dX, dW of a layer with the activation mask of its forward output
             "fresh"      a graph that is used once: prepare, one Y = A X, destroy
             "changed"    a graph that changes: plan update, Y = A X, update back, Y = A X (``changed`` rows)
    graph    "power"      symmetrised Chung-Lu power law + self-loops (``n``, ``edges``, ``gamma``, ``max_degree``, 0 = sqrt(edges))
             "blocks"     stochastic block model (``n`` nodes in blocks of 64, ``p_in``, 4 edges per node between blocks)
             "mixed"      blocks (``n_blocks`` nodes) followed by a power law (``n`` nodes)
    gcn      edge values D^-1/2 (A) D^-1/2 instead of ones
    d        width of the aggregated features (X's for spmm, fresh, changed and aggregate, W's columns for layer and backward)
    d_other  the layer's other width
    x, y, t  "f32", "bf16" or "f16"

The listed sizes are those of the benchmark's configurations (workloads/graphs.py); graphs are made on the GPU with
the same recipes.
"""
import math

import torch

import paper_2412_08902_amd.binding as hc

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
CODES = {"f32": hc.HCSPMM_F32, "bf16": hc.HCSPMM_BF16, "f16": hc.HCSPMM_F16}
BYTES = {"f32": 4, "bf16": 2, "f16": 2}
BLOCK = 64
INTER_DEGREE = 4


def listed():
    c1 = {"graph": "power", "n": 2708, "edges": 10556, "gamma": 2.1, "max_degree": 0, "gcn": False}
    c2 = {"graph": "power", "n": 169343, "edges": 2300000, "gamma": 2.0, "max_degree": 13000, "gcn": True}
    c3 = {"graph": "blocks", "n": 131072, "p_in": 0.25, "gcn": False}
    c4 = {"graph": "power", "n": 2449029, "edges": 123700000, "gamma": 2.2, "max_degree": 0, "gcn": True}
    c5 = {"graph": "power", "n": 232965, "edges": 114600000, "gamma": 1.9, "max_degree": 0, "gcn": True}
    c6 = {"graph": "mixed", "n": 169343, "edges": 2300000, "gamma": 2.0, "max_degree": 13000, "n_blocks": 131072,
          "p_in": 0.75, "gcn": True}
    return [
        # a citation graph of a few thousand nodes: the smallest call, bound by launches
        {"name": "spmm_small", "op": "spmm", **c1, "d": 32, "x": "f32", "y": "f32"},
        # the ordinary call: a medium power-law graph at hidden width 128
        {"name": "spmm_medium", "op": "spmm", **c2, "d": 128, "x": "f32", "y": "f32"},
        # community graph with 16-bit activations in and out, as in a chain of 16-bit layers
        {"name": "spmm_community_bf16", "op": "spmm", **c3, "d": 64, "x": "bf16", "y": "bf16"},
        # the large call: 126 M non-zeros at a narrow width
        {"name": "spmm_large", "op": "spmm", **c4, "d": 32, "x": "f32", "y": "f32"},
        # dense communities next to a power-law part: both kinds of row windows in one graph
        {"name": "spmm_mixed", "op": "spmm", **c6, "d": 128, "x": "f32", "y": "f32"},
        # a number of classes for a width and a node count that no tile divides
        {"name": "spmm_ragged", "op": "spmm", "graph": "power", "n": 50021, "edges": 1400000, "gamma": 2.15,
         "max_degree": 0, "gcn": True, "d": 47, "x": "f32", "y": "f32"},
        # the forward pass of a GCN's first layer on a dense graph: 602 features to 128
        {"name": "layer_dense", "op": "layer", **c5, "d": 128, "d_other": 602, "t": "f32", "y": "f32"},
        # the same with the intermediate and the output in bf16
        {"name": "layer_dense_bf16", "op": "layer", **c5, "d": 128, "d_other": 602, "t": "bf16", "y": "bf16"},
        # aggregate, then update (GIN), 16-bit in and out
        {"name": "aggregate_medium_bf16", "op": "aggregate", **c2, "d": 128, "d_other": 64, "x": "bf16", "y": "bf16"},
        # the backward pass of a hidden layer
        {"name": "backward_medium", "op": "backward", **c2, "d": 128, "d_other": 128},
        # a sampled subgraph: prepared, used once, dropped
        {"name": "fresh_subgraph", "op": "fresh", "graph": "power", "n": 16934, "edges": 230000, "gamma": 2.0,
         "max_degree": 0, "gcn": True, "d": 128, "x": "f32", "y": "f32"},
        # a graph that gains and loses edges between calls
        {"name": "changed_graph", "op": "changed", **c2, "changed": 1000, "d": 128, "x": "f32", "y": "f32"},
    ]


def _log_between(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    op = rng.choice(["spmm", "spmm", "spmm", "layer", "layer", "aggregate", "backward", "backward", "fresh", "changed"])
    # widths: hidden sizes (multiples of 16) as often as anything in between
    def width(lo, hi):
        w = int(round(_log_between(rng, lo, hi)))
        return max(16, (w + 8) // 16 * 16) if rng.random() < 0.6 else w

    d = width(8, 256)
    c = {"op": op, "d": d}
    kind = rng.choice(["power", "power", "power", "blocks", "mixed"])
    # non-zeros: up to the dense configuration's work (nnz * d), and less for paths that prepare or multiply as well
    budget = 1.4e10 if op in ("spmm", "layer", "aggregate") else (6e9 if op == "backward" else 4e8)
    most = min(1.1e8, budget / d)
    n = int(round(_log_between(rng, 2000, min(2.4e6, max(4000.0, most / 8)))))
    if kind == "power":
        degree = _log_between(rng, 4, min(500.0, n / 16.0, max(5.0, most / n)))
        c.update(graph="power", n=n, edges=int(n * degree) // 2 * 2, gamma=round(rng.uniform(1.9, 2.3), 2), max_degree=0,
                 gcn=rng.random() < 0.7)
    else:
        p_in = round(rng.uniform(0.1, 0.9), 2)
        nb = max(2 * BLOCK, int(min(n, 300000, most / 2 / (BLOCK * p_in + INTER_DEGREE))) // BLOCK * BLOCK)
        if kind == "blocks":
            c.update(graph="blocks", n=nb, p_in=p_in, gcn=rng.random() < 0.5)
        else:
            n = min(n, int(most / 2 / 14))
            c.update(graph="mixed", n=n, edges=int(n * rng.uniform(4, 14)) // 2 * 2, gamma=round(rng.uniform(1.9, 2.3), 2),
                     max_degree=0, n_blocks=nb, p_in=p_in, gcn=True)
    if op in ("spmm", "fresh", "changed", "aggregate"):
        # 16-bit features come in widths of whole 8-byte pieces
        c["x"] = rng.choice(["f32", "f32", "bf16", "f16"]) if d % 4 == 0 else "f32"
        c["y"] = rng.choice(["f32", c["x"]])
    if op == "layer":
        c["t"] = rng.choice(["f32", "f32", "bf16", "f16"]) if d % 4 == 0 else "f32"
        c["y"] = rng.choice(["f32", c["t"]])
        c["d_other"] = width(16, 602)
    if op in ("aggregate", "backward"):
        c["d_other"] = width(16, 256)
    if "d_other" in c:      # dense products: up to the dense configuration's multiply-adds
        nodes = c["n"] + c.get("n_blocks", 0)
        c["d_other"] = max(16, min(c["d_other"], int((9e9 if op == "backward" else 1.8e10) / (nodes * d))))
    if op == "changed":
        c["changed"] = int(round(_log_between(rng, 1, max(2.0, min(5000.0, c["n"] / 20.0)))))
    return c


# ---- graphs --------------------------------------------------------------------------------------

def _offset_for_cap(n, alpha, ratio):
    """i0 >= 0 with w_1 / sum(w) == ratio for w_i = (i + i0)^-alpha."""
    idx = torch.arange(1, n + 1, dtype=torch.float64, device="cuda")

    def share(i0):
        w = (idx + i0) ** (-alpha)
        return float(w[0] / w.sum())

    if share(0.0) <= ratio:
        return 0.0
    lo, hi = 0.0, 1.0
    while share(hi) > ratio:
        hi *= 4.0
    for _ in range(30):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if share(mid) > ratio else (lo, mid)
    return hi


_offsets = {}       # i0 of a degree law: depends on the case's sizes alone


def _distinct(draw_keys, target, gen):
    """Exactly ``target`` distinct keys, ascending: more are drawn until there are enough, then a random subset stays."""
    keys = torch.unique(draw_keys(int(target * 1.08) + 64))
    while keys.numel() < target:
        keys = torch.unique(torch.cat([keys, draw_keys(int((target - keys.numel()) * 1.5) + 64)]))
    if keys.numel() > target:
        keep = torch.ones(keys.numel(), dtype=torch.bool, device=keys.device)
        keep[torch.randperm(keys.numel(), generator=gen, device=keys.device)[target:]] = False
        keys = keys[keep]
    return keys


def _power_pairs(n, edges, gamma, max_degree, gen):
    alpha = 1.0 / (gamma - 1.0)
    at = (n, edges, gamma, max_degree)
    if at not in _offsets:
        _offsets[at] = _offset_for_cap(n, alpha, (max_degree or math.isqrt(edges)) / edges)
    w = (torch.arange(1, n + 1, dtype=torch.float64, device="cuda") + _offsets[at]) ** (-alpha)
    cdf = torch.cumsum(w, 0)
    cdf /= cdf[-1].clone()

    def endpoint(count):
        u = torch.rand(count, dtype=torch.float64, device="cuda", generator=gen)
        return torch.searchsorted(cdf, u).clamp_(max=n - 1)

    def keys(count):
        a, b = endpoint(count), endpoint(count)
        k = torch.minimum(a, b) * n + torch.maximum(a, b)
        return k[a != b]

    k = _distinct(keys, edges // 2, gen)
    return k // n, k % n


def _block_pairs(n, p_in, gen):
    nb = n // BLOCK
    i, j = torch.triu_indices(BLOCK, BLOCK, 1, device="cuda")
    present = torch.rand((nb, i.numel()), device="cuda", generator=gen) < p_in
    blk, at = present.nonzero(as_tuple=True)
    inner = (blk * BLOCK + i[at]) * n + blk * BLOCK + j[at]

    def keys(count):
        a = torch.randint(0, n, (count,), device="cuda", generator=gen)
        b = torch.randint(0, n, (count,), device="cuda", generator=gen)
        k = torch.minimum(a, b) * n + torch.maximum(a, b)
        return k[a // BLOCK != b // BLOCK]

    k = torch.cat([inner, _distinct(keys, n * INTER_DEGREE // 2, gen)])
    return k // n, k % n


def _csr(n, u, v, loops, gcn):
    """Pairs u != v, each once -> symmetric CSR with ascending columns (int32) and fp32 values."""
    parts = [u * n + v, v * n + u]
    if loops is not None:
        parts.append(loops * n + loops)
    key = torch.sort(torch.cat(parts)).values
    del parts
    row = key // n
    col = (key - row * n).to(torch.int32)
    rowptr = torch.searchsorted(row, torch.arange(n + 1, device="cuda")).to(torch.int32)
    if gcn:
        s = torch.diff(rowptr).clamp_(min=1).to(torch.float64).rsqrt_()
        vals = (s[row] * s[col.long()]).to(torch.float32)
    else:
        vals = torch.ones(col.numel(), dtype=torch.float32, device="cuda")
    return rowptr, col, vals


def _graph(case, gen):
    n = case["n"]
    if case["graph"] == "power":
        u, v = _power_pairs(n, case["edges"], case["gamma"], case["max_degree"], gen)
        return (n, *_csr(n, u, v, torch.arange(n, device="cuda"), case["gcn"]))
    if case["graph"] == "blocks":
        u, v = _block_pairs(n, case["p_in"], gen)
        return (n, *_csr(n, u, v, None, case["gcn"]))
    nb = case["n_blocks"]
    bu, bv = _block_pairs(nb, case["p_in"], gen)
    pu, pv = _power_pairs(n, case["edges"], case["gamma"], case["max_degree"], gen)
    loops = torch.arange(nb, nb + n, device="cuda")
    return (nb + n, *_csr(nb + n, torch.cat([bu, pu + nb]), torch.cat([bv, pv + nb]), loops, case["gcn"]))


def _sizes(case):
    """(nodes, non-zeros) of the case's graph; blocks by their expectation."""
    power = case["edges"] + case["n"] if case["graph"] != "blocks" else 0
    nb = {"power": 0, "blocks": case["n"], "mixed": case.get("n_blocks", 0)}[case["graph"]]
    nodes = nb if case["graph"] == "blocks" else nb + case["n"]
    return nodes, power + nb * ((BLOCK - 1) * case.get("p_in", 0.0) + INTER_DEGREE)


# ---- the cases' interface --------------------------------------------------------------------------

def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    op, d, other = case["op"], case["d"], case.get("d_other", 0)
    n, rowptr, colind, vals = _graph(case, gen)
    s = {"op": op, "n": n, "d": d, "csr": (rowptr, colind, vals), "y": case.get("y", "f32")}

    def normal(rows, cols, dtype="f32"):
        return torch.randn((rows, cols), device="cuda", generator=gen).to(DTYPES[dtype])

    def glorot(rows, cols):
        a = math.sqrt(6.0 / (rows + cols))
        return (torch.rand((rows, cols), device="cuda", generator=gen) * 2.0 - 1.0) * a

    def workspace(size):
        return torch.empty(max(size, 256), dtype=torch.uint8, device="cuda")

    # the plan is made for the type and width that its aggregation reads
    kind = case["t"] if op == "layer" else case.get("x", "f32")
    s["options"] = {"d_hint": d, "mfma_dtype": CODES[kind]}
    if op != "fresh":
        s["plan"] = hc.hcspmm_prepare(n, n, rowptr, colind, vals, **s["options"])
    if op == "layer":
        s["X"], s["W"], s["t"] = normal(n, other), glorot(other, d), CODES[case["t"]]
        s["ws"] = workspace(hc.hcspmm_gcn_workspace_bytes(s["plan"], other, d))
        s["Y"] = torch.empty((n, d), dtype=DTYPES[s["y"]], device="cuda")
    elif op == "aggregate":
        s["X"], s["W"] = normal(n, d, kind), glorot(d, other)
        s["ws"] = workspace(hc.hcspmm_aggregate_update_workspace_bytes(s["plan"], d, other))
        s["Y"] = torch.empty((n, other), dtype=DTYPES[s["y"]], device="cuda")
    elif op == "backward":
        s["G"], s["X"], s["W"] = normal(n, d), normal(n, other).relu_(), glorot(other, d)
        s["Yf"] = normal(n, d).relu_()
        s["ws"] = workspace(hc.hcspmm_layer_backward_workspace_bytes(s["plan"], other, d))
        s["dX"], s["dW"] = torch.empty((n, other), device="cuda"), torch.empty((other, d), device="cuda")
    else:
        s["X"] = normal(n, d, kind)
        s["Y"] = torch.empty((n, d), dtype=DTYPES[s["y"]], device="cuda")
    if op == "changed":
        # the last neighbour of each changed row moves to the next column (rows stay sorted and free of duplicates)
        rows = torch.randperm(n, generator=gen, device="cuda")[: case["changed"]].sort().values
        last = rowptr[rows + 1].long() - 1
        ok = (rowptr[rows + 1] > rowptr[rows]) & (colind[last.clamp(min=0)] < n - 1)
        rows, last = rows[ok], last[ok]
        moved = colind.clone()
        moved[last] += 1
        s["rows"], s["moved"] = rows.to(torch.int32).cpu().numpy(), moved
        s["Y2"] = torch.empty_like(s["Y"])
    return s


def run(s):
    op = s["op"]
    if op == "spmm":
        return hc.hcspmm_spmm(s["plan"], s["X"], s["Y"])
    if op == "layer":
        return hc.hcspmm_gcn_layer_ex(s["plan"], s["X"], s["W"], s["Y"], s["ws"], t_dtype=s["t"])
    if op == "aggregate":
        return hc.hcspmm_aggregate_update(s["plan"], s["X"], s["W"], s["Y"], s["ws"])
    if op == "backward":
        return hc.hcspmm_layer_backward(s["plan"], s["G"], s["X"], s["W"], s["dX"], s["dW"], s["ws"], Y_fwd=s["Yf"])
    rowptr, colind, vals = s["csr"]
    if op == "fresh":
        plan = hc.hcspmm_prepare(s["n"], s["n"], rowptr, colind, vals, **s["options"])
        hc.hcspmm_spmm(plan, s["X"], s["Y"])
        plan.destroy()
        return s["Y"]
    hc.hcspmm_plan_update(s["plan"], rowptr, s["moved"], vals, s["rows"])
    hc.hcspmm_spmm(s["plan"], s["X"], s["Y"])
    hc.hcspmm_plan_update(s["plan"], rowptr, colind, vals, s["rows"])
    hc.hcspmm_spmm(s["plan"], s["X"], s["Y2"])
    return s["Y"], s["Y2"]


def work(case):
    n, nnz = _sizes(case)
    op, d, other = case["op"], case["d"], case.get("d_other", 0)
    csr = 4.0 * (n + 1) + 8.0 * nnz
    agg = 2.0 * nnz * d
    if op == "layer":
        return {"bytes": csr + 4.0 * (n * other + other * d) + BYTES[case["y"]] * n * d, "flops": agg + 2.0 * n * other * d}
    if op == "aggregate":
        return {"bytes": csr + BYTES[case["x"]] * n * d + 4.0 * d * other + BYTES[case["y"]] * n * other,
                "flops": agg + 2.0 * n * d * other}
    if op == "backward":     # G, forward output, X, W -> dX, dW
        return {"bytes": csr + 4.0 * (2 * n * d + 2 * n * other + 2 * other * d), "flops": agg + 4.0 * n * d * other}
    once = {"bytes": csr + (BYTES[case["x"]] + BYTES[case["y"]]) * n * d, "flops": agg}
    return {k: 2 * v for k, v in once.items()} if op == "changed" else once


def tolerance(case):
    # fp32 sums of up to some ten thousand terms; with 16-bit features, intermediates or outputs one rounding of those
    kinds = {case.get("x", "f32"), case.get("y", "f32"), case.get("t", "f32")}
    if "bf16" in kinds:
        return {"rel": 1e-2, "max": 5e-2}
    if "f16" in kinds:
        return {"rel": 2e-3, "max": 1e-2}
    return {"rel": 1e-5, "max": 4e-4}
