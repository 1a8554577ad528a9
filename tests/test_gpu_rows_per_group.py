"""Several rows to a lane group (launches that would pass 2^32 threads otherwise): the same results as one row to a group,
bit for bit.  The row count per group is a process-wide experiment knob, so the runs with it are a child process."""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHAPES = [(5001, 8, "f32"), (5003, 33, "f32"), (7000, 128, "f32"), (5009, 260, "f32"), (7001, 64, "bf16"), (7001, 96, "f16")]


def results():
    import torch
    import paper_2412_08902_amd.binding as hc
    out = []
    for n, d, kind in SHAPES:
        rng = np.random.default_rng(n + d)
        lens = rng.integers(0, 60, n)
        lens[rng.integers(0, n, 20)] = 700
        rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        colind = rng.integers(0, n, rowptr[-1]).astype(np.int32)
        dev = [torch.from_numpy(a).cuda() for a in (rowptr, colind, rng.standard_normal(rowptr[-1]).astype(np.float32))]
        X = torch.from_numpy(rng.standard_normal((n, d)).astype(np.float32)).cuda()
        X = X.to({"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[kind])
        plan = hc.hcspmm_prepare(n, n, *dev, route_mode=1, d_hint=d, mfma_dtype={"f32": 0, "bf16": 1, "f16": 2}[kind])
        Y = torch.full((n, d), -777.0, device="cuda")
        hc.hcspmm_spmm(plan, X, Y)
        torch.cuda.synchronize()
        out.append(Y.cpu().numpy())
        plan.destroy()
    return out


def test_rows_per_group(tmp_path):
    want = results()
    for rows in ("2", "7"):
        path = str(tmp_path / (rows + ".npz"))
        env = dict(os.environ, HCSPMM_TUNE_RPG=rows, PYTHONPATH=os.pathsep.join([ROOT, os.path.join(ROOT, "tests")]))
        code = "import numpy as np, test_gpu_rows_per_group as t; np.savez(%r, *t.results())" % path
        subprocess.run([sys.executable, "-c", code], env=env, cwd=ROOT, check=True, timeout=100)
        got = np.load(path)
        for i, w in enumerate(want):
            assert np.array_equal(got["arr_%d" % i], w), (rows, SHAPES[i])
