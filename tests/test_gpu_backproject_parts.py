"""A^T r by parts of 32 segments (calls of up to 16384 rows) and of 8 (more rows):
paths of one segment less and more than a part, the last call of the one and the
first of the other, and parts with more lines of voxels than the table holds.

Tolerances: chords are FP64 on both sides, 1e-10 of the sum of magnitudes, and
3e-9 mm where a bent path grazes a plane (a coordinate's 3e-14 mm over slopes from
1e-5); with FP32 results one rounding of every product and of every sum on the
way, n + 2 of the sum of magnitudes for n rows."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_01070_amd import api, synth
from test_gpu_row_walk import records

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    ((40, 40, 6), 15.5, 257),        # 31 segments
    ((40, 40, 6), 16.0, 257),        # 32
    ((40, 40, 6), 16.5, 257),        # 33
    ((120, 120, 20), 60.0, 512),     # 256 unordered rows: more lines than keys
    ((40, 40, 6), 16.5, 16384),
    ((40, 40, 6), 16.5, 16385),
]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dims,r,n", CASES)
def test_backprojection_by_parts(dims, r, n, dtype):
    grid = synth.Grid(*dims)
    mlp = synth.MLPModel(u_in=-r, u_out=r)
    p, _ = records(grid, mlp, n, 51)
    res = np.random.Generator(np.random.PCG64(52)).standard_normal(n).astype(np.float32)
    ref = oracle.backproject(grid, mlp, p, res.astype(np.float64))
    size = oracle.backproject(grid, mlp, p, np.abs(res).astype(np.float64))
    plan = api.Plan(grid, mlp, DEV)
    pr = api.Protons(p, DEV)
    g = api.pct_backproject(plan, pr, torch.from_numpy(res).to(DEV, dtype)).double().cpu().numpy()
    tol = 1e-10 if dtype == torch.float64 else 1e-10 + (n + 2) * 2.0 ** -24
    assert (np.abs(g - ref) <= tol * size + 3e-9).all()
