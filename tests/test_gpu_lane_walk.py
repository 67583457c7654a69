"""The lane-per-row walk behind A x, its row norms and A^T r: paths of fewer
segments than the back projection takes at a time and one more or less than
that, segments that cross several planes, workgroups with idle lanes, more
voxels than the back projection's table holds, a last line of voxels that is
not full, and a path that comes back to voxels within a slab.

Tolerances: chords are FP64 on both sides, 1e-10 relative to the sum of
magnitudes; with FP32 results one rounding of y and n2 (6e-8), and for A^T r one
of every product and one of every sum on the way, n + 2 roundings of the sum of
magnitudes for n rows."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_01070_amd import api, synth
from test_gpu_row_walk import records

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    ((12, 12, 3), (1.0, 1.0, 1.0), 3.5, 1.0, 1, 0.0),      # 7 segments, one row
    ((12, 12, 3), (1.0, 1.0, 1.0), 4.0, 1.0, 255, 0.0),    # 8
    ((12, 12, 3), (1.0, 1.0, 1.0), 4.5, 1.0, 257, 0.0),    # 9
    ((41, 43, 7), (1.0, 1.0, 1.0), 26.0, 500.0, 64, 0.0),  # one segment
    ((37, 91, 9), (1.7, 0.6, 2.5), 30.0, 1.0, 300, 0.0),   # several planes a segment along y
    ((131, 129, 5), (0.3, 0.3, 0.4), 25.0, 2.0, 700, 0.0),  # along every axis
    ((131, 129, 5), (0.3, 0.3, 0.4), 25.0, 0.5, 700, 18.0),  # inside a hull
    ((40, 40, 6), (1.0, 1.0, 1.0), 31.5, 1.0, 300, 14.0),
    ((1, 41, 5), (3.0, 1.0, 1.0), 25.0, 1.0, 100, 0.0),    # a grid one voxel wide
]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dims,pitch,r,step,n,hull", CASES)
def test_linear_operators_match_the_oracle(dims, pitch, r, step, n, hull, dtype):
    grid = synth.Grid(*dims, pitch=pitch)
    mlp = synth.MLPModel(u_in=-r, u_out=r, step=step)
    p, b = records(grid, mlp, n, 8)
    rng = np.random.Generator(np.random.PCG64(9))
    x = rng.uniform(-1.0, 1.0, grid.nvox).astype(np.float32)
    res = rng.standard_normal(n).astype(np.float32)
    plan = api.Plan(grid, mlp, DEV)
    oracle.set_hull(hull or None)
    if hull:
        plan.set_hull(hull)
    try:
        ry, rn2, _ = oracle.forward(grid, mlp, p, x.astype(np.float64))
        size = oracle.forward(grid, mlp, p, np.abs(x).astype(np.float64))[0]
        rg = oracle.backproject(grid, mlp, p, res.astype(np.float64))
        gsize = oracle.backproject(grid, mlp, p, np.abs(res).astype(np.float64))
    finally:
        oracle.set_hull(None)
    pr = api.Protons(p, DEV)
    xd, rd = torch.from_numpy(x).to(DEV, dtype), torch.from_numpy(res).to(DEV, dtype)
    one = 1e-10 if dtype == torch.float64 else 1e-10 + 2.0 ** -24
    y = api.pct_forward(plan, pr, xd).double().cpu().numpy()
    y2, n2 = (v.double().cpu().numpy() for v in api.pct_forward(plan, pr, xd, with_norm=True))
    assert (np.abs(y - ry) <= one * size + 1e-12).all()
    assert np.array_equal(y, y2)
    assert (np.abs(n2 - rn2) <= one * rn2 + 1e-12).all()
    g = api.pct_backproject(plan, pr, rd).double().cpu().numpy()
    many = 1e-10 if dtype == torch.float64 else 1e-10 + (n + 2) * 2.0 ** -24
    assert (np.abs(g - rg) <= many * gsize + 1e-12).all()


@pytest.mark.parametrize("bend", [0.3, 0.6])
def test_norms_of_paths_that_come_back_within_a_slab(bend):
    """Bows whose tops lie inside a thick slab: up to eight pieces before the
    voxels are met again on the way down."""
    grid = synth.Grid(3, 220, 3, pitch=(8.0, 0.1, 4.0))
    mlp = synth.MLPModel(u_in=-12.0, u_out=12.0)
    n = 65
    p = {k: np.zeros(n, np.float32) for k in ("t_in", "v_in", "th_in", "ph_in", "t_out", "v_out", "th_out", "ph_out",
                                              "gantry")}
    p["t_in"] = p["t_out"] = np.linspace(-1.0, 1.0, n).astype(np.float32)
    p["th_in"] = np.full(n, bend, np.float32)
    p["th_out"] = -p["th_in"]
    x = np.ones(grid.nvox)
    _, ref, _ = oracle.forward(grid, mlp, p, x)
    plan = api.Plan(grid, mlp, DEV)
    _, n2 = api.pct_forward(plan, api.Protons(p, DEV), torch.ones(grid.nvox, dtype=torch.float64, device=DEV),
                            with_norm=True)
    assert api.pct_device_status(plan) == 0
    assert np.allclose(n2.cpu().numpy(), ref, rtol=1e-10, atol=0.0)
