"""Hull paths whose straight parts are a whole number of steps long up to
rounding: every row moves on along its axis, so no route may flag it as turning
back (PCT_DEV_REENTRY), and the results are the oracle's.

Tolerances as for the other operators and DROP tests: 1e-10 in FP64, 1e-5 of
max(|x|, 0.05) for FP32 x."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_01070_amd import api, synth
from test_gpu_row_walk import error

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("step,radius,r", [(0.3, 91.3, 100.0), (1.0, 92.0, 100.0), (0.1, 12.3, 20.0), (0.7, 12.3, 20.0)])
def test_whole_steps_outside_the_hull_are_not_a_turn(step, radius, r):
    n = 360
    p = {k: np.zeros(n, np.float32) for k in ("t_in", "v_in", "th_in", "ph_in", "t_out", "v_out", "th_out", "ph_out")}
    p["v_in"] = p["v_out"] = np.linspace(-1.4, 1.3, n).astype(np.float32)
    p["gantry"] = (np.arange(n) * (2.0 * np.pi / n)).astype(np.float32)
    b = np.linspace(0.8, 1.2, n).astype(np.float32) * np.float32(2.0 * radius)
    side = int(2.0 * r)
    # (an origin that keeps the rays through the axis off the voxel planes)
    grid = synth.Grid(side, side, 3, origin=(-r + 0.25, -r + 0.4, -1.5))
    mlp = synth.MLPModel(u_in=-r, u_out=r, step=step)
    oracle.set_hull(radius)
    try:
        x0 = np.linspace(0.5, 1.5, grid.nvox)
        ry, rn2, _ = oracle.forward(grid, mlp, p, x0)
        ref = oracle.drop(grid, mlp, p, b, 1.0, block=90, lam=0.5, n_iter=1)
    finally:
        oracle.set_hull(None)
    plan = api.Plan(grid, mlp, DEV).set_hull(radius)
    pr, bd = api.Protons(p, DEV), torch.from_numpy(b).to(DEV)
    y, n2 = (v.cpu().numpy() for v in api.pct_forward(plan, pr, torch.from_numpy(x0).to(DEV), with_norm=True))
    assert api.pct_device_status(plan) == 0
    assert np.abs(y - ry).max() <= 1e-10 * 3.0 * r
    assert np.abs(n2 - rn2).max() <= 1e-10 * 3.0 * r
    for dtype, tol in ((torch.float64, 1e-10), (torch.float32, 1e-5)):
        x = torch.ones(grid.nvox, dtype=dtype, device=DEV)
        api.pct_drop_iterate(plan, pr, bd, x, block=90, lam=0.5, n_iter=1)
        assert api.pct_device_status(plan) == 0
        assert error(x, ref) <= tol
