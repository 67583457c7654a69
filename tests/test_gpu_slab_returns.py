"""Rows that meet voxels again far down their list: bows whose tops lie inside a
slab many voxels thick, so that a voxel comes back up to dozens of pieces after
the path left it, in one window of records and across two.

DROP must give the oracle's iterate, which counts the row once per voxel and its
norm with both visits, or say that it did not (PCT_DEV_REENTRY); rows that turn
nowhere may be as long in a slab as they like.  Tolerances as for the other DROP
tests: relative to max(|x|, 0.05), 1e-10 for FP64 x and 1e-5 for FP32 x."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_01070_amd import api, synth
from paper_1802_01070_amd._lib import PCT_DROP_FUSED_COMMIT, PCT_DROP_SEPARATE_COMMIT
from test_gpu_row_walk import error

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
PCT_DEV_REENTRY = 0x4

ROUTES = [(torch.float64, 0, 0), (torch.float64, 0, 1), (torch.float32, 0, 0), (torch.float32, 0, 1),
          (torch.float32, PCT_DROP_SEPARATE_COMMIT, 0), (torch.float32, PCT_DROP_FUSED_COMMIT, 0)]


def bows(n, bend, lateral):
    """Paths that rise (laterally, or along z) with slope `bend` and fall again."""
    p = {k: np.zeros(n, np.float32) for k in ("t_in", "v_in", "th_in", "ph_in", "t_out", "v_out", "th_out", "ph_out",
                                              "gantry")}
    pos, slope = ("t", "th") if lateral else ("v", "ph")
    p[pos + "_in"] = p[pos + "_out"] = np.linspace(-0.9, 0.93, n).astype(np.float32)
    p[slope + "_in"] = np.full(n, bend, np.float32)
    p[slope + "_out"] = -p[slope + "_in"]
    return p, np.linspace(5.0, 20.0, n).astype(np.float32)


def run(grid, mlp, p, b, dtype, flags, lanes):
    plan = api.Plan(grid, mlp, DEV, n_hint=64)
    x = torch.ones(grid.nvox, dtype=dtype, device=DEV)
    api.pct_drop_iterate(plan, api.Protons(p, DEV), torch.from_numpy(b).to(DEV), x, block=40, lam=0.5, n_iter=2,
                         flags=flags, lanes=lanes)
    return x, api.pct_device_status(plan)


@pytest.mark.parametrize("dtype,flags,lanes", ROUTES)
@pytest.mark.parametrize("pitch,bend,lateral", [
    (0.1, 0.3, True), (0.1, 0.6, True), (0.1, 1.5, True),      # up to 4, 8 and 20 pieces back
    (0.05, 0.8, True), (0.05, 1.5, False), (0.02, 1.5, False),
])
def test_rows_that_come_back_late_count_once(pitch, bend, lateral, dtype, flags, lanes):
    dims = (3, 5 + int(22.0 / pitch), 3) if lateral else (3, 3, 5 + int(22.0 / pitch))
    grid = synth.Grid(*dims, pitch=(8.0, pitch, 4.0) if lateral else (8.0, 4.0, pitch))
    mlp = synth.MLPModel(u_in=-12.0, u_out=12.0)
    p, b = bows(65, bend, lateral)
    ref = oracle.drop(grid, mlp, p, b, 1.0, block=40, lam=0.5, n_iter=2)
    x, status = run(grid, mlp, p, b, dtype, flags, lanes)
    assert status & ~PCT_DEV_REENTRY == 0
    if lanes == 0 and pitch >= 0.05:
        assert status == 0          # a wave sees the whole slab (at 0.02 the outer slabs do not fit a window)
    if status == 0:
        assert error(x, ref) <= (1e-10 if dtype == torch.float64 else 1e-5)


@pytest.mark.parametrize("dtype,flags,lanes", ROUTES)
def test_a_slab_longer_than_the_window_is_told(dtype, flags, lanes):
    """A slab whose records take several windows: rows that turn there are
    flagged (or right), rows that do not turn are right and not flagged."""
    grid = synth.Grid(1, 1, 9000, pitch=(40.0, 8.0, 0.004))
    mlp = synth.MLPModel(u_in=-12.0, u_out=12.0)
    p, b = bows(65, 2.0, False)
    ref = oracle.drop(grid, mlp, p, b, 1.0, block=40, lam=0.5, n_iter=2)
    x, status = run(grid, mlp, p, b, dtype, flags, lanes)
    tol = 1e-10 if dtype == torch.float64 else 1e-5
    assert status == PCT_DEV_REENTRY or (status == 0 and error(x, ref) <= tol)
    p["ph_out"] = p["ph_in"] = np.full(65, 1.2, np.float32)
    p["v_in"] = np.linspace(-15.0, -13.0, 65).astype(np.float32)
    p["v_out"] = p["v_in"] + np.float32(24.0 * 1.2)
    ref = oracle.drop(grid, mlp, p, b, 1.0, block=40, lam=0.5, n_iter=2)
    x, status = run(grid, mlp, p, b, dtype, flags, lanes)
    assert status == 0
    assert error(x, ref) <= tol
