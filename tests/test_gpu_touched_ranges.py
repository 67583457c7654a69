"""Commits over a block's touched range, on either side of the volumes from which
the fused (2^22 voxels) and the separate schedule (2^24) take it: blocks that
touch a few slices each, in rising and falling order, one block that touches
nothing, a last block that is not full, an odd and an even number of blocks a
sweep, and recorded sweeps replayed.

FP32 block sums are whole numbers, so every schedule without compensation gives
the same bits.  FP64 against the oracle: the paths lie nearly in the slices (slopes
from 1e-4), where the 1e-13 mm that a vertex rounds to moves a crossing by up to
1e-9 mm along the path; with rho_i below 1 that is 1e-9 of x, 2e-8 of
max(|x|, 0.05)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_01070_amd import api, synth
from paper_1802_01070_amd._lib import (PCT_DROP_DETERMINISTIC, PCT_DROP_FUSED_COMMIT, PCT_DROP_NO_COMPENSATION,
                                      PCT_DROP_SEPARATE_COMMIT)
from test_gpu_row_walk import error, records

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def scan(nz, blocks, block, n):
    """Rows of block t around one height; block 1 passes above the volume."""
    grid = synth.Grid(256, 256, nz)
    mlp = synth.MLPModel(u_in=-120.0, u_out=120.0, step=2.0)
    p, b = records(grid, mlp, n, 21)
    heights = np.linspace(float(grid.lo[2]) + 8.0, float(grid.hi[2]) - 8.0, blocks)
    heights[::2] = heights[::2][::-1]
    for t in range(blocks):
        rows = slice(t * block, min(n, (t + 1) * block))
        z = np.float32(heights[t] if t != 1 else float(grid.hi[2]) + 500.0)
        p["v_in"][rows] = z + 0.01 * p["v_in"][rows]
        p["v_out"][rows] = z + 0.01 * p["v_out"][rows]
        p["ph_in"][rows] *= np.float32(0.1)
        p["ph_out"][rows] *= np.float32(0.1)
    return grid, mlp, p, b


@pytest.mark.parametrize("nz", [63, 64, 255, 256])
@pytest.mark.parametrize("blocks,n_iter", [(4, 2), (5, 1), (5, 4)])
def test_schedules_agree(nz, blocks, n_iter):
    block = 24
    grid, mlp, p, b = scan(nz, blocks, block, blocks * block - 5)
    plan = api.Plan(grid, mlp, DEV, n_hint=block)
    pr, bd = api.Protons(p, DEV), torch.from_numpy(b).to(DEV)
    rows = api.Rows(plan, pr, "f32")

    def traced(flags, dtype=torch.float32, chord="f32", calls=2):
        x = torch.ones(grid.nvox, dtype=dtype, device=DEV)
        for _ in range(calls):
            api.pct_drop_iterate(plan, pr, bd, x, block=block, lam=0.5, n_iter=n_iter, chord=chord, flags=flags)
        return x

    def stored(lanes):
        x = torch.ones(grid.nvox, device=DEV)
        for _ in range(2):
            api.pct_drop_iterate_rows(plan, rows, bd, x, block=block, lam=0.5, n_iter=n_iter, lanes=lanes)
        return x

    ref = traced(PCT_DROP_NO_COMPENSATION)
    assert int((ref != 1.0).sum()) > 1000
    for flags in (PCT_DROP_SEPARATE_COMMIT, PCT_DROP_FUSED_COMMIT):
        assert torch.equal(traced(flags), ref)
    by_atomics = stored(64)
    assert torch.equal(stored(0), by_atomics)
    # (the stored norms are summed in another order)
    assert (by_atomics - ref).abs().max().item() <= 1e-5
    want = oracle.drop(grid, mlp, p, b, 1.0, block=block, lam=0.5, n_iter=n_iter)
    for flags in (0, PCT_DROP_DETERMINISTIC):
        assert error(traced(flags, torch.float64, "f64", calls=1), want) <= 2e-8
