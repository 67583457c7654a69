"""Stored-row sweeps by slab bins against the lane-per-row schedule: the block
sums are the same whole numbers, so x is the same bits, for rows that the bins
hold, rows with more pieces in a slab than they hold, rows longer than a wave
keeps in registers, rows whose slabs do not follow each other, rows that start
without a first visit, and blocks of one row."""
import numpy as np
import pytest
import torch

from paper_1802_01070_amd import api, synth
from test_gpu_row_walk import records

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    ((40, 40, 6), (1.0, 1.0, 1.0), 31.5, 24, 24),      # not packed, both axes
    ((40, 40, 6), (1.0, 1.0, 1.0), 31.5, 200, 16),     # packed
    ((33, 65, 35), (1.0, 1.0, 0.5), 32.0, 40, 1),      # blocks of one row
    ((20, 300, 4), (4.0, 0.2, 1.0), 30.0, 100, 40),    # more than four pieces a slab
    ((500, 500, 2), (0.1, 0.1, 3.0), 30.0, 60, 20),    # rows of more than 512 pieces
    ((1, 40, 5), (3.0, 1.0, 1.0), 25.0, 50, 20),       # a grid one voxel wide
]


@pytest.mark.parametrize("order", ["path", "turned", "shifted"])
@pytest.mark.parametrize("dims,pitch,r,n,block", CASES)
def test_binned_rows_match_the_lane_schedule(dims, pitch, r, n, block, order):
    grid = synth.Grid(*dims, pitch=pitch)
    mlp = synth.MLPModel(u_in=-r, u_out=r)
    p, b = records(grid, mlp, n, 11)
    plan = api.Plan(grid, mlp, DEV, n_hint=64)
    rows = api.Rows(plan, api.Protons(p, DEV), "f16")
    bd = torch.from_numpy(b).to(DEV)
    off = rows.offsets.cpu().numpy()
    if order != "path":
        # the same pieces of every row in another order
        to = np.arange(int(off[-1]))
        for a, e in zip(off[:-1], off[1:]):
            if order == "turned":
                to[a + (e - a) // 2:e] = to[a + (e - a) // 2:e][::-1]
            elif e > a:
                to[a:e] = np.roll(to[a:e], 1)
        to = torch.from_numpy(to).to(DEV)
        rows.vox.copy_(rows.vox[to])
        rows.chord.copy_(rows.chord[to])

    def run(lanes):
        x = torch.linspace(0.5, 1.5, grid.nvox, device=DEV)
        api.pct_drop_iterate_rows(plan, rows, bd, x, block=block, lam=0.5, n_iter=2, lanes=lanes)
        return x

    assert torch.equal(run(0), run(64))
    assert api.pct_device_status(plan) == 0
