"""Stored rows by slab bins and by atomics, the routes of a call without named
lanes: either side of the rules that choose (the length of paths at 45 degrees, the
rows of a block against the volume, the time that either takes), and what the
bins' kernel treats apart, on volumes that take it: rows with more pieces in a
slab than the bins hold, rows of more pieces than a wave keeps in registers, rows
whose slabs do not follow each other or that start without a first visit, calls
with and without the packed iterate.

The separate commit kernel of a profiled call tells its route.  Both form the same
whole-number sums, so x is the same bits."""
import numpy as np
import pytest
import torch

from paper_1802_01070_amd import api, synth
from paper_1802_01070_amd._lib import PCT_DROP_PROFILE
from test_gpu_row_walk import records

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # (dims, pitch, r, rows, block, by bins, the longest row at least)
    ((362, 362, 60), (1.0, 1.0, 4.0), 176.0, 1300, 650, True, 430),    # 500 pieces at 45 degrees
    ((380, 380, 60), (1.0, 1.0, 4.0), 184.0, 1420, 710, False, 430),   # 523
    ((256, 256, 128), (1.0, 1.0, 1.0), 110.0, 1364, 682, True, 200),   # 2^23 voxels, 682 rows a block
    ((256, 256, 128), (1.0, 1.0, 1.0), 110.0, 1362, 681, False, 200),  # 681
    ((128, 128, 32), (1.0, 1.0, 1.0), 58.0, 12000, 8000, True, 100),   # blocks of many rows
    ((128, 128, 32), (1.0, 1.0, 1.0), 58.0, 6000, 3000, False, 100),
    ((40, 40, 6), (1.0, 1.0, 1.0), 31.5, 200, 24, False, 40),
    ((20, 300, 800), (4.0, 0.2, 1.0), 30.0, 800, 400, True, 100),      # more than four pieces a slab
    ((30, 30, 5000), (1.0, 1.0, 0.003), 20.0, 800, 400, True, 513),    # more than 512 pieces a row
]


@pytest.mark.parametrize("order", ["path", "turned", "shifted"])
@pytest.mark.parametrize("dims,pitch,r,n,block,bins,longest", CASES)
def test_both_routes_give_the_same_bits(dims, pitch, r, n, block, bins, longest, order):
    grid = synth.Grid(*dims, pitch=pitch)
    mlp = synth.MLPModel(u_in=-r, u_out=r)
    p, b = records(grid, mlp, n, 31)
    plan = api.Plan(grid, mlp, DEV, n_hint=block)
    rows = api.Rows(plan, api.Protons(p, DEV), "f16")
    off = rows.offsets.cpu().numpy()
    assert int(np.diff(off).max()) >= longest
    if order != "path":
        # the same pieces of every row in another order
        to = np.arange(int(off[-1]))
        for a, e in zip(off[:-1], off[1:]):
            if order == "turned":
                to[a + (e - a) // 2:e] = to[a + (e - a) // 2:e][::-1]
            elif e > a:
                to[a:e] = np.roll(to[a:e], 1)
        to = torch.from_numpy(to).to(DEV)
        rows.vox[:rows.nnz] = rows.vox[to]
        rows.chord[:rows.nnz] = rows.chord[to]
    bd = torch.from_numpy(b).to(DEV)

    def run(lanes, n_iter, flags=0):
        x = torch.linspace(0.5, 1.5, grid.nvox, device=DEV)
        api.pct_drop_iterate_rows(plan, rows, bd, x, block=block, lam=0.5, n_iter=n_iter, lanes=lanes, flags=flags)
        return x

    profiled = run(0, 1, PCT_DROP_PROFILE)
    assert (api.pct_profile_read(plan)[1][1] > 0) == bins
    assert torch.equal(profiled, run(64, 1))
    assert torch.equal(run(0, 8), run(64, 8))
    assert api.pct_device_status(plan) == 0
