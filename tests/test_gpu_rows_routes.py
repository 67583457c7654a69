"""Stored rows on either side of the rules that choose slab bins or atomics for a
call without named lanes: the length of a path at 45 degrees (512 pieces), and the
rows of a block against the volume (one for 16384 voxels); and, by bins, rows of
more pieces than the rule reckons with.  Both routes form the same whole-number
sums, so x is the same bits."""
import pytest
import torch

from paper_1802_01070_amd import api, synth
from test_gpu_row_walk import records

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # (dims, pitch, r, rows, block, the longest row at least)
    ((380, 380, 2), (1.0, 1.0, 4.0), 180.0, 90, 30, 430),     # 511 pieces at 45 degrees: bins
    ((386, 386, 2), (1.0, 1.0, 4.0), 184.0, 90, 30, 430),     # 522: atomics
    ((128, 128, 32), (1.0, 1.0, 1.0), 60.0, 96, 32, 100),     # 2^19 voxels, 32 rows: bins
    ((128, 128, 32), (1.0, 1.0, 1.0), 60.0, 93, 31, 100),     # 31: atomics
    ((30, 30, 2000), (1.0, 1.0, 0.003), 20.0, 250, 128, 513),   # steep and finely sliced, by bins
]


@pytest.mark.parametrize("chord", ["f32", "bf16"])
@pytest.mark.parametrize("dims,pitch,r,n,block,longest", CASES)
def test_both_routes_give_the_same_bits(dims, pitch, r, n, block, longest, chord):
    grid = synth.Grid(*dims, pitch=pitch)
    mlp = synth.MLPModel(u_in=-r, u_out=r)
    p, b = records(grid, mlp, n, 31)
    plan = api.Plan(grid, mlp, DEV, n_hint=block)
    rows = api.Rows(plan, api.Protons(p, DEV), chord)
    assert int(rows.offsets.diff().max()) >= longest
    bd = torch.from_numpy(b).to(DEV)

    def run(lanes):
        x = torch.linspace(0.5, 1.5, grid.nvox, device=DEV)
        api.pct_drop_iterate_rows(plan, rows, bd, x, block=block, lam=0.5, n_iter=3, lanes=lanes)
        return x

    assert torch.equal(run(0), run(64))
    assert api.pct_device_status(plan) == 0
