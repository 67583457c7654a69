"""Rounding of the FP64 row norms against the same polylines cut in extended
precision, on a grid whose voxel sizes are no binary fractions.

Vertices lie up to 127 mm from the origin, where a coordinate rounds by 4e-15 mm
rms (2^-46 / sqrt 12), and a chord's two ends take about one and a half such errors
each: over the 250 chords of 0.6 mm of a row the squares sum up to 1.6e-13 in 100,
1.6e-15 rms.  2.2e-15 leaves room for the directions' sines; coordinates that are
scaled to voxels on the way (rounded once more, and 1 / pitch with them) give
3.2e-15."""
import numpy as np
import pytest
import torch

from paper_1802_01070_amd import api, synth
from test_gpu_row_walk import records

pytestmark = pytest.mark.gpu
L = np.longdouble


def squares(grid, mlp, table, p, i):
    """||a_i||^2 of row i, consecutive parts in a voxel merged."""
    f = {k: L(v[i]) for k, v in p.items()}
    gantry = float(p["gantry"][i])
    cs, sn = L(np.cos(gantry)), L(np.sin(gantry))
    u = np.minimum(mlp.u_in + mlp.step * np.arange(table.shape[0]), mlp.u_out).astype(L)
    c = table.T.astype(L)
    t = c[0] * f["t_in"] + c[1] * f["th_in"] + c[2] * f["t_out"] + c[3] * f["th_out"]
    v = c[0] * f["v_in"] + c[1] * f["ph_in"] + c[2] * f["v_out"] + c[3] * f["ph_out"]
    w = np.stack([u * cs - t * sn, u * sn + t * cs, v], 1)
    total, voxel, chord = L(0), None, L(0)
    for a, b in zip(w[:-1], w[1:]):
        d = b - a
        cuts = [L(0), L(1)]
        for ax in range(3):
            at = (np.array([a[ax], b[ax]]) - L(grid.lo[ax])) / L(grid.pitch[ax])
            for k in range(int(np.floor(at.min())), int(np.ceil(at.max())) + 1):
                cut = (L(grid.lo[ax]) + k * L(grid.pitch[ax]) - a[ax]) / d[ax]
                if 0 < cut < 1:
                    cuts.append(cut)
        cuts.sort()
        for lo, hi in zip(cuts[:-1], cuts[1:]):
            middle = a + L(0.5) * (lo + hi) * d
            at = tuple(int(np.floor((middle[ax] - L(grid.lo[ax])) / L(grid.pitch[ax]))) for ax in range(3))
            if at != voxel:
                total += chord * chord
                voxel, chord = at, L(0)
            if all(0 <= k < n for k, n in zip(at, (grid.nx, grid.ny, grid.nz))):
                chord += (hi - lo) * np.sqrt((d * d).sum())
    return total + chord * chord


def test_row_norms_round_no_more_than_their_vertices():
    assert np.finfo(L).eps < 1e-18
    grid = synth.Grid(190, 170, 20, pitch=(0.7, 1.3, 2.5))
    mlp = synth.MLPModel(u_in=-90.0, u_out=90.0)
    n = 300
    p, _ = records(grid, mlp, n, 41)
    # nothing comes back to a voxel: the squares of consecutive parts are the norm
    for k in ("ph_in", "ph_out"):
        p[k] = np.abs(p[k]) * 0.2 + np.float32(0.01)
    p["v_out"] = p["v_in"] + np.float32(0.5 * mlp.depth) * (p["ph_in"] + p["ph_out"])
    plan = api.Plan(grid, mlp, "cuda:0")
    vox, _, nnz = (v.cpu().numpy() for v in api.pct_mlp_trace(plan, api.Protons(p), max_nnz=1024))
    single = np.array([len(set(vox[i, :nnz[i]])) == nnz[i] for i in range(n)])
    assert single.sum() > 250
    x = torch.ones(grid.nvox, dtype=torch.float64, device="cuda:0")
    n2 = api.pct_forward(plan, api.Protons(p), x, with_norm=True)[1].cpu().numpy()
    rows = np.flatnonzero(single & (nnz > 0))
    ref = np.array([squares(grid, mlp, plan.table(), p, i) for i in rows])
    diff = n2[rows].astype(L) - ref
    assert float(np.sqrt((diff * diff).sum() / (ref * ref).sum())) <= 2.2e-15
