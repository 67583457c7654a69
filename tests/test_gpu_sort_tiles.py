"""The sort at the edges of its tiles and of the sizes where its digits are 8
bits for want of room for counts (up to 2048 records, and some sizes below
14337): the order and the records are bit-exact."""
import numpy as np
import pytest

from paper_1802_01070_amd import synth
from test_gpu_sort_scan import check_sorted, edge_records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2048, 2049, 4608, 4609, 9217, 14336, 14337])
@pytest.mark.parametrize("n_angles,slab_mm", [(40, 4.0), (4096, 30.0 / 4096)])
def test_tile_edges(n, n_angles, slab_mm):
    grid = synth.Grid(16, 16, 20, pitch=(1.0, 1.0, 1.5))
    rng = np.random.default_rng(n)
    check_sorted(grid, edge_records(n, rng, grid), rng.random(n).astype(np.float32), n_angles, slab_mm)
