"""GPU test of the cell grid on either side of 1,048,576 cells, where the order
of a cell's slots is made by another pass: count, start and the stable order
equal the oracle's bit for bit, sparse, ordinary and with one crowded cell."""

import numpy as np
import pytest

from tests import gpu_util as G

pytestmark = pytest.mark.gpu


# 101^3 = 1030301 and 102^3 = 1061208 cells
@pytest.mark.parametrize("L", [283.0, 286.0])
@pytest.mark.parametrize("n,most", [(70001, 0), (3000017, 0), (300007, 4096), (300007, 4500)])
def test_bin_cells_on_large_grids(ref, L, n, most):
    rng = np.random.default_rng(n + most)
    q = rng.random((n, 3)) * L
    if most:
        side = L / int(L / 2.8)
        q[rng.permutation(n)[:most]] = (np.array([50, 7, 100]) + 0.02 + 0.96 * rng.random((most, 3))) * side
    s = G.Standalone(q, L, cell_stride=16)
    cell_of, count, start, order, _ = s.bin()
    r_cell, r_count, r_start, r_order = ref.bin_cells(q, L, s.grid.ncell)
    assert np.array_equal(cell_of, r_cell) and np.array_equal(count, r_count)
    assert np.array_equal(start, r_start) and np.array_equal(order, r_order)
