"""GPU test of the cell grid at the sizes where its passes change.

One block up to 16384 particles and 4096 cells (4 slots per thread up to 4096
particles, 16 beyond), a one-launch scan up to 8192 cells, 16 or 128 cells per
block of the sort on either side of 131072 cells, and cells too crowded for the
sort's LDS: count, start and the stable order equal the oracle's bit for bit.
"""

import numpy as np
import pytest

import lj_inputs as li
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# (particles, box side): cells per axis = floor(side / 2.8)
CASES = [(1, 9.0), (65, 9.0), (4096, 20.0), (4097, 20.0), (16384, 33.0), (16385, 33.0),
         (5000, 45.0),      # 16^3 = 4096 cells, one block
         (5000, 48.0),      # 17^3, several launches
         (30000, 57.5),     # 20^3 = 8000 cells, one-launch scan
         (30000, 59.0),     # 21^3 = 9261
         (20000, 9.0),      # 27 cells of ~740: past the sort's LDS
         (150000, 141.0),   # 50^3 = 125000 cells
         (150000, 145.0)]   # 51^3 = 132651


@pytest.mark.parametrize("n,L", CASES)
def test_bin_cells_at_the_edges(ref, n, L):
    q = li.uniform_box(n, L, seed=n)
    s = G.Standalone(q, L)
    cell_of, count, start, order, _ = s.bin()
    r_cell, r_count, r_start, r_order = ref.bin_cells(q, L, s.grid.ncell)
    assert np.array_equal(cell_of, r_cell)
    assert np.array_equal(count, r_count)
    assert np.array_equal(start, r_start)
    assert np.array_equal(order, r_order)


@pytest.mark.parametrize("d", [1, 23, 24, 25, 40, 64])
def test_bin_cells_with_many_cells_in_a_wave(ref, d):
    # 64 slots in a row fall into d cells, each cell coming up again and again:
    # the lanes past the first 24 cells of a wave add to the counts alone
    n, L, m = 20011, 57.5, 20
    i = np.arange(n)
    c = (i // 64 * 37 + i % 64 % d * 13) % m**3
    corner = np.stack([c // (m * m), c // m % m, c % m], axis=1)
    q = (corner + 0.05 + 0.9 * np.random.default_rng(d).random((n, 3))) * (L / m)
    s = G.Standalone(q, L)
    assert s.grid.ncell == (m, m, m)
    cell_of, count, start, order, _ = s.bin()
    r_cell, r_count, r_start, r_order = ref.bin_cells(q, L, s.grid.ncell)
    assert np.array_equal(cell_of, r_cell)
    assert np.array_equal(count, r_count)
    assert np.array_equal(start, r_start)
    assert np.array_equal(order, r_order)
