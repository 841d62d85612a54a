"""GPU test of the list build's register sets and wave splits.

The build holds 384, 512, 768 or 1280 candidates in registers, chosen by the
mean neighbourhood, and gives a cell one wave or (grids of up to 1024 cells)
four.  Each set, on either side of that grid size, and a density past the
largest set: the slot rows equal the oracle's neighbour sets in the documented
order, and the tiled rows equal the slot rows entry by entry.
"""

import numpy as np
import pytest
import torch

import lj_inputs as li
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# (fcc cells, density): cells per axis and mean neighbourhood in the comment
CASES = [
    (7, 0.5),     # 5^3 cells, 296: four waves, 512
    (9, 0.8),     # 5^3, 631: four waves, 768
    (8, 0.8),     # 4^3, 864: four waves, 1280
    (12, 2.2),    # 5^3, 1493: past the largest set
    (16, 0.5),    # 11^3, 332: one wave, 512 in its tail
    (17, 0.5),    # 12^3, 306: one wave, 384
    (18, 0.7),    # 11^3, 473: one wave, 768
    (19, 0.7),    # 12^3, 429: one wave, 512
    (24, 1.6),    # 11^3, 1121: one wave, 1280
]


@pytest.mark.parametrize("n_fcc,rho", CASES)
def test_rows_of_every_register_set(ref, n_fcc, rho):
    from paper_1012_2677_amd import Engine

    a = li.lattice_constant(rho)
    q, L = li.jittered_fcc(n_fcc, amp=0.06 * a, rho=rho, seed=n_fcc)
    q, _, _ = li.shuffle_labels(q[:-5], seed=n_fcc)
    n = q.shape[0]
    keys = np.sort(np.random.default_rng(1).choice(n, 300, replace=False))

    s = G.Standalone(q, L)
    cell_of = s.bin()[0]
    s.build()
    k, p, code = G.rows_for_slots(s.plist, keys)
    rows = ref.neighbors_sample(q, L, keys, rs=2.8)
    order = np.where(code >= 13, code - 13, code + 14)     # own cell, then codes 14 .. 26, then 0 .. 12
    for i in range(len(keys)):
        r = p[k == i]
        assert np.array_equal(np.sort(r), rows[i])
        assert np.array_equal(np.lexsort((r, order[k == i])), np.arange(len(r)))
        assert np.all((cell_of[r] == cell_of[keys[i]]) == (code[k == i] == 13))

    v = li.maxwell_boltzmann(n, seed=2)
    t = Engine(q, v, L, precision="mixed", tile_cells=2)
    f = Engine(q, v, L, precision="mixed", list_layout="slots")
    t.prepare()
    f.prepare()
    assert int(t.state.list_tiled) == 1 and torch.equal(t.id, f.id)
    kt, pt = G.rows_for_slots_state(t, keys)
    kf, pf = G.rows_for_slots_state(f, keys)
    assert np.array_equal(kt, kf) and np.array_equal(pt, pf)
