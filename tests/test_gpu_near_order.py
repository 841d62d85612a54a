"""GPU test of slot lists of a state that re-sorts now and then.

Between two re-sorts the passes walk the keys as the slots lie for the first
rebuilds (48 in FP64) and in cell order after those: energy and virial of the
state reached equal the oracle's at its positions, and a short FP64 run tracks
the oracle's, on shuffled labels.
"""

import numpy as np
import pytest
import torch  # noqa: F401  (loads the HIP runtime that the package then shares)

import lj_inputs as li
from paper_1012_2677_amd import Engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,resort_every,steps,least", [
    ("fp64", 3, 60, 4), ("fp64", 1000, 400, 50), ("mixed", 3, 60, 4), ("mixed", 1000, 100, 8)])
def test_state_between_resorts_matches_oracle(ref, precision, resort_every, steps, least):
    q, L = li.fcc_lattice(10)
    v = li.maxwell_boltzmann(q.shape[0], T=1.0, seed=8)
    q, v, _ = li.shuffle_labels(q, v, seed=9)
    e = Engine(q, v, L, device="cuda:0", precision=precision, resort_every=resort_every)
    e.step(steps)
    assert e.state.rebuilds > least and e.state.resorts < e.state.rebuilds
    en = e.energies()
    _, pe, w = ref.forces(e.positions(), L)
    tol = 1e-12 if precision == "fp64" else 1e-5
    assert en[1] == pytest.approx(pe, rel=tol)
    assert en[2] == pytest.approx(w, rel=tol, abs=tol * abs(pe))
    if precision == "fp64" and steps <= 60:
        rq = ref.run(q, v, L, steps, dt=0.005, sample_every=steps)[0]
        d = e.positions() - rq
        assert np.abs(d - np.rint(d / L) * L).max() < 1e-8
