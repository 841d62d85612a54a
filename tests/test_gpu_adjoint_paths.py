"""GPU test of the two forms of the adjoint pass.

With FP64 parameters that never re-sort and at least 16384 particles the
workspace has room for records of each slot's position and u, which the pass
gathers; otherwise it gathers from the arrays.  Both forms against the oracle,
from one isolated pair to shuffled boxes on either side of that number, and
against each other.

Tolerance: each sum has at most a few hundred FP64 terms of the scale of
hvp_scale, so its rounding is below 1e-13 of that scale; 1e-12 is the bar.
"""

import numpy as np
import pytest
import torch

import lj_inputs as li
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", ["pair", "below", "first", "shuffled"])
def test_records_and_arrays_agree_with_oracle(ref, case):
    from paper_1012_2677_amd.engine import Workspace, make_params

    if case == "pair":
        q, L = np.array([[0.2, 5.0, 5.0], [9.4, 5.1, 4.9]]), 10.0
    else:
        q, L = li.jittered_fcc(16, amp=0.12, seed=4)      # 16384
        if case != "first":
            q, _, _ = li.shuffle_labels(q, seed=4)
        if case == "below":
            q = q[:-1]
        if case == "shuffled":
            q = np.concatenate([q, [[0.5, 0.5, 0.5]]])
    n = len(q)
    rng = np.random.default_rng(5)
    u, out0 = rng.standard_normal((n, 3)), rng.standard_normal((n, 3))
    coef = (1.0, -0.3, 0.2, 0.7, -0.4)
    pairs = ref.pairs_brute(q, L, 2.5) if case == "pair" else ref.pairs_cells(q, L, 2.5)
    scale = np.maximum(G.hvp_scale(q, L, u, pairs), 1.0)
    Hr, dpr = ref.hvp(q, L, u)
    got = []
    for resort in (0, 1):
        s = G.Standalone(q, L)
        s.params = make_params(n, L, precision="fp64", resort_every=resort)
        s.ws = Workspace(s.params, G.device())
        s.bin()
        s.build()
        Hu, dp = s.hvp(u)
        assert G.elementwise_error(Hu, Hr, scale) <= 1e-12
        assert np.abs(dp - dpr).max() <= 1e-12 * max(np.abs(dpr).max(), scale.sum())
        got.append((Hu, *s.adjoint_kick(u, out0, coef)))
    for a, b in zip(*got):
        assert np.abs(a - b).max() <= 1e-12 * max(1.0, np.abs(a).max())
