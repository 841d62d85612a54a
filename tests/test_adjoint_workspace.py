"""Workspace sizes and what the adjoint calls do with them.

The workspace that every call takes does not depend on resort_every, so one made
for some parameters serves the same ones with another; the records of the
adjoint passes are extra room that a caller may give.  md_hvp without dparam
leaves the workspace alone, so that such calls may share one across streams.
"""

import numpy as np
import pytest
import torch

import lj_inputs as li
from tests import gpu_util as G


def _params(n, L, **kw):
    from paper_1012_2677_amd.engine import make_params

    return make_params(n, L, **kw)


@pytest.mark.parametrize("n", [4000, 16383, 16384, 1_000_000])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_sizes(n, precision):
    from paper_1012_2677_amd import _abi as A

    L = (n / 0.5) ** (1.0 / 3.0)
    p = [_params(n, L, precision=precision, resort_every=r) for r in (0, 1, 10)]
    base = [A.md_workspace_bytes(x) for x in p]
    assert base[0] == base[1] == base[2] > 0
    for x in p:
        more = A.md_adjoint_workspace_bytes(x) - base[0]
        assert 48 * n <= more < 48 * n + 512 if n >= 16384 else more == 0
    assert A.md_adjoint_workspace_bytes(_params(n, 1.0)) == 0     # refused parameters


@pytest.mark.gpu
@pytest.mark.parametrize("resort", [0, 1])
def test_hvp_without_parameters_leaves_the_workspace(resort):
    from paper_1012_2677_amd import _abi as A
    from paper_1012_2677_amd.engine import Workspace

    q, L = li.jittered_fcc(17, amp=0.1, seed=6)
    s = G.Standalone(q, L)
    s.bin()
    s.build()
    s.params = _params(len(q), L, precision="fp64", resort_every=resort)
    s.ws = Workspace(s.params, G.device(), adjoint=True)
    u = torch.from_numpy(np.random.default_rng(7).standard_normal((3, len(q)))).to(G.device())
    Hu, dp = torch.empty_like(u), torch.empty(2, dtype=torch.float64, device=G.device())
    s.ws.buf.fill_(0x5A)

    def call(dparam):
        A.md_hvp(s.params, s.pos.data_ptr(), s.grid.c, s.plist.l, u.data_ptr(), Hu.data_ptr(), dparam, s.ws.ptr,
                 s.ws.nbytes, s.stream)
        torch.cuda.synchronize()
        return Hu.clone()

    alone = call(None)
    assert bool((s.ws.buf == 0x5A).all())
    both = call(dp.data_ptr())
    assert not bool((s.ws.buf == 0x5A).all())
    assert (alone - both).abs().max() <= 1e-12 * both.abs().max()


@pytest.mark.gpu
def test_a_workspace_serves_any_resort_every(ref):
    # made for parameters that re-sort, used with ones that do not
    from paper_1012_2677_amd.engine import Workspace

    q, L = li.jittered_fcc(17, amp=0.1, seed=8)
    u = np.random.default_rng(8).standard_normal((len(q), 3))
    out = []
    for adjoint in (False, True):
        s = G.Standalone(q, L)
        s.ws = Workspace(_params(len(q), L, precision="fp64", resort_every=1), G.device(), adjoint=adjoint)
        assert s.params.resort_every == 0
        s.bin()
        s.build()
        F, pw = s.forces()
        out.append((F, pw, *s.hvp(u), *s.adjoint_kick(u, u[::-1], (1.0, -0.3, 0.2, 0.7, -0.4)), s.param_grad()))
    for a, b in zip(*out):
        assert np.abs(a - b).max() <= 1e-12 * np.abs(a).max()
    Hr, dpr = ref.hvp(q, L, u)
    assert np.abs(out[0][2] - Hr).max() <= 1e-11 * np.abs(Hr).max()


@pytest.mark.gpu
def test_engines_carry_no_records():
    from paper_1012_2677_amd import Engine, _abi as A
    from paper_1012_2677_amd.autograd import Field

    q, L = li.jittered_fcc(17, amp=0.1, seed=9)
    e = Engine(q, np.zeros_like(q), L, precision="fp64", resort_every=0, device="cuda:0")
    assert e.ws.nbytes == A.md_workspace_bytes(e.params)
    assert Field(len(q), L, 1.0, 1.0).ws.nbytes == A.md_adjoint_workspace_bytes(e.params)
