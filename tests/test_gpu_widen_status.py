"""GPU test of the list's status when a state has to widen its list.

A state with room for 16-bit entries that comes to a rebuild without a re-sort
stops with MD_ERR_CAPACITY and asks for 32-bit room.  No list was built then: the
status still holds the last list's totals and the stride it needs, with its
overflow word clear, and after the widening the steps go on as those of a state
that had the room from the start.
"""

import pytest
import torch

import lj_inputs as li

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_fcc", [10, 40])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_status_survives_the_request_for_room(n_fcc, precision):
    from paper_1012_2677_amd import Engine, _abi as A

    q, L = li.jittered_fcc(n_fcc, amp=0.08, seed=15)
    v = li.maxwell_boltzmann(len(q), T=1.5, seed=15)
    kw = dict(precision=precision, resort_every=3, cell_stride=1600, device="cuda:0")
    e, wide = Engine(q, v, L, **kw), Engine(q, v, L, **kw)
    wide.plist.resize(1600, 32)
    wide.plist.fill(wide.state.list)
    e.prepare()
    had = e.plist.status.cpu()
    assert e.state.list_tiled and int(had[0]) > len(q) and 0 < int(had[1]) <= 1600 and int(had[2]) == 0
    with pytest.raises(A.MdError) as err:
        A.md_step(e.params, e.state, 100, 0, None, e.stream())
    e._sync_pointers()
    assert err.value.code == A.MD_ERR_CAPACITY and 0 < e.step_count < 100
    assert torch.equal(e.plist.status.cpu(), had)
    e.plist.handle_capacity_error()
    e.plist.fill(e.state.list)
    e.step(40 - e.step_count)
    wide.step(40)
    assert torch.equal(e.pos, wide.pos) and torch.equal(e.vel, wide.vel)
