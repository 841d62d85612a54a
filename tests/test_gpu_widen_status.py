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


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("resort_every", [2, 5])
def test_a_list_that_overflows_and_then_needs_room_settles(precision, resort_every):
    # 64 entries per cell: the first, tiled build overflows; the next one, without a
    # re-sort, asks for room.  Its overflow word must not be the first one's, or
    # a caller would grow the stride for ever and never widen.
    from paper_1012_2677_amd import Engine, _abi as A

    q, L = li.jittered_fcc(10, amp=0.08, seed=16)
    v = li.maxwell_boltzmann(len(q), T=1.0, seed=16)
    e = Engine(q, v, L, precision=precision, resort_every=resort_every, cell_stride=64, device="cuda:0")
    seen = []
    for _ in range(6):
        try:
            A.md_prepare(e.params, e.state, e.stream())
            break
        except A.MdError as err:
            e._sync_pointers()
            assert err.code == A.MD_ERR_CAPACITY
            seen.append(int(e.plist.status.cpu()[2]))
            e.plist.handle_capacity_error()
            e.plist.fill(e.state.list)
    else:
        raise AssertionError(f"not settled: {seen}")
    assert seen[:2] == [1, 0]
    e._sync_pointers()
    e.prepared = True
    e.step(30)
    w = Engine(q, v, L, precision=precision, resort_every=1, device="cuda:0")
    w.step(30)
    d = e.positions() - w.positions()
    assert abs(d - L * (d / L).round()).max() < (1e-8 if precision == "fp64" else 1e-4)


def test_a_droplet_in_an_empty_box(ref):
    # tiles of many cells at the mean density and few of them full
    import numpy as np
    from paper_1012_2677_amd import Engine

    q, L = li.jittered_fcc(16, amp=0.05, rho=0.8, seed=3)
    d = q - L / 2
    q = q[(d * d).sum(1) < (0.45 * L) ** 2] + L
    box = 3 * L
    q, v, _ = li.shuffle_labels(q, li.maxwell_boltzmann(len(q), T=0.7, seed=3), seed=4)
    for precision, tol in (("fp64", 1e-12), ("mixed", 1e-5)):
        for resort_every in (0, 1, 5):
            e = Engine(q, v, box, precision=precision, resort_every=resort_every, device="cuda:0")
            e.step(40)
            _, pe, w = ref.forces(e.positions(), box)
            en = e.energies()
            assert en[1] == pytest.approx(pe, rel=tol) and en[2] == pytest.approx(w, rel=tol, abs=tol * abs(pe))
            assert np.isfinite(e.velocities()).all()
