"""GPU test of the two ways in which queued steps learn that the run has stopped.

Passes of up to 8192 blocks read the step before's maxima themselves, larger ones
look at a gate that a pass of its own sets.  The same box as 21,952 one-cell
tiles (gate) and as the automatic tiles (folded) must take the same steps
bitwise, rebuild at the same ones, and equal a wait after every step; slot lists
on either side of the limit against a wait after every step.

The host reads a run's flags from pinned memory that the device writes, or, given
ordinary memory or none, by a copy: the same steps either way.
"""

import pytest
import torch

import lj_inputs as li

pytestmark = pytest.mark.gpu


def _run(q, v, L, steps, **kw):
    from paper_1012_2677_amd import Engine

    e = Engine(q, v, L, device="cuda:0", **kw)
    e.step(steps, sample_every=7)
    return e


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_gate_and_fold_take_the_same_steps(precision):
    q, L = li.jittered_fcc(40, amp=0.08, seed=2)
    v = li.maxwell_boltzmann(len(q), T=1.5, seed=2)
    # (a stride that no cell outgrows: an overflow counts one more rebuild)
    runs = [_run(q, v, L, 25, precision=precision, cell_stride=1600, **kw)
            for kw in (dict(tile_cells=1), dict(), dict(step_run=1), dict(tile_cells=1, step_run=3))]
    assert runs[0].state.tile_cells == 1 and runs[1].state.tile_cells > 1
    assert runs[0].rebuilds > 2
    for r in runs[1:]:
        assert r.rebuilds == runs[0].rebuilds
        assert torch.equal(r.id, runs[0].id)
        assert torch.equal(r.pos, runs[0].pos) and torch.equal(r.vel, runs[0].vel)


@pytest.mark.parametrize("n_fcc", [20, 82])
def test_slot_lists_on_either_side_of_the_fold(n_fcc):
    q, L = li.jittered_fcc(n_fcc, amp=0.08, seed=3)
    v = li.maxwell_boltzmann(len(q), T=1.5, seed=3)
    a = _run(q, v, L, 14, precision="fp64", resort_every=0)
    b = _run(q, v, L, 14, precision="fp64", resort_every=0, step_run=1)
    assert a.rebuilds == b.rebuilds > 1
    assert torch.equal(a.pos, b.pos) and torch.equal(a.vel, b.vel)


@pytest.mark.parametrize("rule", ["half_skin", "dutc_ldc"])
def test_flags_through_pinned_ordinary_and_no_memory(rule):
    from paper_1012_2677_amd import Engine

    q, L = li.jittered_fcc(10, amp=0.08, seed=5)
    v = li.maxwell_boltzmann(len(q), T=1.5, seed=5)
    runs = []
    for memory in ("pinned", "ordinary", "none"):
        e = Engine(q, v, L, precision="fp64", rebuild_rule=rule, device="cuda:0")
        if memory != "pinned":
            e.host_scratch = torch.zeros(16, dtype=torch.int64) if memory == "ordinary" else None
            e.state.host_scratch = e.host_scratch.data_ptr() if memory == "ordinary" else None
        log = e.step(60, sample_every=10)
        runs.append((e, log))
    for e, log in runs[1:]:
        assert e.rebuilds == runs[0][0].rebuilds > 3
        assert (log == runs[0][1]).all() and torch.equal(e.pos, runs[0][0].pos)
