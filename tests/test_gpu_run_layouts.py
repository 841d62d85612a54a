"""GPU test of queued steps across changes of the list's layout inside one call.

A state that re-sorts at every second or tenth rebuild has a tiled list after a
re-sort and slot entries at the other rebuilds.  Where the tiles outnumber the
8192 blocks up to which the passes of a step check the run themselves and the
slot passes do not (or, with eight keys per wave, the other way round), the
runs of one call change between that and the gate.  A gate that such a run left
set must not stop the next: one call of many steps has to take the same steps,
bit for bit, as one call per step, and track the oracle.

The list has room for slot entries from the start, so that no call ends early
to widen it.  Tolerance against the oracle: two FP64 runs differ by the order of
their sums, 1e-15 of a force at a step, which 40 steps of 0.005 at T = 1.5 grow
by less than e^(40 * 0.005 * 5) and a factor of a few hundred in the count of
terms; 1e-8 of a position is the bar, energies 1e-10 relative.
"""

import numpy as np
import pytest
import torch

import lj_inputs as li

pytestmark = pytest.mark.gpu


def _engine(q, v, L, **kw):
    from paper_1012_2677_amd import Engine

    e = Engine(q, v, L, device="cuda:0", **kw)
    e.plist.resize(e.plist.cell_stride, 32)
    e.plist.fill(e.state.list)
    e.prepare()
    return e


def _start(n_fcc, seed):
    q, L = li.jittered_fcc(n_fcc, amp=0.08, seed=seed)
    return q, li.maxwell_boltzmann(len(q), T=1.5, seed=seed), L


def _same(a, b):
    assert (a.rebuilds, int(a.state.resorts), a.step_count) == (b.rebuilds, int(b.state.resorts), b.step_count)
    assert torch.equal(a.id, b.id) and torch.equal(a.pos, b.pos) and torch.equal(a.vel, b.vel)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("step_run", [0, 1, 3])
def test_one_call_equals_a_call_per_step(precision, step_run):
    # 21^3 cells: 9261 one-cell tiles (gate), 1688 blocks of slot entries (folded)
    q, v, L = _start(30, seed=11)
    kw = dict(precision=precision, resort_every=2, tile_cells=1, cell_stride=1600)
    one = _engine(q, v, L, **kw)
    log1 = np.concatenate([one.step(1, sample_every=5) for _ in range(60)])
    assert one.rebuilds > 6
    many = _engine(q, v, L, step_run=step_run, **kw)
    log = many.step(60, sample_every=5)
    _same(many, one)
    assert log.shape == log1.shape == (12, 4)
    # (the sampled step's kick runs in another pass there, the sums do not)
    assert np.allclose(log, log1, rtol=1e-12, atol=0.0)


def test_one_call_tracks_the_oracle(ref):
    q, v, L = _start(30, seed=12)
    e = _engine(q, v, L, precision="fp64", resort_every=2, tile_cells=1, cell_stride=1600)
    log = e.step(40, sample_every=10)
    assert e.rebuilds > 4
    rq, rv, rlog, _ = ref.run(q, v, L, 40, dt=0.005, sample_every=10)
    d = e.positions() - rq
    assert np.abs(d - np.rint(d / L) * L).max() < 1e-8
    assert np.abs(e.velocities() - rv).max() < 1e-7
    assert np.allclose(log, rlog, rtol=1e-10, atol=1e-10 * np.abs(rlog).max())


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_recorded_frames_across_changes(precision):
    q, v, L = _start(30, seed=13)
    kw = dict(precision=precision, resort_every=2, tile_cells=1, cell_stride=1600)
    many, one = _engine(q, v, L, **kw), _engine(q, v, L, **kw)
    _, frames, built = many.step_record(40)
    for k in range(40):
        before = one.rebuilds
        one.step(1)
        assert built[k] == (one.rebuilds > before)
        at = torch.empty_like(one.pos)
        at[one.id.long()] = one.pos
        assert torch.equal(frames[k, :, :3], at[:, :3])
    assert built.sum() > 4
    _same(many, one)


def test_natural_size_across_resorts():
    # 1,314,036 particles: 9604 tiles (gate) against 5133 blocks (folded)
    q, v, L = _start(69, seed=14)
    kw = dict(precision="fp64", resort_every=10)
    one = _engine(q, v, L, **kw)
    for _ in range(25):
        one.step(4)
    assert one.state.resorts > 1
    many = _engine(q, v, L, **kw)
    many.step(100)
    assert torch.equal(many.id, one.id) and torch.equal(many.pos, one.pos) and torch.equal(many.vel, one.vel)
