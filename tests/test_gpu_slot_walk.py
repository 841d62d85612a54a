"""GPU test of the slot-list passes' two walks: as the slots lie, and in cell order.

A build without a re-sort measures how far apart slots lie that follow one
another: the library's sum equals the same sum over the grid's cells, and slots
in lattice order fall on one side of the rule, shuffled ones on the other, in
each precision.  On either walk the fused step passes take the same steps
whatever the host's waits, track the oracle (FP64) or the FP64 run (mixed), and
keep energy and virial at the oracle's; md_forces, which measures for itself
from 1,572,864 particles on, gives the oracle's forces and the same bits twice.

Tolerances: FP64 sums of up to a few hundred terms per particle, 1e-12 of their
scale; mixed pair terms carry 2^-24 each, 1e-5 of the scale.  A mixed run's
positions part from the FP64 run's by the force error, 1e-5 of a force of about
50 at a step, over 30 steps of 0.005: 30^2 / 2 * 0.005^2 * 5e-4 = 6e-6, times the
growth of e^(30 * 0.005 * 5); 1e-4 is the bar.
"""

import numpy as np
import pytest
import torch

import lj_inputs as li
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _box(n_fcc, shuffled, drop=0, seed=4):
    q, L = li.jittered_fcc(n_fcc, amp=0.08, seed=seed)
    v = li.maxwell_boltzmann(len(q), T=1.0, seed=seed)
    if shuffled:
        q, v, _ = li.shuffle_labels(q, v, seed=seed)
    return q[:len(q) - drop].copy(), v[:len(q) - drop].copy(), L


def _spread(cell_xyz, nc, samples=1024):
    n = len(cell_xyz)
    i = np.arange(samples, dtype=np.int64) * (n - 1) // samples
    j = np.minimum(i + 1, n - 1)
    d2 = 0
    for axis in range(3):
        a, b = (cell_xyz[k] >> (10 * axis) & 1023 for k in (i, j))
        d = np.abs(a - b)
        d = np.minimum(d, nc[axis] - d)
        d2 = d2 + d * d
    return int(np.minimum(d2, 64).sum())


def _engine(q, v, L, **kw):
    from paper_1012_2677_amd import Engine

    return Engine(q, v, L, device="cuda:0", **kw)


@pytest.mark.parametrize("case", ["one", "pair", "few", "ragged", "lattice", "shuffled", "slab"])
def test_spread_is_the_sum_over_the_cells(case):
    L = 9.0
    if case == "one":
        q = np.array([[1.0, 2.0, 3.0]])
    elif case == "pair":
        q = np.array([[0.2, 5.0, 5.0], [8.9, 8.9, 5.0]])
    elif case == "few":
        q = li.uniform_box(255, 40.0, seed=1) * 1.0
        L = 40.0
    elif case == "slab":
        L = np.array([9.0, 60.0, 17.0])
        q = np.random.default_rng(2).random((1500, 3)) * L
        q = q[np.argsort(q[:, 1])]
    else:
        q, _, L = _box(12, case == "shuffled", drop=1 if case == "ragged" else 0)
    # (an ideal gas: the particles of the uniform boxes overlap)
    e = _engine(q, np.zeros_like(q), L, resort_every=0, eps=1e-300)
    e.prepare()
    got = int(e.state.slot_spread)
    assert got == _spread(e.grid.cell_xyz.cpu().numpy().astype(np.int64), e.grid.ncell)
    if case == "lattice":
        assert got < 1024
    if case == "shuffled":
        assert got > 8 * 1024


# 1, 4 and 8 rounds per wave; particle numbers that fill no block
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("n_fcc,drop", [(10, 3), (34, 5), (42, 7)])
def test_states_on_either_walk(ref, precision, shuffled, n_fcc, drop):
    q, v, L = _box(n_fcc, shuffled, drop)
    kw = dict(precision=precision, resort_every=0)
    e = _engine(q, v, L, **kw)
    log = e.step(30, sample_every=10)
    limit = (1.25 if precision == "fp64" else 8.0) * 1024
    assert (e.state.slot_spread > limit) == shuffled
    assert e.rebuilds > 1 and e.state.resorts == 0
    # the same steps with a wait after each
    w = _engine(q, v, L, step_run=1, **kw)
    wlog = w.step(30, sample_every=10)
    assert torch.equal(e.pos, w.pos) and torch.equal(e.vel, w.vel) and np.array_equal(log, wlog)
    en = e.energies()
    at = e.positions()
    _, pe, vir = ref.forces(at, L)
    tol = 1e-12 if precision == "fp64" else 1e-5
    assert en[1] == pytest.approx(pe, rel=tol)
    assert en[2] == pytest.approx(vir, rel=tol, abs=tol * abs(pe))
    assert log[-1, 1] == pytest.approx(pe, rel=tol)
    if n_fcc == 10 or precision == "mixed":
        if precision == "fp64":
            rq = ref.run(q, v, L, 30, dt=0.005, sample_every=30)[0]
        else:
            r = _engine(q, v, L, precision="fp64", resort_every=0)
            r.step(30)
            rq = r.positions()
        d = at - rq
        assert np.abs(d - np.rint(d / L) * L).max() < (1e-8 if precision == "fp64" else 1e-4)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shuffled", [False, True])
def test_recorded_frames_on_either_walk(precision, shuffled):
    q, v, L = _box(16, shuffled, drop=3)
    kw = dict(precision=precision, resort_every=0)
    a, b = _engine(q, v, L, **kw), _engine(q, v, L, **kw)
    _, frames, _ = a.step_record(20)
    for k in range(20):
        b.step(1)
        assert torch.equal(frames[k, :, :3], b.pos[:, :3])
    assert torch.equal(a.pos, b.pos) and torch.equal(a.vel, b.vel)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("n", [1572863, 1572864, 1590001])
def test_forces_on_either_side_of_the_measured_size(ref, precision, shuffled, n):
    q, _, L = _box(74, shuffled)        # 1,620,896
    q = q[:n]
    s = G.Standalone(q, L, precision=precision)
    s.bin()
    s.build()
    F, pw = s.forces()
    F2, pw2 = s.forces()
    assert np.array_equal(F, F2) and np.array_equal(pw, pw2)
    sample = np.unique(np.random.default_rng(n).integers(0, n, 400))
    Fr, S, _, _, _ = ref.forces_sample(q, L, sample)
    assert G.force_error(F[sample], Fr, S) < (1e-12 if precision == "fp64" else 1e-5)
    # the other order of the same particles: the same sums in another order
    if n == 1590001:
        back = np.random.default_rng(9).permutation(n) if not shuffled else np.argsort(np.floor(q[:, 0]), kind="stable")
        o = G.Standalone(q[back], L, precision=precision)
        o.bin()
        o.build()
        G2, pw3 = o.forces()
        assert np.allclose(pw3, pw, rtol=1e-11 if precision == "fp64" else 1e-6)
        S2 = np.maximum(np.linalg.norm(F[back], axis=1), 1.0)
        assert (np.linalg.norm(G2 - F[back], axis=1) / S2).max() < (1e-10 if precision == "fp64" else 1e-3)


@pytest.mark.parametrize("n_fcc,shuffled", [(20, False), (20, True), (82, False)])
def test_mixed_slot_steps_on_either_side_of_the_fold(n_fcc, shuffled):
    # 1000 blocks check the run themselves, 8616 read the gate
    q, v, L = _box(n_fcc, shuffled, seed=3)
    v *= np.sqrt(1.5)
    a = _engine(q, v, L, precision="mixed", resort_every=0)
    a.step(14)
    b = _engine(q, v, L, precision="mixed", resort_every=0, step_run=1)
    b.step(14)
    assert a.rebuilds == b.rebuilds > 1
    assert torch.equal(a.pos, b.pos) and torch.equal(a.vel, b.vel)
