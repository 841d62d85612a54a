"""The work that programs have this package do, as cases that can be timed.

Four kinds, each through the package's public entry points:

  step    a simulation advanced by `Engine.step` with the energy sampled, as a
          production run advances it between two stored frames
  list    the C ABI on one stored configuration: pack, bin, pair list, forces
  energy  `LJEnergy` forward and backward (force matching: a gradient through
          the energy and the forces)
  traj    `TrajectoryMeanPE` forward and backward (a gradient through a run)

Sizes span a few thousand particles to 32 million.  Particles start on an fcc
lattice with every coordinate displaced uniformly by at most 8% of the lattice
constant (a disordered input without overlaps) and Maxwell-Boltzmann
velocities at T = 1; `missing` of the sites are left empty, which makes the
particle number odd and the density ragged, and `shuffled` particles come in
random order.
"""

import math

import numpy as np
import torch

from paper_1012_2677_amd import Engine, Grid, LJEnergy, PairList, TrajectoryMeanPE, Workspace, make_params, stream_handle
from paper_1012_2677_amd import _abi as A

RC, RS, DT = 2.5, 2.8, 0.005
BASIS = ((0.0, 0.0, 0.0), (0.5, 0.5, 0.0), (0.5, 0.0, 0.5), (0.0, 0.5, 0.5))


def _case(kind, nx, ny, nz, rho=0.5, missing=0.0, shuffled=False, precision="fp64", resort=1, steps=0, sample=0, ckpt=0,
          name=None):
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, rho=rho, missing=missing, shuffled=shuffled, precision=precision,
             resort=resort, steps=steps, sample=sample, ckpt=ckpt)
    return c if name is None else dict(name=name, **c)


def listed():
    return [
        # lj4k: the smallest workload, where launches and waits are the time
        _case("step", 10, 10, 10, steps=100, sample=10, name="step_4k_fp64"),
        # a dense liquid in a ragged box, particle number not round, mixed
        _case("step", 15, 14, 13, rho=0.8, missing=0.01, precision="mixed", steps=50, sample=10,
              name="step_11k_liquid_mixed"),
        # lj256k, the mid-size box
        _case("step", 40, 40, 40, steps=40, sample=20, name="step_256k_fp64"),
        # the paper's 500,000-particle box without the re-sort (ids are slots)
        _case("step", 50, 50, 50, resort=0, steps=20, sample=20, name="step_500k_unsorted_fp64"),
        # lj4m, double precision throughout
        _case("step", 100, 100, 100, steps=20, sample=20, name="step_4m_fp64"),
        # lj32m, the headline workload
        _case("step", 200, 200, 200, precision="mixed", steps=20, sample=20, name="step_32m_mixed"),
        # analysis of one stored configuration in arbitrary particle order
        _case("list", 66, 67, 65, missing=0.003, shuffled=True, precision="mixed", name="list_1m_shuffled_mixed"),
        # force matching on a small box, as in a fitting loop over many boxes
        _case("energy", 8, 8, 8, name="energy_2k"),
        # force matching on a liquid whose particles come in no order
        _case("energy", 25, 24, 26, rho=0.8, missing=0.01, shuffled=True, name="energy_62k_liquid_shuffled"),
        # and on a large box
        _case("energy", 64, 64, 64, name="energy_1m"),
        # a gradient through a short run of a small box
        _case("traj", 10, 10, 10, steps=40, ckpt=20, name="traj_4k"),
        # and of lj256k with its checkpoint interval
        _case("traj", 40, 40, 40, steps=60, ckpt=20, name="traj_256k"),
    ]


def draw(rng):
    kind = rng.choice(["step", "step", "step", "list", "energy", "traj"])
    most = {"step": 4.0e6, "list": 2.0e6, "energy": 1.0e6, "traj": 2.5e5}[kind]
    rho = rng.choice([0.5, 0.5, rng.uniform(0.4, 0.85)])
    # at least three cells of side RS on every axis
    least = math.ceil(3.0 * RS / (4.0 / rho) ** (1.0 / 3.0)) + 1
    n = math.exp(rng.uniform(math.log(2048.0), math.log(most)))
    side = (n / 4.0) ** (1.0 / 3.0)
    nx, ny = (max(least, round(side * rng.uniform(0.8, 1.25))) for _ in range(2))
    nz = max(least, round(n / 4.0 / (nx * ny)))
    c = _case(kind, nx, ny, nz, rho=rho, missing=rng.choice([0.0, rng.uniform(0.001, 0.05)]),
              shuffled=rng.random() < 0.4)
    if kind in ("step", "list"):
        c["precision"] = rng.choice(["fp64", "mixed"])
    if kind == "step":
        c["resort"] = rng.choice([1, 1, 1, 10, 0])
        c["steps"] = rng.randrange(10, 41)
        c["sample"] = rng.choice([5, 10, 20])
    if kind == "traj":
        c["steps"] = rng.randrange(20, 61)
        c["ckpt"] = rng.choice([10, 20])
    return c


# -- inputs -----------------------------------------------------------------------
def _lattice(case):
    return (4.0 / case["rho"]) ** (1.0 / 3.0)


def _box(case):
    a = _lattice(case)
    return [case["nx"] * a, case["ny"] * a, case["nz"] * a]


def _count(case):
    sites = 4 * case["nx"] * case["ny"] * case["nz"]
    return sites - int(case["missing"] * sites)


def _inputs(case, seed):
    """Positions in the box and velocities (N, 3), float64, on the GPU."""
    dev = torch.device("cuda")
    g = torch.Generator(dev).manual_seed(int(seed))
    f = dict(dtype=torch.float64, device=dev)
    a = _lattice(case)
    axes = [torch.arange(case[k], **f) for k in ("nx", "ny", "nz")]
    corners = torch.stack(torch.meshgrid(*axes, indexing="ij"), dim=-1).reshape(-1, 1, 3)
    q = ((corners + torch.tensor(BASIS, **f)) * a).reshape(-1, 3)
    q += (0.16 * a) * (torch.rand(q.shape, generator=g, **f) - 0.5)
    if case["missing"] > 0.0 or case["shuffled"]:
        pick = torch.randperm(q.shape[0], generator=g, device=dev)[:_count(case)]
        q = q[pick if case["shuffled"] else pick.sort().values]
    box = torch.tensor(_box(case), **f)
    q -= box * torch.floor(q / box)
    q = torch.where(q >= box, q - box, q)
    v = torch.randn(q.shape, generator=g, **f)
    v -= v.mean(dim=0)
    v *= math.sqrt(3.0 * (q.shape[0] - 1) / float((v * v).sum()))
    return q.contiguous(), v


def _parameters():
    f = dict(dtype=torch.float64, device="cuda")
    return torch.tensor(1.0, **f), torch.tensor(1.0, **f)


def _cotangents(case, n, seed):
    """What a loss hands back for the energy and the forces."""
    dev = torch.device("cuda")
    g = torch.Generator(dev).manual_seed(int(seed) + 7919)
    return (torch.tensor(0.3, dtype=torch.float64, device=dev),
            torch.randn((n, 3), generator=g, dtype=torch.float64, device=dev))


def prepare(case, seed):
    q, v = _inputs(case, seed)
    s = dict(case=case)
    if case["kind"] == "step":
        eng = Engine(q.cpu().numpy(), v.cpu().numpy(), _box(case), rc=RC, rs=RS, dt=DT, precision=case["precision"],
                     resort_every=case["resort"])
        eng.prepare()
        s["engine"] = eng
    elif case["kind"] == "list":
        n = q.shape[0]
        p = make_params(n, _box(case), rc=RC, rs=RS, precision=case["precision"], resort_every=0)
        grid = Grid(p, q.device)
        s.update(q=q, params=p, grid=grid, plist=PairList(p, grid.ncell, q.device), ws=Workspace(p, q.device),
                 pos=torch.empty((n, 4), dtype=torch.float64, device=q.device),
                 force=torch.empty((3, n), dtype=torch.float32 if case["precision"] == "mixed" else torch.float64,
                                   device=q.device),
                 pe_w=torch.empty(2, dtype=torch.float64, device=q.device))
    else:
        eps, sigma = _parameters()
        s.update(q=q.requires_grad_(True), v=v, eps=eps.requires_grad_(True), sigma=sigma.requires_grad_(True))
        if case["kind"] == "energy":
            s["cot"] = _cotangents(case, q.shape[0], seed)
    return s


# -- one pass ---------------------------------------------------------------------
def run(state):
    case = state["case"]
    return {"step": _run_step, "list": _run_list, "energy": _run_energy, "traj": _run_traj}[case["kind"]](case, state)


def _run_step(case, s):
    eng = s["engine"]
    log = eng.step(case["steps"], sample_every=case["sample"])
    # the frame a program stores: positions and velocities in the original
    # particle order, in single precision after a mixed-precision run
    ids = eng.id.long()
    pos, vel = torch.empty_like(eng.pos), torch.empty_like(eng.vel)
    pos[ids] = eng.pos
    vel[:, ids] = eng.vel
    if case["precision"] == "mixed":
        return dict(pos=pos[:, :3].float(), vel=vel.float(), energy=log.astype(np.float32))
    return dict(pos=pos[:, :3], vel=vel, energy=log)


def _run_list(case, s):
    p, grid, plist, ws = s["params"], s["grid"], s["plist"], s["ws"]
    st = stream_handle(s["q"].device)
    A.md_pack_positions(p, s["q"].data_ptr(), s["pos"].data_ptr(), st)
    A.md_bin_cells(p, s["pos"].data_ptr(), grid.c, ws.ptr, ws.nbytes, st)
    A.md_build_pairlist(p, s["pos"].data_ptr(), grid.c, plist.l, ws.ptr, ws.nbytes, st)
    A.md_forces(p, s["pos"].data_ptr(), grid.c, plist.l, s["force"].data_ptr(), s["pe_w"].data_ptr(), ws.ptr, ws.nbytes,
                st)
    energy = s["pe_w"].float() if case["precision"] == "mixed" else s["pe_w"]
    return dict(force=s["force"], energy=energy, start=grid.start, order=grid.order, counts=plist.counts)


def _run_energy(case, s):
    U, F = LJEnergy.apply(s["q"], s["eps"], s["sigma"], _box(case), RC, RS)
    gq, ge, gs = torch.autograd.grad((U, F), (s["q"], s["eps"], s["sigma"]), s["cot"])
    return dict(U=U, F=F, q=gq, eps=ge, sigma=gs)


def _run_traj(case, s):
    O = TrajectoryMeanPE.apply(s["q"], s["v"], s["eps"], s["sigma"], _box(case), case["steps"], case["ckpt"], DT, RC, RS)
    gq, ge, gs = torch.autograd.grad(O, (s["q"], s["eps"], s["sigma"]))
    return dict(O=O, q=gq, eps=ge, sigma=gs)


# -- what a pass cannot do without ------------------------------------------------
def work(case):
    """Bytes: positions and velocities read and written once per step (their
    adjoints too on the way back); list and energy read positions and write
    forces (energy: reads cotangents and writes the position gradient as well).
    Operations: 30 per pair within rc of one force evaluation, 60 of its
    adjoint; 10 per candidate pair of a list within rs."""
    n = _count(case)
    density = n / float(np.prod(_box(case)))
    half = lambda r: 0.5 * n * density * 4.0 / 3.0 * math.pi * r ** 3  # noqa: E731
    pairs, listed_pairs = half(RC), half(RS)
    if case["kind"] == "step":
        return dict(bytes=96.0 * n * case["steps"], flops=(30.0 * pairs + 30.0 * n) * case["steps"])
    if case["kind"] == "list":
        # the list itself is an output: four bytes per entry, both directions
        return dict(bytes=n * (24.0 + (12.0 if case["precision"] == "mixed" else 24.0) + 16.0) + 8.0 * listed_pairs,
                    flops=30.0 * pairs + 10.0 * listed_pairs)
    if case["kind"] == "energy":
        return dict(bytes=96.0 * n, flops=90.0 * pairs + 10.0 * listed_pairs)
    # a forward run, its recomputation from the checkpoints, and the sweep back
    return dict(bytes=(96.0 * 2 + 120.0) * n * case["steps"], flops=(30.0 * 2 + 60.0) * pairs * case["steps"])


# -- the same in plain torch, 64 bits ---------------------------------------------
class _Pairs:
    """Pairs i < j within `reach` by cells, minimum-image; kept while no
    particle has moved more than (reach - RC) / 2."""

    def __init__(self, box, reach):
        self.box, self.reach, self.at = box, reach, None

    def __call__(self, q):
        if self.at is not None:
            d = q - self.at
            d = d - self.box * torch.round(d / self.box)
            if 2.0 * float(d.square().sum(1).max().sqrt()) < self.reach - RC:
                return self.i, self.j
        self.at = q.clone()
        self.i, self.j = self._find(q)
        return self.i, self.j

    def _find(self, q):
        dev, n = q.device, q.shape[0]
        nc = torch.floor(self.box / self.reach).long().clamp(min=1)
        if int(nc.min()) < 3:
            i, j = torch.triu_indices(n, n, 1, device=dev)
            return self._close(q, i, j)
        dims = [int(x) for x in nc]
        inside = q - self.box * torch.floor(q / self.box)
        c = torch.minimum((inside * (nc / self.box)).long(), nc - 1)
        cell = (c[:, 0] * dims[1] + c[:, 1]) * dims[2] + c[:, 2]
        ncell = dims[0] * dims[1] * dims[2]
        order = torch.argsort(cell, stable=True)
        count = torch.bincount(cell, minlength=ncell)
        start = torch.cumsum(count, 0) - count
        width = int(count.max())
        table = torch.full((ncell, width), -1, dtype=torch.long, device=dev)
        cs = cell[order]
        table[cs, torch.arange(n, device=dev) - start[cs]] = order
        every = torch.arange(ncell, device=dev)
        xyz = torch.stack([every // (dims[1] * dims[2]), (every // dims[2]) % dims[1], every % dims[2]], 1)
        out_i, out_j = [], []
        chunk = max(1, 20_000_000 // (width * width))
        for code in range(13, 27):
            shift = torch.tensor([code // 9 - 1, (code // 3) % 3 - 1, code % 3 - 1], device=dev)
            m = (xyz + shift) % nc
            other = (m[:, 0] * dims[1] + m[:, 1]) * dims[2] + m[:, 2]
            for k in range(0, ncell, chunk):
                a, b = table[k:k + chunk], table[other[k:k + chunk]]
                i = a[:, :, None].expand(-1, -1, width).reshape(-1)
                j = b[:, None, :].expand(-1, width, -1).reshape(-1)
                keep = (i >= 0) & (j >= 0)
                if code == 13:
                    keep &= i < j
                i, j = self._close(q, i[keep], j[keep])
                out_i.append(i)
                out_j.append(j)
        return torch.cat(out_i), torch.cat(out_j)

    def _close(self, q, i, j):
        d = q[j] - q[i]
        d = d - self.box * torch.round(d / self.box)
        near = d.square().sum(1) < self.reach ** 2
        return i[near], j[near]


def _energy(q, eps, sigma, box, pairs):
    """(U, W) of the truncated Lennard-Jones potential, differentiable."""
    i, j = pairs(q.detach())
    d = q[j] - q[i]
    d = d - box * torch.round(d / box)
    r2 = d.square().sum(1)
    r2 = r2[r2 < RC * RC]
    x2 = (sigma / RC) ** 2
    c2, c0 = 6.0 * x2 ** 7 - 3.0 * x2 ** 4, 4.0 * x2 ** 3 - 7.0 * x2 ** 6
    s2 = r2 / sigma ** 2
    s6 = s2 ** -3
    U = (4.0 * eps * (s6 * s6 - s6 + c2 * s2 + c0)).sum()
    W = (4.0 * eps * (12.0 * s6 * s6 - 6.0 * s6 - 2.0 * c2 * s2)).sum()
    return U, W


def _energy_force(q, eps, sigma, box, pairs):
    with torch.enable_grad():
        x = q.detach().requires_grad_(True)
        U, W = _energy(x, eps, sigma, box, pairs)
        (g,) = torch.autograd.grad(U, x)
    return U.detach(), W.detach(), -g


def exact(case, seed):
    n = _count(case)
    if n > 5_000_000 or (case["kind"] == "traj" and n * case["steps"] > 20_000_000):
        return None
    q, v = _inputs(case, seed)
    eps, sigma = _parameters()
    box = torch.tensor(_box(case), dtype=torch.float64, device=q.device)
    if case["kind"] == "step":
        return _exact_step(case, q, v, eps, sigma, box)
    pairs = _Pairs(box, RS)
    if case["kind"] == "list":
        U, W, F = _energy_force(q, eps, sigma, box, pairs)
        return dict(force=F.t().contiguous(), energy=torch.stack([U, W]), start=None, order=None, counts=None)
    q.requires_grad_(True)
    eps.requires_grad_(True)
    sigma.requires_grad_(True)
    if case["kind"] == "energy":
        gU, gF = _cotangents(case, n, seed)
        U, _ = _energy(q, eps, sigma, box, pairs)
        (g,) = torch.autograd.grad(U, q, create_graph=True)
        gq, ge, gs = torch.autograd.grad((U, -g), (q, eps, sigma), (gU, gF))
        return dict(U=U.detach(), F=-g.detach(), q=gq, eps=ge, sigma=gs)
    return _exact_traj(case, q, v, eps, sigma, box)


def _exact_step(case, q, v, eps, sigma, box):
    pairs = _Pairs(box, RC + 0.5)
    rows = []
    _, _, F = _energy_force(q, eps, sigma, box, pairs)
    for k in range(1, case["steps"] + 1):
        v = v + 0.5 * DT * F
        q = q + DT * v
        q = q - box * torch.floor(q / box)
        U, W, F = _energy_force(q, eps, sigma, box, pairs)
        v = v + 0.5 * DT * F
        if case["sample"] > 0 and k % case["sample"] == 0:
            ke = 0.5 * v.square().sum()
            rows.append(torch.stack([ke, U, W, ke + U]))
    log = torch.stack(rows).cpu().numpy() if rows else np.zeros((0, 4))
    return dict(pos=q, vel=v.t().contiguous(), energy=log)


def _exact_traj(case, q, v, eps, sigma, box):
    """The run and, backwards, torch's own vector-Jacobian product of each step."""
    pairs = _Pairs(box, RC + 0.5)

    def step(q, v):
        (g,) = torch.autograd.grad(_energy(q, eps, sigma, box, pairs)[0], q, create_graph=True)
        w = v - 0.5 * DT * g
        x = q + DT * w
        U, _ = _energy(x, eps, sigma, box, pairs)
        (g,) = torch.autograd.grad(U, x, create_graph=True)
        return x, w - 0.5 * DT * g, U

    K = case["steps"]
    states, total = [(q.detach(), v)], 0.0
    for _ in range(K):
        a, b = states[-1]
        x, w, U = step(a.clone().requires_grad_(True), b)
        states.append((x.detach(), w.detach()))
        total = total + U.detach()
    aq, av = torch.zeros_like(q), torch.zeros_like(v)
    ge, gs = torch.zeros_like(eps), torch.zeros_like(sigma)
    for k in range(K - 1, -1, -1):
        a, b = (t.clone().requires_grad_(True) for t in states[k])
        x, w, U = step(a, b)
        aq, av, de, ds = torch.autograd.grad((x, w, U), (a, b, eps, sigma), (aq, av, torch.full_like(U, 1.0 / K)))
        ge, gs = ge + de, gs + ds
    return dict(O=total / K, q=aq, eps=ge.detach(), sigma=gs.detach())
