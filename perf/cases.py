"""Timed cases of the library: what a user's program has it do, through the
public entry points of `paper_1710_09421_amd.ek`.

A case is a dict of plain values.  Its `kind` says which call it is:

  step      time steps of one context (`Context.step`), and the read-out that
            a program takes between them
  ensemble  time steps of many replicas in one persistent launch
            (`Ensemble.step`), and the chains' and potentials' read-out
  poisson   one stand-alone solve (`Context.poisson_solve`)
  forward   the warm-start network's guess for one right-hand side
  train     one optimiser step of the network: a batch of accumulated
            gradients, then Adam

Fields of a context with float32 populations are returned in float32, the
precision that its state has; a float64 context's and the solver's results are
returned as the library gives them.
"""
import functools
import math

import numpy as np
import torch

from paper_1710_09421_amd import ek, learned, workloads

METHOD = {"sor": ek.EK_POISSON_SOR, "mg": ek.EK_POISSON_MG}
PRECISION = {"float32": ek.EK_FP32, "float64": ek.EK_FP64}
START = {"zero": ek.EK_WS_ZERO, "previous": ek.EK_WS_PREV, "linear": ek.EK_WS_EXTRAP,
         "quadratic": ek.EK_WS_EXTRAP2}
KT, BJERRUM = 1.0 / 3.0, 0.7


def _step(nx, ny, nz, **kw):
    """Defaults of a step case: a charged pore with salt 0.01 and a field."""
    case = dict(kind="step", nx=nx, ny=ny, nz=nz, slab=8, radius=4, salt=0.01, field=0.01,
                walls="periodic", beads=0, bead_charge=-1.0, bond="fene", coupling="trilinear",
                precision="float32", method="mg", start="quadratic", tol=1e-8, kT=KT,
                fluctuations=False, steps=10, read="system")
    case.update(kw)
    return case


def listed():
    return [
        # the smallest whole calls: the periodic box without walls in float64
        # with the paper's own solver to 1e-10 ...
        _step(32, 32, 32, name="plain-32-f64-sor", slab=0, field=0.0, precision="float64",
              method="sor", start="previous", tol=1e-10, steps=2, read="moments"),
        # ... and the pore that the parity tests run, bound by launches
        _step(24, 24, 32, name="pore-24x24x32", slab=6, beads=8, steps=20, read="moments"),
        # one translocation cell as the benchmark runs it
        _step(64, 64, 128, name="pore-64x64x128", slab=10, radius=5, beads=32, steps=20),
        # the paper's own set-up: harmonic bonds, sigma 2, one MD step per
        # lattice step, sides that stop halving at 3
        _step(96, 96, 160, name="translocation-96x96x160", slab=40, radius=6, salt=0.0075,
              beads=100, bead_charge=-0.1, bond="harmonic", steps=10),
        # the largest box that one context is used for here
        _step(256, 256, 512, name="pore-256x256x512", slab=20, radius=10, salt=0.005, field=0.02,
              beads=256, bead_charge=-0.1, steps=8),
        # thermal fluctuations on, at a lattice kT at which the chain holds
        _step(64, 64, 128, name="fluctuating-64x64x128", slab=10, radius=5, beads=8,
              bead_charge=-0.1, kT=1e-5, fluctuations=True, steps=10),
        # insulating walls (only SOR solves those) with the occupation cube
        _step(48, 48, 64, name="insulating-48x48x64", walls="insulating", beads=16,
              bead_charge=-0.1, coupling="theta", method="sor", start="previous", steps=2,
              read="moments"),
        # the statistics of many translocation events
        dict(name="ensemble-64x48x48x96", kind="ensemble", nx=48, ny=48, nz=96, replicas=64,
             steps=20),
        # stand-alone solves: the paper's solver at its usual tolerance, and
        # multigrid as training pairs are made (1e-10), on sides that no
        # power of two divides far
        dict(name="solve-sor-64x64x128", kind="poisson", nx=64, ny=64, nz=128, method="sor",
             tol=1e-8, check_every=1),
        dict(name="solve-mg-120x120x200", kind="poisson", nx=120, ny=120, nz=200, method="mg",
             tol=1e-10, check_every=1),
        # the network's guess, and one optimiser step of its training
        dict(name="network-forward-64x64x128", kind="forward", nx=64, ny=64, nz=128),
        dict(name="network-train-64x64x128", kind="train", nx=64, ny=64, nz=128, batch=8),
    ]


def _even(rng, lo, hi, of=2):
    """A multiple of `of` between lo and hi, spread over the logarithm."""
    return max(lo, min(hi, of * round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / of)))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "ensemble", "sor", "mg", "forward", "train"])
    if kind == "step":
        variant = rng.choice(["plain", "pore", "pore", "chain", "chain", "fluctuating",
                              "insulating", "harmonic"])
        big = variant not in ("insulating", "harmonic")
        nx, ny = _even(rng, 24, 128 if big else 64), _even(rng, 24, 128 if big else 64)
        nz = _even(rng, 32, 256 if big else 96)
        common = dict(slab=rng.randrange(4, 11), radius=rng.randrange(3, 8),
                      salt=round(rng.uniform(0.002, 0.05), 4), steps=rng.randrange(4, 13),
                      field=round(rng.uniform(0.0, 0.02), 4),
                      start=rng.choice(["previous", "linear", "quadratic"]))
        if variant == "plain":
            n = _even(rng, 16, 48)
            return _step(n, n, n, slab=0, radius=0, salt=common["salt"], field=0.0,
                         precision="float64", method=rng.choice(["sor", "mg"]), start="previous",
                         tol=1e-10, steps=2, read="moments")
        if variant == "chain":
            return _step(nx, ny, nz, **common, beads=rng.randrange(4, 49), bead_charge=-0.1)
        if variant == "fluctuating":
            return _step(nx, ny, nz, **common, kT=1e-5, fluctuations=True)
        if variant == "insulating":
            common.update(start="previous", steps=2)
            return _step(nx, ny, nz, **common, walls="insulating", method="sor", read="moments")
        if variant == "harmonic":
            common.update(radius=6, slab=rng.randrange(10, 17))
            return _step(nx, ny, nz, **common, beads=rng.randrange(6, 17), bead_charge=-0.1,
                         bond="harmonic")
        return _step(nx, ny, nz, **common)
    if kind == "ensemble":
        return dict(kind="ensemble", nx=_even(rng, 24, 48, 8), ny=_even(rng, 24, 48, 8),
                    nz=_even(rng, 48, 96, 8), replicas=rng.randrange(4, 65),
                    steps=rng.randrange(8, 17))
    if kind in ("sor", "mg"):
        top = 64 if kind == "sor" else 160
        return dict(kind="poisson", nx=_even(rng, 16, top), ny=_even(rng, 16, top),
                    nz=_even(rng, 24, 2 * top), method=kind, tol=1e-8 if kind == "sor" else 1e-10,
                    check_every=rng.choice([1, 1, 4]) if kind == "sor" else 1)
    if kind == "forward":
        return dict(kind="forward", nx=_even(rng, 16, 128, 4), ny=_even(rng, 16, 128, 4),
                    nz=_even(rng, 16, 256, 4))
    return dict(kind="train", nx=_even(rng, 16, 64, 4), ny=_even(rng, 16, 64, 4),
                nz=_even(rng, 16, 128, 4), batch=rng.randrange(1, 9))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
@functools.lru_cache(maxsize=4)
def _pore(nx, ny, nz, slab, radius, sites):
    """Solid mask, charged wall sites and last solid layer (no seed in them)."""
    shape = (nz, ny, nx)
    if slab == 0:
        solid = np.zeros(shape, dtype=np.uint8)
        return solid, np.zeros(shape, dtype=bool), 0
    solid, k0, k1 = workloads.pore_geometry(shape, slab, radius)
    lo, hi = k0 - 1, k1 + 2            # the sites with a fluid neighbour lie in these layers
    part = solid[lo:hi]
    near = workloads.boundary_sites(part) if sites == "links" else \
        workloads.face_boundary_sites(part)
    walls = np.zeros(shape, dtype=bool)
    walls[k0:k1 + 1] = near[1:-1]
    return solid, walls, k1


def _fields(case, seed, n_beads=0, bead_charge=0.0, slab=None, radius=None, salt=0.01):
    """Geometry, wall charge and neutral densities [3, z, y, x] of a pore."""
    slab = case.get("slab", 8) if slab is None else slab
    radius = case.get("radius", 4) if radius is None else radius
    sites = "faces" if case.get("walls") == "insulating" else "links"
    solid, wall_sites, top = _pore(case["nx"], case["ny"], case["nz"], slab, radius, sites)
    wall_q = np.where(wall_sites, -0.01, 0.0)
    fluid = solid == 0
    gen = torch.Generator(device="cuda").manual_seed(seed)
    noise = torch.rand((2,) + solid.shape, dtype=torch.float64, device="cuda", generator=gen)
    on = torch.from_numpy(fluid).cuda()
    ions = salt * (1.0 + 0.01 * (2.0 * noise - 1.0)) * on
    excess = wall_q.sum() + bead_charge * n_beads + float((ions[0] - ions[1]).sum())
    ions[0] -= on * (excess / float(fluid.sum()))
    n0 = np.empty((3,) + solid.shape)
    n0[0] = fluid
    n0[1:] = ions.cpu().numpy()
    return solid, wall_q, n0, top


def _chain(case, seed, solid, top, n_beads, harmonic=False):
    """A chain grown from the pore's mouth, at mechanical rest."""
    nx, ny = case["nx"], case["ny"]
    rng = np.random.default_rng(seed)
    clear = 2.0 ** (1.0 / 6.0) * 2.0 + 0.06 if harmonic else 1.5
    kw = dict(bond=2.0, min_dist=clear) if harmonic else {}
    start = np.array([(nx - 1) / 2.0, (ny - 1) / 2.0, top + clear])
    for _ in range(20):
        try:
            return workloads.random_walk_chain(n_beads, start, solid.astype(bool),
                                               top - 1.0 + clear if harmonic else top, rng, **kw)
        except RuntimeError:           # a walk that caught itself: another one
            continue
    raise RuntimeError("no room for the chain")


def _prepare_step(case, seed):
    nb = case["beads"]
    solid, wall_q, n0, top = _fields(case, seed, nb, case["bead_charge"], salt=case["salt"])
    harmonic = case["bond"] == "harmonic"
    p = ek.make_params(solid.shape, precision=PRECISION[case["precision"]], kT=case["kT"],
                       bjerrum=2 * BJERRUM if harmonic else BJERRUM,
                       E_ext=(0.0, 0.0, case["field"]), poisson_method=METHOD[case["method"]],
                       poisson_tol=case["tol"],
                       poisson_max_iter=200 if case["method"] == "mg" else 100000,
                       warm_start=START[case["start"]], walls=case["walls"],
                       fluctuations=int(case["fluctuations"]), seed=seed)
    ctx = ek.Context(p, max_beads=nb)
    ctx.set_geometry(solid, wall_q)
    for s in range(3):
        ctx.set_species_density(s, n0[s])
    if nb:
        pos = _chain(case, seed, solid, top, nb, harmonic)
        chain = dict(M=10.0, eps=KT, sigma=2.0, gamma=2.0, n_sub=1, bond="harmonic", k_bond=1.0,
                     l_bond=2.0) if harmonic else {}
        ctx.set_polymer(pos, np.zeros_like(pos), np.full(nb, case["bead_charge"]),
                        coupling=case["coupling"], **chain)
    state = dict(kind="step", ctx=ctx, steps=case["steps"], beads=nb, read=case["read"],
                 single=case["precision"] == "float32")
    if case["read"] == "system":
        state["rhs"] = torch.empty(solid.shape, dtype=torch.float64, device="cuda")
        state["psi"] = torch.empty_like(state["rhs"])
    return state


def _prepare_ensemble(case, seed):
    rng = np.random.default_rng(seed)
    shape, slab, radius = (case["nz"], case["ny"], case["nx"]), 8, 4
    chains = [(16, 24, 32, 48, 64)[r % 5] for r in range(case["replicas"])]
    p = ek.make_params(shape, poisson_method=ek.EK_POISSON_MG, poisson_max_iter=200,
                       warm_start=ek.EK_WS_EXTRAP)
    ens = ek.Ensemble(p, case["replicas"], max_beads=max(chains))
    q = workloads.STABLE_BEAD_CHARGE
    for r, nb in enumerate(chains):
        solid, wall_q, n0, top = _fields(case, seed + 1000 * r, nb, q, slab=slab, radius=radius)
        if r == 0:
            ens.set_geometry(solid, wall_q)
        pos = _chain(case, seed + 1000 * r, solid, top, nb)
        ens.set_replica(r, (0.0, 0.0, float(rng.uniform(0.01, 0.1))), n0, pos,
                        np.zeros_like(pos), np.full(nb, q))
    ens.set_threads(512)               # the launch shape that the benchmark's tuning picks
    ens.set_group(4)
    return dict(kind="ensemble", ens=ens, steps=case["steps"], replicas=case["replicas"])


def _charge(case, seed):
    """Charge density of a pore and its solid mask, on the GPU."""
    slab, radius = min(10, case["nz"] // 3), min(5, min(case["nx"], case["ny"]) // 4)
    solid, wall_q, n0, _ = _fields(case, seed, slab=slab, radius=radius)
    rho = torch.from_numpy(n0[1] - n0[2] + wall_q).cuda()
    return rho, torch.from_numpy(solid).cuda()


def _prepare_poisson(case, seed):
    rho, _ = _charge(case, seed)
    p = ek.make_params(tuple(rho.shape), poisson_method=METHOD[case["method"]],
                       poisson_tol=case["tol"], poisson_check_every=case["check_every"],
                       poisson_max_iter=400 if case["method"] == "mg" else 100000)
    return dict(kind="poisson", ctx=ek.Context(p), rho=rho, psi=torch.zeros_like(rho))


def _spectrum(shape):
    """Eigenvalues of the 7-point Laplacian on the periodic box."""
    k = [torch.cos(2.0 * math.pi * torch.fft.fftfreq(n, dtype=torch.float64, device="cuda"))
         for n in shape]
    return 2.0 * (k[0][:, None, None] + k[1][None, :, None] + k[2][None, None, :]) - 6.0


def _solved(rho, kT=KT, bjerrum=BJERRUM):
    """Mean-free solution of the discrete Poisson equation, by the spectrum."""
    lam = _spectrum(rho.shape)
    lam[0, 0, 0] = 1.0
    hat = torch.fft.fftn(-rho * (4.0 * math.pi * bjerrum * kT)) / lam
    hat[0, 0, 0] = 0.0
    return torch.fft.ifftn(hat).real.contiguous()


def _rhs(rho):
    return -(rho - rho.mean()) * (4.0 * math.pi * BJERRUM * KT)


def _prepare_forward(case, seed):
    rho, solid = _charge(case, seed)
    net = ek.UNet(tuple(rho.shape), training=False)
    params, scale, _ = learned.load_model()
    net.set_params(params, scale)
    return dict(kind="forward", net=net, rhs=_rhs(rho), solid=solid, guess=torch.empty_like(rho))


def _prepare_train(case, seed):
    pairs = []
    for i in range(case["batch"]):
        rho, solid = _charge(case, seed + 1000 * i)
        pairs.append((_rhs(rho), solid, _solved(rho)))
    net = ek.UNet(tuple(rho.shape), training=True)
    net.set_params(learned.init_params(seed), 10.0)
    return dict(kind="train", net=net, pairs=pairs)


def prepare(case, seed):
    return {"step": _prepare_step, "ensemble": _prepare_ensemble, "poisson": _prepare_poisson,
            "forward": _prepare_forward, "train": _prepare_train}[case["kind"]](case, seed)


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _run_step(state):
    ctx, out = state["ctx"], {}
    ctx.step(state["steps"])
    kept = np.float32 if state["single"] else np.float64
    if state["read"] == "system":      # a snapshot of the field, kept on the GPU
        ctx.poisson_system(state["rhs"], state["psi"])
        out["rhs"], out["psi"] = state["rhs"].float(), state["psi"].float()
    else:                              # every field, on the host
        for s in range(3):
            n, u = ctx.moments(s)
            out[f"n{s}"], out[f"u{s}"] = n.astype(kept), u.astype(kept)
        out["psi"] = ctx.potential().astype(kept)
    if state["beads"]:
        pos, vel = ctx.beads(state["beads"])
        out["pos"], out["vel"] = pos.astype(kept), vel.astype(kept)
    return out


def _run_ensemble(state):
    ens, pos, vel, psi = state["ens"], [], [], []
    ens.step(state["steps"])
    for r in range(state["replicas"]):
        p, v = ens.beads(r)
        pos.append(p)
        vel.append(v)
        psi.append(ens.potential(r).astype(np.float32))
    return dict(pos=np.concatenate(pos).astype(np.float32),
                vel=np.concatenate(vel).astype(np.float32), psi=np.stack(psi))


def _run_poisson(state):
    state["ctx"].poisson_solve(state["rho"], state["psi"], ek.EK_WS_ZERO)
    return state["psi"]


def _run_forward(state):
    state["net"].forward(state["rhs"], state["solid"], state["guess"])
    return state["guess"].float()


def _run_train(state):
    net = state["net"]
    for rhs, solid, psi in state["pairs"]:
        net.accumulate(rhs, solid, psi)
    grad = net.gradient()
    net.adam_step(1e-4, grad_scale=1.0 / len(state["pairs"]))
    loss, _ = net.read_loss()
    return dict(grad=grad, loss=loss)


def run(state):
    return {"step": _run_step, "ensemble": _run_ensemble, "poisson": _run_poisson,
            "forward": _run_forward, "train": _run_train}[state["kind"]](state)


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
_NETWORK_FLOPS = 2 * (27 * 2 * 16 + 27 * 16 + (27 * 16 * 32 + 32 * 16) / 8
                      + (27 * 32 * 64 + 64 * 32) / 64)      # per site


def work(case):
    n = case["nx"] * case["ny"] * case["nz"]
    if case["kind"] == "step":
        width = 8 if case["precision"] == "float64" else 4
        # per step and site: 57 populations read and written, the link word,
        # the potential and the charge read and written once
        return dict(bytes=float(case["steps"] * n * (2 * 57 * width + 4 + 4 * 8)),
                    flops=float(case["steps"] * n * 1500))
    if case["kind"] == "ensemble":
        m = n * case["replicas"] * case["steps"]
        return dict(bytes=float(m * (2 * 57 * 4 + 4 + 4 * 8)), flops=float(m * 1500))
    if case["kind"] == "poisson":      # charge in, potential out
        return dict(bytes=float(16 * n), flops=float(100 * n))
    if case["kind"] == "forward":
        return dict(bytes=float(17 * n), flops=float(_NETWORK_FLOPS * n))
    return dict(bytes=float(case["batch"] * 17 * n), flops=float(case["batch"] * 3 * _NETWORK_FLOPS * n))


# ---------------------------------------------------------------------------
# The same in 64 bits, by torch
# ---------------------------------------------------------------------------
_C = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
      (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1),
      (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]
_OPPOSITE = [0, 2, 1, 4, 3, 6, 5, 8, 7, 10, 9, 12, 11, 14, 13, 16, 15, 18, 17]


def _exact_step(case, seed):
    """The time step in float64: no chain, no noise, periodic potential."""
    solid, wall_q, n0, _ = _fields(case, seed, salt=case["salt"])
    solid = torch.from_numpy(solid).cuda().bool()
    fluid, wall = ~solid, torch.from_numpy(wall_q).cuda()
    c = torch.tensor(_C, dtype=torch.float64, device="cuda")
    w = torch.tensor([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12, dtype=torch.float64, device="cuda")
    z = torch.tensor([0.0, 1.0, -1.0], dtype=torch.float64, device="cuda")
    dims = (-3, -2, -1)
    behind = [torch.roll(solid, (v[2], v[1], v[0]), dims=dims) for v in _C]
    f = w[None, :, None, None, None] * torch.from_numpy(n0).cuda()[:, None] * fluid

    def moments(f):
        return f.sum(1), torch.einsum("pk,spzyx->skzyx", c, f)

    for _ in range(case["steps"]):
        n, j = moments(f)
        rho = (z[:, None, None, None] * n).sum(0) + wall
        psi = _solved(rho, case["kT"])
        e = torch.stack([-0.5 * (torch.roll(psi, -1, -1 - k) - torch.roll(psi, 1, -1 - k))
                         for k in range(3)])
        e[2] += case["field"]
        g = z[:, None, None, None, None] * e[None]
        safe = torch.where(fluid, n, 1.0)
        b = j / safe[:, None] + 0.5 * g
        # drag rates of 1: a half step of them moves u halfway to the mean
        x = safe / safe.sum(0)
        mean = (x[:, None] * b).sum(0)
        u = (b + 0.5 * mean) / 1.5
        phi = g - (u - mean)
        cu = torch.einsum("pk,skzyx->spzyx", c, u)
        cf = torch.einsum("pk,skzyx->spzyx", c, phi)
        uu, fu = (u * u).sum(1)[:, None], (u * phi).sum(1)[:, None]
        wn = w[None, :, None, None, None] * safe[:, None]
        # relaxation time 1: the equilibrium and half of the forcing are left
        post = wn * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu
                     + 0.5 * (3.0 * cf + 9.0 * cu * cf - 3.0 * fu)) * fluid
        f = torch.stack([torch.where(behind[p], post[:, _OPPOSITE[p]],
                                     torch.roll(post[:, p], (v[2], v[1], v[0]), dims=dims))
                         for p, v in enumerate(_C)], dim=1) * fluid
    if case["read"] == "system":
        b = -rho * (4.0 * math.pi * BJERRUM * case["kT"])
        return dict(rhs=b - b.mean(), psi=psi)
    n, j = moments(f)
    out = dict(psi=psi)
    for s in range(3):
        out[f"n{s}"], out[f"u{s}"] = n[s], j[s] / torch.where(fluid, n[s], 1.0)
    return out


def _network(params, x):
    """The network in float64 on channels-last fields [z, y, x, c]."""
    at = 0

    def layer(x, taps, cin, cout):
        nonlocal at
        w = params[at:at + taps * cin * cout].reshape(taps, cin, cout)
        bias = params[at + taps * cin * cout:at + taps * cin * cout + cout]
        at += taps * cin * cout + cout
        if taps == 1:
            return x @ w[0] + bias
        y = bias
        for t in range(27):
            shift = (1 - t // 9, 1 - (t // 3) % 3, 1 - t % 3)
            y = y + torch.roll(x, shift, dims=(0, 1, 2)) @ w[t]
        return y

    def pool(x):
        nz, ny, nx, ch = x.shape
        return x.reshape(nz // 2, 2, ny // 2, 2, nx // 2, 2, ch).mean(dim=(1, 3, 5))

    def up(x):
        for d in range(3):
            x = x.repeat_interleave(2, dim=d)
        return x

    a1 = torch.relu(layer(x, 27, 2, 16))
    a2 = torch.relu(layer(pool(a1), 27, 16, 32))
    a3 = torch.relu(layer(pool(a2), 27, 32, 64))
    c2 = torch.relu(up(layer(a3, 1, 64, 32)) + a2)
    c1 = torch.relu(up(layer(c2, 1, 32, 16)) + a1)
    return layer(c1, 27, 16, 1)[..., 0]


def _network_input(rhs, solid):
    s = float(rhs.std(unbiased=False))
    return torch.stack([(rhs - rhs.mean()) / s, solid.double()], dim=-1), s


def exact(case, seed):
    if case["kind"] == "poisson":
        return _solved(_charge(case, seed)[0])
    if case["kind"] == "forward":
        rho, solid = _charge(case, seed)
        params, scale, _ = learned.load_model()
        with torch.no_grad():
            x, s = _network_input(_rhs(rho), solid)
            return s * scale * _network(torch.from_numpy(params).cuda().double(), x)
    if case["kind"] == "train":
        p = torch.from_numpy(learned.init_params(seed)).cuda().double().requires_grad_()
        total = 0.0
        for i in range(case["batch"]):
            rho, solid = _charge(case, seed + 1000 * i)
            x, s = _network_input(_rhs(rho), solid)
            loss = ((_network(p, x) - _solved(rho) / (s * 10.0)) ** 2).mean()
            loss.backward()
            total += float(loss.detach())
        return dict(grad=p.grad, loss=total / case["batch"])
    if case["kind"] == "step" and not case["beads"] and not case["fluctuations"] \
            and case["walls"] == "periodic" and case["nx"] * case["ny"] * case["nz"] <= 1 << 21:
        return _exact_step(case, seed)
    return None                        # a chain, noise or insulating walls: a second library
