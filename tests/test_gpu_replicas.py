"""The ensemble's launched steps (direct Poisson solve) against the persistent
kernel (multigrid), which takes an ensemble whose cycles are limited to fewer
than 20: boxes whose sites leave a remainder of the 1,024 a block sums, sides
with a prime factor, rows longer than a plane that fits LDS, chains of none to
64 beads; and the ways a solve ends."""
import numpy as np
import pytest

from paper_1710_09421_amd import workloads
from tests.parity import density_error, field_error, velocity_error

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ek():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1710_09421_amd import ek as binding
    binding.lib()
    return binding


def replica(shape, beads, field, seed):
    return workloads.pore_system(shape, shape[0] // 4, min(shape[1:]) // 4, 0.01, field, -0.01,
                                 beads, seed, bead_q=workloads.STABLE_BEAD_CHARGE)


def run(ek, wls, steps, **kw):
    ens = ek.ensemble_from_workloads(wls, precision=ek.EK_FP32, poisson_tol=1e-10, **kw)
    ens.step(steps)
    out = [([ens.moments(r, s) for s in range(3)], ens.potential(r), ens.beads(r), ens.stats(r))
           for r in range(len(wls))]
    ens.close()
    return out


# The two agree to the Poisson tolerance (1e-10) and to roundings of the
# float32 populations that it flips (6e-8 of a deviation each, at most one per
# site and step): 1e-6 for all fields, as between an ensemble and contexts.
@pytest.mark.parametrize("shape,beads", [
    ((16, 12, 10), (0, 0)),          # 1,920 sites
    ((26, 14, 22), (3, 0, 8)),       # primes 13, 7 and 11
    ((24, 24, 24), (8, 16, 5)),
    ((16, 136, 12), (4,)),
    ((56, 32, 32), (64, 1)),
    ((16, 148, 150), (6,)),          # planes beyond LDS: rows and columns apart
])
@pytest.mark.parametrize("start", ["previous", "extrapolated"])
def test_launched_steps_match_the_persistent_kernel(ek, shape, beads, start):
    ws = ek.EK_WS_PREV if start == "previous" else ek.EK_WS_EXTRAP
    wls = [replica(shape, nb, 0.01 * (r + 1), 31 + r) for r, nb in enumerate(beads)]
    a = run(ek, wls, 6, warm_start=ws, poisson_max_iter=200)
    b = run(ek, wls, 6, warm_start=ws, poisson_max_iter=19)
    for r, wl in enumerate(wls):
        fluid = wl.solid == 0
        (ma, pa, ba, sa), (mb, pb, bb, sb) = a[r], b[r]
        err = {"psi": field_error(pa, pb)}
        for s in range(3):
            err[f"n{s}"] = density_error(ma[s][0], mb[s][0], fluid)
            err[f"u{s}"] = velocity_error(ma[s][1], mb[s][1], fluid)
            err[f"m{s}"] = abs(sa["mass"][s] / sb["mass"][s] - 1.0)
        if beads[r]:
            err["R"] = float(np.abs(ba[0] - bb[0]).max())
        print(shape, r, {k: f"{v:.1e}" for k, v in err.items()}, sa["poisson_iters"],
              sb["poisson_iters"], f"{sa['poisson_residual']:.1e}", flush=True)
        assert sa["step"] == sb["step"] == 6
        assert abs(pa.mean()) <= 1e-12 * np.abs(pa).max()
        assert max(err.values()) < 1e-6, err


def test_a_limit_that_no_cycle_meets(ek):
    """Ends as not converged and names the replica, which stays at its step."""
    wls = [replica((24, 24, 24), nb, 0.02, 7 + nb) for nb in (0, 6)]
    ens = ek.ensemble_from_workloads(wls, precision=ek.EK_FP32, poisson_tol=1e-17,
                                     poisson_max_iter=30)
    with pytest.raises(ek.EKError) as e:
        ens.step(4)
    assert e.value.status == ek.EK_ENOCONV and "replica 0" in str(e.value)
    assert "30 cycles" in str(e.value)
    assert ens.stats(0)["step"] == 0
    ens.close()


@pytest.mark.parametrize("steps", [1, 3])
def test_a_second_cycle(ek, steps):
    """A start 1e7 times too large leaves its rounding (1e-16 of it) above the
    tolerance after one cycle: the replica pauses, has a second one, and goes
    on; the other one does not wait and neither differs from a fresh run."""
    wls = [replica((24, 24, 24), nb, 0.02, 7 + nb) for nb in (0, 6)]
    ref = run(ek, wls, steps)
    ens = ek.ensemble_from_workloads(wls, precision=ek.EK_FP32, poisson_tol=1e-10)
    n0 = wls[0].n0.copy()
    x = np.arange(24.0)
    n0[1] += (wls[0].solid == 0) * 1e7 * 0.01 * (1.0 + np.cos(2.0 * np.pi * x / 24.0))
    n0[2] += (wls[0].solid == 0) * 1e7 * 0.01
    ens.set_replica(0, wls[0].E_ext, n0)
    ens.step(1)
    scale = np.abs(ens.potential(0)).max() / np.abs(ref[0][1]).max()
    assert scale > 1e5
    ens.set_replica(0, wls[0].E_ext, wls[0].n0)   # the potential stays as the start
    ens.step(steps)
    fresh = run(ek, wls, steps + 1)[1]
    st = ens.stats(0)
    print(st["poisson_iters"], st["poisson_residual"], scale)
    assert st["step"] == steps and st["poisson_iters"] == (2 if steps == 1 else 1)
    assert field_error(ens.potential(0), ref[0][1]) < 1e-8
    assert ens.stats(1)["step"] == steps + 1
    assert np.array_equal(ens.potential(1), fresh[1])
    assert np.array_equal(ens.beads(1)[0], fresh[2][0])
    ens.close()


def test_neutral_replica_keeps_a_zero_potential(ek):
    wl = replica((16, 16, 16), 0, 0.0, 3)
    wl.n0[1:] = 0.01 * (wl.solid == 0)
    wl.wall_q[:] = 0.0
    (m, psi, _, st), = run(ek, [wl], 3)
    assert not psi.any() and st["step"] == 3
