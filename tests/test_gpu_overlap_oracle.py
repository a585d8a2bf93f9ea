"""The lattice update beside the chain against the float64 oracle, for a chain
across the periodic boundary of a small box: with the timers on the mode is taken
at every size, and the timed sites show that it was."""
import numpy as np
import pytest

from oracle import step as ostep
from tests.parity import density_error, field_error, velocity_error
from tests.test_gpu_launch_modes import _wrapping_chain

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ek():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1710_09421_amd import ek as binding
    binding.lib()
    return binding


@pytest.mark.parametrize("overlap", [True, False])
def test_wrapping_chain_matches_oracle(ek, overlap):
    wl, steps = _wrapping_chain(), 6
    ctx = ek.from_workload(wl, precision=ek.EK_FP64, poisson_tol=1e-10, poisson_check_every=1)
    ctx.set_launch_mode(graphs=True, overlap=overlap)
    ctx.set_timing(True)
    p = ostep.Params(valence=wl.valence, tau=wl.tau, omega_drag=wl.omega_drag,
                     bjerrum=wl.bjerrum, E_ext=wl.E_ext, poisson_tol=1e-10)
    sim = ostep.Simulation(p, wl.solid.astype(bool), wl.wall_q, wl.n0,
                           beads=(wl.beads_R, wl.beads_V, wl.polymer))
    ctx.step(steps)
    sim.run(steps)
    fluid = wl.solid == 0
    err = {}
    for s in range(3):
        n, u = ctx.moments(s)
        err[f"n{s}"] = density_error(n, sim.densities()[s], fluid)
        err[f"u{s}"] = velocity_error(u, sim.velocities()[s], fluid)
    err["psi"] = field_error(ctx.potential(), sim.psi)
    err["R"] = float(np.abs(ctx.beads(4)[0] - sim.R).max())
    sites = ctx.timing()["lb_sites"]
    print(err, sites)
    # beside the chain the fused kernel leaves the sites of the beads' boxes out
    assert sites < steps * wl.fluid_sites if overlap else sites == steps * wl.fluid_sites
    assert max(err.values()) < 1e-8, err
    ctx.close()
