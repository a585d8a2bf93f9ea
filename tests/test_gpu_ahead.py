"""The time loop enqueues the rest of a step behind the direct solve before it
has seen the solve's result; with the phase timers on it looks first.  Both
give the same bits, also where a solve needs a second cycle and the rest of
that step is done again."""
import numpy as np
import pytest

from paper_1710_09421_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ek():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1710_09421_amd import ek as binding
    binding.lib()
    return binding


@pytest.mark.parametrize("start", ["previous", "linear", "zero"])
@pytest.mark.parametrize("beads,overlap", [(0, True), (6, True), (6, False)])
@pytest.mark.parametrize("graphs", [True, False])
def test_same_bits_as_looking_first(ek, start, beads, overlap, graphs):
    ws = {"previous": ek.EK_WS_PREV, "linear": ek.EK_WS_EXTRAP, "zero": ek.EK_WS_ZERO}[start]
    wl = workloads.pore_system((24, 24, 24), 6, 4, 0.01, 0.01, -0.01, beads, 61,
                               bead_q=workloads.STABLE_BEAD_CHARGE)
    z = np.cos(2.0 * np.pi * np.arange(24.0) / 24.0)
    strong = wl.n0.copy()
    strong[1] += (wl.solid == 0) * 1e5 * (1.0 + z)
    strong[2] += (wl.solid == 0) * 1e5
    out = []
    for timed in (False, True):
        ctx = ek.from_workload(wl, precision=ek.EK_FP32, poisson_method=ek.EK_POISSON_MG,
                               poisson_tol=1e-10, poisson_max_iter=200, warm_start=ws)
        ctx.set_launch_mode(graphs=graphs, overlap=overlap)
        ctx.set_timing(timed)
        iters = []
        for n0, steps, q in ((strong, 1, 0.0), (wl.n0, 2, 1.0)):
            for s in range(3):             # the potential stays: a start 1e7 times too large
                ctx.set_species_density(s, n0[s])
            if beads:
                pp = wl.polymer
                ctx.set_polymer(wl.beads_R, wl.beads_V, q * pp["q"], M=pp["M"], n_sub=pp["n_sub"])
            for _ in range(steps):
                ctx.step(1)
                iters.append(ctx.stats()["poisson_iters"])
        ctx.step(4)
        st = ctx.stats()
        fields = [a for s in range(3) for a in ctx.moments(s)] + [ctx.potential()]
        if beads:
            fields += list(ctx.beads(beads))
        out.append((iters, st, fields))
        ctx.close()
    (ia, sa, fa), (ib, sb, fb) = out
    print(start, beads, ia, flush=True)
    assert ia == ib
    if start == "previous":
        assert ia[1] == 2                   # the step that is done again
    assert all(np.array_equal(a, b) for a, b in zip(fa, fb))
    for k in ("step", "poisson_iters", "poisson_residual"):
        assert sa[k] == sb[k], k
    # summed in another order where the timed steps update the lattice beside the chain
    assert np.allclose(sa["mass"], sb["mass"], rtol=1e-12, atol=0.0)
    assert np.allclose(sa["momentum"], sb["momentum"], rtol=1e-9, atol=1e-12)


def test_a_failing_solve_leaves_the_chain(ek):
    wl = workloads.pore_system((24, 24, 24), 6, 4, 0.01, 0.01, -0.01, 6, 62,
                               bead_q=workloads.STABLE_BEAD_CHARGE)
    ctx = ek.from_workload(wl, precision=ek.EK_FP32, poisson_method=ek.EK_POISSON_MG,
                           poisson_tol=1e-17, poisson_max_iter=25)
    with pytest.raises(ek.EKError) as e:
        ctx.step(3)
    assert e.value.status == ek.EK_ENOCONV and "25 cycles" in str(e.value)
    R, V = ctx.beads(6)
    assert np.array_equal(R, wl.beads_R) and np.array_equal(V, wl.beads_V)
    ctx.close()
