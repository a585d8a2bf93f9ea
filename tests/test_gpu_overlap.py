"""The lattice update beside the chain, at boxes on both sides of the size from
which it is taken: a chain whose beads' boxes overlap and wrap around the box
gives the same bits with and without it."""
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


@pytest.mark.parametrize("shape,beads,precision", [
    ((64, 80, 80), 70, "EK_FP32"),        # 409,600 sites: beside the chain
    ((62, 80, 80), 70, "EK_FP32"),        # 396,800: after it
    ((52, 62, 64), 5, "EK_FP64"),         # 206,336 sites of twice the time
    ((48, 64, 64), 130, "EK_FP64")])      # 196,608
def test_same_bits_beside_and_after_the_chain(ek, shape, beads, precision):
    wl = workloads.pore_system(shape, 10, 5, 0.01, 0.01, -0.01, beads, 71,
                               bead_q=workloads.STABLE_BEAD_CHARGE)
    wl.beads_R = wl.beads_R + np.array([shape[2] / 2 + 0.3, -shape[1] / 2 + 0.2, 0.0])
    out = []
    for overlap in (True, False):
        ctx = ek.from_workload(wl, precision=getattr(ek, precision),
                               poisson_method=ek.EK_POISSON_MG, poisson_tol=1e-8)
        ctx.set_launch_mode(graphs=True, overlap=overlap)
        ctx.step(3)
        out.append([a for s in range(3) for a in ctx.moments(s)] + [ctx.potential()] +
                   list(ctx.beads(beads)) + [ctx.stats()["mass"]])
        ctx.close()
    *a, ma = out[0]
    *b, mb = out[1]
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
    assert np.allclose(ma, mb, rtol=1e-12, atol=0.0)   # summed in another order
