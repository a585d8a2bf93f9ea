"""A cycle limit below 20 keeps the time loop on multigrid cycles: replayed from
recorded graphs they give the bits of the same launches one by one, with the fused
finest level too.  More than one cycle a solve shows that none was direct."""
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


WORKLOADS = {
    "small": lambda: workloads.pore_system((32, 24, 24), 6, 4, 0.01, 0.01, -0.01, 8, 32),
    "single-pore": workloads.single_pore,
    # sweeps marching up z on 64 x 8 tiles, with the restriction, correction and
    # norms fused into them
    "fused": lambda: workloads.pore_system((256, 128, 128), 12, 8, 0.01, 0.01, -0.01, 8, 34),
}


@pytest.mark.parametrize("size", list(WORKLOADS))
def test_replayed_cycles_match_single_launches(ek, size):
    wl = WORKLOADS[size]()
    nbd = wl.beads_R.shape[0]
    ctxs = []
    for graphs in (True, False):
        c = ek.from_workload(wl, precision=ek.EK_FP32, poisson_method=ek.EK_POISSON_MG,
                             poisson_tol=1e-8, poisson_max_iter=19)
        c.set_launch_mode(graphs=graphs, overlap=True)
        ctxs.append(c)
    a, b = ctxs
    for t in range(5):
        a.step(1)
        b.step(1)
        sa, sb = a.stats(), b.stats()
        print(size, t, sa["poisson_iters"], sa["poisson_residual0"], sa["poisson_residual"])
        assert sa["poisson_iters"] == sb["poisson_iters"] > 1
        for k in ("poisson_residual0", "poisson_residual"):
            assert sa[k] == sb[k]
        assert sa["poisson_residual"] <= 1e-8
        assert np.array_equal(sa["mass"], sb["mass"])
        assert np.array_equal(a.potential(), b.potential())
        assert all(np.array_equal(x, y) for s in range(3)
                   for x, y in zip(a.moments(s), b.moments(s)))
        assert all(np.array_equal(x, y) for x, y in zip(a.beads(nbd), b.beads(nbd)))
    a.close()
    b.close()
