"""An ensemble whose workspace's memory still has work pending on its stream."""
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


def replica(shape, seed):
    return workloads.pore_system(shape, shape[0] // 4, min(shape[1:]) // 4, 0.01, 0.02, -0.01, 0,
                                 seed)


def ensemble(ek, wls, stream=None, **kw):
    p = ek.make_params(wls[0].shape, poisson_method=ek.EK_POISSON_MG, **kw)
    ens = ek.Ensemble(p, len(wls), stream=stream)
    ens.set_geometry(wls[0].solid, wls[0].wall_q)
    for r, wl in enumerate(wls):
        ens.set_replica(r, wl.E_ext, wl.n0)
    return ens


def test_workspace_with_work_pending_on_the_stream(ek):
    """The memory of a tensor freed on the stream, whose fill has not run yet
    when the ensemble is made."""
    wls = [replica((24, 24, 24), 5), replica((24, 24, 24), 6)]
    ref = ensemble(ek, wls, poisson_max_iter=200)
    nbytes = ref.workspace.numel()
    ref.step(3)
    want = [ref.potential(r) for r in range(2)]
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for _ in range(2):             # the first one warms up what the second one times
            held = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
            side.synchronize()
            torch.cuda._sleep(20_000_000)
            held.fill_(255)
            ptr = held.data_ptr()
            del held
            ens = ensemble(ek, wls, stream=side, poisson_max_iter=200)
            assert ens.workspace.data_ptr() == ptr
            ens.step(3)
            got = [ens.potential(r) for r in range(2)]
            ens.close()
            del ens
            assert all(np.array_equal(a, b) for a, b in zip(got, want))
    ref.close()
