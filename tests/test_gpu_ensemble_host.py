"""The ensemble's host side: a workspace whose memory still has work pending on
the ensemble's stream, the tuner where there is no launch shape to choose, and
the solver that a message names."""
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


@pytest.mark.parametrize("threads,group", [(256, 1), (1024, 2), (512, 4)])
def test_tuning_launched_steps_keeps_the_shape(ek, threads, group):
    """Steps launched over all replicas are the same with every shape."""
    ens = ensemble(ek, [replica((16, 16, 16), 9)], poisson_max_iter=200)
    ens.set_threads(threads)
    ens.set_group(group)
    res = ens.autotune(steps=2)
    assert (res["threads"], res["group"]) == (threads, group)
    assert 0 < res["ms_per_step"] < 1e3
    assert ens.stats(0)["step"] == 9 * (1 + 2 + 2)
    ens.close()


@pytest.mark.parametrize("cycles,name", [(30, "the direct solve"), (19, "multigrid")])
def test_no_convergence_names_the_solver(ek, cycles, name):
    ens = ensemble(ek, [replica((16, 16, 16), 9)], poisson_max_iter=cycles, poisson_tol=1e-17)
    with pytest.raises(ek.EKError) as e:
        ens.step(1)
    assert e.value.status == ek.EK_ENOCONV
    assert f"replica 0: {name} did not reach 1e-17 in {cycles} cycles" in str(e.value)
    ens.close()
