"""The persistent ensemble kernel (a cycle limit below 20) in its launch shapes
against the oracle: workgroup sizes, and teams of workgroups that meet at
barriers.  More than one cycle a solve shows that the steps were not launched
with the direct solve."""
import numpy as np
import pytest

from tests.test_gpu_ensemble import errors, oracle_sim, replicas

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(256, 1), (512, 1), (1024, 1), (256, 4), (512, 2), (512, 4), (1024, 2)]


@pytest.fixture(scope="module")
def ek():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1710_09421_amd import ek as binding
    binding.lib()
    return binding


def _run(ek, wls, threads, group, steps, ws):
    ens = ek.ensemble_from_workloads(wls, precision=ek.EK_FP32, poisson_tol=1e-8,
                                     poisson_max_iter=19, warm_start=ws)
    ens.set_threads(threads)
    ens.set_group(group)
    ens.step(1)
    assert all(ens.stats(r)["poisson_iters"] > 1 for r in range(len(wls)))
    ens.step(steps - 1)
    return ens


@pytest.fixture(scope="module")
def reference():
    wls = replicas()
    sims = {}
    for r in (0, 3):
        sims[r] = oracle_sim(wls[r], 1e-8)
        sims[r].run(20)
    return wls, sims


@pytest.mark.parametrize("start", ["previous", "extrapolated"])
@pytest.mark.parametrize("threads,group", SHAPES)
def test_launch_shapes_match_the_oracle(ek, reference, threads, group, start):
    wls, sims = reference
    ws = ek.EK_WS_PREV if start == "previous" else ek.EK_WS_EXTRAP
    ens = _run(ek, wls, threads, group, 20, ws)
    for r, sim in sims.items():
        err = errors(lambda s: ens.moments(r, s), lambda: ens.potential(r), sim, wls[r])
        err["R"] = float(np.abs(ens.beads(r)[0] - sim.R).max())
        print(threads, group, start, r, err, flush=True)
        assert max(err.values()) < 1e-5, (r, err)
    assert all(ens.stats(r)["step"] == 20 for r in range(len(wls)))
    ens.close()


@pytest.mark.parametrize("threads,group", [(256, 1), (512, 4)])
def test_a_launch_shape_is_deterministic(ek, threads, group):
    wls = replicas()
    out = []
    for _ in range(2):
        ens = _run(ek, wls, threads, group, 6, ek.EK_WS_PREV)
        out.append([a for r in range(len(wls)) for s in range(3) for a in ens.moments(r, s)] +
                   [ens.potential(r) for r in range(len(wls))] + list(ens.beads(3)))
        ens.close()
    assert all(np.array_equal(a, b) for a, b in zip(*out))
