"""Contexts alive together share their device's side stream: interleaved steps,
from one thread and from two, give the bits of contexts alone, and contexts
come and go in any order."""
import threading

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


def make(ek, seed):
    wl = workloads.pore_system((80, 72, 72), 10, 5, 0.01, 0.01, -0.01, 8, seed,
                               bead_q=workloads.STABLE_BEAD_CHARGE)   # 414,720 sites
    return ek.from_workload(wl, precision=ek.EK_FP32, poisson_method=ek.EK_POISSON_MG,
                            poisson_tol=1e-8)


def state(ctx):
    return [a for s in range(3) for a in ctx.moments(s)] + [ctx.potential()] + list(ctx.beads(8))


@pytest.mark.parametrize("threads", [1, 2])
def test_contexts_alive_together(ek, threads):
    ref = []
    for seed in (81, 82):
        ctx = make(ek, seed)
        ctx.step(6)
        ref.append(state(ctx))
        ctx.close()
    gone = make(ek, 83)
    gone.step(1)
    pair = [make(ek, seed) for seed in (81, 82)]
    gone.close()                           # the first user goes before the others start
    if threads == 1:
        for _ in range(3):
            for ctx in pair:
                ctx.step(2)
    else:
        errors = []

        def work(ctx):
            try:
                for _ in range(3):
                    ctx.step(2)
            except Exception as e:         # seen by the test's own thread
                errors.append(e)

        ts = [threading.Thread(target=work, args=(ctx,)) for ctx in pair]
        for t in ts:
            t.start()
        for t in ts:
            t.join(timeout=60)
        assert not errors, errors
    for ctx, want in zip(pair, ref):
        assert all(np.array_equal(a, b) for a, b in zip(state(ctx), want))
        ctx.close()
