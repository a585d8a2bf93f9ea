"""Batches of SOR iterations that end without a result (a wait gives up, a launch
is refused) hand the solve to single launches where they stand: bits, iteration
counts and residuals are those of single launches all along."""
import ctypes

import numpy as np
import pytest

from paper_1710_09421_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NEVER, LIMIT = -1, 1 << 20


@pytest.fixture(scope="module")
def ek():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1710_09421_amd import ek as binding
    binding.lib()
    return binding


def _ends(ek, ctx, limit=LIMIT, limit_from=0, refuse_at=NEVER):
    """A wait of launch `limit_from` on gives up after `limit` looks; launch
    `refuse_at` is refused (0: single launches only)."""
    fn = ek.lib().ek_test_sor_batches
    fn.restype, fn.argtypes = None, [ctypes.c_void_p] + [ctypes.c_int] * 3
    fn(ctx._h, limit, limit_from, refuse_at)


ENDS = [dict(limit=0), dict(limit=0, limit_from=1), dict(limit=0, limit_from=2),
        dict(refuse_at=0), dict(refuse_at=1), dict(refuse_at=2), dict(refuse_at=3)]


@pytest.mark.parametrize("end", ENDS, ids=lambda e: "-".join(f"{k}={v}" for k, v in e.items()))
@pytest.mark.parametrize("shape,check", [((24, 16, 20), 1),    # one batch and its second run
                                         ((64, 64, 64), 1),    # two batches
                                         ((64, 64, 64), 7)])
def test_solve_goes_on_with_single_launches(ek, shape, check, end):
    rng = np.random.default_rng(sum(shape))
    p = ek.make_params(shape, precision=ek.EK_FP64, poisson_method=ek.EK_POISSON_SOR,
                       poisson_tol=1e-10, poisson_max_iter=20000, poisson_check_every=check)
    ctx = ek.Context(p)
    _ends(ek, ctx, **end)
    for _ in range(2):             # the second solve takes single launches from its start
        rho = torch.tensor(rng.normal(size=shape) * 0.01, dtype=torch.float64, device="cuda")
        start = torch.tensor(rng.normal(size=shape) * 0.1, dtype=torch.float64, device="cuda")
        psi, ref = start.clone(), start.clone()
        rep = ctx.poisson_solve(rho, psi, ek.EK_WS_PREV)
        want = ek.poisson_solve_noalloc(p, rho, ref, ek.EK_WS_PREV)
        print(shape, end, rep, flush=True)
        assert rep == want
        assert torch.equal(psi, ref)
    ctx.close()


@pytest.mark.parametrize("end", [dict(limit=0), dict(limit=0, limit_from=1), dict(refuse_at=2)],
                         ids=lambda e: "-".join(f"{k}={v}" for k, v in e.items()))
def test_insulating_steps_go_on_with_single_launches(ek, end):
    wl = workloads.pore_system((32, 24, 24), 6, 4, 0.01, 0.01, -0.01, 0, 12, charge_sites="faces")
    out = []
    for e in (end, dict(refuse_at=0)):
        ctx = ek.from_workload(wl, precision=ek.EK_FP64, poisson_method=ek.EK_POISSON_SOR,
                               poisson_tol=1e-8, poisson_max_iter=20000,
                               walls=ek.EK_WALLS_INSULATING)
        _ends(ek, ctx, **e)
        ctx.step(3)
        st = ctx.stats()
        out.append(([a for s in range(3) for a in ctx.moments(s)] + [ctx.potential()],
                    st["poisson_iters"], st["poisson_residual"]))
        ctx.close()
    (a, ia, ra), (b, ib, rb) = out
    assert (ia, ra) == (ib, rb)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
