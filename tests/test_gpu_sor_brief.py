"""Solves about as short as single launches are cheaper for: after one of them a
solve begins with single launches and goes on with batches where they do not
suffice.  Bits, counts and residuals are those of single launches."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ek():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1710_09421_amd import ek as binding
    binding.lib()
    return binding


@pytest.mark.parametrize("check", [1, 2, 4, 7])
@pytest.mark.parametrize("shape", [(24, 16, 20), (48, 32, 64)])
def test_short_and_long_solves_in_turn(ek, shape, check):
    rng = np.random.default_rng(sum(shape) + check)
    p = ek.make_params(shape, precision=ek.EK_FP64, poisson_method=ek.EK_POISSON_SOR,
                       poisson_tol=1e-6, poisson_max_iter=20000, poisson_check_every=check)
    ctx = ek.Context(p)
    rho = torch.tensor(rng.normal(size=shape) * 0.01, dtype=torch.float64, device="cuda")
    noise = torch.tensor(rng.normal(size=shape), dtype=torch.float64, device="cuda")
    # starts: far, then next to the solution of a charge that hardly changes (some
    # iterations), then far again, and close to it
    solved = torch.zeros_like(rho)
    ek.poisson_solve_noalloc(p, rho, solved, ek.EK_WS_ZERO)
    counts = []
    for k, away in enumerate((1.0, 1e-6, 1e-7, 1e-6, 1.0, 1e-7, 1e-2, 3e-6, 3e-6)):
        start = solved + away * noise * solved.abs().max()
        psi, ref = start.clone(), start.clone()
        rep = ctx.poisson_solve(rho, psi, ek.EK_WS_PREV)
        want = ek.poisson_solve_noalloc(p, rho, ref, ek.EK_WS_PREV)
        counts.append(rep["iterations"])
        assert rep == want, (k, away)
        assert torch.equal(psi, ref), (k, away)
    print(shape, check, counts, flush=True)
    assert min(counts) * (1 + 1 / check) <= 20 < max(counts)
    ctx.close()


@pytest.mark.parametrize("limit", [6, 9, 30, 40])
def test_the_limit_after_a_short_solve(ek, limit):
    """A solve that begins with single launches and meets its cycle limit there or
    in the batches after them."""
    shape = (24, 16, 20)
    rng = np.random.default_rng(limit)
    p = ek.make_params(shape, precision=ek.EK_FP64, poisson_method=ek.EK_POISSON_SOR,
                       poisson_tol=1e-6, poisson_max_iter=limit)
    ctx = ek.Context(p)
    rho = torch.tensor(rng.normal(size=shape) * 0.01, dtype=torch.float64, device="cuda")
    noise = torch.tensor(rng.normal(size=shape), dtype=torch.float64, device="cuda")
    long = ek.make_params(shape, precision=ek.EK_FP64, poisson_method=ek.EK_POISSON_SOR,
                          poisson_tol=1e-6, poisson_max_iter=20000)
    solved = torch.zeros_like(rho)
    ek.poisson_solve_noalloc(long, rho, solved, ek.EK_WS_ZERO)
    psi = solved + 1e-7 * noise * solved.abs().max()
    first = ctx.poisson_solve(rho, psi, ek.EK_WS_PREV)["iterations"]
    assert 0 < first <= 6
    out = []
    for solve in (ctx.poisson_solve, lambda r, s, w: ek.poisson_solve_noalloc(p, r, s, w)):
        psi = solved + noise * solved.abs().max()
        with pytest.raises(ek.EKError) as e:
            solve(rho, psi, ek.EK_WS_PREV)
        assert e.value.status == ek.EK_ENOCONV
        out.append((str(e.value), psi))
    print(limit, first, out[0][0], flush=True)
    assert out[0][0] == out[1][0]
    assert torch.equal(out[0][1], out[1][1])
    ctx.close()
