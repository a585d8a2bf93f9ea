"""SOR iterations run in batches of one launch (tiles in LDS, faces exchanged
between workgroups) against the same iterations launched half sweep by half
sweep: the no-allocation solve takes the latter and must give the same bits,
iteration counts and residuals.  Insulating walls against the oracle's
iterates."""
import numpy as np
import pytest

from oracle import poisson as opoisson
from paper_1710_09421_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ek():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1710_09421_amd import ek as binding
    binding.lib()
    return binding


def _both(ek, shape, tol, check, max_iter, seed, warm, repeats=2):
    rng = np.random.default_rng(seed)
    p = ek.make_params(shape, precision=ek.EK_FP64, poisson_method=ek.EK_POISSON_SOR,
                       poisson_tol=tol, poisson_max_iter=max_iter, poisson_check_every=check)
    ctx = ek.Context(p)
    for k in range(repeats):       # the second solve's batches follow the first one's count
        rho = torch.tensor(rng.normal(size=shape) * 0.01, dtype=torch.float64, device="cuda")
        start = torch.tensor(rng.normal(size=shape) * 0.1, dtype=torch.float64, device="cuda")
        out = []
        for solve in (ctx.poisson_solve, lambda r, s, w: ek.poisson_solve_noalloc(p, r, s, w)):
            psi = start.clone()
            try:
                rep = solve(rho, psi, ek.EK_WS_PREV if warm else ek.EK_WS_ZERO)
            except ek.EKError as e:
                assert e.status == ek.EK_ENOCONV
                rep = str(e)
            out.append((psi.cpu().numpy(), rep))
        print(shape, k, out[0][1])
        assert out[0][1] == out[1][1]
        assert np.array_equal(out[0][0], out[1][0]), shape
    ctx.close()


@pytest.mark.parametrize("shape", [
    (2, 2, 2), (4, 2, 6), (2, 6, 4),      # one row or plane per tile, a tile its own neighbour
    (34, 58, 62),                         # sides with few divisors
    (32, 32, 32), (64, 64, 64),           # one site of a colour per thread
    (128, 64, 64), (64, 128, 96)])        # two and three
def test_batches_give_the_bits_of_single_launches(ek, shape):
    _both(ek, shape, 1e-8, 1, 20000, sum(shape), True)


@pytest.mark.parametrize("check,max_iter", [(1, 20000), (3, 20000), (7, 20000), (100, 20000),
                                            (1, 1), (1, 5), (4, 70), (1, 64), (1, 65)])
def test_tests_and_limits_fall_where_single_launches_put_them(ek, check, max_iter):
    _both(ek, (24, 16, 20), 1e-10, check, max_iter, 7 + check + max_iter, False)


@pytest.mark.parametrize("shape", [(32, 24, 24), (128, 64, 64), (64, 96, 128)])
def test_insulating_iterates_match_the_oracle(ek, shape):
    """The iterate after a fixed number of iterations (a tolerance out of
    reach): a few roundings per iteration, so 1e-12 of the largest |psi|."""
    iterations = 3
    wl = workloads.pore_system(shape, 6, 4, 0.01, 0.0, -0.01, 0, 11, charge_sites="faces")
    ctx = ek.from_workload(wl, precision=ek.EK_FP64, poisson_method=ek.EK_POISSON_SOR,
                           poisson_tol=1e-30, poisson_max_iter=iterations,
                           walls=ek.EK_WALLS_INSULATING)
    with pytest.raises(ek.EKError) as e:
        ctx.step(1)
    assert e.value.status == ek.EK_ENOCONV
    solid = wl.solid.astype(bool)
    eps = 1.0 / (4 * np.pi * wl.bjerrum / 3.0)
    b = opoisson.neumann_rhs(wl.n0[1] - wl.n0[2], wl.wall_q, solid, eps)
    ref, _, _ = opoisson.sor_neumann(b, np.zeros(shape), ~solid, 0.0, 0, iterations=iterations)
    got = np.where(solid, 0.0, ctx.potential())
    err = np.abs(got - ref).max() / np.abs(ref).max()
    print(shape, err)
    assert err < 1e-12
    ctx.close()
