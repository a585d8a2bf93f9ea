"""Paths of the chain kernel against the float64 oracle: a single substep
(all pairs, no list), chains whose pairs and bonds have nearest images across
the box, beads that change their cell within a step, wall sites within the
long reach of sigma = 2, for 8, 4 and 2 lanes per bead."""
import numpy as np
import pytest

from paper_1710_09421_amd import workloads
from tests.test_gpu_md import ek, errors, oracle_sim  # noqa: F401  (ek is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def compare(ek, wl, steps):
    ctx = ek.from_workload(wl, precision=ek.EK_FP64, poisson_tol=1e-10, poisson_check_every=1)
    sim = oracle_sim(wl, 1e-10)
    ctx.step(steps)
    sim.run(steps)
    err = errors(ctx, sim, wl)
    print({k: f"{v:.1e}" for k, v in err.items()}, flush=True)
    ctx.close()
    assert max(err.values()) < 1e-8, err     # as the other float64 comparisons
    return sim


def pore(n_beads, seed, shape=(48, 32, 32), **poly):
    wl = workloads.pore_system(shape, 8, 5, 0.01, 0.01, -0.01, n_beads, seed,
                               bead_q=workloads.STABLE_BEAD_CHARGE, steps=10)
    wl.polymer.update(poly)
    return wl


@pytest.mark.parametrize("n_beads", [2, 40, 80, 140])
@pytest.mark.parametrize("n_sub", [1, 2])
def test_few_substeps(ek, n_beads, n_sub):  # noqa: F811
    compare(ek, pore(n_beads, 51, M=2000.0, gamma=2.0, n_sub=n_sub), 3)


@pytest.mark.parametrize("n_beads", [9, 64, 70, 140])
@pytest.mark.parametrize("wrapped", [False, True])
def test_chain_across_the_box(ek, n_beads, wrapped):  # noqa: F811
    wl = pore(n_beads, 52)
    wl.beads_R = wl.beads_R + np.array([15.8, -16.3, 0.0])
    if wrapped:
        wl.beads_R[:, :2] %= 32.0
        assert np.abs(np.diff(wl.beads_R, axis=0)).max() > 16.0
    compare(ek, wl, 3)


@pytest.mark.parametrize("n_beads", [12, 64])
def test_beads_change_cells_within_a_step(ek, n_beads):  # noqa: F811
    wl = pore(n_beads, 53, gamma=0.5)
    v = np.random.default_rng(8).normal(size=wl.beads_R.shape)
    wl.beads_V = 0.35 * v / np.linalg.norm(v, axis=1, keepdims=True)
    cell = np.floor(wl.beads_R)
    sim = compare(ek, wl, 2)
    assert (np.floor(sim.R) != cell).any()


@pytest.mark.parametrize("n_beads", [6, 30])
@pytest.mark.parametrize("n_sub", [1, 8])
def test_walls_in_long_reach(ek, n_beads, n_sub):  # noqa: F811
    """sigma = 2, beads on a spiral half in the pore, 2.0 to 2.2 from its wall
    sites and the slab's face: the wall terms act on most of them."""
    wl = pore(n_beads, 54, shape=(48, 32, 32))
    k = np.arange(n_beads)
    z0 = wl.beads_R[0, 2] - 4.0
    ang = 2.1 * k / 2.9
    wl.beads_R = np.stack([15.5 + 2.9 * np.cos(ang), 15.5 + 2.9 * np.sin(ang), z0 + 0.55 * k], axis=1)
    wl.beads_V = np.zeros_like(wl.beads_R)
    wl.polymer.update(M=50.0, sigma=2.0, eps=0.05, gamma=2.0, n_sub=n_sub, bond="harmonic", k_bond=1.0,
                      l_bond=2.0)
    sim = compare(ek, wl, 3)
    assert np.abs(sim.V).max() > 1e-4
