"""Kernel caches and diagonal of heterogeneous media (plan set-up) against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ev():
    from paper_1610_00835_amd import ertvie
    ertvie.load()
    return ertvie


@pytest.mark.parametrize("n,h", [((9, 13), 0.1), ((2, 2), 0.3), ((5, 4, 6), 1.0 / 48), ((2, 3, 2), 0.25)])
def test_diagonal_of_rough_medium(ev, oracle_mod, n, h):
    """Independent cell values over three decades: every octant of every cell has its own
    coefficients, faces and corners of the grid included.  Bar: the diagonal's, 1e-13."""
    N = int(np.prod(n))
    st = 10.0 ** np.random.default_rng(N).uniform(-1.0, 2.0, size=N)
    P = oracle_mod.Problem(len(n), n, h, 1, st, 0.9 * st)
    with ev.Plan(len(n), n, h, st, 0.9 * st, kernel=1) as plan:
        np.testing.assert_allclose(plan.diag(), P.diag(), rtol=1e-13, atol=0)
