"""FP64 homogeneous 2D applies: the few-launch form against the general passes (which a plan
with fixed execution forms takes, and which the oracle parity tests check).  Both evaluate the
same compressed operator in FP64 with sums in different orders: at most a few thousand terms
per value, 2^-53 sqrt(4000) = 7e-15 relative to the absolute sums; the bar is 1e-12."""
import numpy as np
import pytest

from paper_1610_00835_amd import inputs
from tests.gpu_util import gpu_apply, rel_l2

pytestmark = pytest.mark.gpu


# leaf lattices: 3 x 3 (one far level, the launches end on it), 3 x 1, 5 x 9 with ragged cells
# (odd boxes on every level), 16 x 2, 33 x 17 (six levels, an odd step), 64 x 64 (row tiles
# together); every order
@pytest.mark.parametrize("n,order", [((24, 24), 8), ((17, 8), 2), ((39, 70), 3), ((128, 9), 4), ((260, 133), 5),
                                     ((260, 133), 8), ((100, 100), 7), ((512, 512), 6), ((511, 505), 8)])
@pytest.mark.parametrize("scheme", [0, 1])
def test_hom2d_equals_general_passes(n, order, scheme):
    from paper_1610_00835_amd import ertvie
    if scheme == 1 and max(n) > 128:
        pytest.skip("one small size per form is enough for the second kernel")
    N = n[0] * n[1]
    h = 1.0 / max(n)
    rng = np.random.default_rng(7)
    ss = rng.uniform(0.0, 3.0, N)
    X = inputs.random_vector(N, 3, nrhs=3)
    kw = dict(method="fmm", prec="fp64", cheb_n=order, nrhs_max=3, scheme=scheme)
    with ertvie.Plan(2, n, h, np.full(N, 3.0), ss, form=(1, 1), **kw) as a, \
            ertvie.Plan(2, n, h, np.full(N, 3.0), ss, **kw) as b:
        assert b.fmm_info()["form_near"] == -1
        assert b.fmm_info()["rank"] == a.fmm_info()["rank"]
        for op in (ertvie.OP_G, ertvie.OP_GS, ertvie.OP_A):
            ya = gpu_apply(a, X[:, 0], op)
            for _ in range(4):                      # eager, captured, replayed
                yb = gpu_apply(b, X[:, 0], op)
                assert rel_l2(yb, ya) <= 1e-12
        Ya = gpu_apply(a, X, ertvie.OP_A)
        for _ in range(3):
            Yb = gpu_apply(b, X, ertvie.OP_A)
            assert max(rel_l2(Yb[:, k], Ya[:, k]) for k in range(3)) <= 1e-12
        # uncompressed translations
    with ertvie.Plan(2, n, h, np.full(N, 3.0), ss, form=(1, 1), svd_tol=-1.0, **kw) as a, \
            ertvie.Plan(2, n, h, np.full(N, 3.0), ss, svd_tol=-1.0, **kw) as b:
        assert rel_l2(gpu_apply(b, X[:, 1], ertvie.OP_GS), gpu_apply(a, X[:, 1], ertvie.OP_GS)) <= 1e-12


@pytest.mark.parametrize("n", [(24, 24), (39, 70), (264, 264)])
def test_stage_profile(n):
    """Every stage that the plan has is timed: near field, P2M, translations and L2P on any tree,
    M2M and L2L above a second far level; the results stay those of an unprofiled apply."""
    from paper_1610_00835_amd import ertvie
    N = n[0] * n[1]
    x = inputs.random_vector(N, 3)
    with ertvie.Plan(2, n, 1.0 / max(n), np.full(N, 3.0), np.full(N, 2.0), method="fmm", cheb_n=6) as plan:
        levels = plan.fmm_info()["levels"]
        want = gpu_apply(plan, x, ertvie.OP_A)
        plan.profile(True)
        got = gpu_apply(plan, x, ertvie.OP_A)
        prof = plan.profile(False)
        assert np.array_equal(got, want)
        for _ in range(3):
            assert np.array_equal(gpu_apply(plan, x, ertvie.OP_A), want)
    stages = {"near", "p2m", "m2l", "l2p"} | ({"m2m", "l2l"} if levels > 2 else set())
    assert {k for k, v in prof.items() if v[0] > 0.0 and v[1] > 0} == stages


@pytest.mark.parametrize("n,order", [((260, 133), 5), ((264, 264), 8)])
def test_hom2d_second_kernel_on_larger_trees(n, order):
    """The kernel of cell integrals (scheme 1) on trees of five and six levels; same bar."""
    from paper_1610_00835_amd import ertvie
    N = n[0] * n[1]
    ss = np.random.default_rng(7).uniform(0.0, 3.0, N)
    X = inputs.random_vector(N, 3, nrhs=3)
    kw = dict(method="fmm", prec="fp64", cheb_n=order, nrhs_max=3, scheme=1)
    with ertvie.Plan(2, n, 1.0 / max(n), np.full(N, 3.0), ss, form=(1, 1), **kw) as a, \
            ertvie.Plan(2, n, 1.0 / max(n), np.full(N, 3.0), ss, **kw) as b:
        assert b.fmm_info()["form_near"] == -1
        for op in (ertvie.OP_G, ertvie.OP_A):
            ya, yb = gpu_apply(a, X, op), gpu_apply(b, X, op)
            assert max(rel_l2(yb[:, k], ya[:, k]) for k in range(3)) <= 1e-12
