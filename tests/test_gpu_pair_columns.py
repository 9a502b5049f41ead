"""FP64 products over the heterogeneous caches for several right-hand sides: every column of
a many-column apply equals the one-column apply of the same plan (streamed, the form that the
oracle parity tests check).  Both add the same FP32-stored values times FP64 vectors in FP64,
in different orders: sums of at most 27 x 512 + 189 x 512 terms differ by less than
2^-53 sqrt(1.1e5) relative to their absolute sum, 4e-14; the bar is 1e-12."""
import numpy as np
import pytest

from paper_1610_00835_amd import inputs
from tests.gpu_util import gpu_apply, rel_l2

pytestmark = pytest.mark.gpu


# block sizes (leaf cells, nodes): 512 and 216; 64 and 64; 216 and 128 (125 padded); 8 and 8;
# 343 (not whole 16-byte pieces: streamed) and 352; 2D 64 and 36; 2D 36 and 16; 512 and 512
@pytest.mark.parametrize("n,leaf,order", [((30, 25, 34), 8, 6), ((18, 20, 17), 4, 4), ((25, 24, 26), 6, 5),
                                          ((9, 10, 8), 2, 2), ((29, 28, 30), 7, 7), ((50, 37), 8, 6),
                                          ((40, 31), 6, 4), ((32, 26, 28), 8, 8)])
def test_columns_equal_single_applies(n, leaf, order):
    from paper_1610_00835_amd import ertvie
    case = inputs.make_case("c3", n=n, seed=2)
    case["h"] = 1.0 / 64
    N = int(np.prod(n))
    X = inputs.random_vector(N, 5, nrhs=67)
    with ertvie.plan_from_case(case, method="fmm", prec="fp64", leaf=leaf, cheb_n=order, nrhs_max=67) as plan:
        one = np.stack([gpu_apply(plan, np.ascontiguousarray(X[:, b]), ertvie.OP_A) for b in range(67)], axis=1)
        assert np.isfinite(one).all()
        for nrhs in (2, 3, 4, 5, 16, 17, 32, 33, 48, 49, 64, 67):
            Y = gpu_apply(plan, np.asfortranarray(X[:, :nrhs]), ertvie.OP_A)
            assert max(rel_l2(Y[:, b], one[:, b]) for b in range(nrhs)) <= 1e-12, nrhs


# few blocks, where 33 columns and more take one pass of 64, and blocks of 512 rows whose rounds of
# workgroups end nearly empty, where 3 and 4 columns are streamed (64 leaves: 532 pairs)
@pytest.mark.parametrize("n,order", [((16, 16, 16), 6), ((20, 17, 24), 6), ((32, 32, 32), 4)])
def test_columns_of_few_blocks(n, order):
    from paper_1610_00835_amd import ertvie
    case = inputs.make_case("c3", n=n, seed=2)
    case["h"] = 1.0 / 32
    N = int(np.prod(n))
    X = inputs.random_vector(N, 5, nrhs=100)
    with ertvie.plan_from_case(case, method="fmm", prec="fp64", cheb_n=order, nrhs_max=100) as plan:
        one = np.stack([gpu_apply(plan, np.ascontiguousarray(X[:, b]), ertvie.OP_A) for b in range(100)], axis=1)
        for nrhs in (3, 4, 5, 33, 48, 49, 100, 36):
            Y = gpu_apply(plan, np.asfortranarray(X[:, :nrhs]), ertvie.OP_A)
            assert max(rel_l2(Y[:, b], one[:, b]) for b in range(nrhs)) <= 1e-12, nrhs
