"""FP64 products for several right-hand sides when the device memory holds the staging rows of a
whole pass for one product but not for the other: the apply runs in passes of four, with the
results of the whole pass."""
import numpy as np
import pytest

from paper_1610_00835_amd import inputs
from tests.gpu_util import rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu


def test_short_staging_memory():
    import torch
    from paper_1610_00835_amd import ertvie
    nrhs, n = 15, (64, 64, 64)
    case = inputs.make_case("c3", n=n, seed=2)
    case["h"] = 1.0 / 64
    N = int(np.prod(n))
    X = to_dev(inputs.random_vector(N, 5, nrhs=nrhs))
    Y = torch.empty_like(X)
    with ertvie.plan_from_case(case, method="fmm", cheb_n=4, nrhs_max=nrhs) as plan:
        want = to_host(plan.apply(X, Y, op=ertvie.OP_A)).copy()
    Y.zero_()
    with ertvie.plan_from_case(case, method="fmm", cheb_n=4, nrhs_max=nrhs) as plan:
        info = plan.fmm_info()
        leaves, cells = (n[0] // 8) ** 3, 8 ** 3
        vectors = 2 * nrhs * 8 * (leaves * cells + 2 * leaves * info["nodes_padded"])
        far = nrhs * 8 * max(info["far_pairs"]) * info["nodes_padded"]
        near = nrhs * 8 * leaves * 27 * cells
        torch.cuda.empty_cache()
        # the far rows fit whole, the near ones not, and four rows of each (4/15) do
        room = vectors + far + near // 8
        assert room > vectors + (far + near) * 4 // nrhs + (64 << 20)
        hold = []
        for _ in range(8):                       # memory freed before may come back late
            free = torch.cuda.mem_get_info()[0]
            if free <= room + (8 << 20):
                break
            hold.append(torch.empty(free - room, dtype=torch.uint8, device="cuda"))
        else:
            pytest.skip("the free memory does not settle")
        got = to_host(plan.apply(X, Y, op=ertvie.OP_A))
        again = to_host(plan.apply(X, Y, op=ertvie.OP_A))
        del hold
    torch.cuda.empty_cache()
    assert max(rel_l2(got[:, b], want[:, b]) for b in range(nrhs)) <= 1e-12
    assert np.array_equal(got, again)
