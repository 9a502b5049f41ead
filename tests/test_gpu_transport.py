"""GPU parity of Algorithm 1 step S.3 (ert_vie_transport) against its reference
(oracle/transport.py): the same step-characteristic sums in FP64 on both sides,
so the bar is relative L2 <= 1e-12 per direction (summation order and the
interpolation's h vs 1/h scaling differ)."""
import numpy as np
import pytest

from oracle import transport as T
from paper_1610_00835_amd import inputs
from tests.gpu_util import log, rel_l2, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ev():
    from paper_1610_00835_amd import ertvie
    ertvie.load()
    return ertvie


def _dirs(dim, k, seed):
    rng = np.random.default_rng(seed)
    d = rng.standard_normal((k, dim))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    return np.concatenate([d, np.eye(dim), -np.eye(dim)[:1]])


def _run(ev, case, U, f, dirs):
    import torch
    with ev.plan_from_case(case, method="direct", prec="fp64") as plan:
        phi = torch.empty((len(dirs), plan.N), dtype=torch.float64, device="cuda")
        plan.transport(to_dev(U) if U is not None else None, to_dev(f) if f is not None else None, dirs, phi)
        torch.cuda.synchronize()
        return phi.cpu().numpy()


@pytest.mark.parametrize("name,n", [("c1", (16, 12)), ("c2", (8, 8, 8)), ("c3", (10, 9, 8)), ("c5", (12, 12, 12))])
def test_transport_matches_reference(ev, name, n):
    case = inputs.make_case(name, n=n, seed=2)
    N = int(np.prod(n))
    rng = np.random.default_rng(3)
    U = rng.uniform(0, 1, N)
    dirs = _dirs(case["dim"], 5, 4)
    got = _run(ev, case, U, case["f"], dirs)
    ref = T.recover(U, case["f"], case["sigma_t"], case["sigma_s"], case["n"], case["h"], dirs)
    errs = [rel_l2(got[k], ref[:, k]) for k in range(len(dirs))]
    log("S.3", name, n, "max rel L2 over directions", max(errs))
    assert max(errs) <= 1e-12
    # the source alone, and U alone
    g2 = _run(ev, case, None, case["f"], dirs[:2])
    assert rel_l2(g2[0], T.sweep(case["f"], case["sigma_t"], case["n"], case["h"], dirs[0])) <= 1e-12


def test_transport_full_size_sampled_cells(ev):
    """The 128^3 many-scattering medium, 6 directions, 300 sampled cells."""
    case = inputs.make_case("c5", n=(128, 128, 128), seed=0)
    N = 128 ** 3
    U = np.random.default_rng(5).uniform(0, 1, N)
    dirs = _dirs(3, 3, 6)
    got = _run(ev, case, U, case["f"], dirs)
    cells = np.random.default_rng(7).choice(N, size=300, replace=False)
    ref = T.recover(U, case["f"], case["sigma_t"], case["sigma_s"], case["n"], case["h"], dirs, cells=cells)
    errs = [rel_l2(got[k][cells], ref[:, k]) for k in range(len(dirs))]
    log("S.3 128^3 sampled cells, max rel L2", max(errs))
    assert max(errs) <= 1e-12


def test_transport_rejects_non_unit_directions(ev):
    import torch
    case = inputs.make_case("c1", n=(8, 8))
    with ev.plan_from_case(case, method="direct", prec="fp64") as plan:
        phi = torch.empty((1, 64), dtype=torch.float64, device="cuda")
        with pytest.raises(ev.ErtError) as ei:
            plan.transport(None, to_dev(case["f"]), np.array([[1.0, 0.1]]), phi)
        assert ei.value.status == ev.EINVAL


@pytest.mark.parametrize("n,scale", [((17, 8, 5), 1.0), ((9, 9, 9), 10.0), ((1, 9, 33), 100.0), ((70, 3, 2), 10.0),
                                     ((2, 2), 1.0), ((33, 17), 10.0), ((1, 70), 100.0), ((65, 40), 1.0)])
def test_transport_tiles_and_step_ranges(ev, n, scale):
    """Grids around and below a tile of cells (thin ones too), independent cell values, steps of
    an optical depth about 0.05, 0.5 and 5 (the three ranges of the step's integral)."""
    N, h = int(np.prod(n)), 0.1
    rng = np.random.default_rng(N)
    st = scale * rng.uniform(0.5, 1.5, N)
    case = {"dim": len(n), "n": n, "h": h, "kernel": 1, "sigma_t": st, "sigma_s": 0.9 * st, "f": rng.uniform(0, 1, N)}
    U = rng.uniform(0, 1, N)
    dirs = _dirs(len(n), 3, 4)
    got = _run(ev, case, U, case["f"], dirs)
    ref = T.recover(U, case["f"], st, 0.9 * st, n, h, dirs)
    assert max(rel_l2(got[k], ref[:, k]) for k in range(len(dirs))) <= 1e-12


@pytest.mark.parametrize("n", [(1, 1, 600), (2, 2, 300), (600, 1, 1), (1, 700, 1), (3, 2, 129), (2, 260, 1), (1, 30, 80),
                               (1, 600), (700, 1), (2, 300), (150, 3), (2, 70, 90)])
def test_transport_thin_grids(ev, n):
    """Tiles up to a line of 512 cells and short rays (small windows), axis-parallel directions
    among them; independent cell values."""
    N, h, d = int(np.prod(n)), 0.1, len(n)
    rng = np.random.default_rng(N)
    st = rng.uniform(0.5, 8.0, N)
    case = {"dim": d, "n": n, "h": h, "kernel": 1, "sigma_t": st, "sigma_s": 0.9 * st, "f": rng.uniform(0, 1, N)}
    U = rng.uniform(0, 1, N)
    dirs = np.concatenate([_dirs(d, 5, 4), np.eye(d), -np.eye(d)])
    got = _run(ev, case, U, case["f"], dirs)
    ref = T.recover(U, case["f"], st, 0.9 * st, n, h, dirs)
    assert max(rel_l2(got[k], ref[:, k]) for k in range(len(dirs))) <= 1e-12
