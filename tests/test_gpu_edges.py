"""GPU kernels at the sizes where their tiles, lane groups and dispatch rules
change, against the oracle or the plain definition of each result."""
import numpy as np
import pytest

from oracle import gomea_ref as G
from paper_2202_11001_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2202_11001_amd import dsm  # noqa: E402

DEV = "cuda:0"


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.fixture(scope="module")
def tiny_problem():
    w = W.tiny()
    return w, dsm.Problem.from_workload(w, max_solutions=512, max_fos_points=4)


def _random_population(w, S, seed):
    """Lattice coordinates with full-rank spread; feasibility plays no part."""
    rng = np.random.default_rng(seed)
    base = W.regular_grid(w.dims, w.mesh).astype(np.float64)
    d = rng.normal(0, 2.0, (S, 2, w.P, 3)) * W.free_mask(w.mesh)[None, None]
    return W.snap(np.clip(base[None, None] + d, -0.5, np.array(w.dims) - 0.5))


# one staging tile of 192 selected solutions: below, exactly one, one more, three with skipped indices among them
@pytest.mark.parametrize("n_sel", [30, 192, 193, 500])
def test_estimate_tiles(tiny_problem, n_sel):
    w, gp = tiny_problem
    X = _random_population(w, 512, n_sel)
    sel = np.random.default_rng(n_sel).permutation(512)[:n_sel].astype(np.int32)
    if n_sel == 500:
        sel[[0, 191, 192, 499]] = [-1, 512, 600, -7]
    tets = gp.topology()["tets"]
    off = np.array([0, 4, 7, 9, 10, 14], dtype=np.int32)  # 4, 3, 2, 1 points and 4 again
    pts = np.concatenate([tets[0], tets[20][:3], tets[30][:2], [13], tets[47]]).astype(np.int32)
    mean, chol = gp.estimate_elements(_t(X), _t(sel), _t(off), _t(pts))
    rmean, _, rchol = G.estimate_elements(X, sel, off, pts, w.mesh)
    np.testing.assert_allclose(mean.cpu().numpy(), rmean, rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(chol.cpu().numpy(), np.array([G.packed_lower(L) for L in rchol]), rtol=1e-8, atol=1e-10)
    p1 = np.arange(w.P, dtype=np.int32)
    mean, chol = gp.estimate_distributions(_t(X), _t(sel), _t(p1))
    rmean, _, rchol = G.estimate(X, sel, p1, w.mesh)
    np.testing.assert_allclose(mean.cpu().numpy(), rmean, rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(chol.cpu().numpy(), np.array([G.packed_lower(L) for L in rchol]), rtol=1e-9, atol=1e-12)
