"""Matrix rows with more than 32 entries (a cell coupled to 31, 32, 40 or 75
others): the products with A in a solve, the residual of the smoother and the
true residual that a solve reports take every entry.

Tolerances: x to 1e-8 of a dense solve after a solve to 1e-12 (condition below
1e3); the reported residual ||b - A x|| / ||b|| to 1e-13 of numpy's on the
returned x (both are sums of at most 80 products per row, of size about 1)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2607_22905_amd as am  # noqa: E402
from tests._problems import dense_csr  # noqa: E402

pytestmark = pytest.mark.gpu


def _hub_matrix(others, seed=0):
    """300 cells in a chain, five subdomains of 60; cell 150 is coupled to
    `others` further cells, those of its own subdomain first."""
    rng = np.random.default_rng(seed)
    n = 300
    D = np.zeros((n, n))
    i = np.arange(n - 1)
    D[i, i + 1] = -rng.uniform(0.5, 1.0, n - 1)
    near = np.argsort(np.abs(np.arange(n) - 150.2), kind="stable")
    near = near[np.abs(near - 150) > 1][:others]
    D[np.minimum(near, 150), np.maximum(near, 150)] = -rng.uniform(0.5, 1.0, others)
    D = D + D.T
    D[np.arange(n), np.arange(n)] = np.abs(D).sum(1) + 0.05
    return dense_csr(D), D, np.repeat(np.arange(5), 60).astype(np.int32)


@pytest.mark.parametrize("smooth", [False, True])
@pytest.mark.parametrize("nrhs", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("others", [29, 30, 40, 75])
def test_solve(others, nrhs, smooth):
    A, D, part = _hub_matrix(others)
    assert int(np.diff(A.row_ptr).max()) == others + 3
    h = am.AlgMortar(A, part, 5, max_nrhs=nrhs)
    if smooth:
        h.set_smoother(part // 2, 3, 1)
    B = np.random.default_rng(nrhs).standard_normal((nrhs, A.n))
    X, info, _ = h.pcg(torch.as_tensor(B if nrhs > 1 else B[0], device="cuda:0"), 1e-12)
    X = X.cpu().numpy().reshape(nrhs, -1)
    for k in range(nrhs):
        ref = np.linalg.solve(D, B[k])
        true = np.linalg.norm(B[k] - D @ X[k]) / np.linalg.norm(B[k])
        assert np.linalg.norm(X[k] - ref) <= 1e-8 * np.linalg.norm(ref), k
        assert info[k]["converged"] == 1 and abs(info[k]["true_rel_res"] - true) <= 1e-13, k
    h.close()
