"""A stored zero inside a subdomain, further from the diagonal than the band,
that new values make nonzero.  The order of the rows was chosen without it; it
counts in A but is not part of the local operators, whose factors, couplings
and basis functions leave it out.  Against dense solves without it, to the
bars of the other local solves and applications (FP64 1e-12, FP32 2e-6)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2607_22905_amd as am  # noqa: E402
from oracle import AlgMortarCPU  # noqa: E402
from tests._problems import dense_csr  # noqa: E402
from tests.test_gpu_block_inverse import BOX, _band_matrix, _local_reference  # noqa: E402
from workloads.tpfa import CSR  # noqa: E402

pytestmark = pytest.mark.gpu


def _gpu(x):
    return torch.as_tensor(x, dtype=torch.float64, device="cuda:0")


@pytest.mark.parametrize("nrhs", [1, 8])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 2e-6)])
def test_stored_zero_becomes_a_coupling(prec, tol, nrhs):
    sizes = (300, 64, 321)
    _, D, part = _band_matrix(sizes, BOX, 11)
    n = part.size
    pairs = [(20, 250), (5, 140), (400, 600)]
    for i, j in pairs:  # room on the diagonals
        D[i, i] += 1.0
        D[j, j] += 1.0
    F = D.copy()
    for i, j in pairs:
        F[i, j] = F[j, i] = -0.75
    full = dense_csr(F)
    rows = np.repeat(np.arange(n), np.diff(full.row_ptr))
    A = CSR(n, full.row_ptr, full.col, D[rows, full.col])  # zeros at the pairs
    h = am.AlgMortar(A, part, len(sizes), prec=prec, max_nrhs=nrhs)
    h.update_values(full)
    r = np.random.default_rng(1).standard_normal(n)
    z = h.local_solve(_gpu(r)).cpu().numpy()
    ref = _local_reference(D, part, r)
    assert np.linalg.norm(z - ref) <= tol * np.linalg.norm(ref)
    # the interfaces are untouched: the application is that of the matrix
    # without the pairs
    ora = AlgMortarCPU(dense_csr(D), part)
    R = np.random.default_rng(2).standard_normal((nrhs, n))
    Z = h.apply(_gpu(R if nrhs > 1 else R[0])).cpu().numpy().reshape(nrhs, -1)
    for k in range(nrhs):
        ref = ora.apply(R[k])
        assert np.linalg.norm(Z[k] - ref) <= tol * np.linalg.norm(ref), k
    # a solve is one with all entries
    B = np.random.default_rng(3).standard_normal((nrhs, n))
    X, info, _ = h.pcg(_gpu(B if nrhs > 1 else B[0]), 1e-12)
    X = X.cpu().numpy().reshape(nrhs, -1)
    for k in range(nrhs):
        x = np.linalg.solve(F, B[k])
        assert np.linalg.norm(X[k] - x) <= 1e-9 * np.linalg.norm(x), k
    h.close()
