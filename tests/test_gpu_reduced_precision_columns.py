"""Reduced-precision applications of 8 and 16 columns (matrix cores) against
those of one column on the same handle, column by column, on subdomains of 1
to 15 blocks with full and ragged last blocks."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2607_22905_amd as am  # noqa: E402
from tests._problems import dense_csr  # noqa: E402
from tests.test_gpu_block_inverse import BOX, CASES, _band_matrix  # noqa: E402

pytestmark = pytest.mark.gpu


def _gpu(x):
    return torch.as_tensor(x, dtype=torch.float64, device="cuda:0")


@pytest.mark.parametrize("separate", [False, True])
@pytest.mark.parametrize("nrhs", [8, 16])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_apply(case, prec, nrhs, separate):
    """The same stored factors and FP32 arithmetic in another order: the
    roundings of two sweeps over at most 15 blocks on matrices of condition
    below 30, 2e-6 as for the solves against dense ones."""
    sizes, offsets = CASES[case]
    A, D, part = _band_matrix(sizes, offsets, 40 + case)
    h = am.AlgMortar(A, part, len(sizes), prec=prec, max_nrhs=nrhs, separate_iface=separate)
    R = _gpu(np.random.default_rng(nrhs).standard_normal((nrhs, A.n)))
    Z = h.apply(R).cpu().numpy()
    for k in range(nrhs):
        z = h.apply(R[k].contiguous()).cpu().numpy()
        assert np.linalg.norm(Z[k] - z) <= 2e-6 * np.linalg.norm(z), k
    h.close()


@pytest.mark.parametrize("separate", [False, True])
@pytest.mark.parametrize("nrhs", [5, 8, 16])
def test_reconstruction_is_fp64(nrhs, separate):
    """z = pbar + sum eta phat in FP64, whatever the factors: on a nearly
    singular system (one cell held, by 1e-6) the coarse part is some 1e5 times
    the local one, so that FP32 roundings of pbar (at most 1e-5 relative, all
    sums being of one sign) do not show in z, and those of the FP32 sums and
    products of the coarse part (3e-8) would.  (FP32 factors: with BF16 ones the
    interface matrix of so singular a system is refused.  Both run the same
    code.)"""
    sizes = (64, 65, 130, 200, 31)
    _, D, part = _band_matrix(sizes, BOX, 3)
    n = part.size
    D[np.arange(n), np.arange(n)] = 0.0
    D[np.arange(n), np.arange(n)] = np.abs(D).sum(1)
    D[5, 5] += 1e-6
    A = dense_csr(D)
    h = am.AlgMortar(A, part, len(sizes), prec="fp32", max_nrhs=nrhs, separate_iface=separate)
    R = _gpu(np.random.default_rng(nrhs).uniform(0.5, 1.0, (nrhs, n)))
    Z = h.apply(R).cpu().numpy()
    for k in range(nrhs):
        z = h.apply(R[k].contiguous()).cpu().numpy()
        pbar = h.local_solve(R[k].contiguous()).cpu().numpy()
        tol = 1e-5 * np.abs(pbar).max() / np.abs(z).min() + 1e-13
        assert tol < 1e-9
        assert np.abs(Z[k] / z - 1.0).max() <= tol, k
    h.close()


@pytest.mark.parametrize("case", range(len(CASES)))
def test_bf16_products(case):
    """BF16 x BF16 products: 16 columns (matrix cores) and one (vector units)
    round the same operands and keep the diagonals and what they multiply in
    FP32; the products are exact in FP32.  Sums in another order differ by some
    1e-7, which moves an operand of three in 1e5 over a rounding boundary, by
    2^-8: 1e-5 in the norm.  A rounded diagonal would show as 5e-4 and more."""
    sizes, offsets = CASES[case]
    A, D, part = _band_matrix(sizes, offsets, 60 + case)
    h = am.AlgMortar(A, part, len(sizes), prec="bf16", max_nrhs=16, separate_iface=True,
                     bf16_products=True)
    R = _gpu(np.random.default_rng(case).standard_normal((16, A.n)))
    Z = h.apply(R).cpu().numpy()
    for k in range(16):
        z = h.apply(R[k].contiguous()).cpu().numpy()
        assert np.linalg.norm(Z[k] - z) <= 1e-4 * np.linalg.norm(z), k
    h.close()
