"""Local solves with FP32 and BF16 factors where a conductive body lies inside
a subdomain.  The inverse of a block is then nearly of rank one over the body,
and rounding its entries would lose its small eigenvalues, or their sign; the
set-up keeps such a subdomain's blocks as triangular factors, whose product is
definite whatever the rounding.

Iterations: at most five more than with rounded unit triangular band factors
(LIMITS: that form in numpy, FP32 arithmetic, on the same systems), whose
preconditioner is definite for any rounding, too.

Local solves of a positive right-hand side: the inverse of an M-matrix is made
of sums of nonnegative products throughout, so each component's relative error
is at most the number of roundings on a path: 2^-24 for each of some 30 blocks
of 140 operations in FP32, of which they average out to a few per cent: 1e-5;
2^-9 for each of the two factors of up to 30 blocks with BF16 factors: 0.12."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2607_22905_amd as am  # noqa: E402
from tests._problems import dense_csr  # noqa: E402
from tests.test_gpu_block_inverse import BOX, WIDE, _local_reference  # noqa: E402
from workloads.configs import cartesian_problem  # noqa: E402

pytestmark = pytest.mark.gpu

DIR = [(0, 0, 1.0), (0, 1, 0.0)]
# (body, precision, contrast): iterations to 1e-8 with triangular band factors
LIMITS = {
    ("cube", "bf16", 1e1): 17, ("cube", "bf16", 1e2): 19, ("cube", "bf16", 1e3): 21,
    ("cube", "bf16", 1e4): 26, ("cube", "bf16", 1e6): 77,
    ("cube", "fp32", 1e4): 12, ("cube", "fp32", 1e6): 12, ("cube", "fp32", 1e8): 20,
    ("cube", "fp32", 1e10): 25, ("cube", "fp64", 1e12): 16,
    ("plate", "bf16", 1e2): 18, ("plate", "bf16", 1e3): 21, ("plate", "bf16", 1e4): 27,
    ("plate", "bf16", 1e6): 48,
    ("plate", "fp32", 1e4): 13, ("plate", "fp32", 1e6): 13, ("plate", "fp32", 1e8): 16,
    ("plate", "fp32", 1e10): 24, ("plate", "fp64", 1e12): 14,
}


def _body(kind, contrast, n=16, box=8):
    """16^3 cells in 8^3 boxes, a body of the given contrast in each: a cube
    of 4^3 cells or a plate of 1 x 6 x 6."""
    g = np.zeros((n, n, n))
    w = (slice(2, 6),) * 3 if kind == "cube" else (slice(3, 4), slice(1, 7), slice(1, 7))
    for a in range(0, n, box):
        for b in range(0, n, box):
            for c in range(0, n, box):
                g[a:a + box, b:b + box, c:c + box][w] = np.log(contrast)
    P = cartesian_problem("body", n, n, n, g, DIR, None, (box,) * 3, 1e-8)
    part, m = am.partition_blocks(P.dims, (box,) * 3)
    return P, part, m


def _gpu(x):
    return torch.as_tensor(x, dtype=torch.float64, device="cuda:0")


PRODUCTS = {"separate_iface": True, "bf16_products": True}  # an option of the BF16 form
FORMS = [(c, nrhs, {}) for c in LIMITS for nrhs in (1, 2, 4, 8, 16)] + \
        [(c, nrhs, PRODUCTS) for c in LIMITS for nrhs in (1, 16) if c[1] == "bf16"]


@pytest.mark.parametrize("case,nrhs,kw", FORMS, ids=["%s-%s-%.0e-%d%s" % (*c, n, "-products" if k else "")
                                                     for c, n, k in FORMS])
def test_solve(case, nrhs, kw):
    kind, prec, contrast = case
    P, part, m = _body(kind, contrast)
    h = am.AlgMortar(P.A, part, m, prec=prec, max_nrhs=nrhs, **kw)
    B = np.random.default_rng(nrhs).standard_normal((nrhs, P.n))
    B[0] = P.b
    X, info, status = h.pcg(_gpu(B if nrhs > 1 else B[0]), 1e-8, 300, raise_on_error=False)
    assert status == 0 and all(i["converged"] == 1 for i in info), info
    if not kw:  # (vectors rounded to BF16 in the products: iterations of their own)
        assert info[0]["iterations"] <= LIMITS[case] + 5, info[0]
    h.close()


def _contrast_matrix(sizes, offsets, seed):
    """As the band matrices of the well-conditioned tests, but with the middle
    half of every subdomain 1e6 times as conductive and hardly any dominance."""
    rng = np.random.default_rng(seed)
    part = np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)
    n = int(part.size)
    start = np.repeat(np.cumsum(sizes) - sizes, sizes)
    size = np.repeat(sizes, sizes)
    pos = np.arange(n) - start
    body = (4 * pos >= size) & (4 * pos < 3 * size)
    D = np.zeros((n, n))
    for o in offsets:
        i = np.arange(n - o)
        i = i[part[i] == part[i + o]]
        D[i, i + o] = -rng.uniform(0.1, 1.0, i.size) * np.where(body[i] & body[i + o], 1e6, 1.0)
    ends = np.cumsum(sizes)[:-1]
    D[ends - 1, ends] = -rng.uniform(0.1, 1.0, ends.size)
    D = D + D.T
    D[np.arange(n), np.arange(n)] = np.abs(D).sum(1) + np.where(body, 0.0, 0.05)
    return dense_csr(D), D, part


SIZES = [((1, 2, 63, 64, 65), BOX), ((127, 128, 129, 191, 193), WIDE), ((511, 512, 513), BOX),
         ((576, 577, 640, 641), WIDE), ((575, 705, 895, 950), BOX)]


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-5), ("bf16", 0.12)])
@pytest.mark.parametrize("tile", [0, 1, 2])
@pytest.mark.parametrize("case", range(len(SIZES)))
def test_local_solves(case, tile, prec, tol, monkeypatch):
    monkeypatch.setenv("ALGMORTAR_TILE", str(tile))
    sizes, offsets = SIZES[case]
    A, D, part = _contrast_matrix(sizes, offsets, case)
    h = am.AlgMortar(A, part, len(sizes), prec=prec)
    r = np.random.default_rng(7).uniform(0.5, 1.0, A.n)
    z = h.local_solve(_gpu(r)).cpu().numpy()
    ref = _local_reference(D, part, r)
    assert np.abs(z / ref - 1.0).max() <= tol
    h.close()


@pytest.mark.parametrize("nrhs", [2, 4, 8, 16])
@pytest.mark.parametrize("prec,tol", [("fp32", 1e-5), ("bf16", 0.12)])
@pytest.mark.parametrize("case", range(len(SIZES)))
def test_columns(case, prec, tol, nrhs):
    """Every column count's kernel: the columns of an application against those
    of the one-column kernel on the same handle (a positive right-hand side:
    the coarse part is positive, too)."""
    sizes, offsets = SIZES[case]
    A, D, part = _contrast_matrix(sizes, offsets, 20 + case)
    h = am.AlgMortar(A, part, len(sizes), prec=prec, max_nrhs=nrhs)
    R = _gpu(np.random.default_rng(nrhs).uniform(0.5, 1.0, (nrhs, A.n)))
    Z = h.apply(R).cpu().numpy()
    for k in range(nrhs):
        z = h.apply(R[k].contiguous()).cpu().numpy()
        assert np.abs(Z[k] / z - 1.0).max() <= 1e-5, k
    h.close()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_update_values(prec, monkeypatch):
    """The form follows the values: to a body, and back, each like a fresh
    set-up, bit for bit."""
    monkeypatch.setenv("ALGMORTAR_TILE", "0")
    (P0, part, m), (P1, _, _) = _body("cube", 2.0), _body("cube", 1e8)
    h = am.AlgMortar(P0.A, part, m, prec=prec)
    r = _gpu(np.random.default_rng(3).standard_normal(P0.n))
    for P in (P1, P0, P1):
        h.update_values(P.A)
        fresh = am.AlgMortar(P.A, part, m, prec=prec)
        assert torch.equal(h.apply(r), fresh.apply(r))
        fresh.close()
    h.close()


@pytest.mark.parametrize("prec,contrast", [("bf16", 1e4), ("fp32", 1e8)])
def test_smoothing_blocks(prec, contrast):
    """The smoother's block solves with a body inside the blocks."""
    P, part, m = _body("cube", contrast)
    h = am.AlgMortar(P.A, part, m, prec=prec)
    _, plain, _ = h.pcg(_gpu(P.b), 1e-8, 300)
    h.set_smoother(part // 2, m // 2, 1)
    _, info, _ = h.pcg(_gpu(P.b), 1e-8, 300)
    assert info[0]["converged"] == 1 and info[0]["iterations"] <= plain[0]["iterations"]
    h.close()
