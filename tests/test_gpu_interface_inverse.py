"""The explicit inverse of the interface matrix at the edges of its 64 x 64
tiles: chains of subdomains with 1 to 321 basis functions (one tile, one row
short of and beyond a tile, an even and an odd number of tiles) and a grid
whose dissection has several blocks, in the fused, the dense and the
dissection form, against numpy on the exported S.

Tolerance: the backward error bound of an elimination, n eps cond(S) relative
to the inverse."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2607_22905_amd as am  # noqa: E402
from tests.test_gpu_block_inverse import _band_matrix  # noqa: E402
from workloads import make_config  # noqa: E402

pytestmark = pytest.mark.gpu


def _check(h):
    S, X = h.export_interface("S"), h.export_interface("Sinv")
    ref = np.linalg.inv(S)
    n = S.shape[0]
    tol = n * np.finfo(float).eps * np.linalg.cond(S)
    assert np.linalg.norm(X - ref) <= max(tol, 1e-15) * np.linalg.norm(ref)
    assert np.array_equal(X, X.T)
    h.close()


@pytest.mark.parametrize("form", [{}, {"separate_iface": True},
                                  {"separate_iface": True, "dense_iface": True}],
                         ids=["fused", "dissection", "dense"])
@pytest.mark.parametrize("n_iface", [1, 63, 64, 65, 127, 128, 129, 191, 193, 321])
def test_chain(n_iface, form):
    A, _, part = _band_matrix([3] * (n_iface + 1), (1,), 100 + n_iface)
    _check(am.AlgMortar(A, part, n_iface + 1, **form))


@pytest.mark.parametrize("form", [{"separate_iface": True},
                                  {"separate_iface": True, "dense_iface": True}],
                         ids=["dissection", "dense"])
def test_grid(form):
    P = make_config("c2", nx=30, ny=25, nz=20)
    part, m = am.partition_blocks(P.dims, (5, 5, 5))
    _check(am.AlgMortar(P.A, part, m, **form))
