"""Applications and the exported inverse at the interface sizes where the
dissection form changes (one block, blocks of one row short of and beyond a
64-row tile, blocks with separators above them), 1 to 16 columns.  The export
of this form is what its solve makes of the unit vectors, so an error in the
block inverses, in the Schur complement's or in the couplings shows in it.

Tolerances: applications 1e-12 against the oracle, as elsewhere; the inverse
within n eps cond(S) of numpy's, the backward error bound of an elimination."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2607_22905_amd as am  # noqa: E402
from oracle import AlgMortarCPU  # noqa: E402
from tests.test_gpu_block_inverse import _band_matrix  # noqa: E402
from workloads import make_config  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [1, 2, 4, 16])
@pytest.mark.parametrize("n_iface", [1, 63, 64, 65, 128, 129, 193, 321])
def test_chain(n_iface, nrhs):
    A, _, part = _band_matrix([3] * (n_iface + 1), (1,), 200 + n_iface)
    ora = AlgMortarCPU(A, part)
    h = am.AlgMortar(A, part, n_iface + 1, separate_iface=True, max_nrhs=nrhs)
    R = np.random.default_rng(nrhs).standard_normal((nrhs, A.n))
    Z = h.apply(torch.as_tensor(R if nrhs > 1 else R[0], device="cuda:0")).cpu().numpy()
    for k, z in enumerate(Z.reshape(nrhs, -1)):
        ref = ora.apply(R[k])
        assert np.linalg.norm(z - ref) <= 1e-12 * np.linalg.norm(ref), k
    h.close()


@pytest.mark.parametrize("nrhs", [1, 2, 8])
def test_export_leaves_a_running_application_alone(nrhs):
    """A grid whose dissection has blocks and separators: the exported inverse,
    and applications queued around the export."""
    P = make_config("c2", nx=30, ny=25, nz=20)
    part, m = am.partition_blocks(P.dims, (5, 5, 5))
    order, blk, ntop = am.interface_nd(P.A, part, m, nrhs)
    assert blk.size > 2 and ntop > 0
    h = am.AlgMortar(P.A, part, m, separate_iface=True, max_nrhs=nrhs)
    r = torch.as_tensor(np.random.default_rng(0).standard_normal((nrhs, P.n)), device="cuda:0")
    z0 = h.apply(r)
    S = h.export_interface("S")
    for _ in range(20):
        z1 = h.apply(r)
    X = h.export_interface("Sinv")
    z2 = h.apply(r)
    assert torch.equal(z0, z1) and torch.equal(z0, z2)
    ref = np.linalg.inv(S)
    tol = S.shape[0] * np.finfo(float).eps * np.linalg.cond(S)
    assert np.linalg.norm(X - ref) <= tol * np.linalg.norm(ref)
    h.close()
