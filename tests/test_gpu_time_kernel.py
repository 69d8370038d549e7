"""Timing the interface solve of a handle with a small interface system: in
the local kernel for few columns (nothing to time), a launch of its own for
more."""
import pytest

pytest.importorskip("torch")

import paper_2607_22905_amd as am  # noqa: E402
from workloads import make_config  # noqa: E402

pytestmark = pytest.mark.gpu


def test_interface_solve_by_columns():
    P = make_config("c2", nx=32, ny=32, nz=32)
    part, m = am.partition_blocks(P.dims, P.partition[1])
    h = am.AlgMortar(P.A, part, m, max_nrhs=8)
    with pytest.raises(am.AlgMortarError) as e:
        h.time_kernel("gemv", nrhs=1)
    assert e.value.status_name == "AM_ERR_ARG"
    ms, by = h.time_kernel("gemv", nrhs=8)
    assert 0.0 < ms < 1.0
    assert by == 8.0 * h.n_iface * (h.n_iface + 3 * 8)
    h.close()
