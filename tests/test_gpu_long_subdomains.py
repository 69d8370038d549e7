"""Basis functions of chains as long as, and longer than, the basis-function
kernel keeps on chip (4096 rows), against their exact values.

In a chain with conductances c between cells, the local operator closes the
couplings to the neighbouring subdomains with twice their conductance, and the
basis function of the left interface falls from 1 with the resistance passed:
phat_k = 1 - (1/(2 c_left) + sum of 1/c up to cell k) / the whole resistance.
The conductances are multiples of 1/64, so that the matrix is exact.

Tolerance: the values are corrected once for their residual in twice the
working precision, which leaves the rounding of the result: 1e-15.  (The
uncorrected ones are off by the chain's condition, 1e7, times 1e-16.)"""
import numpy as np
import pytest

pytest.importorskip("torch")

import paper_2607_22905_amd as am  # noqa: E402
from workloads.tpfa import CSR  # noqa: E402

pytestmark = pytest.mark.gpu


def _chain(sizes, seed):
    n = int(sum(sizes))
    c = np.random.default_rng(seed).integers(32, 128, n - 1) / 64.0
    d = np.zeros(n)
    d[:-1] += c
    d[1:] += c
    d[0] += 1.0
    rp = np.concatenate([[0], np.cumsum(np.r_[2, np.full(n - 2, 3), 2])]).astype(np.int64)
    col = np.empty(rp[-1], np.int32)
    val = np.empty(rp[-1])
    for i in range(n):
        js = [j for j in (i - 1, i, i + 1) if 0 <= j < n]
        col[rp[i]:rp[i + 1]] = js
        val[rp[i]:rp[i + 1]] = [d[i] if j == i else -c[min(i, j)] for j in js]
    return CSR(n, rp, col, val), c, np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)


@pytest.mark.parametrize("sizes", [(64, 4096, 70), (64, 4097, 70), (4161, 4096, 9000, 30)])
def test_basis_functions(sizes):
    A, c, part = _chain(sizes, len(sizes))
    h = am.AlgMortar(A, part, len(sizes))
    end = np.cumsum(sizes)
    for s in range(1, len(sizes) - 1):  # interface s - 1 on the left, s on the right
        a, b = int(end[s - 1]), int(end[s])
        r = 1.0 / c.astype(np.longdouble)
        passed = r[a - 1] / 2 + np.concatenate([[0], np.cumsum(r[a:b - 1])])
        fall = passed / (passed[-1] + r[b - 1] / 2)
        for iface, ref in ((s - 1, 1 - fall), (s, fall)):
            v = h.export_mbf(iface, s, sizes[s])
            assert np.abs(v - ref).max() <= 1e-15, (s, iface)
    h.close()
