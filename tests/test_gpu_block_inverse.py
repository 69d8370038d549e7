"""The block-inverse local solves (bands within 64 rows) at the sizes where
they change form: subdomains of 1 to 15 blocks of 64 rows with full and ragged
last blocks (one block; two, whose second half has none; nine, kept whole in
registers; ten and more, whose outer blocks are streamed), rows with up to
nine couplings to the neighbouring block, 1 to 16 columns, every layout of
the kernel, FP64 and the reduced precisions, against dense solves.

Tolerances.  FP64: the bar of the other applies, 1e-12 relative.  FP32: 64
products and two sweeps over at most 15 blocks of rounding 2^-24 each, on
matrices of condition below 30: 2e-6.  BF16 factors: 2^-9 per stored entry and
the same condition: 0.05."""
import numpy as np
import pytest

import paper_2607_22905_amd as am
from workloads.tpfa import CSR

pytestmark = pytest.mark.gpu


def _band_matrix(sizes, offsets, seed):
    """Subdomains of the given sizes in a row: symmetric M-matrix with random
    negative couplings at the index distances `offsets` inside a subdomain
    and one link between consecutive ones; rows dominated by 10%."""
    rng = np.random.default_rng(seed)
    part = np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)
    n = int(part.size)
    D = np.zeros((n, n))
    for o in offsets:
        i = np.arange(n - o)
        ok = part[i] == part[i + o]
        D[i[ok], i[ok] + o] = -rng.uniform(0.1, 1.0, ok.sum())
    ends = np.cumsum(sizes)[:-1]
    D[ends - 1, ends] = -rng.uniform(0.1, 1.0, ends.size)
    D = D + D.T
    D[np.arange(n), np.arange(n)] = 1.1 * np.abs(D).sum(1) + 0.05
    row, col = np.nonzero(D)
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(row, minlength=n), out=rp[1:])
    return CSR(n, rp, col.astype(np.int32), D[row, col]), D, part


def _local_reference(D, part, r):
    x = np.zeros_like(r)
    for p in range(part.max() + 1):
        om = np.flatnonzero(part == p)
        rest = np.setdiff1d(np.arange(part.size), om)
        A = D[np.ix_(om, om)] - np.diag(D[np.ix_(om, rest)].sum(1))
        x[om] = np.linalg.solve(A, r[om])
    return x


WIDE = (1, 2, 7, 31, 40, 50, 57, 61, 63, 64)   # up to nine couplings a side
BOX = (1, 8, 64)                               # one
CASES = [
    ((1, 2, 63, 64, 65), BOX),
    ((127, 128, 129, 191, 193), WIDE),
    ((511, 512, 513), BOX),
    ((576, 577, 640, 641), BOX),
    ((575, 705, 895, 950), WIDE),
]
TOL = {"fp64": 1e-12, "fp32": 2e-6, "bf16": 0.05}


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("tile", [0, 1, 2])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_local_solves(case, tile, prec, monkeypatch):
    import torch
    monkeypatch.setenv("ALGMORTAR_TILE", str(tile))
    sizes, offsets = CASES[case]
    A, D, part = _band_matrix(sizes, offsets, case)
    h = am.AlgMortar(A, part, len(sizes), prec=prec)
    r = np.random.default_rng(7).standard_normal(A.n)
    z = h.local_solve(torch.as_tensor(r, device="cuda:0")).cpu().numpy()
    ref = _local_reference(D, part, r)
    for p in range(len(sizes)):  # each subdomain on its own
        om = part == p
        assert np.linalg.norm(z[om] - ref[om]) <= TOL[prec] * np.linalg.norm(ref[om]), (p, sizes[p])
    h.close()


@pytest.mark.parametrize("separate", [False, True])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 8, 16])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_apply_columns(case, nrhs, separate):
    """Every column count's kernel, the interface solve inside the local
    launch, as one launch (more columns), or as the dissection launches."""
    import torch
    from oracle import AlgMortarCPU
    sizes, offsets = CASES[case]
    A, D, part = _band_matrix(sizes, offsets, 20 + case)
    ora = AlgMortarCPU(A, part)
    h = am.AlgMortar(A, part, len(sizes), max_nrhs=nrhs, separate_iface=separate)
    R = np.random.default_rng(nrhs).standard_normal((nrhs, A.n))
    Z = h.apply(torch.as_tensor(R if nrhs > 1 else R[0], device="cuda:0")).cpu().numpy().reshape(nrhs, -1)
    for k in range(nrhs):
        ref = ora.apply(R[k])
        assert np.linalg.norm(Z[k] - ref) <= 1e-12 * np.linalg.norm(ref)
    h.close()
