"""The bound by which the set-up decides how a rounded block inverse is kept,
in numpy: with S a symmetric M-matrix, D = diag(S), X = S^{-1} and E the change
of X by the rounding of its entries, row sums of D^{1/2} |E| D^{1/2} of at most
tau keep E within -2 tau X and 2 tau X; and the triangular form K^T D K is
definite for any rounding, where the rounded X is not."""
import numpy as np
import pytest
import scipy.linalg as sla


def _bf16(x):
    u = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) >> 16 << 16
    return u.astype(np.uint32).view(np.float32).astype(float)


def _fp32(x):
    return np.asarray(x, np.float32).astype(float)


def _block(contrast, seed):
    """64 cells of an 8 x 8 grid with a conductive body in the middle."""
    rng = np.random.default_rng(seed)
    c = np.ones((8, 8))
    c[2:6, 2:6] = contrast
    S = np.zeros((64, 64))
    idx = np.arange(64).reshape(8, 8)
    for a, b, w in ((idx[:, 1:], idx[:, :-1], np.minimum(c[:, 1:], c[:, :-1])),
                    (idx[1:], idx[:-1], np.minimum(c[1:], c[:-1]))):
        w = w * rng.uniform(0.5, 1.0, w.shape)
        S[a, b] = S[b, a] = -w
    S[np.arange(64), np.arange(64)] = -S.sum(1) + rng.uniform(0.0, 0.2, 64)
    return S


@pytest.mark.parametrize("seed", range(3))
@pytest.mark.parametrize("contrast", [1.0, 1e1, 1e2, 1e3, 1e4, 1e6, 1e8])
@pytest.mark.parametrize("rounded,tau", [(_bf16, 1 / 4), (_fp32, 1 / 1024)])
def test_bound(rounded, tau, contrast, seed):
    S = _block(contrast, seed)
    X = np.linalg.inv(S)
    X = (X + X.T) / 2
    dg = np.diag(X)
    E = rounded(X - np.diag(dg)) + np.diag(_fp32(dg)) - X
    d = np.sqrt(np.diag(S))
    bound = (d[:, None] * np.abs(E) * d).sum(1).max()
    # (the least eigenvalues are accurate to about cond(X) eps only)
    slack = 1e-13 * np.linalg.cond(X)
    lam = sla.eigvalsh(d[:, None] * X * d)
    assert lam[0] >= 0.5 - slack
    if bound <= tau:
        ev = sla.eigvalsh(E, X)
        assert max(-ev[0], ev[-1]) <= 2 * bound + slack and 2 * bound <= 0.5
    L = np.linalg.cholesky(S)
    p = np.diag(L)
    K = rounded(np.tril(sla.solve_triangular(L / p, np.eye(64), lower=True, unit_diagonal=True), -1))
    K += np.eye(64)
    assert np.all(1 / p**2 > 0) and np.linalg.matrix_rank(K) == 64


def test_symmetric_form_loses_definiteness():
    """What the bound is there for: BF16 entries at a contrast of 1e4."""
    S = _block(1e4, 0)
    X = np.linalg.inv(S)
    R = _bf16(X - np.diag(np.diag(X))) + np.diag(_fp32(np.diag(X)))
    d = np.sqrt(np.diag(S))
    assert (d[:, None] * np.abs(R - X) * d).sum(1).max() > 1 / 4
    assert sla.eigvalsh((R + R.T) / 2)[0] < 0
