"""Principal components of data with fewer nonzero singular values than the
subspace has columns (few cases, repeated rows, whole spaces): the columns
beyond the rank are rounding noise that has to stay orthogonal to the others.
Against the FP64 SVD.  The subspace holds every component after one step, so
singular values agree to rounding (1e-12 of the largest), vectors are unit,
orthogonal (1e-10) and eigenvectors of C^T C (residual 1e-10 of its norm)."""
import numpy as np
import pytest
import torch

from oracle import extras
from oracle.prep import impute_column_means

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


def check(cc, X, M, r, iters):
    _, S0, _ = extras.pca(X, M, r)
    Xt = impute_column_means(X, M)
    C = Xt - Xt.mean(axis=0)
    m = None if M is None else torch.tensor(M.astype(np.uint8), device="cuda")
    V, S, _ = cc.pca(torch.tensor(np.nan_to_num(X), device="cuda"), m, r=r, iters=iters)
    V = V.cpu().numpy()
    assert np.abs(S - S0).max() <= 1e-12 * S0[0], (S, S0)
    live = S0 > 1e-9 * S0[0]
    W = V[:, live]
    assert np.abs(W.T @ W - np.eye(live.sum())).max() < 1e-10
    assert np.abs(C.T @ (C @ W) - W * S[live] ** 2).max() < 1e-10 * S0[0] ** 2


@pytest.mark.parametrize("n", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("p", [5, 30, 271, 3000])
@pytest.mark.parametrize("masked", [False, True])
def test_few_cases(cc, n, p, masked):
    rng = np.random.default_rng(n * p)
    X = rng.standard_normal((n, p))
    M = None
    if masked:
        M = rng.random((n, p)) < 0.7
        M[0] = True
    for r in sorted({1, 2, min(4, n, p)}):
        for iters in (2, 100):
            check(cc, X, M, r, iters)


# distinct rows repeated (rank: one less), and a rank-4 matrix in 16 and 24 columns
@pytest.mark.parametrize("n,p,distinct,r", [(300, 40, 2, 1), (300, 40, 4, 2), (1000, 600, 3, 3), (64, 12, 12, 4),
                                            (2000, 500, 5, 8), (90, 700, 5, 16)])
def test_repeated_rows(cc, n, p, distinct, r):
    rng = np.random.default_rng(n + p)
    X = rng.standard_normal((distinct, p))[rng.permutation(np.arange(n) % distinct)]
    check(cc, X, None, r, 50)
