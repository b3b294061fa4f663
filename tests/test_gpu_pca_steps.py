"""The subspace iteration of cc_pca where its steps differ: nearly dependent
columns (Gram-Schmidt in place of Cholesky), fewer nonzero singular values
than subspace columns, one to three groups of eight columns, several row
groups per chunk.  Against the FP64 SVD.  With singular values in the ratio
q between neighbours, the squared iteration leaves a vector off by about
2^-52 q^2 per step that its gap does not remove, far below 1e-7 here."""
import numpy as np
import pytest
import torch

from oracle import extras

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


def spectrum(rng, n, p, sv):
    """n x p with zero column means and the given singular values."""
    k = len(sv)
    A = rng.standard_normal((n, k))
    U, _ = np.linalg.qr(A - A.mean(0))
    V, _ = np.linalg.qr(rng.standard_normal((p, k)))
    return (U * np.asarray(sv)) @ V.T


@pytest.mark.parametrize("n,p,r,sv", [
    (60, 40, 2, [1e4, 1e2, 1.0, 1e-2, 1e-4]),                  # steep: dependent columns at the start
    (6, 40, 2, [5.0, 3.0, 2.0, 1.5, 1.0]),                     # 5 nonzero values, 10 columns
    (70, 33, 1, list(2.0 ** -np.arange(20.0))),                # 9 columns
    (257, 129, 8, list(1.5 ** -np.arange(40.0))),              # 16 columns
    (200, 130, 16, list(1.4 ** -np.arange(60.0))),             # 24 columns
    (30, 7, 3, [4.0, 3.0, 2.0, 1.0]),                          # the whole space
    (20000, 600, 2, list(1.3 ** -np.arange(30.0))),            # several row groups per chunk
])
def test_steps(cc, n, p, r, sv):
    X = spectrum(np.random.default_rng(n + p), n, p, sv) + 0.25
    V0, S0, c0 = extras.pca(X, None, r)
    V, S, c = cc.pca(torch.tensor(X, device="cuda"), r=r, iters=60)
    assert np.allclose(S, S0, rtol=1e-9, atol=0), (S, S0)
    assert np.abs(V.cpu().numpy() - V0).max() < 1e-7
    assert np.abs(c.cpu().numpy() - c0).max() < 1e-12


def test_single_column_and_constant(cc):
    X = torch.arange(12, dtype=torch.float64, device="cuda").reshape(12, 1)
    V, S, _ = cc.pca(X, r=1)
    assert float(V[0, 0]) == 1.0 and S[0] == pytest.approx(float((X - X.mean()).norm()), rel=1e-14)
    V, S, _ = cc.pca(torch.ones(9, 5, dtype=torch.float64, device="cuda"), r=2)
    assert np.all(S == 0.0)
