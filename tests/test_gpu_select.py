"""The neighbour selection, its tie and wide-list paths, the column moments
and the median rule of the kNN weights at the edges of their ranges, against
the FP64 oracle.  The edge set is exact; weights differ by the rounding of
FP64 sums of p squares and of exp, 1e-12 relative with room to spare."""
import numpy as np
import pytest
import torch

from oracle import weights

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


def check(cc, X, M, k, phi, normalize=False):
    e0, w0, phi0 = weights.knn_weights(X, M, k, phi)
    if normalize:
        w0 = w0 / w0.sum()
    m = None if M is None else torch.tensor(M.astype(np.uint8), device="cuda")
    e, w, phi1 = cc.build_knn_weights(torch.tensor(X, device="cuda"), m, k=k, phi=phi, normalize=normalize)
    assert np.array_equal(e.cpu().numpy(), e0)
    assert np.allclose(w.cpu().numpy(), w0, rtol=1e-12, atol=0)
    assert phi1 == pytest.approx(phi0, rel=1e-12)


# keys per thread change at 256, 1024, 2048 and 4096 rows
@pytest.mark.parametrize("n", [2, 3, 65, 256, 257, 1024, 1025, 2048, 2049, 4097])
def test_rows_at_the_edges_of_the_selection(cc, n):
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 3))
    check(cc, X, None, min(n - 1, 7), -0.5, normalize=n % 2 == 1)


# more candidates than a block has threads, than its list holds, all rows
@pytest.mark.parametrize("n,k", [(700, 120), (700, 128), (700, 300), (700, 699), (1100, 600)])
def test_many_neighbours(cc, n, k):
    rng = np.random.default_rng(k)
    check(cc, rng.standard_normal((n, 5)), None, k, -0.5)


# integer points: most distances are tied, at the boundary of the candidates
# too, and repeated points are at distance zero
@pytest.mark.parametrize("n,side", [(300, 3), (900, 2), (640, 40)])
def test_ties_go_to_the_lower_row(cc, n, side):
    rng = np.random.default_rng(side)
    check(cc, rng.integers(0, side, size=(n, 2)).astype(np.float64), None, 6, 0.25)


# 4 and 16 columns per block, rows past a thread's first batch, a column with
# one observed entry
@pytest.mark.parametrize("n,p", [(5, 1), (40, 1023), (40, 1030), (2100, 9), (3000, 2)])
def test_column_moments(cc, n, p):
    rng = np.random.default_rng(n + p)
    X = rng.standard_normal((n, p)) * 3.0 + 5.0
    M = rng.random((n, p)) < 0.7
    M[:, 0] = False
    M[n // 2, 0] = True
    M[np.arange(n), rng.integers(0, p, n)] = True
    Z = np.where(M, X, 0.0)
    cnt = np.maximum(M.sum(0), 1)
    mean = Z.sum(0) / cnt
    sd = np.sqrt((np.where(M, X - mean, 0.0) ** 2).sum(0) / cnt)
    want = np.where(M, (X - mean) * np.where(sd > 0, 1.0 / np.where(sd > 0, sd, 1.0), 0.0), X)
    got = cc.standardize_columns(torch.tensor(X, device="cuda"), torch.tensor(M.astype(np.uint8), device="cuda"))
    assert np.allclose(got.cpu().numpy(), want, rtol=0, atol=1e-12 * 20)


# spread distances, many equal ones, and ranges of many binary orders
@pytest.mark.parametrize("kind", ["spread", "equal", "orders"])
def test_median_rule(cc, kind):
    rng = np.random.default_rng(3)
    n = 1500
    if kind == "spread":
        X = rng.standard_normal((n, 4))
    elif kind == "equal":
        X = np.stack([np.arange(n) % 30, np.arange(n) // 30], 1).astype(np.float64)
    else:
        X = np.exp(rng.uniform(-8.0, 8.0, n))[:, None] * rng.standard_normal((n, 2))
    check(cc, X, None, 5, -0.5)
