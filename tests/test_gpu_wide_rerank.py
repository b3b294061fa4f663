"""Rows with hundreds of others within FP32 rounding of their k-th neighbour:
the wider passes re-rank thousands of exact distances per row, counting ranks
or finding the k smallest in turn.  Edges and their order are exact against
the FP64 oracle; weights to 1e-12 relative, as for the other builds."""
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


# n rows around `groups` places, `spread` apart within a place (0: equal
# rows, whose ties go to the lower row); small k, and k so large that ranks
# are counted in the wide passes too
@pytest.mark.parametrize("n,groups,spread,k", [(700, 1, 0.0, 1), (900, 2, 0.0, 10), (1300, 1, 1e-9, 5),
                                               (1300, 2, 1e-9, 11), (1600, 2, 1e-10, 200), (2100, 3, 1e-9, 23),
                                               (900, 1, 1e-9, 899)])
def test_wide_passes_rank_exactly(cc, n, groups, spread, k):
    rng = np.random.default_rng(n + k)
    X = rng.standard_normal((groups, 3))[rng.integers(0, groups, n)] + spread * rng.standard_normal((n, 3))
    e0, w0, phi0 = weights.knn_weights(X, None, k, 0.5)
    e, w, phi = cc.build_knn_weights(torch.tensor(X, device="cuda"), None, k=k, phi=0.5)
    assert np.array_equal(e.cpu().numpy(), e0)
    assert np.allclose(w.cpu().numpy(), w0, rtol=1e-12, atol=0)
    assert phi == phi0


def test_more_neighbours_than_half_the_candidates(cc):
    """7000 neighbours of 14010 rows: twice k is more than a pass takes, so it
    ranks 12288 candidates.  The neighbours of some rows against the oracle's
    lists of those rows and of the rows they meet."""
    n, k = 14010, 7000
    rng = np.random.default_rng(5)
    X = rng.standard_normal((n, 2))
    e = cc.build_knn_weights(torch.tensor(X, device="cuda"), None, k=k, phi=0.5)[0]
    for i in (0, 77, n - 1):
        lists = weights.knn_rows(X, k, [i])
        nb = torch.cat([e[e[:, 0] == i, 1], e[e[:, 1] == i, 0]]).cpu().numpy()
        assert len(set(nb)) == len(nb) and set(lists[0]) <= set(nb)
        extra = np.setdiff1d(nb, lists[0])
        out = np.setdiff1d(np.arange(n), np.append(nb, i))
        for js, there in ((extra, True), (out, False)):
            for j in rng.permutation(js)[:5]:
                assert (i in weights.knn_rows(X, k, [j])[0]) == there
