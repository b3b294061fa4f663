"""Wide rows: the LDS-slab point sweep (tiles of 32 features, groups of
points, several tiles per block, lists of 0 to more than 64 neighbours) and
the edge sweep over whole rows (a wave or a block per edge), against the
oracle's FP64 trajectory: 1e-11 relative for FP64 states, 2e-6 and 2e-5 for
the mixed and FP32 states over these few iterations."""
import numpy as np
import pytest
import torch

from oracle import mm, weights
from tests._gpu import as_f32_values, rel_max, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


def problem(n, p, k, masked, hubs=0):
    rng = np.random.default_rng(n + 3 * p + k)
    X = as_f32_values(rng.standard_normal((n, p)) + 2.0 * (np.arange(n) % 4)[:, None])
    M = None
    if masked:
        M = rng.random((n, p)) < 0.9
        M[0, :] = True
    E, w, _ = weights.knn_weights(X, M, k, -0.5)
    if hubs:  # points joined to many others, and one joined to none
        E = {tuple(e) for e in E}
        for h in range(hubs):
            E |= {(h, j) for j in range(h + 1, min(n, h + 30 + 20 * h))}
        E = np.array(sorted(e for e in E if n - 1 not in e), dtype=np.int64)
        w = 0.5 + rng.random(len(E))
    return X, M, E, w


def follow(cc, X, M, E, w, precision, gamma, iters, tol):
    prob = mm.Problem(X, M, E, w)
    dtype = torch.float64 if precision == "f64" else torch.float32
    Xt, m, e, wt = to_dev(X, M, E, w, dtype)
    with cc.Problem(Xt, m, e, wt, precision=precision) as g:
        st, _ = prob.solve(gamma, mm.Opts(tol=0, max_iter=iters, proj="jacobi:1", test_every=5))
        g.solve(gamma, tol=0.0, max_iter=iters, test_every=5)
        U, A, s = (t.cpu().numpy() for t in g.get_state())
    assert rel_max(U, st.U) < tol and rel_max(A, st.A) < tol
    if precision == "f64":
        assert np.abs(s - st.s).max() < 1e-9


# tiles and rows that do not fill their blocks, one group and several, FP64
# slabs of twice the size
@pytest.mark.parametrize("n,p,k,masked,hubs", [(3, 5, 1, False, 0), (40, 33, 5, True, 0), (128, 64, 6, False, 0),
                                               (129, 70, 6, True, 0), (300, 150, 8, True, 4), (500, 36, 5, False, 3)])
def test_slab_point_sweep(cc, monkeypatch, n, p, k, masked, hubs):
    monkeypatch.setenv("CCMI_SLAB_F", "32")
    follow(cc, *problem(n, p, k, masked, hubs), "f64", 3.0, 23, 1e-11)


# as chosen by size: several tiles per block, two groups
@pytest.mark.parametrize("n,p,precision,tol", [(256, 8300, "f64", 1e-11), (300, 9001, "mixed", 2e-6),
                                               (260, 16390, "f32", 2e-5)])
@pytest.mark.parametrize("masked", [False, True])
def test_slab_by_size(cc, n, p, precision, tol, masked):
    follow(cc, *problem(n, p, 4, masked), precision, 3.0, 7, tol)


@pytest.mark.parametrize("precision", ["f32", "mixed", "f64"])
def test_slab_warm_starts(cc, monkeypatch, precision):
    """Two solves by slabs, the second from the first's state, against waves."""
    X, M, E, w = problem(200, 90, 6, True)
    monkeypatch.setenv("CCMI_RESIDENT", "0")
    out = []
    for slab in ("0", "32"):
        monkeypatch.setenv("CCMI_SLAB_F", slab)
        Xt, m, e, wt = to_dev(X, M, E, w, torch.float64 if precision == "f64" else torch.float32)
        with cc.Problem(Xt, m, e, wt, precision=precision) as g:
            g.solve(1.0, tol=0.0, max_iter=20)
            g.solve(4.0, tol=0.0, max_iter=20)
            out.append([t.cpu().numpy() for t in g.get_state()])
    tol = {"f32": 2e-5, "mixed": 2e-6, "f64": 1e-11}[precision]
    for a, b in zip(*out):
        assert rel_max(a, b) < tol


# a block per edge (few edges, long rows) and a wave per edge; rows beyond a
# lane's first chunks, ragged ends, more edges than partial rows
@pytest.mark.parametrize("n,p,k,precision,tol", [(2, 1025, 1, "f64", 1e-11), (12, 1500, 2, "f64", 1e-11),
                                                 (12, 9000, 2, "f64", 1e-11), (40, 1025, 6, "f64", 1e-11),
                                                 (120, 1203, 20, "f64", 1e-11), (150, 2051, 9, "mixed", 2e-6)])
def test_edge_rows(cc, n, p, k, precision, tol):
    follow(cc, *problem(n, p, k, n % 4 == 0), precision, 3.0, 15, tol)
