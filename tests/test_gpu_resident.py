"""Small problems solved in one workgroup (CCMI_RESIDENT=0 turns that off):
the FP64 trajectory follows the oracle's at the edges of the range, with the
tolerances of the other sweeps (1e-11 relative for FP64 states, whose
rounding per step is 2^-53; 2e-6 and 2e-5 for the mixed and FP32 states);
launches of any length and the stopping test end in the same state."""
import numpy as np
import pytest
import torch

from oracle import mm, weights
from tests._gpu import as_f32_values, oracle_jacobi, plain_problem, reduced_expression, rel_max, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


def _gpu(cc, X, mask, edges, w, precision):
    dtype = torch.float64 if precision == "f64" else torch.float32
    Xt, m, e, wt = to_dev(X, mask, edges, w, dtype)
    return cc.Problem(Xt, m, e, wt, precision=precision)


def state(g):
    return [t.cpu().numpy() for t in g.get_state()]


# one piece per point and several, below and above 256 pieces, hubs, ragged
# rows, a wave's lanes sharing 1 to 8 edges, the largest work and beyond it
@pytest.mark.parametrize("n,p,k", [(2, 1, 1), (5, 4, 2), (64, 4, 5), (65, 5, 3), (30, 33, 4), (52, 40, 5),
                                   (40, 130, 6), (200, 10, 10), (370, 10, 10), (200, 24, 10), (150, 61, 9)])
@pytest.mark.parametrize("masked", [False, True])
def test_trajectory(cc, n, p, k, masked):
    rng = np.random.default_rng(n * 7 + p)
    X = rng.standard_normal((n, p)) + 3.0 * (np.arange(n) % 3)[:, None]
    M = None
    if masked:
        M = rng.random((n, p)) < 0.8
        M[0, :] = True
    E, w, _ = weights.knn_weights(X, M, min(k, n - 1), -0.5)
    st, info = mm.Problem(X, M, E, w).solve(3.0, mm.Opts(tol=0, max_iter=70, proj="jacobi:1", record=True))
    with _gpu(cc, X, M, E, w, "f64") as g:
        gi = g.solve(3.0, tol=0.0, max_iter=70, record_objective=1)
        U, A, s = state(g)
        F = g.trace()
    assert gi["iters"] == 70 and gi["converged"] == 0
    assert rel_max(U, st.U) < 1e-11 and rel_max(A, st.A) < 1e-11
    assert np.abs(s - st.s).max() < 1e-9 and np.array_equal(s == 0, st.s == 0)
    assert np.allclose(F, info.trace_F, rtol=1e-10, atol=0)
    assert gi["d"] == pytest.approx(info.d, rel=1e-10)


@pytest.mark.parametrize("precision,tol", [("mixed", 2e-6), ("f32", 2e-5)])
def test_reduced_precision(cc, precision, tol):
    X, M, E, w, _ = reduced_expression(n=120, p=30)
    st, _ = oracle_jacobi(X, M, E, w).solve(3.0, mm.Opts(tol=0, max_iter=200, proj="jacobi:1"))
    with _gpu(cc, X, M, E, w, precision) as g:
        g.solve(3.0, tol=0.0, max_iter=200)
        U, A, _ = state(g)
    assert rel_max(U, st.U) < tol and rel_max(A, st.A) < tol


# windows of 1, 5 and 64 iterations; iteration caps below, at and past a
# launch's 4096 sweeps
@pytest.mark.parametrize("window,tol,cap", [(1, 1e-4, 3000), (5, 1e-5, 3000), (64, 1e-5, 9000),
                                            (64, 0.0, 4095), (64, 0.0, 4096), (64, 0.0, 8200), (7, 0.0, 1)])
def test_stop_and_launch_length(cc, window, tol, cap):
    X = plain_problem()[0][:60]
    E, w, _ = weights.knn_weights(X, None, 6, 0.1)
    st, info = oracle_jacobi(X, None, E, w).solve(
        2.0, mm.Opts(proj="jacobi:1", tol=tol, max_iter=cap, test_every=window))
    with _gpu(cc, X, None, E, w, "f64") as g:
        gi = g.solve(2.0, tol=tol, max_iter=cap, test_every=window)
        U, A, s = state(g)
    assert gi["converged"] == int(info.converged) and gi["iters"] == info.iters
    assert rel_max(U, st.U) < 1e-10 and rel_max(A, st.A) < 1e-10 and np.abs(s - st.s).max() < 1e-8
    if cap >= window:  # a window ended: the oracle has no stopping quantity before
        assert gi["rel_change"] == pytest.approx(info.rel_change, rel=1e-6)


@pytest.mark.parametrize("precision", ["f32", "mixed", "f64"])
def test_between_other_sweeps(cc, monkeypatch, precision):
    """A resident solve, one by launches (two projection sweeps), a batch and
    a resident solve again, each from the state the one before left: as by
    launches throughout, to the precision's rounding over the few steps."""
    X, M, E, w, _ = reduced_expression(n=90, p=20)
    out = []
    for res in ("0", "1"):
        monkeypatch.setenv("CCMI_RESIDENT", res)
        with _gpu(cc, X, M, E, w, precision) as g:
            g.solve(1.0, tol=0.0, max_iter=33)
            g.solve(2.0, tol=0.0, max_iter=20, proj_sweeps=2)
            g.solve(3.0, tol=0.0, max_iter=17)
            with cc.Batch([g], [[4.0, 5.0]], autotune=False, max_iter=21, tol=0.0) as bt:
                bt.run()
            g.solve(6.0, tol=0.0, max_iter=25)
            blob = g.export_state()
            g.solve(7.0, tol=0.0, max_iter=25)
            g.import_state(blob)
            g.solve(7.0, tol=0.0, max_iter=25)
            out.append(state(g))
    tol = {"f32": 1e-5, "mixed": 1e-6, "f64": 1e-12}[precision]
    for a, b in zip(*out):
        assert rel_max(a, b) < tol


def test_no_edges_and_repeat(cc):
    X, M, E, w, _ = reduced_expression(n=80, p=20)
    with _gpu(cc, X, M, np.zeros((0, 2), int), np.zeros(0), "mixed") as g:
        g.solve(5.0, tol=0.0, max_iter=10)
        U = g.U(torch.float64).cpu().numpy()
    assert np.array_equal(U[M], X[M])
    outs = []
    for _ in range(2):
        with _gpu(cc, X, M, E, w, "mixed") as g:
            g.solve(5.0, tol=0.0, max_iter=300)
            outs.append(state(g))
    assert all(np.array_equal(a, b) for a, b in zip(*outs))
