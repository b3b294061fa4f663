"""The stopping test, its windows and the non-finite status on the paths that
take them from other sums: LDS slabs, whole-row edges beyond one turn of the
waves, and one workgroup with missing entries.  Against the oracle's FP64
trajectory: states 1e-10 relative over some hundred iterations, the stopping
quantity (a difference of iterates) 1e-6 relative, as for the other paths."""
import numpy as np
import pytest
import torch

from oracle import mm, weights
from tests._gpu import oracle_jacobi, reduced_expression, rel_max, to_dev
from tests.test_gpu_wide import follow, problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


def stops_as_the_oracle(cc, X, M, E, w, window, tol, cap, gamma=2.0):
    st, info = oracle_jacobi(X, M, E, w).solve(
        gamma, mm.Opts(proj="jacobi:1", tol=tol, max_iter=cap, test_every=window))
    Xt, m, e, wt = to_dev(X, M, E, w, torch.float64)
    with cc.Problem(Xt, m, e, wt, precision="f64") as g:
        gi = g.solve(gamma, tol=tol, max_iter=cap, test_every=window)
        U, A, s = (t.cpu().numpy() for t in g.get_state())
    assert gi["converged"] == int(info.converged) and gi["iters"] == info.iters
    assert rel_max(U, st.U) < 1e-10 and rel_max(A, st.A) < 1e-10 and np.abs(s - st.s).max() < 1e-8
    assert gi["rel_change"] == pytest.approx(info.rel_change, rel=1e-6)
    return gi


# windows of 1, 5 and 64 iterations, ended by the test and by the cap
WINDOWS = [(1, 3e-2, 1500), (5, 3e-2, 1500), (64, 3e-2, 1500), (64, 0.0, 130), (5, 0.0, 23)]


@pytest.mark.parametrize("window,tol,cap", WINDOWS)
@pytest.mark.parametrize("masked", [False, True])
def test_slab_stopping_test(cc, monkeypatch, window, tol, cap, masked):
    monkeypatch.setenv("CCMI_SLAB_F", "32")
    X, M, E, w = problem(60, 45, 5, masked)
    gi = stops_as_the_oracle(cc, X, M, E, w, window, tol, cap)
    assert gi["converged"] == (tol > 0)


@pytest.mark.parametrize("window,tol,cap", WINDOWS)
def test_resident_windows_with_missing_entries(cc, window, tol, cap):
    X, M, E, w, _ = reduced_expression(n=60, p=12)
    gi = stops_as_the_oracle(cc, X, M, E, w, window, tol, cap)
    assert gi["converged"] == (tol > 0)


# 4096 edges are one turn of the waves of 512 blocks
@pytest.mark.parametrize("precision,tol", [("f64", 1e-11), ("mixed", 2e-6), ("f32", 2e-5)])
def test_more_edges_than_waves(cc, precision, tol):
    X, M, E, w = problem(130, 1100, 60, True)
    assert len(E) > 4096
    follow(cc, X, M, E, w, precision, 3.0, 12, tol)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_state_by_slabs(cc, monkeypatch, bad):
    """CC_ERR_NUMERIC, then a solve from the initial state, bitwise as a fresh
    problem's."""
    monkeypatch.setenv("CCMI_SLAB_F", "32")
    X, M, E, w = problem(60, 45, 5, True)
    Xt, m, e, wt = to_dev(X, M, E, w, torch.float32)
    with cc.Problem(Xt, m, e, wt) as g:
        g.solve(3.0, tol=0.0, max_iter=20)
        want = g.U(torch.float64)
    with cc.Problem(Xt, m, e, wt) as g:
        U, A, s = (t.cpu().numpy() for t in g.get_state())
        U[5, 3] = bad
        g.set_state(U, A, s)
        with pytest.raises(cc.CCError) as ei:
            g.solve(3.0, max_iter=100)
        assert ei.value.status == 4
        g.solve(3.0, tol=0.0, max_iter=20)
        assert torch.equal(g.U(torch.float64), want)
