"""Sampled timing of solves by one workgroup: every sample_every-th sweep of
all that run, over solves of any length (a solve that reports I iterations
runs sweeps 0..I, whose last one's sums end it)."""
import pytest
import torch

from tests._gpu import reduced_expression, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


@pytest.mark.parametrize("every", [1, 7, 50, 1000])
def test_every_kth_sweep_over_several_solves(cc, every):
    """Solves ended by the stopping test, by the cap, in one launch of up to
    4096 sweeps and in several."""
    X, M, E, w, _ = reduced_expression(n=60, p=12)
    Xt, m, e, wt = to_dev(X, M, E, w, torch.float64)
    with cc.Problem(Xt, m, e, wt, precision="f64") as g:
        g.profile(every)
        sweeps = 0
        for gamma, opts in ((1.0, dict(tol=1e-3, max_iter=20000)), (2.0, dict(tol=0.0, max_iter=9)),
                            (3.0, dict(tol=0.0, max_iter=9000)), (4.0, dict(tol=1e-3, max_iter=20000)),
                            (5.0, dict(tol=0.0, max_iter=4095)), (6.0, dict(tol=0.0, max_iter=4096))):
            sweeps += g.solve(gamma, **opts)["iters"] + 1
        ks = g.kernel_stats()
    for name in ("point_sweep", "edge_stage"):
        assert ks[name]["launches"] == (sweeps + every - 1) // every
