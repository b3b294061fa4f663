"""A problem's scalars change slots with every launch pair but stay in one slot
through a resident solve.  Whatever the numbers of launches and sweeps before
it, creating a batch leaves the problem's state alone (bitwise), and its run
starts from that state: as by launches throughout, FP64 to 1e-10 relative."""
import numpy as np
import pytest
import torch

from tests._gpu import reduced_expression, rel_max, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


def state(g):
    return [t.cpu().numpy() for t in g.get_state()]


# launch pairs of the first solve: 2, 3 and 19; resident sweeps: 1 to 3 and more
@pytest.mark.parametrize("first", [0, 1, 17])
@pytest.mark.parametrize("sweeps", [1, 2, 3, 40])
def test_batch_after_launches_and_a_resident_solve(cc, monkeypatch, first, sweeps):
    X, M, E, w, _ = reduced_expression(n=70, p=20)
    Xt, m, e, wt = to_dev(X, M, E, w, torch.float64)
    out = []
    for res in ("0", "1"):
        monkeypatch.setenv("CCMI_RESIDENT", res)
        with cc.Problem(Xt, m, e, wt, precision="f64") as g:
            if first:
                g.solve(1.0, tol=0.0, max_iter=first, proj_sweeps=2)
            g.solve(3.0, tol=0.0, max_iter=sweeps)
            before = state(g)
            with cc.Batch([g], [[0.0, 2.0]], autotune=False, max_iter=15, tol=0.0) as bt:
                assert all(np.array_equal(a, b) for a, b in zip(before, state(g)))
                bt.run()
                out.append(state(g))
                # a solve between two runs, and one after them
                g.solve(1.0, tol=0.0, max_iter=sweeps + 1)
                bt.run()
            g.solve(2.0, tol=0.0, max_iter=4)
            out[-1] += state(g)
    for a, b in zip(*out):
        assert rel_max(a, b) < 1e-10
