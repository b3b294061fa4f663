"""Which small problems one workgroup solves, and what the launch-shape
switches turn off.

A solve of I iterations by launches enqueues I + 2 pairs of them, a resident
one runs I + 1 sweeps: the sampled counts tell which ran."""
import pytest
import torch

from tests import test_gpu_lazy_u as lazy_tests
from tests._gpu import plain_problem, reduced_expression, to_dev

pytestmark = pytest.mark.gpu

SWITCHES = ["CCMI_VEC", "CCMI_IPW", "CCMI_EDGE_IPW", "CCMI_POINT_WAVES", "CCMI_SLAB_F", "CCMI_EDGE_ITEMS",
            "CCMI_EDGE_SLAB", "CCMI_EDGE_SLAB_ITEMS", "CCMI_LAZY_U"]


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


def ran_resident(cc, X, M, E, w, precision="mixed"):
    Xt, m, e, wt = to_dev(X, M, E, w, torch.float64 if precision == "f64" else torch.float32)
    with cc.Problem(Xt, m, e, wt, precision=precision) as g:
        g.profile(1)
        g.solve(1.0, tol=0.0, max_iter=3)
        n = g.kernel_stats()["point_sweep"]["launches"]
    assert n in (4, 5)
    return n == 4


def test_small_problems_run_resident(cc, monkeypatch):
    X, M, E, w, _ = reduced_expression(n=60, p=12)
    assert ran_resident(cc, X, M, E, w)
    monkeypatch.setenv("CCMI_RESIDENT", "0")
    assert not ran_resident(cc, X, M, E, w)


@pytest.mark.parametrize("switch", SWITCHES)
def test_launch_shape_switches_ask_for_launches(cc, monkeypatch, switch):
    """A switch that shapes the launches means launches, unless
    CCMI_RESIDENT=1 says otherwise."""
    X, M, E, w, _ = reduced_expression(n=60, p=12)
    monkeypatch.setenv(switch, "1" if switch != "CCMI_SLAB_F" else "0")
    assert not ran_resident(cc, X, M, E, w)
    monkeypatch.setenv("CCMI_RESIDENT", "1")
    assert ran_resident(cc, X, M, E, w)


def test_lazy_u_without_a_mask(cc, monkeypatch):
    """Both sides of the bitwise comparison run the wave sweep."""
    X, M, E, w = plain_problem()
    for lazy in ("0", "1"):
        monkeypatch.setenv("CCMI_LAZY_U", lazy)
        assert not ran_resident(cc, X, M, E, w)
    lazy_tests.test_lazy_u_no_mask_plain(cc, monkeypatch)
