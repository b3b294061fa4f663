"""Small problems by launches over many blocks, which the defaults solve in
one workgroup: the inputs and tolerances of the tests of those solves, with
CCMI_RESIDENT=0, and what the launch-shape switches turn off.

A solve of I iterations by launches enqueues I + 2 pairs of them, a resident
one runs I + 1 sweeps: the sampled counts tell which ran."""
import pytest
import torch

from tests import test_gpu_lazy_u as lazy_tests
from tests import test_gpu_solver as solver_tests
from tests import test_gpu_wide as wide_tests
from tests._gpu import plain_problem, reduced_expression, to_dev

pytestmark = pytest.mark.gpu

SWITCHES = ["CCMI_VEC", "CCMI_IPW", "CCMI_EDGE_IPW", "CCMI_POINT_WAVES", "CCMI_SLAB_F", "CCMI_EDGE_ITEMS",
            "CCMI_EDGE_SLAB", "CCMI_EDGE_SLAB_ITEMS", "CCMI_LAZY_U"]


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


@pytest.fixture
def launches(monkeypatch):
    monkeypatch.setenv("CCMI_RESIDENT", "0")


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


@pytest.mark.parametrize("n,p", [(1, 1), (1, 5), (2, 1), (3, 300), (9, 1)])
def test_tiny_shapes(cc, launches, n, p):
    solver_tests.test_tiny_shapes(cc, n, p)


@pytest.mark.parametrize("iters", [1, 2, 3, 7, 60])
def test_trajectory(cc, launches, iters):
    solver_tests.test_fixed_iterations_f64_match_oracle_trajectory(cc, iters)


def test_stopping_test(cc, launches):
    solver_tests.test_plain_config_f64_gamma_1(cc)


@pytest.mark.parametrize("gamma", [10.0, 1000.0])
def test_converged_mixed(cc, launches, gamma):
    solver_tests.test_plain_config_mixed_converged(cc, gamma)


def test_f32(cc, launches):
    solver_tests.test_f32_precision_plain(cc)


def test_no_edges(cc, launches):
    solver_tests.test_gamma_zero_and_isolated_points(cc)


def test_all_observed_mask(cc, launches):
    solver_tests.test_all_observed_mask_equals_no_mask(cc)


def test_non_finite_state(cc, launches):
    solver_tests.test_non_finite_state_reports_numeric_error(cc)


def test_sampling(cc, launches):
    """Events of every fourth launch pair of 66: 17 samples."""
    solver_tests.test_kernel_stats_sample_every_kth_iteration(cc)
    X, M, E, w = plain_problem()
    Xt, m, e, wt = to_dev(X, M, E, w, torch.float32)
    with cc.Problem(Xt, m, e, wt) as g:
        g.profile(4)
        g.solve(10.0, tol=0.0, max_iter=64)
        assert g.kernel_stats()["edge_stage"]["launches"] == 17


def test_one_wide_edge(cc, launches):
    wide_tests.test_edge_rows(cc, 2, 1025, 1, "f64", 1e-11)


@pytest.mark.parametrize("n,p,resident", [(8, 1024, True), (8, 1025, True), (8, 1152, True), (8, 1153, False),
                                          (2, 2048, True), (2, 2049, False), (3, 3000, False), (10, 1200, False)])
def test_which_wide_rows_run_resident(cc, n, p, resident):
    """Both sides of the lines for rows of more than 1024 features; what runs
    follows the oracle."""
    X, M, E, w = wide_tests.problem(n, p, min(2, n - 1), False)
    assert ran_resident(cc, X, M, E, w) == resident
    wide_tests.follow(cc, X, M, E, w, "mixed", 3.0, 15, 2e-6)
