"""A column of equal observed entries standardises to exactly 0, whatever the
rounding of their sum: compared exactly.  One that nearly is constant keeps
its deviations."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

VALUES = [0.1, 1.0 / 3.0, 1e6 + 0.1, 0.7, -2.3, 1e-5, 3.14159, 0.0, -0.1]


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


# 4 and 16 columns per block, more rows than a block's threads
@pytest.mark.parametrize("n", [1, 2, 3, 5, 7, 10, 50, 257, 611, 1000, 5000])
@pytest.mark.parametrize("p", [9, 1035])
@pytest.mark.parametrize("masked", [False, True])
def test_constant_columns_become_zero(cc, n, p, masked):
    rng = np.random.default_rng(n + p)
    X = np.tile(np.resize(VALUES, p), (n, 1))
    X[:, 4] = rng.standard_normal(n)  # one that is not constant
    M = np.ones((n, p), bool)
    if masked:
        M = rng.random((n, p)) < 0.7
        X = np.where(M, X, rng.standard_normal((n, p)))
    m = torch.tensor(M.astype(np.uint8), device="cuda") if masked else None
    got = cc.standardize_columns(torch.tensor(X, device="cuda"), m).cpu().numpy()
    const = np.arange(p) != 4
    assert (got[:, const][M[:, const]] == 0).all()
    assert np.array_equal(got[~M], X[~M])
    if n > 2 and M[:, 4].sum() > 1:
        z = got[M[:, 4], 4]
        assert abs(z.mean()) < 1e-12 and abs((z * z).mean() - 1.0) < 1e-12



@pytest.mark.parametrize("n", [3, 40, 3000])
def test_nearly_constant_column(cc, n):
    """One entry a rounding away from the others: no 0 / 0 and no zeroing of
    it; the mean is uncertain by about n roundings, so only its being finite
    and told apart from the others is compared."""
    X = np.full((n, 3), 0.7)
    X[n // 2] = np.nextafter(0.7, 1.0)
    got = cc.standardize_columns(torch.tensor(X, device="cuda")).cpu().numpy()
    assert np.isfinite(got).all()
    rest = np.delete(got, n // 2, axis=0)
    assert (rest == rest[0]).all() and (got[n // 2] > rest[0]).all()
