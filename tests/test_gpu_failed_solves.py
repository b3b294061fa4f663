"""What a solve that ends in CC_ERR_NUMERIC leaves behind, by launches and in
one workgroup: infos up to it, the label rows of the gammas before it, and
nothing in its own row (labels are whole numbers: compared exactly)."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1409_2065_amd import _lib
from tests._gpu import reduced_expression, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


# a gamma whose square overflows makes rho, eps and so d infinite
@pytest.mark.parametrize("resident", ["0", "1"])
@pytest.mark.parametrize("good", [0, 1, 2])
def test_failed_gamma_leaves_its_label_row(cc, monkeypatch, resident, good):
    monkeypatch.setenv("CCMI_RESIDENT", resident)
    X, M, E, w, _ = reduced_expression(n=90, p=20)
    Xt, m, e, wt = to_dev(X, M, E, w, torch.float32)
    gammas = np.array([0.5, 4.0][:good] + [1e200, 8.0])
    o = _lib.default_opts(tol=0.0, max_iter=30)
    infos = (_lib.SolveInfo * len(gammas))()
    lab = torch.full((len(gammas), 90), -7, dtype=torch.int32, device="cuda")
    with cc.Problem(Xt, m, e, wt, precision="mixed") as g:
        st = _lib.load().cc_solve_path(g._h, len(gammas), gammas.ctypes.data_as(_lib.P_f64), C.byref(o),
                                       C.c_void_p(lab.data_ptr()), None, infos)
    assert st == _lib.CC_ERR_NUMERIC and infos[good].status == _lib.CC_ERR_NUMERIC
    torch.cuda.synchronize()
    got = lab.cpu().numpy()
    assert (got[good:] == -7).all()
    if good:
        with cc.Problem(Xt, m, e, wt, precision="mixed") as g:
            _, ref, _ = g.solve_path(gammas[:good], tol=0.0, max_iter=30)
        assert np.array_equal(got[:good], ref.cpu().numpy())
        assert [infos[k].n_clusters for k in range(good)] == [len(np.unique(r)) for r in got[:good]]
