"""Cluster counts of a served request whose labels nobody asks for: many
gammas share a bounded scratch in turns.  Whole numbers, compared exactly."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1409_2065_amd import _lib

pytestmark = pytest.mark.gpu


# 9000 rows of 2000 labels are more than the scratch of 64 MiB, 40 rows less
@pytest.mark.parametrize("n,gammas", [(2000, 9000), (70, 40)])
def test_counts_without_labels(n, gammas):
    import paper_1409_2065_amd as cc
    cc.load()
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 2)) + 4.0 * (np.arange(n) % 3)[:, None]
    with cc.Server("mixed", round_iters=1024, tol=0.0, max_iter=1) as srv:
        t = srv.submit(X, k=4, gammas=np.geomspace(0.1, 1e5, gammas))
        for _ in range(1000):
            if srv.step()[2]:
                break
        lab, infos, _ = srv.result(t)
        again = (_lib.SolveInfo * gammas)()
        assert _lib.load().cc_server_result(srv._h, t, None, again, None) == 0
    lab = lab.cpu().numpy()
    want = (lab == np.arange(n)[None, :]).sum(1)
    assert len(set(want)) > 1
    assert [i["n_clusters"] for i in infos] == list(want)
    assert [again[k].n_clusters for k in range(gammas)] == list(want)
