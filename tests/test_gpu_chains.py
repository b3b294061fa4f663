"""Batches of one to seven launch classes (more than the parallel chains of a
batch's graph), with and without tuning, against plain solves of the same
problems: FP64 states over fixed iterations, where only the order of the
block sums differs (1e-9 relative for objectives, labels equal)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

WIDTHS = [900, 20, 400, 100, 200, 700, 130]


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


@pytest.mark.parametrize("count", [1, 3, 5, 7])
@pytest.mark.parametrize("tune", [False, True])
def test_batch_classes_match_plain_solves(cc, count, tune):
    g = torch.Generator(device="cuda").manual_seed(count)
    probs, ref = [], []
    gammas = [0.05, 0.5, 5.0]
    opts = dict(tol=0.0, max_iter=30)
    for q in range(count):
        n = 40 + 17 * q
        X = torch.randn(n, WIDTHS[q], generator=g, device="cuda", dtype=torch.float64)
        X += 2.0 * (torch.arange(n, device="cuda") % 3)[:, None]
        e, w = cc.build_knn_weights(X, k=5, phi=-0.5)[:2]
        with cc.Problem(X, None, e, w, precision="f64") as P:
            infos, lab, _ = P.solve_path(gammas, **opts)
            ref.append((infos, lab.cpu().numpy()))
        probs.append(cc.Problem(X, None, e, w, precision="f64"))
    B = cc.Batch(probs, [gammas] * count, autotune=tune, **opts)
    for _ in range(2):  # a run starts from the problems' current states
        for P in probs:
            P.reset_state()
        labels, infos = B.run()[:2]
        for q in range(count):
            lab = np.stack([np.asarray(torch.as_tensor(x).cpu()) for x in labels[q]])
            assert np.array_equal(lab, ref[q][1])
            for a, b in zip(infos[q], ref[q][0]):
                assert a["iters"] == b["iters"]
                assert abs(a["objective"] - b["objective"]) <= 1e-9 * abs(b["objective"])
    B.close()
