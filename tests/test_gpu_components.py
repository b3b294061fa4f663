"""Labels from LDS and from memory, and problems given their edges out of order."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


def _union_find(n, ei, ej, keep):
    parent = list(range(n))

    def find(a):
        while parent[a] != a:
            parent[a] = parent[parent[a]]
            a = parent[a]
        return a

    for a, b, k in zip(ei, ej, keep):
        if k:
            ra, rb = find(int(a)), find(int(b))
            if ra != rb:
                parent[max(ra, rb)] = min(ra, rb)
    return np.array([find(i) for i in range(n)])


@pytest.mark.parametrize("n", [1, 2, 65, 1025, 16000, 16001])
@pytest.mark.parametrize("shape", ["none", "chain", "random"])
def test_components_against_union_find(cc, n, shape):
    """Labels are whole numbers: they equal the oracle's.  16000 points is the
    most that keep their labels in LDS."""
    rng = np.random.default_rng(n)
    if shape == "none" or n == 1:
        ei, ej, keep = (np.zeros(0, np.int64),) * 3
    elif shape == "chain":  # a path visited in random order: the longest label chains
        o = rng.permutation(n)
        a, b = o[:-1], o[1:]
        ei, ej, keep = np.minimum(a, b), np.maximum(a, b), rng.random(n - 1) < 0.98
    else:
        a, b = rng.integers(0, n, 3 * n), rng.integers(0, n, 3 * n)
        ok = a != b
        e = np.unique(np.stack([np.minimum(a, b)[ok], np.maximum(a, b)[ok]]), axis=1)
        ei, ej, keep = e[0], e[1], rng.random(e.shape[1]) < 0.25
    edges = torch.tensor(np.stack([ei, ej], axis=1).astype(np.int32), device="cuda")
    lab, ncl = cc.components(n, edges, torch.tensor(keep.astype(np.uint8), device="cuda"))
    ref = _union_find(n, ei, ej, keep)
    assert np.array_equal(lab.cpu().numpy(), ref)
    assert ncl == len(np.unique(ref))


@pytest.mark.parametrize("n,p", [(60, 5), (400, 70), (300, 6000)])
def test_edge_order_is_immaterial(cc, n, p):
    """The sums over a point's neighbours run by neighbour index and those over
    edges differ by rounding alone: 1e-9 of the largest entry in FP64."""
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn(n, p, generator=g, device="cuda", dtype=torch.float64)
    edges, w = cc.build_knn_weights(X, k=5, phi=-0.5)[:2]
    perm = torch.randperm(edges.shape[0], generator=torch.Generator().manual_seed(1)).to("cuda")
    gammas = [0.1, 1.0, 10.0]
    out = []
    for e, ww in ((edges, w), (edges[perm].contiguous(), w[perm].contiguous())):
        with cc.Problem(X, None, e, ww, precision="f64") as P:
            res = P.solve_path(gammas, tol=0.0, max_iter=40)
            out.append((P.U(torch.float64), res))
    assert (out[0][0] - out[1][0]).abs().max().item() <= 1e-9 * X.abs().max().item()
    dup = torch.cat([edges[perm], edges[:1]]).contiguous()
    with pytest.raises(cc.CCError):
        cc.Problem(X, None, dup, torch.cat([w[perm], w[:1]]).contiguous(), precision="f64")
