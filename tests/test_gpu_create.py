"""Creating problems with long edge lists: what is uploaded together and what
by itself gives the same solve, and the host holds the lists once."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from oracle import mm
from tests._gpu import rel_max, to_dev

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def cc():
    import paper_1409_2065_amd as P
    P.load()
    return P


@pytest.mark.parametrize("n,hub", [(540, True), (700, False)])
def test_large_and_small_lists(cc, n, hub):
    """A star of 540 points (lists just above 1 MiB, edges far below) and a
    random graph of 150 000 edges (edges and lists above), in FP64 against the
    oracle's trajectory: 1e-11 relative."""
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 6))
    if hub:
        E = np.stack([np.zeros(n - 1, int), np.arange(1, n)], 1)
    else:
        a, b = np.triu_indices(n, 1)
        keep = np.sort(rng.permutation(len(a))[:150000])
        E = np.stack([a[keep], b[keep]], 1)
    w = 0.5 + rng.random(len(E))
    st, _ = mm.Problem(X, None, E, w).solve(2.0, mm.Opts(tol=0, max_iter=12, proj="jacobi:1"))
    Xt, m, e, wt = to_dev(X, None, E, w, torch.float64)
    with cc.Problem(Xt, m, e, wt, precision="f64") as g:
        g.solve(2.0, tol=0.0, max_iter=12)
        U, A, s = (t.cpu().numpy() for t in g.get_state())
    assert rel_max(U, st.U) < 1e-11 and rel_max(A, st.A) < 1e-11
    assert np.abs(s - st.s).max() < 1e-9


CHILD = """
import resource, sys, torch
import paper_1409_2065_amd as cc
def star(n):
    e = torch.stack([torch.zeros(n - 1, dtype=torch.int32), torch.arange(1, n, dtype=torch.int32)], 1).cuda().contiguous()
    cc.Problem(torch.ones(n, 4, device="cuda"), None, e, torch.ones(n - 1, device="cuda", dtype=torch.float64)).close()
peak = lambda: resource.getrusage(resource.RUSAGE_SELF).ru_maxrss * 1024
star(100)
r0 = peak()
star(6000)
print("peak growth", peak() - r0)
"""


def test_host_holds_the_lists_once():
    """A star of 6000 points has 6000 x 5999 list slots of 8 bytes (288 MB):
    creating it raises the process's peak by less than half as much again."""
    out = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stderr[-2000:]
    assert int(out.stdout.split("peak growth")[1]) < 1.5 * 6000 * 5999 * 8
