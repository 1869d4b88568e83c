"""One graph object used by two handles (own streams, own host threads) at once.

The graph records facts of its arrays on first use (degrees, weight range,
whether int16 offsets fit); both threads meet a new graph object at the same
time here, and each result is that of a graph object of its own."""
import threading

import numpy as np
import pytest
import torch

import paper_2105_00578_amd as sx
from tests.gpu_util import random_graph, star_graph, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["short", "hub", "weighted"])
def test_two_handles_share_a_new_graph(which):
    if which == "hub":
        g = star_graph(3000)
    else:
        g = random_graph(800, 0.02, 3, np.float64 if which == "weighted" else None)
    rp, col, w = upload(g)
    X = torch.randn(g.n, 5, dtype=torch.float64, device=rp.device)
    handles = []
    for _ in range(2):
        with torch.cuda.stream(torch.cuda.Stream()):
            handles.append(sx.Handle(0))
    own = sx.Handle(0)
    want = sx.laplacian_apply(own, sx.Graph(own, rp, col, w), X)
    opts = sx.options_default(True, sx.PRECOND_CHEBYSHEV)
    pre = sx.precond_apply(own, sx.Graph(own, rp, col, w), opts, X)
    outs = [(torch.empty_like(X), torch.empty_like(X)) for _ in handles]
    for _ in range(20):
        G = sx.Graph(own, rp, col, w)
        torch.cuda.synchronize()
        gate = threading.Barrier(2)
        errors = []

        def work(h, out):
            try:
                gate.wait(30)
                sx.laplacian_apply(h, G, X, out=out[0])
                sx.precond_apply(h, G, opts, X, out=out[1])
            except Exception as e:          # reported by the test's own thread
                errors.append(e)

        ts = [threading.Thread(target=work, args=a) for a in zip(handles, outs)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert not errors
        torch.cuda.synchronize()
        for a, b in outs:
            assert torch.equal(a, want) and torch.equal(b, pre)
