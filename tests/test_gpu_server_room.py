"""What a served graph takes of the arena: no state of the top-k, of sparse re-evaluation or
of residual splash (32 KiB), which no served schedule uses.
"""
import numpy as np
import pytest

from paper_1909_11469_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1909_11469_amd import bp as mod
    return mod


@pytest.mark.parametrize("H,W", [(8, 9), (32, 33)])
def test_arena_smaller_than_a_graph_of_its_own(bp, H, W):
    prob = inputs.ising_grid(H, W, 2.5, 1)
    kw = dict(eps=1e-5, p=0.5, seed=3, max_iters=60)
    with bp.Graph(prob) as g:
        ref = g.run("rnbp", **kw)
        ref_m = g.marginals()
    # the server's own records (of one graph), flags, counter and tile list: under 4 KiB
    with bp.Server(bp.bp_workspace_bytes(prob) - (16 << 10) + (4 << 10), max_graphs=1) as srv:
        for _ in range(3):  # the room is given back and taken again
            rid = srv.submit(prob, "rnbp", **kw)
            while srv.counts()[2] == 0:
                srv.step(7)
            m, r = srv.result(rid)
            assert r["iterations"] == ref["iterations"] and r["committed"] == ref["committed"]
            assert np.array_equal(m, ref_m)
