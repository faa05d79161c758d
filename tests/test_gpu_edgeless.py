"""K = 2 graphs without edges past the size that one block solves: every tile is empty, the
first evaluation finds nothing to do, and the beliefs are the unaries'.
"""
import numpy as np
import pytest

from paper_1909_11469_amd import inputs

pytestmark = pytest.mark.gpu

N = 5000


@pytest.fixture(scope="module")
def bp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1909_11469_amd import bp as mod
    return mod


def _problem():
    return dict(N=N, K=2, edges=np.zeros((0, 2), np.int32), pair_kind=inputs.PAIR_ISING,
                coupling=np.zeros(0), log_unary=np.random.default_rng(1).standard_normal((N, 2)))


def _check(prob, marg):
    u = np.exp(prob["log_unary"])
    # a sigmoid in FP32: the log-odds rounded once, an exponential and a quotient
    assert np.allclose(marg, u / u.sum(1, keepdims=True), rtol=2e-6, atol=0.0)


@pytest.mark.parametrize("kw", [dict(schedule="lbp"), dict(schedule="rnbp"), dict(schedule="rbp"),
                                dict(schedule="rs"), dict(schedule="rnbp", sparse=1),
                                dict(schedule="rnbp", noalloc=True)])
def test_no_edges(bp, kw):
    prob = _problem()
    with bp.Graph(prob) as g:
        r = g.run(eps=1e-6, p=0.5, seed=1, max_iters=30, **kw)
        assert r["converged"] and r["iterations"] == 0 and r["committed"] == 0
        _check(prob, g.marginals())


def test_no_edges_served(bp):
    prob = _problem()
    with bp.Server(64 << 20, max_graphs=2) as srv:
        rid = srv.submit(prob, "rnbp", eps=1e-6, p=0.5, seed=1, max_iters=30)
        while srv.counts()[2] == 0:
            srv.step(8)
        m, r = srv.result(rid)
    assert r["converged"] and r["iterations"] == 0
    _check(prob, m)
