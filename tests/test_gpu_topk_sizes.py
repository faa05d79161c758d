"""The top-k at the sizes where its launches change: more than one block of 4,096
positions, more keys than one trip of the histogram's blocks (4,194,304), more blocks
than a committing block counts ties for itself (2,048, 8,388,608 positions).

A ring with equal fields and two coupling strengths: from uniform messages the residuals
take two values, so the frontier is known without arithmetic: the strongly coupled
messages first, ties in (target, source) order (residual splash: variables by id).
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


def _ring(n, shuffled):
    ids = np.random.default_rng(n).permutation(n) if shuffled else np.arange(n)
    edges = np.stack([ids, np.roll(ids, -1)], 1).astype(np.int32)
    strong = np.arange(n) % 7 == 3
    return dict(N=n, K=2, edges=edges, log_unary=np.tile([-0.3, 0.3], (n, 1)),
                pair_kind=inputs.PAIR_ISING, coupling=np.where(strong, 0.8, 0.4)), strong


def _first(k, *keys):
    """The first k indices ordered by the keys, most significant first, as a mask."""
    out = np.zeros(len(keys[0]), bool)
    out[np.lexsort(keys[::-1])[:k]] = True
    return out


def _commit_once(bp, prob, schedule, p, **kw):
    with bp.Graph(prob) as g:
        r = g.run(schedule, eps=1e-9, p=p, max_iters=1, **kw)
        m, _ = g.get_state()
    assert r["iterations"] == 1
    return np.any(m != 0.5, axis=1), r


# (n, p): the k-th key among the strong ones and among the weak, in early and late blocks
@pytest.mark.parametrize("n,p", [(2049, 0.9), (30000, 0.01), (30000, 0.12), (30000, 0.5),
                                 (30000, 0.9999), (4200000, 0.13), (4200000, 0.7)])
def test_frontier_of_ties(bp, n, p):
    prob, strong = _ring(n, shuffled=n <= 30000)
    src = prob["edges"].reshape(-1).astype(np.int64)  # rows 2u and 2u + 1: a -> b, b -> a
    dst = prob["edges"][:, ::-1].reshape(-1).astype(np.int64)
    k = int(np.ceil(p * len(src)))
    changed, r = _commit_once(bp, prob, "rbp", p)
    assert r["committed"] == k
    assert np.array_equal(changed, _first(k, ~np.repeat(strong, 2), dst * n + src))


@pytest.mark.parametrize("n,p", [(30000, 0.1), (30000, 0.3), (8400000, 0.1), (8400000, 0.3)])
def test_splash_roots_of_ties(bp, n, p):
    prob, strong = _ring(n, shuffled=n <= 30000)
    src = prob["edges"].reshape(-1).astype(np.int64)
    near = np.zeros(n, bool)                          # variables beside a strong edge
    near[prob["edges"][strong].reshape(-1)] = True
    k = int(np.ceil(p * len(src)))
    changed, _ = _commit_once(bp, prob, "rs", p, splash_depth=0)
    # depth 0: every message out of the roots
    assert np.array_equal(changed, _first(k, ~near, np.arange(n))[src])
