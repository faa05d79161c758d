"""The [E][K] kernel that deals (message, target state) pairs to lanes: per-slot
tables, shared tables over 16 states, nodes over a tile; and the widths up to 16
states that have a kernel of their own.

One LBP sweep from the same FP32 state against the FP64 oracle, per message
max_x |m_gpu - m_ref| / max_x m_ref <= 1e-6 (the one-sweep bar), and runs split
over warm-started runs bitwise equal to one run (outcome-flag rows).
"""
import numpy as np
import pytest

import oracle
from paper_1909_11469_amd import inputs

pytestmark = pytest.mark.gpu

SWEEP_TOL = 1e-6


@pytest.fixture(scope="module")
def bp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1909_11469_amd import bp as mod
    return mod


def _problem(kind, K, seed):
    """A 7 x 9 grid ("sym", "asym": shared table; "dense": a table per edge) with
    two vertices of no edge, or ("star_*") a centre with more messages than one
    tile, and a ring."""
    rng = np.random.default_rng(seed)
    star = kind.startswith("star")
    if star:
        n = 4096 // K + 40
        edges = [(0, i) for i in range(1, n)] + [(i, i + 1) for i in range(1, n - 1)]
    else:
        n = 63 + 2
        edges = [(9 * r + c, 9 * r + c + 1) for r in range(7) for c in range(8)]
        edges += [(9 * r + c, 9 * (r + 1) + c) for r in range(6) for c in range(9)]
    edges = np.array(edges, dtype=np.int32)
    pr = dict(N=n, K=K, edges=edges, log_unary=rng.standard_normal((n, K)))
    if kind.endswith("dense"):
        pr.update(pair_kind=inputs.PAIR_DENSE,
                  pair=np.exp(0.5 * rng.standard_normal((len(edges), K, K))))
    else:
        table = np.exp(0.5 * rng.standard_normal((K, K)))
        pr.update(pair_kind=inputs.PAIR_SHARED, edge_scale=rng.uniform(0.5, 1.5, len(edges)),
                  shared=table if kind.endswith("asym") else 0.5 * (table + table.T))
    return pr


def _state(E, K, seed):
    m = np.random.default_rng(seed).uniform(0.3, 1.0, size=(E, K))
    return (m / m.sum(1, keepdims=True)).astype(np.float32)


@pytest.mark.parametrize("kind,K", [
    ("dense", 3), ("dense", 8), ("dense", 21), ("dense", 63), ("sym", 17), ("sym", 33), ("sym", 63),
    ("asym", 17), ("asym", 48), ("sym", 3), ("asym", 13), ("sym", 15), ("star_dense", 5),
    ("star_sym", 21), ("star_asym", 33), ("star_sym", 32), ("star_sym", 64), ("star_sym", 7)])
def test_single_sweep(bp, kind, K):
    prob = _problem(kind, K, K)
    state = _state(2 * len(prob["edges"]), K, 3)
    with bp.Graph(prob) as g:
        g.set_state(state, t=0, prev_active=-1)
        start, _ = g.get_state()
        g.run("lbp", eps=0.0, max_iters=1, warm_start=True)
        got, _ = g.get_state()
    cand, _ = oracle.evaluate(prob, start.astype(np.float64))
    err = np.max(np.abs(got - cand), axis=1) / np.max(np.abs(cand), axis=1)
    assert err.max() <= SWEEP_TOL, err.max()


@pytest.mark.parametrize("kind,K", [("dense", 21), ("sym", 21), ("asym", 21), ("sym", 13),
                                    ("star_sym", 32)])
def test_dynamic_p_chained_runs_bitwise(bp, kind, K):
    prob = _problem(kind, K, 4)
    kw = dict(eps=1e-6, p=0.5, seed=8, check_every=4)
    with bp.Graph(prob) as g:
        g.run("rnbp", max_iters=24, **kw)
        full, st_full = g.get_state()
    with bp.Graph(prob) as g:
        for i, k in enumerate((1, 2, 8, 13)):
            g.run("rnbp", max_iters=k, warm_start=i > 0, **kw)
        part, st_part = g.get_state()
    assert st_full == st_part
    assert np.array_equal(full.view(np.uint32), part.view(np.uint32))
