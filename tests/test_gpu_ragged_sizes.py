"""Variables with their own numbers of states at the graph sizes where the split of
the work changes: a block for a variable of 1,024 or 4,096 multiply-adds on (up to
1,024 and 4,096 variables), a wave for every variable above.

One LBP sweep from the same FP32 state against the FP64 oracle, each message within
1e-6 of its largest entry (the one-sweep bar).
"""
import numpy as np
import pytest

import oracle
from paper_1909_11469_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1909_11469_amd import bp as mod
    return mod


@pytest.mark.parametrize("n,degree", [(1024, 5.0), (1025, 6.0), (4096, 4.0), (4097, 4.0)])
def test_single_sweep(bp, n, degree):
    prob = inputs.protein_like_graph(n, degree, 5)
    off = oracle.message_offsets(prob)
    rng = np.random.default_rng(n)
    state = rng.uniform(0.2, 1.0, size=int(off[-1]))
    state /= np.repeat(np.add.reduceat(state, off[:-1]), np.diff(off))
    with bp.Graph(prob) as g:
        g.set_state(state.astype(np.float32), t=0, prev_active=-1)
        start, _ = g.get_state()
        g.run("lbp", eps=0.0, max_iters=1, warm_start=True)
        got, _ = g.get_state()
    ref, _ = oracle.evaluate(prob, start.astype(np.float64))
    err = np.maximum.reduceat(np.abs(got - ref), off[:-1]) / np.maximum.reduceat(ref, off[:-1])
    assert err.max() <= 1e-6, err.max()
