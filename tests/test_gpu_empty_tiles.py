"""K = 32 with one symmetric shared table (the matrix-core kernel): tiles without
messages.  128 variables fill a tile, so isolated ones in front make the first tile (or
the first two) empty, with no message before its own; a graph without edges has
nothing but such tiles.
"""
import numpy as np
import pytest

import oracle
from paper_1909_11469_amd import inputs

pytestmark = pytest.mark.gpu

K = 32


@pytest.fixture(scope="module")
def bp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1909_11469_amd import bp as mod
    return mod


def _problem(lead, gap=0, edges=True):
    """`lead` isolated variables, a 6 x 7 grid, `gap` isolated ones, a chain of 9."""
    rng = np.random.default_rng(lead + gap)
    e = []
    if edges:
        e = [(lead + 7 * r + c, lead + 7 * r + c + 1) for r in range(6) for c in range(6)]
        e += [(lead + 7 * r + c, lead + 7 * (r + 1) + c) for r in range(5) for c in range(7)]
        far = lead + 42 + gap
        e += [(far + i, far + i + 1) for i in range(8)]
    n = lead + 42 + gap + 9
    table = np.exp(0.5 * rng.standard_normal((K, K)))
    return dict(N=n, K=K, edges=np.array(e, dtype=np.int32).reshape(-1, 2),
                log_unary=rng.standard_normal((n, K)), pair_kind=inputs.PAIR_SHARED,
                shared=0.5 * (table + table.T), edge_scale=np.ones(len(e)))


LAYOUTS = [(128, 0), (129, 0), (256, 300), (0, 300)]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("lead,gap", LAYOUTS)
def test_single_sweep(bp, lead, gap, bf16):
    prob = _problem(lead, gap)
    E = 2 * len(prob["edges"])
    m = np.random.default_rng(3).uniform(0.3, 1.0, size=(E, K))
    state = (m / m.sum(1, keepdims=True)).astype(np.float32)
    with bp.Graph(prob, flags=bp.BP_FLAG_BF16_MATRIX_CORES if bf16 else 0) as g:
        g.set_state(state, t=0, prev_active=-1)
        start, _ = g.get_state()
        g.run("lbp", eps=0.0, max_iters=1, warm_start=True)
        got, _ = g.get_state()
    cand, _ = oracle.evaluate(prob, start.astype(np.float64))
    err = np.max(np.abs(got - cand), axis=1) / np.max(np.abs(cand), axis=1)
    # FP32: the one-sweep bar; BF16 operands: 8-bit mantissas of table and cavity
    assert err.max() <= (2.0 ** -7 if bf16 else 1e-6), err.max()


@pytest.mark.parametrize("lead,gap", LAYOUTS)
def test_dynamic_p_chained_runs_bitwise(bp, lead, gap):
    prob = _problem(lead, gap)
    kw = dict(eps=1e-6, p=0.5, seed=8)
    with bp.Graph(prob) as g:
        g.run("rnbp", max_iters=24, **kw)
        full, st_full = g.get_state()
    with bp.Graph(prob) as g:
        for i, k in enumerate((1, 2, 8, 13)):
            g.run("rnbp", max_iters=k, warm_start=i > 0, **kw)
        part, st_part = g.get_state()
    assert st_full == st_part
    assert np.array_equal(full.view(np.uint32), part.view(np.uint32))


@pytest.mark.parametrize("schedule,p", [("lbp", 1.0), ("rnbp", 0.5), ("rbp", 0.25)])
@pytest.mark.parametrize("lead", [0, 300])
def test_no_edges(bp, lead, schedule, p):
    prob = _problem(lead, edges=False)
    with bp.Graph(prob) as g:
        r = g.run(schedule, eps=1e-6, p=p, seed=1, max_iters=20)
        got = g.marginals()
    assert r["converged"] and r["iterations"] == 0
    u = np.exp(prob["log_unary"] - prob["log_unary"].max(1, keepdims=True))
    # a softmax in FP32: exponent, sum of 32 and quotient, each within a few ulp
    assert np.allclose(got, u / u.sum(1, keepdims=True), rtol=2e-6, atol=0.0)
