"""Which edge a rejected graph names: the first at fault, whatever comes after it."""
import numpy as np
import pytest

from paper_1909_11469_amd import inputs

N = 40


def _message(edges):
    from paper_1909_11469_amd import bp  # (not at collection: GPU tests load torch first)
    edges = np.array(edges, dtype=np.int32)
    prob = dict(N=N, K=2, edges=edges, log_unary=np.zeros((N, 2)), pair_kind=inputs.PAIR_ISING,
                coupling=np.full(len(edges), 0.5))
    with pytest.raises(bp.BpError) as e:
        bp.bp_workspace_bytes(prob)
    return str(e.value)


GOOD = [(i, i + 1) for i in range(0, 30)]


@pytest.mark.parametrize("bad,text", [
    ({5: (2, 1)}, "edge 5 duplicates"),                       # the other way round
    ({5: (1, 2), 9: (0, N)}, "edge 5 duplicates"),            # before one out of range
    ({5: (-1, 2), 9: (0, 1)}, "edge 5 = (-1, 2) out of range"),
    ({4: (7, 7), 9: (0, 1)}, "edge 4 is a self-loop"),
    ({9: (0, 1), 12: (7, 7)}, "edge 9 duplicates"),
    ({29: (0, 1)}, "edge 29 duplicates"),
    ({8: (30, 0), 20: (0, 30), 25: (30, 0)}, "edge 20 duplicates"),
])
def test_first_bad_edge_is_named(bad, text):
    assert text in _message([bad.get(i, e) for i, e in enumerate(GOOD)])
