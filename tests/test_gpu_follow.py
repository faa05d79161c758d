"""A run that the host follows by the progress word while the device is held up:
other work of the same stream goes first, so that the host waits long and asks the
stream many times.  The result is the undisturbed run's, bit for bit.
"""
import numpy as np
import pytest

from paper_1909_11469_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule,p", [("lbp", 1.0), ("rnbp", 0.5), ("rbp", 1 / 64)])
def test_follow_behind_other_work(schedule, p):
    import torch
    from paper_1909_11469_amd import bp
    prob = inputs.ising_grid(60, 61, 2.5, 3)
    a = torch.randn(8192, 8192, device="cuda")
    b = torch.empty_like(a)
    out = []
    for busy in (False, True):
        with bp.Graph(prob) as g:
            g.run(schedule, eps=1e-5, p=p, seed=4, max_iters=40)  # tunes its launch shape
            if busy:
                for _ in range(12):  # about 0.1 s of the stream
                    torch.mm(a, a, out=b)
            r = g.run(schedule, eps=1e-5, p=p, seed=4, max_iters=40)
            out.append((r["iterations"], r["committed"], g.get_state()[0]))
    assert out[0][:2] == out[1][:2]
    assert np.array_equal(out[0][2].view(np.uint32), out[1][2].view(np.uint32))
