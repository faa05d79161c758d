"""The kernels' short forms of log and exp against the device library's, every float of
their ranges, in the build under test: a wave chooses between the two by all of its
lanes, so a message's bits are its own only if the two agree.
"""
import pytest

pytestmark = pytest.mark.gpu


def test_short_forms_equal_the_library_on_every_float():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1909_11469_amd import bp
    assert bp.bp_check_short_math() == (0, 0)
