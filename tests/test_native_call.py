"""The native form of the launching calls, on the CPU: whatever is not what most calls hand over is left (None) to the Python
form, whose checks and messages stay those of every call."""
import pytest
import torch

import paper_2509_22323_amd as ra
from paper_2509_22323_amd import binding


@pytest.fixture(scope="module")
def native():
    return binding._load_native()


def test_leaves_to_python_what_it_does_not_take(native):
    x = torch.zeros((1, 2, 64, 64), dtype=torch.bfloat16)
    m = torch.ones((1, 2, 1, 1), dtype=torch.uint8)
    assert native.dense(x, x, x, x, None, 0.0) is None                      # not on a GPU
    assert native.dense(None, 1, "q", x, None, 0.0) is None
    assert native.dense(x) is None                                          # another number of arguments
    assert native.block_sparse(x, x, x, x, m, 64, None, 0.0, None) is None
    assert native.select(x, x, m, 64, None, None, 0.9, 0.0, m) is None
    for segments in ([], [(x, x, x)], [(x, x, x, x)] * 3, (x, x, x, x), "segments", [(x, x, x, x)]):
        assert native.joint(segments, None, 64, None, None, 0.0, None) is None
        assert native.joint_select(segments, 64, None, None, None, 0.9, 0.0, None, m) is None
    assert native.store(x, x, x, None) is None and native.reuse(x, x, x, m) is None


def test_refusals_stay_those_of_python():
    x = torch.zeros((1, 2, 64, 64), dtype=torch.bfloat16)
    m = torch.ones((1, 2, 1, 1), dtype=torch.uint8)
    for call in (lambda: ra.rapid_attn_dense(x, x, x, x), lambda: ra.rapid_attn_block_sparse(x, x, x, x, m, 64),
                 lambda: ra.rapid_attn_joint([(x, x, x, x)]), lambda: ra.rapid_mask_select(x, x, m, 64),
                 lambda: ra.rapid_attn_joint_select([(x, x, x, x)]), lambda: ra.rapid_cache_store(x, x, x),
                 lambda: ra.rapid_cache_reuse(x, x, x)):
        with pytest.raises(TypeError):
            call()
    with pytest.raises(ValueError):
        ra.rapid_attn_joint([])
