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


def _refused():
    x = torch.zeros((1, 2, 64, 64), dtype=torch.bfloat16)
    with pytest.raises(TypeError):                                          # (of the Python form: not on a GPU)
        ra.rapid_attn_dense(x, x, x, x)
    with pytest.raises(TypeError):
        ra.rapid_attn_joint_select([(x, x, x, x)])


def test_a_package_without_the_native_form_calls_by_way_of_ctypes(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_native", None)
    monkeypatch.setattr(binding, "_NATIVE_SO", str(tmp_path / "native_call.so"))
    _refused()


@pytest.mark.parametrize("other", ["file", "torch"])
def test_a_native_form_that_does_not_fit_is_not_used(other, monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_native", None)
    if other == "file":
        (tmp_path / "native_call.so").write_bytes(b"not a library")
        monkeypatch.setattr(binding, "_NATIVE_SO", str(tmp_path / "native_call.so"))
    else:
        monkeypatch.setattr(torch, "__version__", "0.0")
    with pytest.warns(RuntimeWarning, match="by way of ctypes"):
        _refused()


def test_the_library_is_built_where_the_native_form_cannot_be(monkeypatch, tmp_path):
    from paper_2509_22323_amd import build
    made, stale = [], tmp_path / "native_call.so"
    stale.write_bytes(b"of other sources")
    monkeypatch.setattr(build, "NATIVE_OUT", str(stale))
    monkeypatch.setattr(build, "_run", lambda cmd, out, verbose: made.append(out) or out)
    monkeypatch.setattr("shutil.which", lambda name: None)
    assert build.build() == build.OUT
    assert build.OUT in made and str(stale) not in made and not stale.exists()


def test_calls_without_a_workspace_are_not_put_to_the_native_form(monkeypatch):
    """It would look at every tensor and hand them back: 0.1 us of a call."""
    class Asked:
        def __getattr__(self, name):
            raise AssertionError(name)

    x = torch.zeros((1, 2, 64, 64), dtype=torch.bfloat16)
    m = torch.ones((1, 2, 1, 1), dtype=torch.uint8)
    monkeypatch.setattr(binding, "_native", Asked())
    for call in (lambda: ra.rapid_attn_block_sparse(x, x, x, x, m, 64), lambda: ra.rapid_attn_joint([(x, x, x, x)], mask=m, block=64),
                 lambda: ra.rapid_mask_select(x, x, m, 64), lambda: ra.rapid_attn_joint_select([(x, x, x, x)])):
        with pytest.raises(TypeError):
            call()
