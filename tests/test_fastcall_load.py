"""The binding without its native entry points: loaded and called all the same, in Python."""
import os
import sys
import warnings

import pytest
import torch

from paper_2401_13660_amd import _binding as B

pytestmark = pytest.mark.skipif(not os.path.exists(B.LIB_PATH), reason="libmbscan.so not built")
NAME = B.__package__ + "._fastcall"


@pytest.fixture
def unloaded(monkeypatch):
    """The binding as before its first call, with no native module imported."""
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_fast", None)
    monkeypatch.delitem(sys.modules, NAME, raising=False)
    monkeypatch.delattr(sys.modules[B.__package__], "_fastcall", raising=False)
    return monkeypatch


def test_used_where_it_is_built_for_this_torch(unloaded):
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        B.load_library()
    assert B._fast is not None and B._fast.torch_version == torch.__version__


def _takes_calls_in_python(match):
    with pytest.warns(RuntimeWarning, match=match):
        lib = B.load_library()
    assert B._fast is None and lib is B._lib and lib.mb_abi_version() > 0
    with warnings.catch_warnings():                      # said once
        warnings.simplefilter("error")
        assert B.load_library() is lib
        with pytest.raises(B.MBScanError, match="u must be"):    # the Python code's own check
            B.scan_fwd(*[torch.zeros(1)] * 5)


def test_absent_or_not_loadable(unloaded):
    unloaded.setitem(sys.modules, NAME, None)            # its import raises ImportError
    _takes_calls_in_python("_fastcall")


def test_built_for_another_torch(unloaded):
    import paper_2401_13660_amd._fastcall as fast
    unloaded.setattr(fast, "torch_version", "0.0")
    _takes_calls_in_python("built for torch 0.0")
