"""The binding without its native form, and when that counts as built (no GPU needed)."""
import sys

import pytest

from paper_2504_12285_amd import binding as bl

torch = pytest.importorskip("torch")


def test_without_the_native_form_calls_run_in_python(monkeypatch):
    import paper_2504_12285_amd as pkg
    monkeypatch.setattr(bl, "_native", None)
    monkeypatch.delattr(pkg, "_bl_torch", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2504_12285_amd._bl_torch", None)      # import raises ImportError
    with pytest.warns(RuntimeWarning, match="run in Python"):
        native = bl._first_native()
    assert bl._native is native
    for call in (native.quant, native.product, native.decode, native.run):
        assert call(1, 2, 3) is NotImplemented
    with pytest.raises(AssertionError):                                           # the Python form's own check
        bl.bl_quant_act_int8(torch.zeros((1, 64), dtype=torch.bfloat16))
