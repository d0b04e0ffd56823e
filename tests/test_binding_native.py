"""The native part of the binding refuses what is no candidate before any call of the library.  No GPU."""
import numpy as np
import pytest
import torch


def test_refusals():
    from paper_2304_14463_amd import _candidates as native
    s, a = torch.zeros(8, dtype=torch.int32), torch.zeros(8, dtype=torch.uint8)
    for bad in ((s, s, a), (s, None, a), (a, s, a), (s, s, s)):   # on the CPU, or of another type
        with pytest.raises(ValueError):
            native.pointers(4, *bad)
        if bad[1] is not None:
            with pytest.raises(ValueError):
                native.evaluate(0, 0, 4, *bad, None, 0, 24, 0)
    for bad in (np.zeros(8, np.int32), None, 3):
        with pytest.raises(TypeError):
            native.pointers(4, bad, s, a)
    with pytest.raises(TypeError):
        native.pointers(4, s, s)
    with pytest.raises(TypeError):
        native.evaluate("moc_eval_batch", 0, 4, s, s, a, None, 0, 24, 0)


def test_results_are_made_like_the_candidates():
    from paper_2304_14463_amd import _candidates as native
    x, at = native.empty(torch.zeros(2), 1, 5, 24)
    assert x.shape == (5, 24) and x.dtype is torch.uint8 and x.data_ptr() == at and x.is_contiguous() and not x.requires_grad
    x, at = native.empty(torch.zeros(2, requires_grad=True), 4, 7)
    assert x.shape == (7,) and x.dtype is torch.int32 and x.data_ptr() == at and not x.requires_grad
    with pytest.raises(RuntimeError):
        native.empty(torch.zeros(2), 1, -1, 24)


@pytest.mark.parametrize("native", [None, 1], ids=["missing", "of another version"])
def test_native_part_that_does_not_fit_the_binding(monkeypatch, native):
    """... is refused with the command that builds it."""
    import sys
    import types

    import paper_2304_14463_amd
    from paper_2304_14463_amd import moccasin
    other = None if native is None else types.ModuleType("paper_2304_14463_amd._candidates")
    if other is not None:
        other.abi_version, other.__file__ = native, "elsewhere.so"
    monkeypatch.setitem(sys.modules, "paper_2304_14463_amd._candidates", other)
    monkeypatch.delattr(paper_2304_14463_amd, "_candidates", raising=False)
    if other is not None:
        monkeypatch.setattr(paper_2304_14463_amd, "_candidates", other, raising=False)
    monkeypatch.setattr(moccasin, "_native", None)
    with pytest.raises(RuntimeError, match="paper_2304_14463_amd.build"):
        moccasin._candidates()


@pytest.mark.gpu
@pytest.mark.parametrize("call", ["moc_eval_batch", "moc_eval_batch_staged", "moc_eval_toggles"])
def test_results_into_a_storage(call):
    """`out` may be whatever has a data_ptr()."""
    from paper_2304_14463_amd import moccasin as moc
    g = moc.moc_graph_upload(3, [0, 0, 1, 2], [0, 1], [5, 6, 7], [1, 1, 1], 100, 1)
    moc.moc_graph_set_order(g, [0, 1, 2])
    s = torch.tensor([0, 2, 5] if call.endswith("staged") else [0, 1, 2], dtype=torch.int32, device="cuda")
    e, a = s + 1, torch.ones(3, dtype=torch.uint8, device="cuda")
    want = getattr(moc, call)(g, s, e, a)
    room = torch.zeros_like(want)
    storage = room.untyped_storage()
    assert getattr(moc, call)(g, s, e, a, out=storage) is storage
    assert (room == want).all() and want.any()
    with pytest.raises(AttributeError):
        getattr(moc, call)(g, s, e, a, out=[0])
    g.free()
