"""The binding's output allocation (host side only): fresh outputs have the asked length and dtype, start at multiples of 16
bytes, do not overlap, own their storage, and caller-provided ones are used and checked."""
import io

import pytest
import torch

binding = pytest.importorskip("paper_2506_02850_amd.binding")


@pytest.mark.parametrize("T,k", [(1, 1), (2, 2), (7, 3), (16, 4), (33, 5)])
def test_fresh_outputs_do_not_overlap(T, k):
    f32, i32, u8 = torch.float32, torch.int32, torch.uint8
    specs = (("a", T, i32), ("b", k + 1, i32), ("c", T + 1, i32), ("d", T, u8), ("e", k, u8), ("f", T, f32), ("g", max(T - 1, 0), f32), ("h", k, f32))
    res = binding._outs(None, "cpu", specs)
    for (name, n, dtype), t in zip(specs, res):
        assert tuple(t.shape) == (n,) and t.dtype == dtype and t.is_contiguous(), name
        if n:
            assert t.data_ptr() % 16 == 0, name
    for i, t in enumerate(res):
        t.fill_(i + 1)
    for i, t in enumerate(res):
        assert bool((t == i + 1).all())


def test_given_outputs_are_used_and_checked():
    mine = torch.zeros(5, dtype=torch.int32)
    a, b = binding._outs({"a": mine, "b": None}, "cpu", (("a", 5, torch.int32), ("b", 3, torch.int32)))
    assert a is mine and tuple(b.shape) == (3,)
    with pytest.raises(ValueError):
        binding._outs({"a": mine}, "cpu", (("a", 6, torch.int32),))


@pytest.mark.parametrize("given", [None, {"kept_idx": torch.zeros(6, dtype=torch.int32)}])
def test_fresh_outputs_are_tensors_of_their_own(given):
    # what a caller may do with one output leaves the others alone: keep it, save it, resize it, work on it with a gradient
    specs = (("kept_idx", 6, torch.int32), ("orig_idx_out", 6, torch.int32), ("frame_score", 8, torch.float32), ("sim", 7, torch.float32))
    res = binding._outs(given, "cpu", specs)
    assert len({t.untyped_storage().data_ptr() for t in res}) == len(res)
    for (_, n, dtype), t in zip(specs, res):
        assert t._base is None and t.untyped_storage().nbytes() == n * t.element_size()
    kept, orig, score, sim = res
    orig.fill_(7)
    kept.resize_(40).fill_(1)
    assert bool((orig == 7).all())
    a, b = io.BytesIO(), io.BytesIO()
    torch.save(sim, a)
    torch.save(sim.clone(), b)
    assert len(a.getvalue()) == len(b.getvalue())
    weight = torch.ones(8, requires_grad=True)
    score.fill_(2.0).mul_(weight)
    score.sum().backward()
    assert bool((weight.grad == 2.0).all())
