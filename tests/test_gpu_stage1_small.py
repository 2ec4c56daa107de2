"""Stage 1 of a small video in one launch: against the oracle and the two separate calls,
on both sides of each line."""
import pytest
import torch

from paper_2506_02850_amd import synth
from tests.stage1_plan import small_video
from tests.test_gpu_stage1_one_call import check, mk

pytestmark = pytest.mark.gpu


# small: in one launch
@pytest.mark.parametrize("T,grid,d,dtype,k,alpha,beta,s1,s2,small", [
    (8, (4, 4), 64, "f32", 4, 0.5, 0.4, 2, 3, True),
    (32, (4, 4), 128, "bf16", 5, 0.5, 0.4, 2, 3, True),       # 32 frames, 512 tokens, 128 KB: the largest
    (33, (3, 5), 128, "bf16", 5, 0.5, 0.4, 2, 3, False),      # one frame too many
    (27, (1, 19), 64, "bf16", 6, 0.5, 0.4, 2, 3, False),      # 513 tokens
    (32, (4, 4), 136, "bf16", 5, 0.5, 0.4, 2, 3, False),      # 136 KB
    (4, (4, 4), 1024, "bf16", 2, 0.5, 0.5, 2, 3, True),       # four rounds of chunks
    (4, (4, 4), 1032, "bf16", 2, 0.5, 0.5, 2, 3, False),      # five
    (4, (2, 2), 4096, "bf16", 2, 0.5, 0.5, 2, 3, False),      # sixteen
    (16, (4, 4), 64, "bf16", 5, 0.5, 0.4, 1, 2, True),        # 2048 pooled chunks
    (17, (4, 4), 64, "bf16", 5, 0.5, 0.4, 1, 2, False),       # 2176
    (32, (4, 4), 128, "bf16", 5, 0.5, 0.4, 1, 2, False),      # 8192
    (2, (3, 3), 8, "bf16", 1, 0.5, 0.4, 2, 3, True),          # one chunk a row: fifteen of sixteen lanes idle
    (5, (7, 5), 24, "f32", 5, 0.3, 0.45, 2, 3, True),         # six chunks; every frame an event; 2, 3, 7 and 7
    (7, (3, 5), 40, "bf16", 3, 0.5, 0.4, 1, 2, True),         # stride 1; a run of frames with one missing
    (1, (4, 4), 64, "bf16", 1, 0.5, 0.4, 2, 3, True),
    (3, (11, 11), 64, "f32", 2, 0.7, 0.3, 3, 4, True),        # 3, 4, 5 and 6: windows with and without code of their own
])
@pytest.mark.parametrize("edge,sim_mode,reduce_", [(0, 0, 0), (1, 1, 1)])
def test_small_shapes(T, grid, d, dtype, k, alpha, beta, s1, s2, small, edge, sim_mode, reduce_):
    assert small_video(T, grid, d, dtype, s1, s2, edge) == small
    v = synth.planted_video(500 + T + d, T, grid, d, k, 1, T, 0.15, dtype)
    for out_dtype in ("f32", "bf16"):
        check(v, grid, k, alpha, beta, s1, s2, out_dtype, sim_mode=sim_mode, edge=edge, reduce_=reduce_)


# every stride 2: one launch where one round of loads is enough, two otherwise
@pytest.mark.parametrize("T,grid,d,dtype,small", [
    (12, (4, 4), 40, "bf16", True), (16, (4, 4), 64, "f32", True),     # 64 tokens of four frames, 1024 pooled chunks: the largest
    (17, (4, 4), 64, "f32", False), (12, (4, 6), 40, "bf16", False), (16, (4, 4), 264, "bf16", False), (16, (2, 2), 256, "bf16", True),
    (1, (2, 2), 8, "bf16", True)])
def test_small_shapes_of_uniform_stride(T, grid, d, dtype, small):
    assert small_video(T, grid, d, dtype, 2, 2, one_pass=True) == small
    v = synth.planted_video(700 + T + d, T, grid, d, min(T, 7), 1, T, 0.15, dtype)
    for out_dtype in ("f32", "bf16"):
        check(v, grid, min(T, 7), 1.0, 1.0, 2, 2, out_dtype, edge=T % 2, reduce_=T % 2)
    check(v, grid, min(T, 7), 1.0, 1.0, 2, 2, "f32", sim_mode=1)       # the adaptive form


@pytest.mark.parametrize("uniform", [False, True])
def test_small_batch_is_its_videos(uniform):
    B = mk()
    g = torch.Generator(device="cuda").manual_seed(3)
    gh, gw = (4, 4) if uniform else (4, 6)
    assert small_video(12, (gh, gw), 64, "bf16", 2, 2 if uniform else 3, one_pass=uniform)
    feats = torch.randn((5, 12, gh * gw, 64), generator=g, device="cuda").bfloat16()
    text = torch.randn((5, 64), generator=g, device="cuda").bfloat16()
    args = (1.0, 1.0, 2, 2) if uniform else (0.5, 0.4, 2, 3)
    many = B.metok_segment_compress_batched(feats, gh, gw, 3, text, *args)
    for b in range(5):
        one = B.metok_segment_compress(feats[b], gh, gw, 3, text[b], *args)
        M = int(one["frame_offsets"][-1])                # rows behind the last pooled one are not written
        for name, t in one.items():
            rows = M if name in ("out_tokens", "token_event") else None
            assert torch.equal(many[name][b][:rows], t[:rows]), (name, b)


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_small_with_a_frame_that_is_not_finite(value):
    B = mk()
    g = torch.Generator(device="cuda").manual_seed(4)
    feats = torch.randn((12, 16, 64), generator=g, device="cuda")
    feats[5, 3, 7] = value
    text = torch.randn((64,), generator=g, device="cuda")
    one = B.metok_segment_compress(feats, 4, 4, 3, text, 0.5, 0.4, 2, 3)
    seg = B.metok_segment_events(feats, 3, text)
    two = B.metok_compress_encoder_tokens(feats, 4, 4, seg["event_start"], 0.5, 0.4, 2, 3, frame_score=seg["frame_score"])
    for name in ("event_start", "frame_event"):
        assert torch.equal(one[name], seg[name]), name
    for name in ("event_is_key", "frame_is_key", "frame_stride", "frame_offsets"):
        assert torch.equal(one[name], two[name]), name
    M = int(one["frame_offsets"][-1])
    assert torch.equal(one["out_tokens"][:M].isnan(), two["out_tokens"][:M].isnan())
    assert torch.equal(one["out_tokens"][:M].nan_to_num(), two["out_tokens"][:M].nan_to_num())


@pytest.mark.parametrize("side", [4, 16])                                # one launch, and a kernel for every name
@pytest.mark.parametrize("uniform,names", [(False, {"FRAME_STATS", "POOL", "SEGMENT", "PLAN"}), (True, {"FRAME_STATS_POOL2", "SEGMENT", "PLAN"})])
def test_names_that_the_trace_hook_brackets(side, uniform, names):
    B = mk()
    assert small_video(8, (side, side), 64, "f32", 2, 2 if uniform else 3, one_pass=uniform) == (side == 4)
    ids = {"FRAME_STATS": 1, "POOL": 2, "FRAME_STATS_POOL2": 3, "SEGMENT": 4, "PLAN": 5, "ROW_STATS": 6}
    feats, text = torch.randn((8, side * side, 64), device="cuda"), torch.randn((64,), device="cuda")
    args = (feats, side, side, 3, text) + ((1.0, 1.0, 2, 2) if uniform else (0.5, 0.4, 2, 3))
    B.metok_segment_compress(*args)
    bracketed = set()
    for name, kernel in ids.items():
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        end.record()
        torch.zeros((1,), device="cuda")
        begin.record()                                                  # after `end` until the call records both
        assert B.lib().metok_trace_kernel(kernel, begin.cuda_event, end.cuda_event) == 0
        try:
            B.metok_segment_compress(*args)
        finally:
            B.lib().metok_trace_kernel(0, None, None)
        torch.cuda.synchronize()
        if begin.elapsed_time(end) > 0:
            bracketed.add(name)
    assert bracketed == names
