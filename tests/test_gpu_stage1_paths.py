"""Stage 1 where its kernels change shape: rows at the edges of the chunk counts per lane, frame counts at the edges of the
ranking and reduction splits, thousands of frames in one call, every pooling stride that has its own window code, the event
ids of uniformly pooled rows on both sides of the planning workgroup's limit, and a frame that is not finite.  Compared with
the CPU oracle with the tolerances of tests/parity.py and, bit for bit, with the two-call path."""
import numpy as np
import pytest
import torch

from oracle import metok_oracle as O
from paper_2506_02850_amd import synth
from tests.parity import RTOL, assert_rel, frame_score_scale
from tests.test_gpu_stage1_one_call import check, mk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,chunks", [("bf16", c) for c in (1, 16, 17, 48, 49, 80, 81, 96, 128, 129, 144, 145, 192, 193, 257, 320, 385)] +
                         [("f32", c) for c in (33, 65, 144, 192, 193, 300, 512, 769)])
def test_row_widths_at_the_edges_of_the_chunk_counts(dtype, chunks):
    d = chunks * (8 if dtype == "bf16" else 4)
    v = synth.planted_video(6000 + chunks, 7, (3, 5), d, 2, 1, 7, 0.1, dtype)
    check(v, (3, 5), 2, 0.5, 0.5, 1, 2, dtype)


@pytest.mark.parametrize("T,k", [(1, 1), (2, 1), (2, 2), (15, 4), (16, 5), (17, 16), (33, 6), (257, 9), (512, 20), (513, 20), (1025, 30)])
def test_frame_counts_at_the_edges_of_the_splits(T, k):
    v = synth.planted_video(7000 + T, T, (2, 3), 64, min(k, 8, T), 1, T, 0.05, "f32")
    # ties do not matter here: the boundaries are compared with the oracle's on the kernel's own similarities
    B = mk()
    feats, text = synth.to_torch(v.feats, "f32", "cuda"), synth.to_torch(v.text_emb, "f32", "cuda")
    got = B.metok_segment_compress(feats, 2, 3, k, text, 0.5, 0.4, 1, 2)
    torch.cuda.synchronize()
    sim = got["sim"].cpu().numpy()
    es, fe = O.event_boundaries(sim, k)
    np.testing.assert_array_equal(got["event_start"].cpu().numpy(), es)
    np.testing.assert_array_equal(got["frame_event"].cpu().numpy(), fe)
    ref = O.compress_encoder_tokens(v.feats, (2, 3), None, es, 0.5, 0.4, 1, 2, frame_score=got["frame_score"].cpu().numpy().astype(np.float64))
    for name in ("frame_stride", "frame_offsets"):
        np.testing.assert_array_equal(got[name].cpu().numpy(), ref[name], err_msg=name)
    M = int(ref["frame_offsets"][-1])
    np.testing.assert_array_equal(got["token_event"][:M].cpu().numpy(), ref["token_event"])
    np.testing.assert_allclose(got["out_tokens"][:M].cpu().numpy(), ref["tokens"], rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("dtype,out_dtype", [("bf16", "bf16"), ("bf16", "f32"), ("f32", "f32"), ("f32", "bf16")])
@pytest.mark.parametrize("grid,s1,s2,alpha", [((7, 9), 1, 2, 0.5), ((13, 12), 2, 3, 0.5), ((13, 11), 3, 4, 0.75), ((14, 13), 3, 5, 0.5),
                                              ((12, 12), 6, 4, 0.5), ((5, 3), 7, 2, 1.0)])
@pytest.mark.parametrize("edge", [O.POOL_FLOOR, O.POOL_CEIL])
def test_every_window_code(grid, s1, s2, alpha, edge, dtype, out_dtype):
    v = synth.planted_video(8000 + grid[0] * 16 + grid[1], 12, grid, 144, 4, 1, 9, 0.1, dtype)
    check(v, grid, 4, alpha, 0.5, s1, s2, out_dtype, edge=edge)


@pytest.mark.parametrize("T,grid", [(60, (4, 6)), (300, (4, 6)), (461, (24, 24))])      # 360, 1800 and 66384 rows
def test_event_ids_of_uniformly_pooled_rows(T, grid):
    v = synth.planted_video(9000 + T, T, grid, 16, 5, 1, T, 0.02, "bf16")
    B = mk()
    feats, text = synth.to_torch(v.feats, "bf16", "cuda"), synth.to_torch(v.text_emb, "bf16", "cuda")
    if T == 60:
        got = B.metok_segment_compress_batched(torch.stack([feats, feats]), *grid, 5, torch.stack([text, text]), 1.0, 1.0, 2, 2)
    else:
        got = B.metok_segment_compress(feats, *grid, 5, text, 1.0, 1.0, 2, 2)
    torch.cuda.synchronize()
    rows = (grid[0] // 2) * (grid[1] // 2)
    events, frames = got["token_event"].cpu().numpy().reshape(-1, T * rows), got["frame_event"].cpu().numpy().reshape(-1, T)
    for te, fe in zip(events, frames):
        np.testing.assert_array_equal(te, np.repeat(fe, rows))


@pytest.mark.parametrize("T,grid,d,s1,s2", [(40, (4, 4), 8, 3, 4), (33, (12, 12), 64, 3, 4), (20, (24, 24), 40, 1, 2), (9, (27, 27), 136, 2, 3)])
def test_few_or_many_pooling_workgroups_per_frame(T, grid, d, s1, s2):
    # 1 chunk, 128, 2880 and 2873 chunks at the smallest stride: one workgroup per frame, one, twelve and twelve
    v = synth.planted_video(9500 + T, T, grid, d, 3, 1, T, 0.2 / d ** 0.5, "bf16")
    check(v, grid, 3, 0.5, 0.4, s1, s2, "bf16")


# partials per frame: 4 tokens each with strides of their own, a 2 x 2 window each with stride 2; one workgroup adds them up for one
# frame per wave (T <= 16) and up to 8192 of those beyond (T - 16 times 512, 529; 8371 for the 17th frame)
@pytest.mark.parametrize("T,grid,s1,s2", [(5, (96, 96), 6, 9), (16, (61, 64), 5, 7), (17, (182, 184), 12, 16), (17, (64, 64), 6, 9),
                                          (32, (32, 64), 5, 7), (32, (46, 46), 5, 7), (32, (46, 46), 2, 2)])
def test_few_frames_of_many_partials(T, grid, s1, s2):
    v = synth.planted_video(9700 + T, T, grid, 16, 4, 1, T, 0.05, "f32")
    alpha, beta = (1.0, 1.0) if s1 == s2 else (0.5, 0.4)
    check(v, grid, 4, alpha, beta, s1, s2, "f32")


def tied_video(T, seed):
    """Frames drawn from four vectors: most adjacent pairs tie exactly in their cosine, most frames in their text score."""
    rng = np.random.default_rng(seed)
    basis = rng.standard_normal((4, 4, 16)).astype(np.float32)
    return basis[rng.integers(0, 4, size=T)], rng.standard_normal(16).astype(np.float32)


@pytest.mark.parametrize("T", [1, 3, 8, 9, 32, 33, 100, 511, 512, 513])     # 64 to 2 threads per frame, then one; totals by one workgroup up to 32
@pytest.mark.parametrize("event_reduce", [O.EVENT_REDUCE_MEAN, O.EVENT_REDUCE_MAX])
def test_short_videos_with_ties(T, event_reduce):
    """Boundaries, key events and key frames of tied similarities and scores: the decisions on the GPU's own values, exactly, from
    one call, from the two calls, and in a batch; k from one event to one per frame."""
    B = mk()
    feats_np, text_np = tied_video(T, 77 + T)
    feats, text = torch.from_numpy(feats_np).cuda(), torch.from_numpy(text_np).cuda()
    for k in sorted({1, max(1, T // 17), max(1, T // 3), T}):
        one = B.metok_segment_compress(feats, 2, 2, k, text, 0.5, 0.45, 1, 2, event_reduce=event_reduce)
        seg = B.metok_segment_events(feats, k, text)
        two = B.metok_compress_encoder_tokens(feats, 2, 2, seg["event_start"], 0.5, 0.45, 1, 2, frame_score=seg["frame_score"], event_reduce=event_reduce)
        many = B.metok_segment_compress_batched(torch.stack([feats] * 3), 2, 2, k, torch.stack([text] * 3), 0.5, 0.45, 1, 2, event_reduce=event_reduce)
        torch.cuda.synchronize()
        es, fe = O.event_boundaries(one["sim"].cpu().numpy(), k)
        np.testing.assert_array_equal(one["event_start"].cpu().numpy(), es)
        np.testing.assert_array_equal(one["frame_event"].cpu().numpy(), fe)
        score = one["frame_score"].cpu().numpy().astype(np.float64)
        ref = O.compress_encoder_tokens(feats_np, (2, 2), None, es, 0.5, 0.45, 1, 2, frame_score=score, event_reduce=event_reduce)
        # float32 sums of up to T scores: relative to the largest score, T ulps at most
        np.testing.assert_allclose(one["event_score"].cpu().numpy(), ref["event_score"], rtol=0, atol=T * 2.0 ** -24 * np.abs(score).max())
        # key events: the rule on the GPU's own event scores (equal events tie), then key frames, strides and offsets follow
        got_es = one["event_score"].cpu().numpy()
        key = np.zeros(k, dtype=np.uint8)
        key[np.lexsort((np.arange(k), -got_es))[:int(np.ceil(0.5 * k - 1e-9))]] = 1
        np.testing.assert_array_equal(one["event_is_key"].cpu().numpy(), key)
        np.testing.assert_array_equal(one["frame_is_key"].cpu().numpy(), ref["frame_is_key"])
        stride = np.where(key[fe] == 1, np.where(ref["frame_is_key"] == 1, 1, 2), np.where(ref["frame_is_key"] == 1, 2, 2))
        np.testing.assert_array_equal(one["frame_stride"].cpu().numpy(), stride)
        np.testing.assert_array_equal(one["frame_offsets"].cpu().numpy(), np.concatenate([[0], np.cumsum(np.where(stride == 1, 4, 1))]))
        M = int(one["frame_offsets"][-1])
        for name in ("sim", "event_start", "frame_event", "frame_score"):
            assert torch.equal(one[name], seg[name]), name
        for name in ("event_is_key", "frame_is_key", "frame_stride", "frame_offsets", "event_score"):
            assert torch.equal(one[name], two[name]), name
        for b in range(3):
            for name, t in one.items():
                rows = slice(0, M) if name in ("out_tokens", "token_event") else slice(None)
                assert torch.equal(many[name][b][rows], t[rows]), (b, name)


@pytest.mark.parametrize("T,k", [(2048, 5), (2049, 5), (5000, 1), (3000, 2999), (4100, 1500), (8192, 61), (8192, 8192)])
@pytest.mark.parametrize("uniform", [False, True])      # three strides after a pass of statistics; stride 2 in one pass
def test_long_videos_in_one_call(T, k, uniform):
    # boundaries by radix select, key frames of events and key events by bisection above 1024, then the plan in the same
    # workgroup and the same LDS; the totals of 64 workgroups over several rounds of frames
    B = mk()
    feats_np, text_np = tied_video(T, T + k)
    feats, text = torch.from_numpy(feats_np).cuda(), torch.from_numpy(text_np).cuda()
    alpha, s1, s2 = (1.0, 2, 2) if uniform else (0.5, 1, 2)
    one = B.metok_segment_compress(feats, 2, 2, k, text, alpha, 0.45, s1, s2)
    torch.cuda.synchronize()
    sim, score = one["sim"].cpu().numpy(), one["frame_score"].cpu().numpy()
    assert_rel(sim, O.adjacent_frame_cosine(feats_np.astype(np.float64)), RTOL["f32"], "sim", scale=1.0)
    assert_rel(score, O.frame_text_score(feats_np, text_np), RTOL["f32"], "frame_score", scale=frame_score_scale(feats_np, text_np))
    # decisions on the GPU's own values, exactly
    es, fe = O.event_boundaries(sim, k)
    np.testing.assert_array_equal(one["event_start"].cpu().numpy(), es)
    np.testing.assert_array_equal(one["frame_event"].cpu().numpy(), fe)
    ref = O.compress_encoder_tokens(feats_np, (2, 2), None, es, alpha, 0.45, s1, s2, frame_score=score.astype(np.float64))
    for name in ("event_is_key", "frame_is_key", "frame_stride", "frame_offsets"):
        np.testing.assert_array_equal(one[name].cpu().numpy(), ref[name], err_msg=name)
    M = int(ref["frame_offsets"][-1])
    np.testing.assert_array_equal(one["token_event"][:M].cpu().numpy(), ref["token_event"])
    np.testing.assert_allclose(one["out_tokens"][:M].cpu().numpy(), ref["tokens"], rtol=1e-5, atol=1e-6)
    if uniform:
        return
    # the two calls, bit for bit
    seg = B.metok_segment_events(feats, k, text)
    two = B.metok_compress_encoder_tokens(feats, 2, 2, seg["event_start"], alpha, 0.45, s1, s2, frame_score=seg["frame_score"])
    torch.cuda.synchronize()
    for name in ("sim", "event_start", "frame_event", "frame_score"):
        assert torch.equal(one[name], seg[name]), name
    for name in ("event_is_key", "frame_is_key", "frame_stride", "frame_offsets", "event_score"):
        assert torch.equal(one[name], two[name]), name
    assert torch.equal(one["out_tokens"][:M], two["out_tokens"][:M]) and torch.equal(one["token_event"][:M], two["token_event"][:M])


@pytest.mark.parametrize("T,k", [(2049, 3), (4100, 1500)])
def test_long_videos_of_a_batch(T, k):
    B = mk()
    videos = [tied_video(T, 10 * T + b) for b in range(3)]
    feats = [torch.from_numpy(f).cuda() for f, _ in videos]
    texts = [torch.from_numpy(t).cuda() for _, t in videos]
    got = B.metok_segment_compress_batched(torch.stack(feats), 2, 2, k, torch.stack(texts), 0.5, 0.45, 1, 2)
    for b in range(3):
        one = B.metok_segment_compress(feats[b], 2, 2, k, texts[b], 0.5, 0.45, 1, 2)
        torch.cuda.synchronize()
        M = int(one["frame_offsets"][-1])
        for name, t in one.items():
            rows = slice(0, M) if name in ("out_tokens", "token_event") else slice(None)
            assert torch.equal(got[name][b][rows], t[rows]), (b, name)


@pytest.mark.parametrize("T", [20, 600, 3000])          # boundaries ranked by several threads, by one, by radix select
def test_a_frame_that_is_not_finite(T):
    """Two pairs without a similarity (NaN): the boundaries are the k - 1 lowest keys of what the kernel wrote, in the order of
    the bits, the events cover the video, and every frame gets its rows."""
    from tests.test_gpu_selection_paths import ordered_key
    B = mk()
    feats_np, text_np = tied_video(T, T)
    feats_np = feats_np.copy()
    feats_np[7, 1, 3] = np.nan
    k = 6
    got = B.metok_segment_compress(torch.from_numpy(feats_np).cuda(), 2, 2, k, torch.from_numpy(text_np).cuda(), 0.5, 0.45, 1, 2)
    torch.cuda.synchronize()
    sim = got["sim"].cpu().numpy()
    assert np.isnan(sim[6:8]).all() and np.isfinite(np.delete(sim, (6, 7))).all()
    cuts = np.sort(np.lexsort((np.arange(T - 1), ordered_key(sim)))[:k - 1]) + 1
    np.testing.assert_array_equal(got["event_start"].cpu().numpy(), np.concatenate([[0], cuts, [T]]))
    stride, offsets = got["frame_stride"].cpu().numpy(), got["frame_offsets"].cpu().numpy()
    assert set(np.unique(stride)) <= {1, 2}
    np.testing.assert_array_equal(np.diff(offsets), np.where(stride == 1, 4, 1))
    starts = got["event_start"].cpu().numpy()
    for a, b in zip(starts[:-1], starts[1:]):
        assert int(got["frame_is_key"][a:b].sum()) == int(np.ceil(0.45 * (b - a) - 1e-9))
