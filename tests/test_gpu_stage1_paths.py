"""Stage 1 where its kernels change shape: rows at the edges of the chunk counts per lane, frame counts at the edges of the
ranking and reduction splits, every pooling stride that has its own window code, and the event ids of uniformly pooled rows
on both sides of the planning workgroup's limit.  Compared with the CPU oracle with the tolerances of tests/parity.py and,
bit for bit, with the two-call path."""
import numpy as np
import pytest
import torch

from oracle import metok_oracle as O
from paper_2506_02850_amd import synth
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
