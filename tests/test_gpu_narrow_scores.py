"""Attention scores with at most 64 query rows per kv head (the narrow kernels) and their neighbours, against the CPU oracle:
row counts at the edges of the 16-row blocks, keys at the edges of the 16-key subtiles and of the eight waves, both softmax
readings, a prefix, and logits so far apart that the sums relative to the first keys leave the range of float."""
import numpy as np
import pytest
import torch

from oracle import metok_oracle as O
from paper_2506_02850_amd import synth
from tests.parity import RTOL, assert_rel
from tests.test_gpu_stage2 import check_prune, i32, make_layer, mk, run_prune

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,dh,Hq,Hkv,Tq", [
    ("bf16", 128, 4, 4, 1), ("bf16", 128, 28, 4, 1), ("bf16", 128, 4, 4, 16), ("bf16", 128, 4, 4, 17), ("bf16", 128, 2, 2, 33),
    ("bf16", 128, 2, 2, 64), ("bf16", 128, 2, 2, 65), ("bf16", 64, 6, 2, 21), ("bf16", 64, 4, 4, 5), ("bf16", 32, 3, 3, 64), ("bf16", 32, 2, 2, 32),
    ("bf16", 256, 2, 2, 8), ("f32", 32, 4, 2, 16), ("f32", 64, 2, 2, 48), ("f32", 64, 3, 3, 2), ("f32", 128, 2, 2, 9), ("f32", 128, 2, 2, 30), ("f32", 128, 2, 2, 61),
    ("bf16", 128, 8, 2, 64), ("bf16", 64, 14, 2, 32), ("f32", 64, 14, 2, 32), ("f32", 32, 6, 2, 40)])          # one row block per wave of the shared-stage kernels
@pytest.mark.parametrize("frames,tokens,vis_start,mode", [(1, 5, 0, 0), (3, 43, 2, 0), (23, 37, 0, 1), (40, 113, 17, 0)])
def test_narrow_scores(dtype, dh, Hq, Hkv, Tq, frames, tokens, vis_start, mode):
    layer = make_layer(4000 + dh + Tq, frames, tokens, min(3, frames), Tq + 3, 16, Hq, Hkv, dh, dtype, vis_start=vis_start)
    seg = np.zeros(layer.n_vis, dtype=np.int32)
    quotas = [layer.n_vis // 2]
    got, q = run_prune(layer, seg, quotas, Tq=Tq, score_mode=mode)
    check_prune(layer, seg, quotas, got, q, score_mode=mode)


# the shared-stage kernels: rows of every length, turned into fragments in one round (up to 16 pieces of 16 bytes) or two (32),
# row counts that leave a block partly empty, fewer blocks than waves, two blocks per wave, several row splits
@pytest.mark.parametrize("dtype,dh,Hq,Hkv,Tq", [
    ("bf16", 32, 5, 1, 13), ("bf16", 64, 22, 2, 9), ("bf16", 128, 23, 1, 3), ("bf16", 128, 27, 1, 19), ("bf16", 256, 1, 1, 1),
    ("bf16", 256, 7, 1, 7), ("bf16", 256, 26, 2, 20), ("f32", 32, 13, 1, 5), ("f32", 64, 21, 1, 20), ("f32", 128, 5, 1, 13), ("f32", 128, 43, 1, 6)])
@pytest.mark.parametrize("frames,tokens,mode", [(3, 11, 0), (30, 97, 1)])
def test_query_rows_of_the_shared_stage_kernels(dtype, dh, Hq, Hkv, Tq, frames, tokens, mode):
    layer = make_layer(4300 + dh + Hq, frames, tokens, 3, Tq + 1, 16, Hq, Hkv, dh, dtype, vis_start=5)
    seg = np.zeros(layer.n_vis, dtype=np.int32)
    quotas = [layer.n_vis // 3]
    got, q = run_prune(layer, seg, quotas, Tq=Tq, score_mode=mode)
    check_prune(layer, seg, quotas, got, q, score_mode=mode)


@pytest.mark.parametrize("Hq,Tq", [(2, 20), (2, 64), (14, 32)])          # narrow with two and four blocks; the shared-stage kernels
def test_logits_far_above_the_first_keys(Hq, Tq):
    # later keys lift the logits by hundreds (log2): a sum relative to the first subtile would overflow
    B = mk()
    rng = np.random.default_rng(Tq)
    n, dh, Hkv, text = 700, 64, 2, Tq
    q = np.abs(rng.standard_normal((Hq, Tq, dh))).astype(np.float32)
    k = 0.1 * rng.standard_normal((Hkv, n + text, dh)).astype(np.float32)
    k[:, 300:310] += 40.0
    k[:, 600] += 60.0
    q, k = synth.bf16_round(q), synth.bf16_round(k)
    hidden = np.zeros((n + text, 8), dtype=np.float32)
    out = B.metok_prefill_prune(synth.to_torch(hidden, "bf16", "cuda"), 0, n, i32(np.zeros(n)), [n // 2],
                                q_text=synth.to_torch(q, "bf16", "cuda"), k_all=synth.to_torch(k, "bf16", "cuda"))
    torch.cuda.synchronize()
    want = O.text_to_visual_attention(q, k, 0, n, 0)
    assert_rel(out["scores"].cpu().numpy(), want, RTOL["bf16"], "scores", scale=want.max())
    assert want[600] > 0.9
