"""Attention scores with more than 64 query rows per kv head on long key ranges, against the CPU oracle: every count of row
blocks around which waves own or share a second one, two uneven row splits, lengths at which pass 1 alone and both passes share
blocks, and sums relative to the first keys that leave the range of float."""
import numpy as np
import pytest
import torch

from oracle import metok_oracle as O
from paper_2506_02850_amd import synth
from tests.parity import RTOL
from tests.test_gpu_stage2 import check_prune, i32, make_layer, mk, run_prune

pytestmark = pytest.mark.gpu

# 32 kv heads share the 256 workgroup slots: 8 workgroups along the keys (4 where the rows are split in two)
KV_HEADS = 32


# rows / 32 rounded up: 9, 10, 11 (the last one partly empty), 13, 14, 14, 15, 16, 14 + 13
@pytest.mark.parametrize("dtype,dh,group,Tq", [
    ("bf16", 64, 9, 32), ("bf16", 128, 5, 64), ("f32", 32, 11, 31), ("bf16", 32, 13, 32), ("bf16", 128, 7, 64), ("f32", 64, 7, 64),
    ("bf16", 64, 15, 31), ("bf16", 64, 8, 64), ("bf16", 64, 27, 32)])
@pytest.mark.parametrize("tokens,vis_start,mode", [(1960, 7, 0), (4200, 0, 1)])      # 4 and 8 to 9 stages of 64 keys a workgroup
def test_row_blocks_of_the_waves(dtype, dh, group, Tq, tokens, vis_start, mode):
    layer = make_layer(5200 + dh + group, 10, tokens // 10, 4, Tq + 3, 16, KV_HEADS * group, KV_HEADS, dh, dtype, vis_start=vis_start)
    seg = np.zeros(layer.n_vis, dtype=np.int32)
    quotas = [layer.n_vis // 2]
    got, q = run_prune(layer, seg, quotas, Tq=Tq, score_mode=mode)
    check_prune(layer, seg, quotas, got, q, score_mode=mode)


@pytest.mark.parametrize("up", [True, False])
@pytest.mark.parametrize("dtype,dh,group,Tq", [("bf16", 64, 7, 64), ("bf16", 128, 9, 32), ("bf16", 64, 4, 64), ("f32", 32, 3, 40)])
def test_sums_that_leave_the_range_of_float(dtype, dh, group, Tq, up):
    """Keys alternate between low and high logits every 64 keys: relative to the largest logit of a lane's first keys, the second
    stage of every workgroup adds terms beyond 2^127 (`up`; the workgroup starts over with a running maximum) or far below the
    smallest float (the other way round).  An infinite or lost sum would spoil every row's normaliser."""
    B = mk()
    rng = np.random.default_rng(dh + Tq + group)
    H, S = KV_HEADS, 2048                                             # 256 keys, four stages a workgroup
    n = S - Tq
    q = np.abs(rng.standard_normal((H * group, Tq, dh))).astype(np.float32) + np.float32(0.1)
    k = (0.3 * rng.standard_normal((H, S, dh))).astype(np.float32)
    k[:, (np.arange(S) // 64) % 2 == (1 if up else 0)] += np.float32(1600 / dh)
    if dtype == "bf16":
        q, k = synth.bf16_round(q), synth.bf16_round(k)
    # the premise, in log2 units: [head, query, pair of stages, stage, key]
    logits = np.matmul(q.reshape(H, group * Tq, dh), k.transpose(0, 2, 1)) / np.sqrt(dh) * 1.4426950408889634
    tops = logits.reshape(H, group * Tq, S // 128, 2, 64).max(axis=4)
    jump = tops[..., 1] - tops[..., 0]
    assert (jump > 130).all() if up else (jump < -130).all()
    size = float(np.abs(logits).max()) / 1.4426950408889634
    del logits
    hidden = torch.zeros((S, 8), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    out = B.metok_prefill_prune(hidden, 0, n, i32(np.zeros(n)), [n // 2], q_text=synth.to_torch(q, dtype, "cuda"),
                                k_all=synth.to_torch(k, dtype, "cuda"))
    torch.cuda.synchronize()
    got, want = out["scores"].cpu().numpy().astype(np.float64), O.text_to_visual_attention(q, k, 0, n, 0)
    # a logit is dh products added in fp32: at most dh 2^-24 of its size off, once in the term and once in the normaliser;
    # the sums and the exponentials as elsewhere (RTOL); below 2^-126 a probability may be zero
    tol = RTOL[dtype] + 2 * dh * 2.0 ** -24 * size
    assert np.isfinite(got).all()
    assert (np.abs(got - want) <= tol * want + 2.0 ** -126).all(), float((np.abs(got - want) / (want + 1e-30)).max())
