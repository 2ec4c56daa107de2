"""Attention scores with at most 64 query rows per kv head (the narrow kernels) and their neighbours, against the CPU oracle:
row counts at the edges of the 16-row blocks, keys at the edges of the 16-key subtiles and of the eight waves, several subtiles
per wave, both softmax readings, a prefix, logits so far apart that a wave's sums relative to its first keys leave the range of
float, and keys that are not finite."""
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
    # later keys lift the logits by hundreds (log2): the partial sums that are merged are that far apart
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


# 32 kv heads share the 256 workgroup slots: 8 workgroups of 256 keys each, so a wave of the narrow kernels walks two 16-key
# subtiles (t = 0, 1) 128 keys apart in a 2048-key sequence, and three in a longer one
MANY_KV_HEADS = 32


@pytest.mark.parametrize("dtype,dh,Tq", [("bf16", 64, 5), ("bf16", 128, 20), ("bf16", 32, 64), ("f32", 64, 31), ("f32", 32, 7)])
@pytest.mark.parametrize("tokens,vis_start,mode", [(2000, 0, 0), (2900, 40, 0), (2900, 40, 1)])
def test_several_subtiles_per_wave(dtype, dh, Tq, tokens, vis_start, mode):
    layer = make_layer(4500 + dh + Tq, 10, tokens // 10, 4, Tq + 3, 16, MANY_KV_HEADS, MANY_KV_HEADS, dh, dtype, vis_start=vis_start)
    seg = np.zeros(layer.n_vis, dtype=np.int32)
    quotas = [layer.n_vis // 2]
    got, q = run_prune(layer, seg, quotas, Tq=Tq, score_mode=mode)
    check_prune(layer, seg, quotas, got, q, score_mode=mode)


@pytest.mark.parametrize("up", [True, False])
@pytest.mark.parametrize("dtype,dh,Tq", [("bf16", 64, 9), ("bf16", 64, 20), ("bf16", 64, 64), ("bf16", 128, 40), ("f32", 32, 9), ("f32", 64, 33)])
def test_sums_that_leave_the_range_of_float(dtype, dh, Tq, up):
    """Keys alternate between low and high logits every 128 keys: relative to the largest logit of its first subtile, the
    second subtile of every wave adds terms beyond 2^127 (`up`; the wave starts over with a running maximum) or far below the
    smallest float (the other way round).  A wave that kept an infinite or lost sum would spoil every row's normaliser."""
    B = mk()
    rng = np.random.default_rng(dh + Tq)
    H, S = MANY_KV_HEADS, 2048
    n = S - Tq
    q = np.abs(rng.standard_normal((H, Tq, dh))).astype(np.float32) + np.float32(0.1)
    k = (0.3 * rng.standard_normal((H, S, dh))).astype(np.float32)
    k[:, (np.arange(S) // 128) % 2 == (1 if up else 0)] += np.float32(1600 / dh)
    if dtype == "bf16":
        q, k = synth.bf16_round(q), synth.bf16_round(k)
    # the premise, in log2 units: [head, query, workgroup, subtile t, wave, key of the subtile]
    logits = np.matmul(q.astype(np.float64), k.astype(np.float64).transpose(0, 2, 1)) / np.sqrt(dh)
    tops = (logits * 1.4426950408889634).reshape(H, Tq, S // 256, 2, 8, 16).max(axis=5)
    jump = tops[:, :, :, 1] - tops[:, :, :, 0]
    assert (jump > 130).all() if up else (jump < -130).all()
    hidden = torch.zeros((S, 8), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    out = B.metok_prefill_prune(hidden, 0, n, i32(np.zeros(n)), [n // 2], q_text=synth.to_torch(q, dtype, "cuda"),
                                k_all=synth.to_torch(k, dtype, "cuda"))
    torch.cuda.synchronize()
    got, want = out["scores"].cpu().numpy().astype(np.float64), O.text_to_visual_attention(q, k, 0, n, 0)
    # a logit is dh products added in fp32: at most dh 2^-24 of its size off, once in the term and once in the normaliser;
    # the sums and the exponentials as elsewhere (RTOL); below 2^-126 a probability may be zero
    tol = RTOL[dtype] + 2 * dh * 2.0 ** -24 * np.abs(logits).max()
    assert np.isfinite(got).all()
    assert (np.abs(got - want) <= tol * want + 2.0 ** -126).all(), float((np.abs(got - want) / (want + 1e-30)).max())


@pytest.mark.parametrize("Hq,Tq", [(4, 20), (4, 64), (28, 10), (28, 64)])          # narrow; the shared-stage kernels with one and two blocks per wave
def test_keys_that_are_not_finite(Hq, Tq):
    """A key with a NaN has a NaN score, and the rows of its kv head, whose normaliser it spoils, add nothing to the other
    keys; a key whose logits are -inf gets no probability and leaves the rest alone; the selection keeps its order."""
    from tests.test_gpu_selection_paths import ordered_key
    B = mk()
    rng = np.random.default_rng(Hq + Tq)
    Hkv, dh, n = 4, 64, 900
    group, S = Hq // Hkv, n + Tq
    q = synth.bf16_round(np.abs(rng.standard_normal((Hq, Tq, dh))).astype(np.float32) + np.float32(0.1))
    k = synth.bf16_round((0.2 * rng.standard_normal((Hkv, S, dh))).astype(np.float32))
    bad = k.copy()
    bad[1, 50, 3] = np.nan
    bad[2, 70, 5] = -np.inf
    hidden = torch.zeros((S, 8), dtype=torch.bfloat16, device="cuda")
    out = B.metok_prefill_prune(hidden, 0, n, i32(np.zeros(n)), [n // 2], q_text=synth.to_torch(q, "bf16", "cuda"),
                                k_all=synth.to_torch(bad, "bf16", "cuda"))
    torch.cuda.synchronize()
    scores = out["scores"].cpu().numpy()
    k[2, 70] = np.float32(-1e5)                                       # probability 0 in 64 bits too
    want = np.zeros(n)
    for h in range(Hkv):
        if h != 1:
            want += O.text_to_visual_attention(q[h * group:(h + 1) * group], k[h:h + 1], 0, n, 0) / Hkv
    others = np.arange(n) != 50
    assert np.isnan(scores[50])
    assert_rel(scores[others], want[others], RTOL["bf16"], "scores")
    order = np.lexsort((np.arange(n), -ordered_key(scores)))
    np.testing.assert_array_equal(out["kept_idx"].cpu().numpy(), np.sort(order[:n // 2]))
