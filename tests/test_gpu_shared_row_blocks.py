"""Attention scores with more than 64 query rows per kv head on long key ranges, against the CPU oracle: every count of row
blocks around which waves own or share a second one, two uneven row splits, lengths at which pass 1 alone and both passes share
blocks, and sums relative to the first keys that leave the range of float."""
import numpy as np
import pytest
import torch

from oracle import metok_oracle as O
from paper_2506_02850_amd import synth
from tests.parity import RTOL, assert_rel
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
    stage of every workgroup adds terms beyond 2^127 (`up`; its blocks are added once more) or far below the smallest float (the
    other way round).  An infinite or lost sum would spoil every row's normaliser."""
    S = 2048                                                          # 256 keys, four stages a workgroup
    check_scores_of_jumps(dtype, dh, group, Tq, S, (np.arange(S) // 64) % 2 == (1 if up else 0), 64, up)


@pytest.mark.parametrize("low", [32, 64, 96, 160, 224])
@pytest.mark.parametrize("dtype,dh,group,Tq", [("bf16", 64, 7, 64), ("bf16", 128, 9, 32), ("bf16", 64, 11, 31), ("f32", 64, 13, 32), ("bf16", 64, 3, 40)])
def test_one_jump_at_every_place_of_a_workgroup(dtype, dh, group, Tq, low):
    """The first `low` keys of every workgroup have low logits and the others high ones, so that the first block beyond the range of
    float is another one each time: of the first or the second subtile of a stage, and of the stages around the ends of the
    pipeline."""
    S = 2048
    check_scores_of_jumps(dtype, dh, group, Tq, S, np.arange(S) % 256 >= low, 32, None)


def check_scores_of_jumps(dtype, dh, group, Tq, S, high, run, up):
    """`high`: the keys with high logits, in runs of a multiple of `run`; up: every second run is above (below) the one before."""
    B = mk()
    rng = np.random.default_rng(dh + Tq + group)
    H = KV_HEADS
    n = S - Tq
    q = np.abs(rng.standard_normal((H * group, Tq, dh))).astype(np.float32) + np.float32(0.1)
    k = (0.3 * rng.standard_normal((H, S, dh))).astype(np.float32)
    k[:, high] += np.float32(1600 / dh)
    if dtype == "bf16":
        q, k = synth.bf16_round(q), synth.bf16_round(k)
    # the premise, in log2 units: [head, query, run, key]
    logits = np.matmul(q.reshape(H, group * Tq, dh), k.transpose(0, 2, 1)) / np.sqrt(dh) * 1.4426950408889634
    tops = logits.reshape(H, group * Tq, S // run, run).max(axis=3)
    jump = np.diff(tops, axis=2)[:, :, np.diff(high.reshape(S // run, run)[:, 0].astype(int)) == (-1 if up is False else 1)]
    assert jump.size and ((jump < -130).all() if up is False else (jump > 130).all())
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


# 14 blocks (two of them shared by two waves each), 16, 9 (one shared), 8, a split of 27, and the narrow kernels
@pytest.mark.parametrize("dtype,dh,group,Tq", [("bf16", 64, 7, 64), ("bf16", 128, 8, 64), ("f32", 64, 9, 32), ("bf16", 64, 4, 64), ("bf16", 64, 27, 32),
                                               ("bf16", 64, 1, 20), ("f32", 32, 2, 32)])
@pytest.mark.parametrize("at", [5, 100, 1030, 1330])                  # the first keys of a workgroup, later ones, among them of a second subtile
def test_keys_that_are_not_finite_on_long_ranges(dtype, dh, group, Tq, at):
    """A key with a NaN has a NaN score, one whose logits are +inf an infinite one; the rows of their kv heads, whose normalisers they
    spoil, add nothing to the other keys.  A key whose logits are -inf gets no probability and leaves the rest alone."""
    B = mk()
    rng = np.random.default_rng(dh + Tq + group)
    H, S = KV_HEADS, 2048
    n = S - Tq
    q = np.abs(rng.standard_normal((H * group, Tq, dh))).astype(np.float32) + np.float32(0.1)
    k = (0.2 * rng.standard_normal((H, S, dh))).astype(np.float32)
    if dtype == "bf16":
        q, k = synth.bf16_round(q), synth.bf16_round(k)
    bad = k.copy()
    bad[1, at, 3], bad[2, at + 40, 5], bad[3, at + 70, 5] = np.nan, -np.inf, np.inf
    hidden = torch.zeros((S, 8), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    out = B.metok_prefill_prune(hidden, 0, n, i32(np.zeros(n)), [n // 2], q_text=synth.to_torch(q, dtype, "cuda"),
                                k_all=synth.to_torch(bad, dtype, "cuda"))
    torch.cuda.synchronize()
    scores = out["scores"].cpu().numpy()
    k[2, at + 40] = np.float32(-1e5)                                  # probability 0 in 64 bits too
    good = [h for h in range(H) if h not in (1, 3)]
    rows = q.reshape(H, group, Tq, dh)[good].reshape(-1, Tq, dh)
    want = O.text_to_visual_attention(rows, k[good], 0, n, 0) * (len(good) / H)
    others = ~np.isin(np.arange(n), (at, at + 70))
    assert np.isnan(scores[at]) and scores[at + 70] == np.inf
    assert_rel(scores[others], want[others], RTOL[dtype], "scores")
