"""Attention scores whose partial statistics are more than pass 2 merges for itself, so that a kernel between the passes does: one and two row
blocks a wave, the products of bf16 parts, a batch, ragged last blocks, against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import metok_oracle as O
from paper_2506_02850_amd import synth
from tests.parity import RTOL, assert_rel
from tests.score_plan import score_plans
from tests.test_gpu_split_products import takes_parts
from tests.test_gpu_stage2 import i32, mk

pytestmark = pytest.mark.gpu

LINE = 256 * 1024


def scores(q, k, n, dtype, batch=0):
    hidden = torch.zeros((max(batch, 1), k.shape[-2], 8), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    q, k = synth.to_torch(q, dtype, "cuda"), synth.to_torch(k, dtype, "cuda")
    B = mk()
    if batch:
        out = B.metok_prefill_prune_batched(hidden, 0, n, i32(np.zeros((batch, n))), [[n // 2]] * batch, q_text=q, k_all=k)
    else:
        out = B.metok_prefill_prune(hidden[0], 0, n, i32(np.zeros(n)), [n // 2], q_text=q, k_all=k)
    return out["scores"].cpu().numpy()


# one kv head: 256 workgroups along the keys.  Row blocks 8, 8 (ragged), 14 in two blocks a wave; fp32 with one subtile a workgroup, parts, two blocks a wave
@pytest.mark.parametrize("dtype,Hq,Hkv,dh,Tq,n,parts", [
    ("bf16", 8, 1, 64, 32, 4500, False), ("bf16", 15, 1, 256, 17, 4500, False), ("bf16", 14, 2, 64, 64, 33000, False),
    ("f32", 8, 1, 64, 32, 4500, False), ("f32", 8, 1, 64, 32, 9000, True), ("f32", 15, 1, 128, 17, 9100, True), ("f32", 14, 2, 32, 64, 33000, False)])
def test_merged_by_a_kernel(dtype, Hq, Hkv, dh, Tq, n, parts):
    S = n + Tq
    plan = score_plans(S, n, Hq, Hkv, dh, Tq, dtype).plan
    assert plan.partials > LINE and (dtype == "f32" and takes_parts(S, n, Hq, Hkv, dh, Tq)) == parts
    rng = np.random.default_rng(41 + dh + n)
    q, k = rng.standard_normal((Hq, Tq, dh)).astype(np.float32), rng.standard_normal((Hkv, S, dh)).astype(np.float32)
    if dtype == "bf16":
        q, k = synth.bf16_round(q), synth.bf16_round(k)
    assert_rel(scores(q, k, n, dtype), O.text_to_visual_attention(q, k, 0, n, 0), RTOL[dtype], "scores")


def test_merged_by_a_kernel_in_a_batch():
    Hq, Hkv, dh, Tq, n, batch = 16, 1, 64, 32, 24468, 3
    S = n + Tq
    assert score_plans(S, n, Hq, Hkv, dh, Tq, batch=batch).plan.partials > LINE
    rng = np.random.default_rng(43)
    q, k = (synth.bf16_round(rng.standard_normal((batch, h, rows, dh)).astype(np.float32)) for h, rows in ((Hq, Tq), (Hkv, S)))
    got = scores(q, k, n, "bf16", batch)
    for b in range(batch):
        assert_rel(got[b], O.text_to_visual_attention(q[b], k[b], 0, n, 0), RTOL["bf16"], "scores")


@pytest.mark.parametrize("at", [3, 40, 100, 8999])                  # of the first stage and of later ones of a workgroup
def test_keys_that_are_not_finite(at):
    """Parts: logits of -inf are probability 0, a NaN spoils its key and its kv head's rows, which add nothing to other keys."""
    Hq, Hkv, dh, Tq, n = 8, 1, 64, 32, 9000
    assert takes_parts(n + Tq, n, Hq, Hkv, dh, Tq) and score_plans(n + Tq, n, Hq, Hkv, dh, Tq, "f32").plan.partials > LINE
    rng = np.random.default_rng(47)
    q = np.abs(rng.standard_normal((Hq, Tq, dh))).astype(np.float32) + np.float32(0.1)
    k = (0.2 * rng.standard_normal((Hkv, n + Tq, dh))).astype(np.float32)
    low, bad = k.copy(), k.copy()
    low[0, at, 5], bad[0, at, 5] = -np.inf, np.nan
    k[0, at] = np.float32(-1e5)
    assert_rel(scores(q, low, n, "f32"), O.text_to_visual_attention(q, k, 0, n, 0), 1e-5, "scores")
    got = scores(q, bad, n, "f32")
    assert np.isnan(got[at]) and (got[np.arange(n) != at] == 0).all()
