"""fp32 attention scores of 65 to 256 query rows per kv head on more than a few keys, whose products are taken on three bf16 parts of
every element: against the CPU oracle, with jumps beyond the range of float, against the error of fp32 products, and with elements that are
large or not finite (fp32 products)."""
import numpy as np
import pytest
import torch

from oracle import metok_oracle as O
from paper_2506_02850_amd import synth
from tests.parity import assert_rel
from tests.score_plan import score_plans
from tests.test_gpu_shared_row_blocks import KV_HEADS, check_scores_of_jumps
from tests.test_gpu_stage2 import check_prune, i32, make_layer, mk, run_prune

pytestmark = pytest.mark.gpu


def takes_parts(S, n_vis, Hq, Hkv, dh, Tq, vis_start=0, mode=0):
    plan = score_plans(S, n_vis, Hq, Hkv, dh, Tq, dtype="f32", vis_start=vis_start, mode=mode).plan
    return 2 < plan.rbw <= 8 and (plan.per1 >= 2 if plan.rbw > 4 else plan.per1 * dh // 8 >= 96)


# row blocks of a workgroup: 3 (the last one ragged), 4, 5, 7, 8, and 7 + 7 split rows; the last stage of a range is ragged
@pytest.mark.parametrize("dh,group,Tq", [(128, 3, 31), (128, 2, 64), (32, 5, 30), (64, 7, 32), (128, 4, 64), (128, 7, 64)])
@pytest.mark.parametrize("tokens,vis_start,mode", [(1960, 7, 0), (2500, 0, 1)])
def test_against_the_oracle(dh, group, Tq, tokens, vis_start, mode):
    layer = make_layer(6100 + dh + group, 10, tokens // 10, 4, Tq + 3, 16, KV_HEADS * group, KV_HEADS, dh, "f32", vis_start=vis_start)
    assert takes_parts(layer.n_vis + vis_start + Tq + 3, layer.n_vis, KV_HEADS * group, KV_HEADS, dh, Tq, vis_start, mode)
    seg = np.zeros(layer.n_vis, dtype=np.int32)
    quotas = [layer.n_vis // 2]
    got, q = run_prune(layer, seg, quotas, Tq=Tq, score_mode=mode)
    check_prune(layer, seg, quotas, got, q, score_mode=mode)


@pytest.mark.parametrize("low", [32, 96, 224])
def test_jumps_beyond_the_range_of_float(low):
    S = 2048
    check_scores_of_jumps("f32", 64, 7, 32, S, np.arange(S) % 256 >= low, 32, None)


def run_scores(q, k, n):
    """Scores of the n keys before the text, and in 64 bits."""
    hidden = torch.zeros((k.shape[1], 8), device="cuda")
    out = mk().metok_prefill_prune(hidden, 0, n, i32(np.zeros(n)), [n // 2], q_text=synth.to_torch(q, "f32", "cuda"), k_all=synth.to_torch(k, "f32", "cuda"))
    return out["scores"].cpu().numpy().astype(np.float64)


# nonzero elements of a query row; ones: the lower halves of all words are ones, whose parts cut off are furthest from their products
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("nonzero,ones", [(1, False), (1, True), (2, False), (4, True), (8, False), (64, False), (64, True)])
def test_error_is_that_of_fp32_products(dh, nonzero, ones):
    """A key of probability 0 in every subtile is -1e5 for parts and -inf for fp32 products; all other scores are of the same numbers, with
    logits of some ten to a hundred, so that the error of the logits is what a score is off."""
    rng = np.random.default_rng(29 + nonzero)
    Hkv, group, Tq, n = 4, 7, 32, 5000
    assert takes_parts(n + Tq, n, Hkv * group, Hkv, dh, Tq)
    q = np.full((Hkv * group, Tq, dh), 1e-30, dtype=np.float32)                  # not 0: -inf stays -inf
    at = np.argsort(rng.random(q.shape), axis=2)[:, :, :nonzero]
    np.put_along_axis(q, at, (100 / nonzero * rng.uniform(1, 4, at.shape)).astype(np.float32), axis=2)
    k = (rng.uniform(1, 2, (Hkv, n + Tq, dh)) * np.sqrt(dh / 64)).astype(np.float32)
    if ones:
        q, k = (q.view(np.uint32) | 0xffff).view(np.float32), (k.view(np.uint32) | 0xffff).view(np.float32)
    k[:, ::32] = -1e5
    want = O.text_to_visual_attention(q, k, 0, n, 0)
    bad = k.copy()
    bad[:, ::32] = -np.inf
    parts, products = run_scores(q, k, n), run_scores(q, bad, n)
    seen = want > 1e-12 * want.max()
    assert (parts[:n:32] == 0).all() and (products[:n:32] == 0).all() and seen.sum() > 500
    rms = lambda got: float(np.sqrt(np.mean((got[seen] / want[seen] - 1) ** 2)))
    # the products that are left out, 0.29 x 2^-24 rms, make one rounding (0.43 x 2^-24) 1.2 of it; parts that are cut off 1.5
    assert rms(parts) <= 1.2 * rms(products)


@pytest.mark.parametrize("big", [2.0 ** 59, 3.4e38])
def test_large_elements(big):
    """An element near the largest, whose nearest bf16 number is infinite, against queries that are tiny there."""
    rng = np.random.default_rng(31)
    Hkv, group, dh, Tq, n = 4, 7, 64, 32, 5000
    q = rng.standard_normal((Hkv * group, Tq, dh)).astype(np.float32)
    k = rng.standard_normal((Hkv, n + Tq, dh)).astype(np.float32)
    q[:, :, 11] = np.float32(2.0 ** -120)
    k[:, :, 11] = 0
    k[1, 77, 11], k[1, 4001, 11], k[2, 3000, 11] = big, -big, big
    assert_rel(run_scores(q, k, n), O.text_to_visual_attention(q, k, 0, n, 0), 1e-5, "scores")
    big_q = q.copy()
    big_q[3, 5, 11], big_q[8, 6, 11] = big, -big                        # against keys that are 0 there
    k[:, :, 11] = 0
    assert_rel(run_scores(big_q, k, n), O.text_to_visual_attention(big_q, k, 0, n, 0), 1e-5, "scores")


def test_elements_that_are_not_finite():
    """A NaN (whose only mantissa bit is the last one) spoils its key and its kv head's rows; -inf in a key, against positive queries, is
    probability 0."""
    rng = np.random.default_rng(17)
    Hkv, group, dh, Tq, n = 4, 7, 64, 32, 5000
    S = n + Tq
    assert takes_parts(S, n, Hkv * group, Hkv, dh, Tq)
    q = np.abs(rng.standard_normal((Hkv * group, Tq, dh))).astype(np.float32) + np.float32(0.1)
    k = (0.2 * rng.standard_normal((Hkv, S, dh))).astype(np.float32)
    bad = k.copy()
    bad[1, 50, 3] = np.array([0x7f800001], dtype=np.uint32).view(np.float32)[0]
    bad[2, 70, 5] = bad[2, 4000, 60] = -np.inf
    scores = run_scores(q, bad, n)
    fixed = k.copy()
    fixed[2, 70] = fixed[2, 4000] = np.float32(-1e5)
    want = sum(O.text_to_visual_attention(q[h * group:(h + 1) * group], fixed[h:h + 1], 0, n, 0) for h in (0, 2, 3)) / Hkv
    others = np.arange(n) != 50
    assert np.isnan(scores[50])
    assert_rel(scores[others], want[others], 1e-5, "scores")


@pytest.mark.parametrize("dh,value", [(64, np.inf), (64, -np.inf), (128, np.inf)])
def test_an_infinite_query_element(dh, value):
    """The logits of its row are infinite with the sign of the key's element: keys of +inf have an infinite score, for the others the
    row adds nothing."""
    rng = np.random.default_rng(19)
    Hkv, group, Tq, n = 4, 7, 32, 5000
    Hq, S = Hkv * group, n + Tq
    assert takes_parts(S, n, Hq, Hkv, dh, Tq)
    q, k = rng.standard_normal((Hq, Tq, dh)).astype(np.float32), rng.standard_normal((Hkv, S, dh)).astype(np.float32)
    want = O.text_to_visual_attention(q, k, 0, n, 0) - O.text_to_visual_attention(q[:1, 9:10], k[:1, :n + 10], 0, n, 0) / (Hq * Tq)
    q[0, 9, 2] = value
    got = run_scores(q, k, n)
    up = k[0, :n, 2] * np.sign(value) > 0
    assert (got[up] == np.inf).all()
    assert_rel(got[~up], want[~up], 1e-5, "scores")


def test_a_query_element_that_is_no_number():
    """A NaN whose only mantissa bit is the last one, which a bf16 number does not have, in a query: its row is NaN for every key."""
    rng = np.random.default_rng(23)
    Hkv, group, dh, Tq, n = 4, 7, 64, 32, 5000
    assert takes_parts(n + Tq, n, Hkv * group, Hkv, dh, Tq)
    q, k = rng.standard_normal((Hkv * group, Tq, dh)).astype(np.float32), rng.standard_normal((Hkv, n + Tq, dh)).astype(np.float32)
    assert np.isfinite(run_scores(q, k, n)).all()
    q[3, 30, 63] = np.array([0x7f800001], dtype=np.uint32).view(np.float32)[0]
    assert np.isnan(run_scores(q, k, n)).all()
