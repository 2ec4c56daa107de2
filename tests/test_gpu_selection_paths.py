"""The one-launch selection (at most 16 classes; at most 40960 tokens, one video of 5 to 16 classes 22528) and its neighbours,
against the CPU oracle: sizes at the edges of its tiles and of its register variants, scores that need more than one digit,
more ties than its candidate list holds, scores that are not finite, tokens without a class, quotas above a class's
population, and the metadata the row mover carries.  All results are integers or copied rows: every comparison is exact."""
import numpy as np
import pytest
import torch

from oracle import metok_oracle as O
from tests.test_gpu_stage2 import i32, mk

pytestmark = pytest.mark.gpu


def scores_of(kind, n, rng):
    if kind == "spread":                       # like attention: all positive, within a few octaves
        return np.exp(rng.standard_normal(n)).astype(np.float32) / n
    if kind == "outlier":                      # one huge value: nearly all keys share the first digit
        x = (1.0 + 1e-6 * rng.integers(0, 4000, size=n)).astype(np.float32)
        x[rng.integers(0, n)] = 3e38
        x[rng.integers(0, n)] = -3e38
        return x
    if kind == "ties":                         # a handful of values: thousands of keys equal the threshold
        return rng.integers(-2, 3, size=n).astype(np.float32)
    return np.full(n, -0.5, dtype=np.float32)  # "equal"


@pytest.mark.parametrize("n,n_seg", [(1, 1), (63, 2), (65, 4), (1023, 5), (1025, 16), (4096, 2), (4097, 16), (12288, 4), (12289, 1),
                                     (20481, 3), (40960, 16), (40961, 16), (5000, 17)])
@pytest.mark.parametrize("kind", ["spread", "outlier", "ties", "equal"])
@pytest.mark.parametrize("in_place", [False, True])
def test_selection_and_carried_metadata(n, n_seg, kind, in_place):
    B = mk()
    rng = np.random.default_rng(n + n_seg)
    D, prefix, text = 8, 3, 5
    scores = scores_of(kind, n, rng)
    seg = rng.integers(0, n_seg, size=n).astype(np.int32)
    event = rng.integers(0, 40, size=n).astype(np.int32)
    orig = rng.permutation(3 * n)[:n].astype(np.int32)
    quotas = [int(rng.integers(0, int((seg == c).sum()) + 1)) for c in range(n_seg)]
    hidden = rng.standard_normal((prefix + n + text, D)).astype(np.float32)
    dev = torch.from_numpy(hidden).cuda()
    rows = prefix + text + sum(quotas)
    out = B.metok_prefill_prune(dev, prefix, n, i32(seg), quotas, scores=torch.from_numpy(scores).cuda(), token_event=i32(event),
                                orig_idx=i32(orig), hidden_out=dev[:rows] if in_place else None)
    torch.cuda.synchronize()
    kept = O.segmented_topk(scores, seg, quotas)
    np.testing.assert_array_equal(out["kept_idx"].cpu().numpy(), kept)
    np.testing.assert_array_equal(out["hidden_out"].cpu().numpy(), O.compact_hidden(hidden, prefix, n, kept))
    np.testing.assert_array_equal(out["token_seg_out"].cpu().numpy(), seg[kept])
    np.testing.assert_array_equal(out["token_event_out"].cpu().numpy(), event[kept])
    np.testing.assert_array_equal(out["orig_idx_out"].cpu().numpy(), orig[kept])


@pytest.mark.parametrize("n_seg", [2, 17])
def test_tokens_without_a_class_and_quotas_above_the_population(n_seg):
    # both selection paths: such tokens are never kept, and the list is padded with index 0 and zero metadata
    B = mk()
    rng = np.random.default_rng(n_seg)
    n = 3000
    scores = rng.standard_normal(n).astype(np.float32)
    seg = rng.integers(0, 2, size=n).astype(np.int32)
    seg[rng.random(n) < 0.2] = -1
    seg[rng.random(n) < 0.2] = n_seg
    event = np.full(n, 9, dtype=np.int32)
    pop = [int((seg == c).sum()) for c in (0, 1)]
    quotas = [pop[0] + 11, pop[1] // 2] + [0] * (n_seg - 2)
    hidden = rng.standard_normal((n, 4)).astype(np.float32)
    out = B.metok_prefill_prune(torch.from_numpy(hidden).cuda(), 0, n, i32(seg), quotas, scores=torch.from_numpy(scores).cuda(),
                                token_event=i32(event))
    torch.cuda.synchronize()
    second = np.nonzero(seg == 1)[0]
    order = second[np.lexsort((second, -scores[second].astype(np.float64)))]
    kept = np.sort(np.concatenate([np.nonzero(seg == 0)[0], order[:quotas[1]]]))
    want = np.concatenate([kept, np.zeros(11, dtype=kept.dtype)])
    real = np.arange(want.size) < kept.size
    np.testing.assert_array_equal(out["kept_idx"].cpu().numpy(), want)
    np.testing.assert_array_equal(out["hidden_out"].cpu().numpy(), hidden[want])
    np.testing.assert_array_equal(out["token_seg_out"].cpu().numpy(), np.where(real, seg[want], 0))
    np.testing.assert_array_equal(out["token_event_out"].cpu().numpy(), np.where(real, 9, 0))
    np.testing.assert_array_equal(out["orig_idx_out"].cpu().numpy(), want)


def test_supplied_scores_of_a_batch_keep_each_video_apart():
    B = mk()
    rng = np.random.default_rng(77)
    batch, n = 5, 9000
    scores = np.stack([scores_of(kind, n, rng) for kind in ("spread", "outlier", "ties", "equal", "spread")])
    seg = rng.integers(0, 6, size=(batch, n)).astype(np.int32)
    quotas = [[int(rng.integers(0, int((seg[b] == c).sum()) + 1)) for c in range(6)] for b in range(batch)]
    hidden = rng.standard_normal((batch, n, 4)).astype(np.float32)
    out = B.metok_prefill_prune_batched(torch.from_numpy(hidden).cuda(), 0, n, i32(seg), quotas, scores=torch.from_numpy(scores).cuda())
    torch.cuda.synchronize()
    for b in range(batch):
        kept = O.segmented_topk(scores[b], seg[b], quotas[b])
        np.testing.assert_array_equal(out["kept_idx"][b, :len(kept)].cpu().numpy(), kept)
        np.testing.assert_array_equal(out["token_seg_out"][b, :len(kept)].cpu().numpy(), seg[b][kept])
        np.testing.assert_array_equal(out["hidden_out"][b, :len(kept)].cpu().numpy(), hidden[b][kept])


def ordered_key(scores):
    """The order of the selection on bit patterns: an unsigned integer that grows with the score (-0 like +0, NaN with the
    sign bit below -inf, without it above +inf, the further the larger the payload)."""
    u = scores.view(np.uint32).copy()
    u[u == 0x80000000] = 0
    return np.where(u & 0x80000000, ~u, u | 0x80000000).astype(np.int64)


# bit patterns: the two NaN at the ends of the order, other NaN, the infinities, the largest and smallest finite values,
# denormals and both zeros
PATTERNS = np.array([0xffffffff, 0x7fffffff, 0xffc00000, 0x7fc00000, 0xff800000, 0x7f800000, 0xff7fffff, 0x7f7fffff,
                     0x80000001, 0x00000001, 0x80000000, 0x00000000, 0xbf800000, 0x3f800000], dtype=np.uint32)


@pytest.mark.parametrize("n_seg", [1, 3, 16, 17])                      # the one-launch selection with either digit width; the general path
@pytest.mark.parametrize("n,top", [(700, 40), (3000, 1500), (13000, 6000)])      # candidates ranked in the list; more equal keys than it holds
@pytest.mark.parametrize("batch", [1, 3])
def test_nan_and_infinite_scores_keep_the_order_of_their_bits(n_seg, n, top, batch):
    # Integers throughout: exactly quota tokens per class, by (key descending, index ascending).  `top` tokens hold the
    # largest key there is, and the quota of class 0 lies inside them, so that the threshold is that key.
    B = mk()
    rng = np.random.default_rng(n + n_seg)
    bits = PATTERNS[rng.integers(0, len(PATTERNS), size=(batch, n))]
    seg = rng.integers(0, n_seg, size=(batch, n)).astype(np.int32)
    for b in range(batch):
        own = rng.permutation(n)[:top]
        bits[b, own], seg[b, own] = 0x7fffffff, 0
        rest = np.setdiff1d(np.arange(n), own)
        bits[b, rest[bits[b, rest] == 0x7fffffff]] = 0xffffffff
    scores = bits.view(np.float32)
    quotas = [[top // 2] + [int(rng.integers(0, int((seg[b] == c).sum()) + 1)) for c in range(1, n_seg)] for b in range(batch)]
    if n_seg > 2:
        for q in quotas:
            q[2] = 0                                                  # a class that keeps nothing beside one whose threshold is the largest key
    hidden = torch.zeros((batch, n, 4), device="cuda")
    if batch == 1:
        out = B.metok_prefill_prune(hidden[0], 0, n, i32(seg[0]), quotas[0], scores=torch.from_numpy(scores[0]).cuda())
        got = [out["kept_idx"].cpu().numpy()]
    else:
        out = B.metok_prefill_prune_batched(hidden, 0, n, i32(seg), quotas, scores=torch.from_numpy(scores).cuda())
        got = [out["kept_idx"][b, :sum(quotas[b])].cpu().numpy() for b in range(batch)]
    for b in range(batch):
        key = ordered_key(scores[b])
        want = []
        for c in range(n_seg):
            members = np.nonzero(seg[b] == c)[0]
            want.append(members[np.lexsort((members, -key[members]))][:quotas[b][c]])
        np.testing.assert_array_equal(got[b], np.sort(np.concatenate(want)), err_msg=f"video {b}")


@pytest.mark.parametrize("batch,n,n_seg", [(1, 22528, 16), (1, 22529, 16), (1, 22529, 4), (2, 40960, 16), (2, 40961, 5), (2, 3000, 17)])
@pytest.mark.parametrize("kind", ["spread", "ties"])
def test_both_sides_of_the_line_between_the_two_selections(batch, n, n_seg, kind):
    B = mk()
    rng = np.random.default_rng(n + n_seg)
    scores = np.stack([scores_of(kind, n, rng) for _ in range(batch)])
    seg = rng.integers(0, n_seg, size=(batch, n)).astype(np.int32)
    quotas = [[int(rng.integers(0, int((seg[b] == c).sum()) + 1)) for c in range(n_seg)] for b in range(batch)]
    hidden = rng.standard_normal((batch, n + 1, 4)).astype(np.float32)
    dev = torch.from_numpy(hidden).cuda()
    if batch == 1:
        out = B.metok_prefill_prune(dev[0], 1, n, i32(seg[0]), quotas[0], scores=torch.from_numpy(scores[0]).cuda())
        out = {name: t[None] for name, t in out.items()}
    else:
        out = B.metok_prefill_prune_batched(dev, 1, n, i32(seg), quotas, scores=torch.from_numpy(scores).cuda())
    torch.cuda.synchronize()
    for b in range(batch):
        kept = O.segmented_topk(scores[b], seg[b], quotas[b])
        np.testing.assert_array_equal(out["kept_idx"][b, :len(kept)].cpu().numpy(), kept)
        np.testing.assert_array_equal(out["token_seg_out"][b, :len(kept)].cpu().numpy(), seg[b][kept])
        np.testing.assert_array_equal(out["hidden_out"][b, :1 + len(kept)].cpu().numpy(), O.compact_hidden(hidden[b], 1, n, kept))
