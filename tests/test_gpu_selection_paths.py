"""The one-launch selection (at most 16 classes, at most 40960 tokens) and its neighbours, against the CPU oracle: sizes at
the edges of its tiles and of its register variants, scores that need more than one digit, more ties than its candidate
list holds, tokens without a class, quotas above a class's population, and the metadata the row mover carries.  All
results are integers or copied rows: every comparison is exact."""
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
