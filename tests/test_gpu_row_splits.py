"""Attention scores on key ranges around the length up to which the query rows of a kv head are split over more workgroups, so
that every wave has one block of rows, against the CPU oracle: row counts of one and several whole-row workgroups, the last
length on the split side and the first on the other, a batch, a split that does not fit the workspace, and what follows the scores
of a split in the workspace.  Every test asserts the plan that it is about."""
import numpy as np
import pytest
import torch

from paper_2506_02850_amd import synth
from tests.score_plan import score_plans
from tests.test_gpu_stage2 import check_prune, i32, make_layer, mk, run_prune
from tests.test_gpu_stage2_batched import layers_of, run_batched

pytestmark = pytest.mark.gpu

KV_HEADS = 32                                                         # share the 256 workgroup slots, 8 workgroups along the keys


# Blocks of 32 rows: 9 (5 + 4), 14 (7 + 7), 16 (8 + 8), and 17 (two whole workgroups of 9 and 8, split 6 + 6 + 5, the last block partly
# empty).  LINE: the last length of the split side, five 32-key subtiles a workgroup (with more than 64 KB of partial statistics
# the line lies at eight).
@pytest.mark.parametrize("dtype,dh,group,Tq,line", [("bf16", 64, 9, 32, 1280), ("bf16", 128, 7, 64, 1280), ("f32", 32, 16, 32, 1280), ("bf16", 32, 13, 40, 640)])
@pytest.mark.parametrize("place,mode", [("short", 0), ("last", 0), ("past", 0), ("last", 1)])
def test_scores_around_the_row_split(dtype, dh, group, Tq, line, place, mode):
    keys = {"short": 200, "last": line, "past": line + 1}[place]
    tokens = keys - Tq if mode == 0 else keys                         # the softmax runs over the whole sequence, or the tokens alone
    assert score_plans(tokens + Tq, tokens, KV_HEADS * group, KV_HEADS, dh, Tq, dtype, mode=mode).split == (place != "past")
    check_level(make_layer(5600 + dh + group, 1, tokens, 1, Tq, 16, KV_HEADS * group, KV_HEADS, dh, dtype), Tq, mode)


def check_level(layer, Tq, mode=0):
    seg = np.zeros(layer.n_vis, dtype=np.int32)
    quotas = [layer.n_vis // 2]
    got, q = run_prune(layer, seg, quotas, Tq=Tq, score_mode=mode)
    check_prune(layer, seg, quotas, got, q, score_mode=mode)


def test_rows_stay_whole_where_the_split_does_not_fit_the_workspace():
    Tq, group, tokens = 32, 9, 58
    plans = score_plans(tokens + Tq, tokens, KV_HEADS * group, KV_HEADS, 64, Tq)
    assert not plans.split and plans.plan.per1 <= 5
    check_level(make_layer(5650, 1, tokens, 1, Tq, 16, KV_HEADS * group, KV_HEADS, 64, "bf16"), Tq)


# what lies behind the column sums of a split: the general selection's state, the source rows of the in-place compaction
@pytest.mark.parametrize("in_place", [True, False])
@pytest.mark.parametrize("classes", [1, 17])
@pytest.mark.parametrize("batch", [0, 3])
def test_selection_and_compaction_behind_a_split(batch, classes, in_place):
    B = mk()
    Tq, group, dh, tokens, D = 64, 7, 64, 900, 64
    Hq, S = KV_HEADS * group // 4, tokens + Tq
    assert score_plans(S, tokens, Hq, KV_HEADS // 4, dh, Tq, batch=max(batch, 1)).split
    layers = [make_layer(5950 + b, 10, tokens // 10, 4, Tq, D, Hq, KV_HEADS // 4, dh, "bf16") for b in range(max(batch, 1))]
    seg = (np.arange(tokens) % classes).astype(np.int32)
    quotas = [[int((seg == c).sum()) // 2 - (b + c) % 3 for c in range(classes)] for b in range(len(layers))]
    join = (lambda get: torch.stack([get(l) for l in layers])) if batch else (lambda get: get(layers[0]))
    hidden = join(lambda l: synth.to_torch(l.hidden, "bf16", "cuda"))
    kw = dict(q_text=join(lambda l: synth.to_torch(l.q_text, "bf16", "cuda")), k_all=join(lambda l: synth.to_torch(l.k_all, "bf16", "cuda")),
              token_event=join(lambda l: i32(l.token_event)), event_weight=join(lambda l: torch.from_numpy(l.event_weight).cuda()))
    segs = join(lambda l: i32(seg))
    if batch:
        out = B.metok_prefill_prune_batched(hidden, 0, tokens, segs, quotas, hidden_out=hidden if in_place else None, **kw)
    else:
        rows = S - tokens + sum(quotas[0])
        out = B.metok_prefill_prune(hidden, 0, tokens, segs, quotas[0], hidden_out=hidden[:rows] if in_place else None, **kw)
    torch.cuda.synchronize()
    for b, layer in enumerate(layers):
        kept = sum(quotas[b])
        got = {}
        for name, t in out.items():
            if isinstance(t, torch.Tensor):
                t = (t[b] if batch else t).float() if t.dtype == torch.bfloat16 else (t[b] if batch else t)
                got[name] = t.cpu().numpy()[:tokens if name == "scores" else S - tokens + kept if name == "hidden_out" else kept]
        check_prune(layer, seg, quotas[b], got, layer.q_text)


@pytest.mark.parametrize("keys", [640, 641])                          # two videos share the slots
def test_batch_around_the_row_split(keys):
    Tq = 64
    assert score_plans(keys, keys - Tq, KV_HEADS * 7, KV_HEADS, 64, Tq, batch=2).split == (keys == 640)
    layers = layers_of([5700, 5800], 1, keys - Tq, 1, Tq, 16, KV_HEADS * 7, KV_HEADS, 64, "bf16")
    segs = [np.zeros(l.n_vis, dtype=np.int32) for l in layers]
    quotas = [[layers[0].n_vis // 2], [layers[1].n_vis // 3]]
    for b, (got, q) in enumerate(run_batched(layers, segs, quotas)):
        check_prune(layers[b], segs[b], quotas[b], got, q)


@pytest.mark.parametrize("keys", [8192, 8193])                        # 8 kv heads, 32 workgroups of eight subtiles along the keys
def test_scores_around_the_row_split_with_many_partials(keys):
    # 14 blocks x 32 partials, 112 KB: beyond 64 KB rows are split up to eight subtiles a workgroup instead of five
    Tq, Hkv = 32, 8
    plans = score_plans(keys, keys - Tq, 14 * Hkv, Hkv, 64, Tq)
    assert plans.split == (keys == 8192) and plans.whole.partials > 65536
    layer = make_layer(5900, 1, keys - Tq, 1, Tq, 16, 14 * Hkv, Hkv, 64, "bf16")
    check_level(layer, Tq)
