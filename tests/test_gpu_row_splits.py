"""Attention scores on key ranges around the length up to which the query rows of a kv head are split over more workgroups, so
that every wave has one block of rows, against the CPU oracle: row counts of one and several whole-row workgroups, the last
length on the split side and the first on the other, and a batch."""
import numpy as np
import pytest

from tests.test_gpu_stage2 import check_prune, make_layer, run_prune
from tests.test_gpu_stage2_batched import layers_of, run_batched

pytestmark = pytest.mark.gpu

# 32 kv heads share the 256 workgroup slots, 8 workgroups along the keys: five 32-key subtiles each are 1280 keys (so few partial
# statistics that pass 2 merges them: with more of them the line lies at eight)
KV_HEADS, LINE = 32, 1280


# 9, 14 and 16 blocks of 32 rows (5 + 4, 7 + 7, 8 + 8), 17 (6 + 6 + 5, with the last block partly empty)
@pytest.mark.parametrize("dtype,dh,group,Tq", [("bf16", 64, 9, 32), ("bf16", 128, 7, 64), ("f32", 32, 16, 32), ("bf16", 32, 13, 40)])
@pytest.mark.parametrize("keys,mode", [(90, 0), (LINE, 0), (LINE + 1, 0), (LINE, 1)])
def test_scores_around_the_row_split(dtype, dh, group, Tq, keys, mode):
    tokens = keys - Tq if mode == 0 else keys                         # the softmax runs over the whole sequence, or the tokens alone
    layer = make_layer(5600 + dh + group, 1, tokens, 1, Tq, 16, KV_HEADS * group, KV_HEADS, dh, dtype)
    seg = np.zeros(layer.n_vis, dtype=np.int32)
    quotas = [layer.n_vis // 2]
    got, q = run_prune(layer, seg, quotas, Tq=Tq, score_mode=mode)
    check_prune(layer, seg, quotas, got, q, score_mode=mode)


@pytest.mark.parametrize("keys", [LINE // 2, LINE // 2 + 1])          # two videos share the slots
def test_batch_around_the_row_split(keys):
    Tq = 64
    layers = layers_of([5700, 5800], 1, keys - Tq, 1, Tq, 16, KV_HEADS * 7, KV_HEADS, 64, "bf16")
    segs = [np.zeros(l.n_vis, dtype=np.int32) for l in layers]
    quotas = [[layers[0].n_vis // 2], [layers[1].n_vis // 3]]
    for b, (got, q) in enumerate(run_batched(layers, segs, quotas)):
        check_prune(layers[b], segs[b], quotas[b], got, q)


@pytest.mark.parametrize("keys", [8192, 8193])                        # 8 kv heads, 32 workgroups of eight subtiles along the keys
def test_scores_around_the_row_split_with_many_partials(keys):
    # 9 blocks x 32 partials are more than pass 2 merges for itself
    Tq, Hkv = 32, 8
    layer = make_layer(5900, 1, keys - Tq, 1, Tq, 16, 9 * Hkv, Hkv, 64, "bf16")
    seg = np.zeros(layer.n_vis, dtype=np.int32)
    quotas = [layer.n_vis // 2]
    got, q = run_prune(layer, seg, quotas, Tq=Tq)
    check_prune(layer, seg, quotas, got, q)
