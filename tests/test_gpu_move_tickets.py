"""The row mover's tiles are drawn from one, two or four counters, by the number of slabs of a (layer, video): bit-exact against the
oracle with many tiles per slab, whose stores wait for earlier tiles of the same counter."""
import numpy as np
import pytest

from tests.test_gpu_stage3 import adversarial_sets, run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,heads,videos", [(6, 2, 2), (6, 4, 1), (6, 5, 2), (43, 2, 1)])      # 43 layers: two launches
def test_counters_of_a_launch(layers, heads, videos):
    S = 700                                                       # rows of 2 KB: tiles of 64 rows
    sets = adversarial_sets(S)
    names = ["stride2", "shift_by_one", "random_half", "prefix_then_tail", "all_tail", "random_eighth"]
    idx = [np.stack([sets[names[l % 6]].astype(np.int32)] * videos) for l in range(layers)]
    run_and_check(layers, videos, heads, S, 1024, "bf16", idx)
