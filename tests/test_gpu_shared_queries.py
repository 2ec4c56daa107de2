"""Narrow attention scores (at most 64 query rows per kv head) whose queries the workgroup shares in LDS, and the kernels beside that line
whose waves load their own: ragged row blocks, ranges with waves that have no keys, against the CPU oracle."""
import numpy as np
import pytest

from tests.test_gpu_stage2 import check_prune, make_layer, run_prune

pytestmark = pytest.mark.gpu


# fragments of 16 rows x 64 bytes: 8, 16 (a row block with one row), 8 (one row missing), 16, 32, 8; not shared: 4 (one row block), 4, 2
@pytest.mark.parametrize("dtype,dh,Tq", [("bf16", 128, 17), ("bf16", 128, 33), ("bf16", 64, 63), ("f32", 128, 18), ("f32", 128, 64), ("f32", 32, 35),
                                         ("bf16", 128, 16), ("bf16", 32, 64), ("bf16", 32, 17)])
@pytest.mark.parametrize("tokens,vis_start", [(70, 0), (900, 13)])
def test_against_the_oracle(dtype, dh, Tq, tokens, vis_start):
    layer = make_layer(7300 + dh + Tq, 10, tokens // 10, 4, Tq + 3, 16, 6, 6, dh, dtype, vis_start=vis_start)
    seg = np.zeros(layer.n_vis, dtype=np.int32)
    quotas = [layer.n_vis // 2]
    got, q = run_prune(layer, seg, quotas, Tq=Tq)
    check_prune(layer, seg, quotas, got, q)
