"""Which row path the planner resolves AUTO to: MFMA for groups of eight over
bf16 or fp8 KV and groups of four over fp8 KV (head_dim 128), the vector ALUs
for every other shape."""

import numpy as np
import pytest

import paper_2512_04013_amd as aug


@pytest.mark.parametrize("kv", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("g", [1, 2, 4, 8])
def test_auto_row_path(kv, d, g):
    if kv == "fp8" and d == 64:
        pytest.skip("fp8 KV needs head_dim 128")
    qd = "f32" if kv == "f32" else "bf16"
    shape = aug.make_shape(2 * g, 2, d, qd, kv, qd, 0.1)
    ctx = np.array([700, 3000, 17])
    bt = np.concatenate([[0], np.cumsum(-(-ctx // 16))])
    info, plan = aug.aug_attn_plan(shape, [0, 1, 2, 3], ctx, bt, int(bt[-1]))
    mfma = d == 128 and ((g == 8 and kv != "f32") or (g == 4 and kv == "fp8"))
    assert info.row_path == (aug.AUG_ROWS_MFMA if mfma else aug.AUG_ROWS_VALU) == plan[61]
