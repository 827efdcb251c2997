"""The end of a row item: lane groups, then waves, then spans merged, for every
combination of head_dim, group size and KV dtype (they differ in lanes per
token row, in heads per lane after each exchange, and in dims per thread).
Contexts of one key, of one block and one key, of fewer blocks than waves
(waves and lane groups without any key) and of several spans."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import attention as oa  # noqa: E402
from synth.attn_inputs import make_batch_from_lengths  # noqa: E402
from tests.gpu_util import compare, say  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

KINDS = [(d, g, dt) for d in (64, 128) for g in (1, 2, 4, 8) for dt in ("f32", "bf16", "fp8")
         if not (dt == "fp8" and d == 64)]


@pytest.mark.parametrize("d,g,dt", KINDS)
def test_row_items_merge_lanes_waves_and_spans(d, g, dt):
    from paper_2512_04013_amd import runtime as rt
    qd = "f32" if dt == "f32" else "bf16"
    ctx = [1, 2, 15, 17, 49, 64, 130, 700]
    b = make_batch_from_lengths("merge", [1] * len(ctx), ctx, num_q_heads=2 * g, num_kv_heads=2, head_dim=d,
                                q_dtype=qd, kv_dtype=dt, out_dtype=qd, n_pool_blocks=128, seed=31, kv_std=1.0)
    want = oa.attention_for(b)
    shape, kv, q, bids = rt.upload_batch(b, staging_bytes=1)
    for row_path in ((1, 2) if d == 128 and g >= 4 and dt != "f32" else (0,)):
        for split in (0, 32):
            say(f"[row merge] d={d} g={g} {dt} split={split} row path {row_path}")
            att = rt.MixedAttention(shape, kv, b.q_start, b.ctx_len, b.bt_start, b.block_ids, bids,
                                    kv_split_tokens=split, row_path=row_path)
            got = rt.to_host_f64(att.run(q))
            torch.cuda.synchronize()
            assert np.isfinite(got).all()
            compare(got, want, qd, what=f"row merge d={d} g={g} {dt} split={split}")
