"""The default prefill tiles over fp8 KV multiply the query as bf16: its
elements count whatever else their row holds.

Each row of every head has one element far above the others, in a dimension
where all keys are zero, so the scores come from the small elements alone. The
sum of 128 exact products in fp32 is off by at most 2^-16 of the sum of their
magnitudes (128 terms, 2^-24 each, and a factor of two), here at most 2^-7 in
the exponent, and bf16 rounds probabilities and outputs by 2^-9: 2 % of the
largest value covers them. A query that keeps only what lies within 2^-22 of its
row's largest magnitude misses it by far."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import attention as oa  # noqa: E402
from synth.attn_inputs import make_batch_from_lengths  # noqa: E402
from tests.gpu_util import say  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("tile_path", [0, 1])
@pytest.mark.parametrize("log2_large", [0, 12, 20, 24])
@pytest.mark.parametrize("hq,hkv", [(4, 4), (16, 2)])
def test_small_elements_beside_a_large_one(hq, hkv, log2_large, tile_path):
    from paper_2512_04013_amd import runtime as rt
    say(f"[tile scores] {hq}/{hkv} heads, one element 2^{log2_large}, tile path {tile_path}")
    b = make_batch_from_lengths("tilescores", [2, 33, 130], [2, 40, 200], num_q_heads=hq, num_kv_heads=hkv, head_dim=128,
                                q_dtype="bf16", kv_dtype="fp8", out_dtype="bf16", n_pool_blocks=32, seed=7, kv_std=1.0)
    q = (b.q.astype(np.uint32) << 16).view(np.float32).copy()
    q[:, :, 77] = np.float32(2.0 ** log2_large)
    b.q = (q.view(np.uint32) >> 16).astype(np.uint16)
    b.k_cache = b.k_cache.copy()
    b.k_cache[..., 77] = 0
    shape, kv, q_dev, bids = rt.upload_batch(b, staging_bytes=1)
    att = rt.MixedAttention(shape, kv, b.q_start, b.ctx_len, b.bt_start, b.block_ids, bids, tile_path=tile_path)
    assert att.info.num_prefill_items == att.info.num_items
    out = att.run(q_dev)
    torch.cuda.synchronize()
    want = oa.attention_for(b)
    err = np.abs(rt.to_host_f64(out) - want).max() / np.abs(want).max()
    assert err < 0.02, err
