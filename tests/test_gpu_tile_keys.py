"""Prefill tiles over fp8 KV with queries of every magnitude, and pools at an
offset that the direct loads to LDS do not take.

A query rounded to one code misses the bf16 gate on these sharp keys (0.1 of an
output)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import attention as oa  # noqa: E402
from synth.attn_inputs import make_batch_from_lengths  # noqa: E402
from tests.gpu_util import compare, say  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _batch(kv, hq, hkv, seed):
    # tile edges: one row short of and past a 128-row tile, chunks that end inside a block, a lone block
    return make_batch_from_lengths(f"tilekeys{seed}", [128 * hkv // hq + 1, 2, 33, 16], [700, 63, 33, 1040], num_q_heads=hq,
                                   num_kv_heads=hkv, head_dim=128, q_dtype="bf16", kv_dtype=kv, out_dtype="bf16",
                                   n_pool_blocks=256, seed=seed, kv_std=1.0)


def _run(b, split, offset=0):
    from paper_2512_04013_amd import runtime as rt
    shape, kv, q, bids = rt.upload_batch(b, staging_bytes=1 << 24)
    if offset:
        def moved(x):
            buf = torch.empty(x.numel() * x.element_size() + 16, dtype=torch.uint8, device=x.device)
            part = buf[offset:offset + x.numel() * x.element_size()].view(x.dtype).view(x.shape)
            part.copy_(x)
            return part
        kv = rt.PagedKV(shape, moved(kv.k_cache), moved(kv.v_cache), kv.k_scale, kv.v_scale, staging_bytes=1 << 24)
        assert kv.k_cache.data_ptr() % 16 == offset
    att = rt.MixedAttention(shape, kv, b.q_start, b.ctx_len, b.bt_start, b.block_ids, bids, kv_split_tokens=split)
    assert att.info.num_prefill_items > 0
    out = att.run(q)
    torch.cuda.synchronize()
    return rt.to_host_f64(out)


@pytest.mark.parametrize("hq,hkv", [(4, 4), (8, 4), (16, 4), (32, 4)])
def test_queries_of_every_range(hq, hkv):
    b = _batch("fp8", hq, hkv, 60 + hq)
    say(f"[tile keys] fp8 G={hq // hkv}")
    rng = np.random.default_rng(hq)
    q = (b.q.astype(np.uint32) << 16).view(np.float32).copy()
    q *= np.exp2(rng.integers(-20, 1, q.shape)).astype(np.float32) * 4        # elements of one row 2^20 apart
    q[1] *= np.float32(2.0 ** -90)                                           # rows far below the scale's clamp, and zero
    q[3] *= np.float32(2.0 ** -118)
    q[5, 0] = 0
    q[7, 0] = 0
    q[7, 0, 5] = np.float32(2.0 ** 6)                                        # a lone large element
    b.q = (q.view(np.uint32) >> 16).astype(np.uint16)
    for split in (0, 48):
        compare(_run(b, split), oa.attention_for(b), "bf16", what=f"G={hq // hkv} split={split}")


@pytest.mark.parametrize("kv", ["fp8", "bf16"])
def test_pools_at_an_odd_offset(kv):
    b = _batch(kv, 32, 8, 91)
    say(f"[tile keys] {kv}, pools 8 bytes into an allocation")
    got = _run(b, 48, offset=8)
    compare(got, oa.attention_for(b), "bf16", what=f"{kv} offset pools")
    assert np.array_equal(got, _run(b, 48))
