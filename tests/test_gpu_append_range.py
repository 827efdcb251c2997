"""fp8 append at the ends of its division's range: block scales inside and
outside the span in which a quotient comes from the reciprocal, quotients on
ties and among the subnormal codes, and a NaN. Every byte as the oracle's."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from oracle import kvappend  # noqa: E402
from synth.attn_inputs import make_batch_from_lengths  # noqa: E402
from tests.gpu_util import say  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("log2_scale,spread", [(0, 0), (0, 14), (-52, 6), (-58, 6), (-90, 6), (50, 6), (80, 6)])
def test_every_scale_range(log2_scale, spread):
    from paper_2512_04013_amd import runtime as rt
    say(f"[append range] rows around 2^{log2_scale}, elements 2^{spread} apart")
    # whole blocks, blocks begun by an earlier step (whose scale grows or is kept), single rows
    b = make_batch_from_lengths("appendrange", [40, 16, 1, 1, 3], [45, 16, 8, 17, 35], num_q_heads=16, num_kv_heads=2, head_dim=128,
                                q_dtype="bf16", kv_dtype="fp8", out_dtype="bf16", n_pool_blocks=32, seed=5)
    b = synth.poison_new_slots(b)
    rng = np.random.default_rng(100 + log2_scale + spread)
    new = []
    for _ in range(2):
        x = rng.standard_normal((61, 2, 128)).astype(np.float32)
        if spread == 0:
            x = rng.integers(-448, 449, x.shape).astype(np.float32)      # the scale is 1 where 448 is drawn: ties
            x[:, :, 0] = 448.0
        x *= np.exp2(log2_scale + rng.integers(-spread, 1, x.shape)).astype(np.float32)
        new.append((x.view(np.uint32) >> 16).astype(np.uint16))
    k_new, v_new = new
    want = kvappend.append(b.k_cache, b.v_cache, b.k_scale, b.v_scale, "fp8", k_new, v_new, b.q_start, b.ctx_len, b.bt_start, b.block_ids)
    shape, kv, _, bids = rt.upload_batch(b)
    att = rt.MixedAttention(shape, kv, b.q_start, b.ctx_len, b.bt_start, b.block_ids, bids)
    att.append(rt.to_device_array(k_new, "bf16", "cuda"), rt.to_device_array(v_new, "bf16", "cuda"))
    torch.cuda.synchronize()
    for name, got, ref in zip(("k_cache", "v_cache", "k_scale", "v_scale"), (kv.k_cache, kv.v_cache, kv.k_scale, kv.v_scale), want):
        g = got.contiguous().view(torch.uint8).cpu().numpy().reshape(-1)
        assert np.count_nonzero(g != np.ascontiguousarray(ref).view(np.uint8).reshape(-1)) == 0, name


def test_a_nan_saturates_and_counts_for_nothing():
    from paper_2512_04013_amd import runtime as rt
    say("[append range] NaN")
    b = make_batch_from_lengths("appendnan", [16], [16], num_q_heads=16, num_kv_heads=2, head_dim=128,
                                q_dtype="bf16", kv_dtype="fp8", out_dtype="bf16", n_pool_blocks=4, seed=5)
    k_new, v_new = synth.make_new_kv(b, seed=2)
    k_new[3, 1, 7] = 0
    want = kvappend.append(b.k_cache, b.v_cache, b.k_scale, b.v_scale, "fp8", k_new, v_new, b.q_start, b.ctx_len, b.bt_start, b.block_ids)
    for bits, code in ((0x7FC0, 0x7E), (0xFFC0, 0xFE)):
        k_new[3, 1, 7] = bits
        shape, kv, _, bids = rt.upload_batch(b)
        att = rt.MixedAttention(shape, kv, b.q_start, b.ctx_len, b.bt_start, b.block_ids, bids)
        att.append(rt.to_device_array(k_new, "bf16", "cuda"), rt.to_device_array(v_new, "bf16", "cuda"))
        ref = np.ascontiguousarray(want[0]).view(np.uint8).reshape(-1, 2, 16, 128).copy()
        ref[int(b.block_ids[0]), 1, 3, 7] = code
        got = kv.k_cache.contiguous().view(torch.uint8).cpu().numpy().reshape(ref.shape)
        assert np.array_equal(got, ref)
