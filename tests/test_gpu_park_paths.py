"""Park and resume through staging and the copy engine against the direct
kernels: the same bytes, for record counts on both sides of the size at which
the direct path ends, for host buffers the kernels cannot take (not 16-byte
aligned, or not pinned) and for every KV dtype. A direct transfer leaves the
staging buffer alone, so the buffer's bytes tell which path ran."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import kvpark  # noqa: E402
from synth.attn_inputs import make_batch_from_lengths  # noqa: E402
from tests.gpu_util import say  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _host(kind, nbytes):
    if kind == "pageable":
        return torch.empty(nbytes, dtype=torch.uint8)
    if kind == "misaligned":
        return torch.empty(nbytes + 16, dtype=torch.uint8, pin_memory=True)[8:8 + nbytes]
    return torch.empty(nbytes, dtype=torch.uint8, pin_memory=True)


def _moved_directly(pool, move):
    pool.staging.fill_(0xA5)
    move()
    torch.cuda.synchronize()
    return bool((pool.staging == 0xA5).all())


@pytest.mark.parametrize("kv,hkv,d", [("f32", 1, 64), ("bf16", 1, 64), ("fp8", 1, 128), ("f32", 8, 64), ("bf16", 8, 128), ("fp8", 8, 128)])
@pytest.mark.parametrize("kind", ["pinned", "misaligned", "pageable"])
@pytest.mark.parametrize("staging_records", [1, 3, 1000])
def test_every_path_moves_the_same_bytes(kv, hkv, d, kind, staging_records):
    from paper_2512_04013_amd import runtime as rt
    qd = "f32" if kv == "f32" else "bf16"
    b = make_batch_from_lengths("park", [1], [100], num_q_heads=2 * hkv, num_kv_heads=hkv, head_dim=d, q_dtype=qd, kv_dtype=kv,
                                out_dtype=qd, n_pool_blocks=48, seed=3, extra_reqs_ctx=[90, 33])
    shape, pool, _, _ = rt.upload_batch(b, staging_bytes=1)
    pool.staging = torch.empty(staging_records * pool.record_bytes, dtype=torch.uint8, device="cuda")
    src = b.park.park_blocks
    used = set(b.block_ids.tolist()) | set(src.tolist())
    dst = np.array(sorted(set(range(48)) - used)[:len(src)], np.int32)
    host = _host(kind, len(src) * pool.record_bytes)
    say(f"[park paths] {kv} {kind} staging={staging_records}")
    src_dev, dst_dev = torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda()
    assert _moved_directly(pool, lambda: pool.park(src, src_dev, host)) == (kind == "pinned")
    assert np.array_equal(host.numpy(), kvpark.park(b.k_cache, b.v_cache, b.k_scale, b.v_scale, kv, src))
    assert _moved_directly(pool, lambda: pool.resume(dst, dst_dev, host)) == (kind == "pinned")
    for t in (pool.k_cache, pool.v_cache, pool.k_scale, pool.v_scale):
        if t is not None:
            raw = t.contiguous().view(torch.uint8).reshape(48, -1).cpu().numpy()
            assert np.array_equal(raw[dst], raw[src])


@pytest.mark.parametrize("blocks", [127, 128, 129, 200])
def test_around_the_direct_limit(blocks):
    """64 KiB records: 128 of them are the largest image that goes direct."""
    from paper_2512_04013_amd import make_shape
    from paper_2512_04013_amd import runtime as rt
    say(f"[park limit] {blocks} blocks")
    g = torch.Generator(device="cuda").manual_seed(blocks)
    k = torch.randn(512, 8, 16, 128, generator=g, device="cuda").bfloat16()
    v = torch.randn(512, 8, 16, 128, generator=g, device="cuda").bfloat16()
    pool = rt.PagedKV(make_shape(32, 8, 128, "bf16", "bf16", "bf16", 0.1), k, v, staging_bytes=50 * 65536)
    ids = torch.randperm(512, generator=g, device="cuda").to(torch.int32)
    src, dst = ids[:blocks].contiguous(), ids[256:256 + blocks].contiguous()
    host = pool.host_buffer(blocks)
    want_k, want_v = k[src.long()].clone(), v[src.long()].clone()
    src_host, dst_host = src.cpu().numpy(), dst.cpu().numpy()
    assert _moved_directly(pool, lambda: pool.park(src_host, src, host)) == (blocks <= 128)
    rec = host.view(torch.bfloat16).reshape(blocks, 2, 8, 16, 128)
    assert torch.equal(rec[:, 0], want_k.cpu()) and torch.equal(rec[:, 1], want_v.cpu())
    assert _moved_directly(pool, lambda: pool.resume(dst_host, dst, host)) == (blocks <= 128)
    assert torch.equal(k[dst.long()], want_k) and torch.equal(v[dst.long()], want_v)
