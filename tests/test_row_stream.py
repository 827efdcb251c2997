"""The planner's flag for K/V loads that leave the caches alone, and that it
changes no bit of a result."""

import numpy as np
import pytest

# before the library: both then use torch's HIP runtime
torch = pytest.importorskip("torch")

import paper_2512_04013_amd as aug  # noqa: E402

HEADER, ITEM = 64, 48
STREAM_BYTES = 100_000_000


def _items(info, plan):
    return plan[HEADER:HEADER + ITEM * info.num_items].reshape(-1, ITEM)


@pytest.mark.parametrize("kv,elem", [("bf16", 2), ("fp8", 1), ("f32", 4)])
def test_flag_follows_the_row_bytes(kv, elem):
    """Row items of a launch are flagged from STREAM_BYTES of K/V up (rows
    only: a chunk's keys do not count), tiles never."""
    qd = "f32" if kv == "f32" else "bf16"
    shape = aug.make_shape(8, 8, 128, qd, kv, qd, 0.1)
    per_key = 8 * 128 * elem * 2
    keys = -(-STREAM_BYTES // per_key)
    for total, want in ((keys - 1, 0), (keys, 1)):
        q_len = np.array([2, 1, 1]) if kv != "f32" else np.array([1, 1])
        ctx = [64] * (len(q_len) - 2) + [total // 2, total - total // 2]
        bt = np.concatenate([[0], np.cumsum([-(-c // 16) for c in ctx])])
        info, plan = aug.aug_attn_plan(shape, np.concatenate([[0], np.cumsum(q_len)]), ctx, bt, int(bt[-1]))
        items = _items(info, plan)
        rows = items[items[:, 2] == 0]
        assert len(rows) and (rows[:, 3] == want).all() and not items[items[:, 2] == 1][:, 3].any()


def test_rows_of_one_chunk_are_not_flagged():
    """fp32 chunks become row items that read the same keys once per row: over
    the limit counted so, far under it counted once."""
    shape = aug.make_shape(8, 2, 128, "f32", "f32", "f32", 0.1)
    q_len, ctx = [64] * 16, [576] * 16
    row_bytes = sum(c * (c + 1) // 2 - (c - q) * (c - q + 1) // 2 for q, c in zip(q_len, ctx)) * 2 * 2 * 128 * 4
    assert sum(ctx) * 2 * 2 * 128 * 4 < STREAM_BYTES // 4 and row_bytes > 4 * STREAM_BYTES
    bt = np.concatenate([[0], np.cumsum([c // 16 for c in ctx])])
    info, plan = aug.aug_attn_plan(shape, np.arange(17) * 64, ctx, bt, int(bt[-1]))
    assert not _items(info, plan)[:, 3].any()
    # beside decodes that stream, they still do not
    q_len, ctx = q_len + [1] * 8, ctx + [20000] * 8
    bt = np.concatenate([[0], np.cumsum([-(-c // 16) for c in ctx])])
    info, plan = aug.aug_attn_plan(shape, np.concatenate([[0], np.cumsum(q_len)]), ctx, bt, int(bt[-1]))
    items = _items(info, plan)
    row0 = np.ascontiguousarray(items[:, 4:8]).view(np.int32)[:, 0]
    assert (items[row0 < 1024, 3] == 0).all() and (items[row0 >= 1024, 3] == 1).all()


@pytest.mark.parametrize("shared,want", [(0, 1), (20, 1), (200, 0)])
def test_blocks_shared_by_requests_count_once(shared, want):
    """64 decodes of 220 blocks whose first `shared` blocks are the same pool
    blocks: 14 MB are read over and over where 200 are shared. Without the
    block table the planner cannot know."""
    shape = aug.make_shape(64, 8, 128, "bf16", "fp8", "bf16", 0.1)
    n, nblk = 64, 220
    own = nblk - shared
    ids = np.concatenate([np.concatenate([np.arange(shared), shared + r * own + np.arange(own)]) for r in range(n)])
    args = shape, np.arange(n + 1), [nblk * 16 - 5] * n, np.arange(n + 1) * nblk, n * nblk
    info, plan = aug.aug_attn_plan(*args, block_ids=ids)
    assert (_items(info, plan)[:, 3] == want).all()
    blind, plan = aug.aug_attn_plan(*args)
    assert (_items(blind, plan)[:, 3] == 1).all()
    assert blind.num_items == info.num_items and blind.workspace_bytes == info.workspace_bytes


@pytest.mark.parametrize("hq,hkv,d,kv,elem", [(32, 8, 128, "bf16", 2), (64, 8, 128, "fp8", 1), (8, 2, 128, "f32", 4),
                                              (16, 4, 64, "bf16", 2), (4, 4, 64, "f32", 4)])
@pytest.mark.parametrize("chunks", [0, 2])
def test_large_launches_start_with_ordinary_loads(hq, hkv, d, kv, elem, chunks):
    """From 640 MB of decodes' K/V the items that start the launch read 320 MB
    through the caches and the rest stream; just below, all stream."""
    qd = "f32" if kv == "f32" else "bf16"
    shape = aug.make_shape(hq, hkv, d, qd, kv, qd, 0.1)
    per_key = hkv * d * elem * 2
    for total, prefix in ((640_000_000 // per_key + 1, 320_000_000), (640_000_000 // per_key - 1, 0)):
        n = 40
        ctx = [total // n + (r % 7 - 3) * 50 for r in range(n)]
        ctx[-1] += total - sum(ctx)
        q_len, ctx = [20] * chunks + [1] * n, [300] * chunks + ctx
        q_start = np.concatenate([[0], np.cumsum(q_len)])
        bt = np.concatenate([[0], np.cumsum([-(-c // 16) for c in ctx])])
        info, plan = aug.aug_attn_plan(shape, q_start, ctx, bt, int(bt[-1]))
        items = _items(info, plan)
        i32 = np.ascontiguousarray(items).view(np.int32).reshape(-1, 12)
        decode = (items[:, 2] == 0) & (i32[:, 1] >= q_start[chunks])
        keys = (i32[:, 4] - i32[:, 3])[decode]
        assert keys.sum() == total * hkv and not items[~decode, 3].any()
        before = (np.cumsum(keys) - keys).astype(np.int64) * d * elem * 2
        assert np.array_equal(items[decode, 3] != 0, before >= prefix)


@pytest.mark.gpu
@pytest.mark.parametrize("d,g,kv,row_path", [(64, 1, "f32", 0), (128, 2, "f32", 0), (64, 4, "bf16", 0), (128, 1, "bf16", 0),
                                             (128, 4, "bf16", 1), (128, 4, "bf16", 2), (128, 8, "bf16", 2),
                                             (128, 2, "fp8", 0), (128, 4, "fp8", 2), (128, 8, "fp8", 2)])
def test_flag_changes_no_bit(d, g, kv, row_path):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2512_04013_amd import runtime as rt
    from synth.attn_inputs import make_batch_from_lengths
    qd = "f32" if kv == "f32" else "bf16"
    # no, one, two, an odd and an even number of blocks a wave; a chunk beside them or not
    for q_lens, ctx in (([1] * 6, [1, 16, 80, 97, 300, 700]), ([1, 1, 9, 1], [33, 400, 40, 1000])):
        b = make_batch_from_lengths("stream", q_lens, ctx, num_q_heads=2 * g, num_kv_heads=2, head_dim=d, q_dtype=qd,
                                    kv_dtype=kv, out_dtype=qd, n_pool_blocks=160, seed=5, kv_std=1.0)
        shape, pool, q, bids = rt.upload_batch(b, staging_bytes=1)
        for split in (0, 160):
            att = rt.MixedAttention(shape, pool, b.q_start, b.ctx_len, b.bt_start, b.block_ids, bids,
                                    kv_split_tokens=split, row_path=row_path)
            plain = att.run(q).clone()
            plan = att.plan_host.numpy()
            items = _items(att.info, plan)
            assert not items[:, 3].any()
            items[items[:, 2] == 0, 3] = 1
            att.plan_dev.copy_(torch.from_numpy(plan))
            att.out.zero_()
            assert torch.equal(att.run(q), plain)
