"""The planner's flag for K/V loads that leave the caches alone, and that it
changes no bit of a result."""

import numpy as np
import pytest

import paper_2512_04013_amd as aug

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


@pytest.mark.gpu
@pytest.mark.parametrize("d,g,kv,row_path", [(64, 1, "f32", 0), (128, 2, "f32", 0), (64, 4, "bf16", 0), (128, 1, "bf16", 0),
                                             (128, 4, "bf16", 1), (128, 4, "bf16", 2), (128, 8, "bf16", 2),
                                             (128, 2, "fp8", 0), (128, 4, "fp8", 2), (128, 8, "fp8", 2)])
def test_flag_changes_no_bit(d, g, kv, row_path):
    torch = pytest.importorskip("torch")
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
