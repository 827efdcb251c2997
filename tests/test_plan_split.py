"""The planner's own split of row items: every key of every row is read by
exactly one span of each KV head whatever split the launch estimate picks, the
partial slots are distinct, equal batches give equal images, and a batch that
fitted the library's scratch array under the split by size still does."""

import numpy as np
import pytest

import paper_2512_04013_amd as aug

SHAPES = [(4, 4, 64, "f32"), (8, 2, 128, "f32"), (16, 8, 64, "bf16"), (32, 8, 128, "bf16"), (64, 8, 128, "bf16"),
          (32, 8, 128, "fp8"), (64, 8, 128, "fp8")]


def _plan(shape, q_len, ctx, **kw):
    q_start = np.concatenate([[0], np.cumsum(q_len)])
    bt = np.concatenate([[0], np.cumsum([-(-c // 16) for c in ctx])])
    info, plan = aug.aug_attn_plan(shape, q_start, ctx, bt, int(bt[-1]), **kw)
    return info, plan, q_start


@pytest.mark.parametrize("seed", range(21))
def test_spans_partition_every_row(seed):
    rng = np.random.default_rng(seed)
    hq, hkv, d, kv = SHAPES[seed % len(SHAPES)]
    qd = "f32" if kv == "f32" else "bf16"
    shape = aug.make_shape(hq, hkv, d, qd, kv, qd, 0.1)
    n = int(rng.choice([1, 2, 5, 17, 60, 300]))
    ctx = np.clip(np.exp(rng.uniform(0, np.log(12000), n)), 1, None).astype(int)
    q_len = np.where(rng.random(n) < 0.2, np.minimum(ctx, rng.integers(1, 40, n)), 1)
    info, plan, q_start = _plan(shape, q_len, ctx)
    again = _plan(shape, q_len, ctx)[1]
    assert np.array_equal(plan, again)
    raw = plan[64:64 + 48 * info.num_items].reshape(-1, 48)
    i32, i16 = raw.view(np.int32).reshape(-1, 12), raw.view(np.int16).reshape(-1, 24)
    row = raw[:, 2] == 0
    parts = i32[row, 7]
    assert len(set(parts[parts >= 0])) == (parts >= 0).sum()
    spans = {}
    for item, kvh in zip(i32[row], i16[row, 0]):
        spans.setdefault((int(item[1]), int(kvh)), []).append((int(item[3]), int(item[4])))
    for r in range(n):
        if q_len[r] > 1 and kv != "f32":
            continue                                     # tiles
        for j in range(q_len[r]):
            for h in range(hkv):
                got = sorted(spans.pop((int(q_start[r]) + j, h)))
                ends = [e for _, e in got]
                assert got[0][0] == 0 and ends[-1] == ctx[r] - q_len[r] + j + 1
                assert [b for b, _ in got[1:]] == ends[:-1] and all(b % 16 == 0 and b < e for b, e in got)
    assert not spans


def test_scratch_limit_is_kept():
    """Prefill tiles whose partials alone nearly fill the library's scratch
    array: the row items beside them take no split that would exceed it."""
    shape = aug.make_shape(64, 8, 128, "bf16", "fp8", "bf16", 0.1)
    seen = 0
    for chunks in range(1, 24):
        for rows in (16, 40, 100):
            q_len, ctx = [rows] * chunks + [1] * 6, [9000] * chunks + [20000] * 6
            info, _, _ = _plan(shape, q_len, ctx)
            nominal, _, _ = _plan(shape, q_len, ctx, kv_split_tokens=info.kv_split_tokens)
            if nominal.workspace_bytes <= aug.NOALLOC_SCRATCH_BYTES:
                assert info.workspace_bytes <= aug.NOALLOC_SCRATCH_BYTES
                seen += info.workspace_bytes > aug.NOALLOC_SCRATCH_BYTES // 2
    assert seen


def test_cut_of_many_items():
    """A launch of 2048 items and more keeps the split by size, one of fewer may
    be cut otherwise, a requested split is taken as given. The benchmark reports
    the cut."""
    from bench import longest_row_item
    shape = aug.make_shape(32, 8, 128, "bf16", "bf16", "bf16", 0.1)
    rng = np.random.default_rng(0)
    ctx = np.clip(rng.lognormal(np.log(1400), 0.8, 256), 1, 16384).astype(int)
    info, plan, _ = _plan(shape, [1] * 256, ctx)
    assert info.num_items >= 2048 and longest_row_item(plan, info) <= info.kv_split_tokens
    few, plan, _ = _plan(shape, [1] * 20, [2000] * 20)
    assert longest_row_item(plan, few) > few.kv_split_tokens
    asked, plan, _ = _plan(shape, [1] * 20, [2000] * 20, kv_split_tokens=few.kv_split_tokens)
    assert longest_row_item(plan, asked) <= asked.kv_split_tokens == few.kv_split_tokens


@pytest.mark.parametrize("layer", SHAPES + [(8, 8, 64, "bf16"), (16, 2, 64, "bf16"), (8, 8, 128, "fp8")])
def test_merges_are_priced(layer):
    """One decode is not cut into spans whose merge outlasts their streaming
    (8000 keys: 10.7 us in 16 spans, 17.5 in 63), nor a short one cut at all
    where a wave reads it in a few blocks (300 keys, eight heads on MFMA)."""
    hq, hkv, d, kv = layer
    qd = "f32" if kv == "f32" else "bf16"
    shape = aug.make_shape(hq, hkv, d, qd, kv, qd, 0.1)
    slow = kv == "f32" and d == 128 and hq > hkv      # few heads' blocks at a time: more spans pay
    for ctx, most in ((8000, 48 if slow else 40), (60000, 120 if slow else 64)):
        info, _, _ = _plan(shape, [1], [ctx])
        assert 4 <= info.num_items // hkv <= most
    info, _, _ = _plan(shape, [1], [100])
    assert info.num_items == hkv
    if hq == 8 * hkv and d == 128:
        assert _plan(shape, [1], [300])[0].num_items == hkv


def test_plain_batch_descriptions_are_taken():
    """The C calls take a description itself, by reference or by pointer, and
    refuse anything else in its place."""
    C, lib = aug.C, aug.lib()
    shape = aug.make_shape(8, 2, 128, "bf16", "bf16", "bf16", 0.1)
    arrays = [np.array(a, np.int32) for a in ([0, 1, 2], [40, 700], [0, 3, 47])]
    desc = aug.aug_batch_desc(2, *(a.ctypes.data_as(C.POINTER(C.c_int32)) for a in arrays), None, 64)
    want, _ = aug.aug_attn_plan(shape, *arrays, 64)
    for d in (desc, C.byref(desc), C.pointer(desc)):
        info, n = aug.aug_attn_plan_info(), C.c_size_t()
        assert lib.aug_attn_plan(shape, d, 0, None, 0, C.byref(info)) == aug.AUG_OK
        assert bytes(info) == bytes(want)
        assert lib.aug_attn_plan_opts(shape, d, aug.aug_plan_options(0, 0, 0), None, 0, C.byref(info)) == aug.AUG_OK
        assert lib.aug_attn_workspace_size(shape, d, 0, C.byref(n)) == aug.AUG_OK and n.value == want.workspace_bytes
    for d in (shape, C.byref(shape), C.addressof(desc)):
        with pytest.raises(C.ArgumentError):
            lib.aug_attn_plan(shape, d, 0, None, 0, C.byref(aug.aug_attn_plan_info()))
