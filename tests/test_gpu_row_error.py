"""Decode rows of four heads per KV head over fp8 KV: the default path is no
further from float64 than the vector rows, down to contexts of a few keys."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("ctx", [1, 2, 5, 16, 17, 64, 250, 1500])
@pytest.mark.parametrize("sharp", [1.0, 6.0])
@pytest.mark.parametrize("chunk", [False, True])
def test_error_against_float64(ctx, sharp, chunk):
    import paper_2512_04013_amd as aug
    from paper_2512_04013_amd import runtime as rt
    from tests.gpu_util import say
    say(f"[row error] ctx={ctx} sharp={sharp} chunk={chunk}")
    n, hq, hkv, d = 48, 32, 8, 128
    nblk = -(-ctx // 16)
    # beside a prefill chunk the rows run on four waves, alone on eight
    q_len, lens = [1] * n + [2] * chunk, [ctx] * n + [16] * chunk
    bt = np.concatenate([[0], np.cumsum([-(-c // 16) for c in lens])]).astype(np.int32)
    pool = int(bt[-1])
    g = torch.Generator(device="cuda").manual_seed(ctx)
    k, v = (torch.randn(pool, hkv, 16, d, generator=g, device="cuda").mul_(80).clamp_(-448, 448).to(torch.float8_e4m3fn)
            for _ in range(2))
    ks, vs = (torch.rand(pool, hkv, generator=g, device="cuda") * 0.003 + 0.011 for _ in range(2))
    shape = aug.make_shape(hq, hkv, d, "bf16", "fp8", "bf16", d ** -0.5)
    kv = rt.PagedKV(shape, k.view(torch.uint8), v.view(torch.uint8), ks, vs, staging_bytes=1)
    ids = torch.randperm(pool, generator=g, device="cuda").to(torch.int32)
    q_start = np.concatenate([[0], np.cumsum(q_len)]).astype(np.int32)
    q = (torch.randn(int(q_start[-1]), hq, d, generator=g, device="cuda") * sharp).bfloat16()
    rows = ids.cpu().numpy()[:n * nblk].reshape(n, nblk)
    err = {}
    for path in (aug.AUG_ROWS_AUTO, aug.AUG_ROWS_VALU):
        att = rt.MixedAttention(shape, kv, q_start, np.array(lens, np.int32), bt, ids.cpu().numpy(), ids, row_path=path)
        out = att.run(q)[:n].double()
        torch.cuda.synchronize()
        num = den = floor = 0.0
        for r in range(n):
            b = torch.from_numpy(rows[r]).cuda().long()
            kk, vv = ((c[b].double() * s[b][:, :, None, None].double()).permute(1, 0, 2, 3).reshape(hkv, -1, d)[:, :ctx]
                      for c, s in ((k, ks), (v, vs)))
            p = torch.softmax(torch.bmm(q[r].double().reshape(hkv, hq // hkv, d), kk.transpose(1, 2).contiguous()) * d ** -0.5, -1)
            want = torch.bmm(p, vv.contiguous()).reshape(hq, d)
            num += float((out[r] - want).square().sum())
            floor += float((want.bfloat16().double() - want).square().sum())
            den += float(want.square().sum())
        err[path] = (num / den) ** 0.5
    floor = (floor / den) ** 0.5
    # the rounding of the output, and its draw (196608 values: 0.2 % of the root
    # mean square) beside probabilities good to 2^-17 and float32 sums
    assert err[aug.AUG_ROWS_AUTO] <= 1.01 * floor + 2.0 ** -16
    assert err[aug.AUG_ROWS_AUTO] <= err[aug.AUG_ROWS_VALU] * 1.01
