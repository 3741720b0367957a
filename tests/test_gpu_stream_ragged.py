"""Batches of decode steps whose contexts differ in length, one launch of the streaming kernel: every item's result is
that of its own call in one split, and the time is one that follows the bytes (workgroups of items with fewer splits that had nothing to do put two of the
others on one compute unit: 4 queries took longer than 8)."""
import pytest
import torch

from paper_2605_03644_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ad():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding
    binding.load_library()
    return binding


def _lens(n, nq):
    return [int(n * (0.9 + 0.2 * ((7 * i) % 11) / 11)) for i in range(nq)]


def _batch(ad, hq, hkv, d, dtype, lens):
    td = torch.float32 if dtype == ad.F32 else torch.bfloat16
    rnd = lambda i, *s: wl.normal_tensor(s, td, "cuda", i)  # noqa: E731
    ctx = ad.Context(1, hq, hkv, d, 1.0e4, dtype, max_position=1 << 16)
    k, v = rnd(1, max(lens), hkv, d), rnd(2, max(lens), hkv, d)
    caches = [ad.Cache(ctx, max(n, 1), with_index=False) for n in lens]
    for c, n in zip(caches, lens):
        c.k[0, :n].copy_(k[:n])
        c.v[0, :n].copy_(v[:n])
        c.c.len = n
    q, ks, vs = rnd(3, len(lens), 1, hq, d), rnd(4, len(lens), 1, hkv, d), rnd(5, len(lens), 1, hkv, d)
    out = torch.empty_like(q)
    items = ctx.pack_attn_items([(i, n, q[i], ks[i], vs[i], n, out[i]) for i, n in enumerate(lens)])
    ctx.keep = (k, v, q, ks, vs)
    return ctx, caches, items, out


@pytest.mark.parametrize("hq,hkv,d,f32", [(28, 4, 128, False), (32, 8, 64, False), (8, 2, 128, True), (3, 3, 8, True)])
@pytest.mark.parametrize("lens", [[0, 700], [65, 1, 0, 640], _lens(800, 32), [1, 2000, 63, 64], [0] * 5 + [129], _lens(300, 33)])
@pytest.mark.parametrize("splits", [0, 3, 64])
def test_items_of_different_lengths(ad, hq, hkv, d, f32, lens, splits):
    ctx, caches, items, out = _batch(ad, hq, hkv, d, ad.F32 if f32 else ad.BF16, lens)
    ctx.set_attn_splits(splits)
    ctx.query_attn_batched(caches, 0, items)
    torch.cuda.synchronize()
    _, _, q, ks, vs = ctx.keep
    tol = 1e-5 if f32 else 2.0 ** -7   # of a bf16 result two roundings, and weights of 16 bits
    for i, n in enumerate(lens):
        ctx.set_attn_splits(1)
        one = ctx.query_attn(caches[i], 0, n, q[i], ks[i], vs[i], n)
        torch.cuda.synchronize()
        assert float((out[i].float() - one.float()).norm()) <= tol * float(one.float().norm()), i


def test_four_queries_take_no_longer_than_eight(ad):
    us = []
    for nq in (4, 8):
        ctx, caches, items, _ = _batch(ad, 28, 4, 128, ad.BF16, _lens(8000, nq))
        for rep in range(2):
            ctx.profile_enable(True)
            for _ in range(20):
                ctx.query_attn_batched(caches, 0, items)
            torch.cuda.synchronize()
            each = sorted(ctx.profile_read_each()["query_attn"])
            ctx.profile_enable(False)
        us.append(1e3 * float(each[len(each) // 2]))
        ctx.close()
    print("us:", us)
    assert us[0] < us[1]
