"""Decode steps of bf16 / head_dim 128 models (at most 16 query rows per kv head) through the streaming kernel, and the
border to the tile kernel: row counts, contexts that end inside a 32-key step, batches of ragged contexts and of more
problems than one launch takes, items that share a cache, contexts beyond the streaming kernel's share."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2605_03644_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
BAR = dict(max_abs=2e-2, rel_fro=1e-2)  # the bf16 bar of every attention test: query, weights and output rounded to bf16


@pytest.fixture(scope="module")
def ad():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding
    binding.load_library()
    return binding


def _model(hq, hkv):
    return dataclasses.replace(wl.WORKLOADS["tiny_fp32"], name=f"decode_{hq}_{hkv}", n_q_heads=hq, n_kv_heads=hkv, head_dim=128,
                               dtype="bf16", rope_theta=5.0e5)


def _random(w, seed, *shape):
    return wl.normal_tensor(shape, w.torch_dtype, "cuda", seed)


def _cache(ad, ctx, w, n, seed):
    c = ad.Cache(ctx, max(n, 1), with_index=False)
    c.k.copy_(_random(w, seed, *c.k.shape))
    c.v.copy_(_random(w, seed + 1, *c.v.shape))
    c.c.len = n
    return c


def _check(oracle_mod, w, c, n, q, ks, vs, pos, out):
    ref = oracle_mod.query_attn(H.to_storage(c.k[0]), H.to_storage(c.v[0]), "bf16", n, H.to_storage(q), H.to_storage(ks),
                                H.to_storage(vs), w.rope_theta, pos)
    H.check_attention(out.float().cpu().numpy(), ref, **BAR)


@pytest.mark.parametrize("hq,hkv,t_q", [(7, 1, 1), (28, 4, 2), (16, 2, 2), (4, 4, 16), (4, 4, 17)])
@pytest.mark.parametrize("n_ctx,splits", [(0, 0), (1, 0), (31, 1), (32, 0), (33, 2), (64, 0), (4161, 0), (4161, 64), (2000, 7)])
def test_decode_edges(ad, oracle_mod, hq, hkv, t_q, n_ctx, splits):
    w = _model(hq, hkv)
    ctx = ad.Context.for_workload(w, max_position=1 << 14)
    c = _cache(ad, ctx, w, n_ctx, 11 + n_ctx)
    q, ks, vs = _random(w, 5, t_q, hq, 128), _random(w, 6, t_q, hkv, 128), _random(w, 7, t_q, hkv, 128)
    ctx.set_attn_splits(splits)
    out = ctx.query_attn(c, 0, n_ctx, q, ks, vs, n_ctx + 3)
    again = ctx.query_attn(c, 0, n_ctx, q, ks, vs, n_ctx + 3)
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    _check(oracle_mod, w, c, n_ctx, q, ks, vs, n_ctx + 3, out)
    ctx.close()


def test_decode_ragged_batch(ad, oracle_mod):
    """35 caches of very different lengths, an empty one among them, in one call."""
    w = _model(8, 2)
    ctx = ad.Context.for_workload(w, max_position=1 << 14)
    lens = [0, 1, 5000, 64, 777] + [int(x) for x in np.random.default_rng(4).integers(1, 900, 30)]
    caches = [_cache(ad, ctx, w, n, 50 + 2 * i) for i, n in enumerate(lens)]
    items = []
    for i, c in enumerate(caches):
        q, ks, vs = _random(w, 500 + 3 * i, 1, 8, 128), _random(w, 501 + 3 * i, 1, 2, 128), _random(w, 502 + 3 * i, 1, 2, 128)
        items.append((i, c.len, q, ks, vs, c.len, torch.empty_like(q)))
    ctx.query_attn_batched(caches, 0, items)
    torch.cuda.synchronize()
    for (i, n, q, ks, vs, pos, out) in items:
        _check(oracle_mod, w, caches[i], n, q, ks, vs, pos, out)
    # the same item twice: the cache is shared, which is the tile kernel's case
    two = [items[2][:6] + (torch.empty_like(items[2][2]),), items[2][:6] + (torch.empty_like(items[2][2]),)]
    ctx.query_attn_batched(caches, 0, two)
    torch.cuda.synchronize()
    assert torch.equal(two[0][6], two[1][6])
    # the two kernels round P and the partials differently; relative to the output, as everywhere, so that a split that is
    # left out is seen (1/79 of 5000 keys: 0.11)
    H.check_attention(two[0][6].float().cpu().numpy(), items[2][6].double().cpu().numpy(), **BAR)
    ctx.close()


def test_decode_beyond_the_streaming_share(ad):
    """Contexts on either side of the border between the two kernels (200 MB), each against a float32 reference.  The bar is
    relative to the output (means over 49k keys are small): one of 64 splits left out would be 0.12 of it."""
    w = _model(32, 8)
    n = 49152   # 201 MB
    ctx = ad.Context.for_workload(w, max_position=1 << 17)
    c = _cache(ad, ctx, w, n, 9)
    q, ks, vs = _random(w, 5, 1, 32, 128), _random(w, 6, 1, 8, 128), _random(w, 7, 1, 8, 128)
    outs = []
    for m, merges in ((n, 1), (n - 512, 0)):           # the tile kernel has a merge of its own
        ctx.profile_enable(True)
        outs.append(ctx.query_attn(c, 0, m, q, ks, vs, n).float())
        torch.cuda.synchronize()
        prof = ctx.profile_read()
        ctx.profile_enable(False)
        assert (prof["query_attn"][1], prof["attn_combine"][1]) == (1, merges)
    kf, vf = c.k[0].float(), c.v[0].float()
    for m, out in zip((n, n - 512), outs):
        got = out[0].view(8, 4, 128)
        # reference in float32 torch over the same cache: the query row rotated to position n, its own key as well
        inv = w.rope_theta ** (-torch.arange(0, 64, dtype=torch.float64, device="cuda") / 64.0) * n
        cs, sn = torch.cos(inv).float(), torch.sin(inv).float()
        rot = lambda x: torch.cat([x[..., :64] * cs - x[..., 64:] * sn, x[..., 64:] * cs + x[..., :64] * sn], -1)  # noqa: E731
        qr, kr = rot(q[0].float()).view(8, 4, 128), rot(ks[0].float())
        for hk in range(8):
            keys, vals = torch.cat([kf[:m, hk], kr[hk:hk + 1]]), torch.cat([vf[:m, hk], vs[0].float()[hk:hk + 1]])
            p = torch.softmax(qr[hk] @ keys.T / 128.0 ** 0.5, dim=-1)
            H.check_attention(got[hk].cpu().numpy(), (p @ vals).double().cpu().numpy(), **BAR)
    ctx.close()
