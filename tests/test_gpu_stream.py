"""The streaming attention kernel (every shape beside bf16 / head_dim 128) at the edges of its decomposition: contexts
that end inside a 16-key step or a 64-key split, row counts that end inside a 16-row block, split counts up to the
largest, more problems than one launch takes, gathered contexts."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2605_03644_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu

# fp32: sums of some hundred products of N(0,1) values in another order, 1e-6 of a result of size 1; bf16: the rotated
# query and the output are rounded to bf16 (2^-9 each of a score and of an output of size 1)
BARS = {"f32": dict(max_abs=1e-4, rel_fro=1e-5), "bf16": dict(max_abs=2e-2, rel_fro=1e-2)}


@pytest.fixture(scope="module")
def ad():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding
    binding.load_library()
    return binding


def _model(dtype, d, hq, hkv):
    return dataclasses.replace(wl.WORKLOADS["tiny_fp32"], name=f"stream_{dtype}_{d}", n_q_heads=hq, n_kv_heads=hkv, head_dim=d,
                               dtype=dtype, rope_theta=5.0e5, n_shots=24, len_lo=30, len_hi=70)


def _random(w, seed, *shape):
    return wl.normal_tensor(shape, w.torch_dtype, "cuda", seed)


def _full_cache(ad, ctx, w, n, seed):
    c = ad.Cache(ctx, max(n, 1), with_index=False)
    c.k.copy_(_random(w, seed, *c.k.shape))
    c.v.copy_(_random(w, seed + 1, *c.v.shape))
    c.c.len = n
    return c


def _ref(oracle_mod, w, c, n, q, ks, vs, pos):
    return oracle_mod.query_attn(H.to_storage(c.k[0]), H.to_storage(c.v[0]), w.dtype, n, H.to_storage(q), H.to_storage(ks),
                                 H.to_storage(vs), w.rope_theta, pos)


@pytest.mark.parametrize("dtype,d,hq,hkv", [("f32", 8, 4, 2), ("f32", 16, 2, 2), ("f32", 32, 3, 1), ("f32", 64, 4, 2),
                                            ("f32", 128, 8, 2), ("bf16", 16, 4, 2), ("bf16", 32, 2, 1), ("bf16", 64, 8, 2),
                                            ("bf16", 256, 4, 2)])
@pytest.mark.parametrize("n_ctx,t_q,splits", [(0, 5, 0), (1, 1, 0), (15, 4, 1), (16, 17, 2), (63, 8, 0), (65, 9, 2), (1000, 33, 0),
                                              (1000, 3, 7), (4300, 2, 64)])
def test_stream_edges(ad, oracle_mod, dtype, d, hq, hkv, n_ctx, t_q, splits):
    w = _model(dtype, d, hq, hkv)
    ctx = ad.Context.for_workload(w, max_position=1 << 14)
    c = _full_cache(ad, ctx, w, n_ctx, 11 + n_ctx)
    q, ks, vs = _random(w, 5, t_q, hq, d), _random(w, 6, t_q, hkv, d), _random(w, 7, t_q, hkv, d)
    ctx.set_attn_splits(splits)
    out = ctx.query_attn(c, 0, n_ctx, q, ks, vs, n_ctx + 3)
    again = ctx.query_attn(c, 0, n_ctx, q, ks, vs, n_ctx + 3)   # the arrival counters are back at zero
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    H.check_attention(out.float().cpu().numpy(), _ref(oracle_mod, w, c, n_ctx, q, ks, vs, n_ctx + 3), **BARS[dtype])
    ctx.close()


@pytest.mark.parametrize("t_q", [70, 300])
def test_stream_two_row_blocks(ad, oracle_mod, t_q):
    """bf16 / 64 with enough rows for two 16-row blocks per workgroup (t_q = 300), and just one (t_q = 70)."""
    w = _model("bf16", 64, 32, 8)
    ctx = ad.Context.for_workload(w, max_position=1 << 14)
    for n_ctx in (130, 901):
        c = _full_cache(ad, ctx, w, n_ctx, 3)
        q, ks, vs = _random(w, 5, t_q, 32, 64), _random(w, 6, t_q, 8, 64), _random(w, 7, t_q, 8, 64)
        out = ctx.query_attn(c, 0, n_ctx, q, ks, vs, n_ctx)
        H.check_attention(out.float().cpu().numpy(), _ref(oracle_mod, w, c, n_ctx, q, ks, vs, n_ctx), **BARS["bf16"])
    ctx.close()


def test_stream_batches_beyond_one_launch(ad, oracle_mod):
    """35 problems of different lengths (empty ones among them) in one call, over two caches."""
    w = _model("f32", 64, 4, 2)
    ctx = ad.Context.for_workload(w, max_position=1 << 14)
    caches = [_full_cache(ad, ctx, w, n, n) for n in (700, 333)]
    items, rng = [], np.random.default_rng(2)
    for i in range(35):
        ci, t_q = int(rng.integers(2)), int(rng.integers(1, 20))
        n = int(rng.choice([0, 1, 64, int(rng.integers(1, caches[ci].len + 1))]))
        q, ks, vs = (_random(w, 100 + 3 * i + k, t_q, h, 64) for k, h in enumerate((4, 2, 2)))
        items.append((ci, n, q, ks, vs, n + i, torch.empty_like(q)))
    ctx.query_attn_batched(caches, 0, items)
    torch.cuda.synchronize()
    for ci, n, q, ks, vs, pos, out in items:
        H.check_attention(out.cpu().numpy(), _ref(oracle_mod, w, caches[ci], n, q, ks, vs, pos), **BARS["f32"])
    ctx.close()


@pytest.mark.parametrize("dtype,d", [("f32", 8), ("f32", 128), ("bf16", 16), ("bf16", 64), ("bf16", 256)])
@pytest.mark.parametrize("m,t_q,splits", [(1, 2, 1), (14, 11, 0), (14, 3, 5)])
def test_stream_gathered_context(ad, oracle_mod, dtype, d, m, t_q, splits):
    """Zero-copy form: the same bits of K as an assembled cache would hold, so the outputs agree with the oracle chain."""
    w = _model(dtype, d, 4, 2)
    k_pool, v_pool, off = wl.make_pool(w, "cuda", n_layers=1)
    ctx = ad.Context.for_workload(w, max_position=1 << 14)
    ctx.pool_register(k_pool, v_pool, off)
    ids = np.random.default_rng(m).permutation(w.n_shots)[:m].astype(np.int32)
    total = int(np.sum(off[ids + 1] - off[ids]))
    q, ks, vs = _random(w, 5, t_q, 4, d), _random(w, 6, t_q, 2, d), _random(w, 7, t_q, 2, d)
    ctx.set_attn_splits(splits)
    out = ctx.query_attn_pool(0, ids, None, q, ks, vs, 29 + total, pos0=29)
    pl = oracle_mod.plan(off, ids, np.arange(m, dtype=np.int32), slot0=0, pos0=29)
    ko, vo, _ = oracle_mod.assemble(H.to_storage(k_pool), H.to_storage(v_pool), dtype, w.rope_theta, 0, pl, 0, total)
    ref = oracle_mod.query_attn(ko[0], vo[0], dtype, total, H.to_storage(q), H.to_storage(ks), H.to_storage(vs), w.rope_theta,
                                29 + total)
    H.check_attention(out.float().cpu().numpy(), ref, **BARS[dtype])
    ctx.close()


@pytest.mark.parametrize("form", ["cache", "pool"])
@pytest.mark.parametrize("dtype,hq,hkv,t_q,n_ctx", [("f32", 32, 8, 256, 350), ("bf16", 32, 8, 64, 2150), ("f32", 32, 8, 4130, 150)])
def test_stream_two_row_blocks_and_many_units(ad, oracle_mod, dtype, hq, hkv, t_q, n_ctx, form):
    """Two row blocks in both element types, over a cache and gathered (bf16: with several splits), and more units than
    arrival counters; 300 sampled outputs."""
    w = _model(dtype, 64, hq, hkv)
    ctx = ad.Context.for_workload(w, max_position=1 << 14)
    c = _full_cache(ad, ctx, w, n_ctx, 3)
    q, ks, vs = _random(w, 5, t_q, hq, 64), _random(w, 6, t_q, hkv, 64), _random(w, 7, t_q, hkv, 64)
    if form == "cache":
        out = ctx.query_attn(c, 0, n_ctx, q, ks, vs, n_ctx)
        kc, vc = H.to_storage(c.k[0]), H.to_storage(c.v[0])
    else:
        off = np.arange(0, n_ctx + 1, 50).astype(np.int64)
        ids = np.random.default_rng(1).permutation(n_ctx // 50).astype(np.int32)
        ctx.pool_register(c.k, c.v, off)
        out = ctx.query_attn_pool(0, ids, None, q, ks, vs, n_ctx)
        pl = oracle_mod.plan(off, ids, np.arange(len(ids), dtype=np.int32), slot0=0, pos0=0)
        ko, vo, _ = oracle_mod.assemble(H.to_storage(c.k), H.to_storage(c.v), dtype, w.rope_theta, 0, pl, 0, n_ctx)
        kc, vc = ko[0], vo[0]
    rng = np.random.default_rng(2)
    pairs = np.stack([rng.integers(0, t_q, 300), rng.integers(0, hq, 300)], axis=1).astype(np.int32)
    pairs[0], pairs[1] = (0, 0), (t_q - 1, hq - 1)
    ref = oracle_mod.query_attn(kc, vc, dtype, n_ctx, H.to_storage(q), H.to_storage(ks), H.to_storage(vs), w.rope_theta, n_ctx,
                                pairs=pairs)
    got = np.stack([out[j, h].float().cpu().numpy() for j, h in pairs])
    H.check_attention(got, ref, **BARS[dtype])
    ctx.close()
