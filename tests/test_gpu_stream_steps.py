"""The streaming attention kernel where its keys come through LDS and where its splits are merged: contexts that end on either
side of a 32-key step, of the eight wavefronts' first steps and of their second ones, own tokens that fill a key block or run
over it, and split counts around the eight that a thread of the merge has in flight and around those where its threads
form two, four and eight groups, for one row up to a full row block."""
import dataclasses

import pytest
import torch

from paper_2605_03644_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu

# as in test_gpu_stream.py: fp32 sums in another order; bf16: query and output rounded to 2^-9
BARS = {"f32": dict(max_abs=1e-4, rel_fro=1e-5), "bf16": dict(max_abs=2e-2, rel_fro=1e-2)}


@pytest.mark.parametrize("dtype,d,hq,hkv", [("bf16", 128, 4, 4), ("bf16", 128, 28, 4), ("bf16", 64, 8, 2), ("f32", 64, 4, 2), ("f32", 128, 8, 2)])
@pytest.mark.parametrize("n_ctx,t_q,splits", [(31, 1, 1), (33, 2, 1), (256, 1, 1), (257, 16, 1), (513, 17, 1), (1100, 4, 2), (1100, 1, 9),
                                              (2200, 2, 17), (4096, 1, 64), (600, 3, 8), (1100, 5, 16), (2112, 4, 32), (2240, 2, 33)])
def test_steps_and_merges(oracle_mod, dtype, d, hq, hkv, n_ctx, t_q, splits):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding as ad
    w = dataclasses.replace(wl.WORKLOADS["tiny_fp32"], name="steps", n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype=dtype, rope_theta=5.0e5)
    t_q = min(t_q, 16 * hkv // hq if (dtype, d) == ("bf16", 128) and hq == 28 else t_q) or 1  # (28/4 heads: the streaming kernel's rows)
    ctx = ad.Context.for_workload(w, max_position=1 << 14)
    c = ad.Cache(ctx, n_ctx, with_index=False)
    c.k.copy_(wl.normal_tensor(tuple(c.k.shape), w.torch_dtype, "cuda", n_ctx))
    c.v.copy_(wl.normal_tensor(tuple(c.v.shape), w.torch_dtype, "cuda", n_ctx + 1))
    c.c.len = n_ctx
    q, ks, vs = (wl.normal_tensor((t_q, h, d), w.torch_dtype, "cuda", 5 + i) for i, h in enumerate((hq, hkv, hkv)))
    ctx.set_attn_splits(splits)
    out = ctx.query_attn(c, 0, n_ctx, q, ks, vs, n_ctx + 3)
    assert torch.equal(out, ctx.query_attn(c, 0, n_ctx, q, ks, vs, n_ctx + 3))
    ref = oracle_mod.query_attn(H.to_storage(c.k[0]), H.to_storage(c.v[0]), dtype, n_ctx, H.to_storage(q), H.to_storage(ks),
                                H.to_storage(vs), w.rope_theta, n_ctx + 3)
    H.check_attention(out.float().cpu().numpy(), ref, **BARS[dtype])
    ctx.close()
