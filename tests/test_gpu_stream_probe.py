"""Probes of bf16 / head_dim 128 models over short contexts, which the streaming kernel takes from the tile kernel: row counts
that end inside a 16-row block, contexts that end inside a step, one split and several, workgroups that fit the chip once and
that do not, on both sides of the border between the kernels."""
import dataclasses

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


def _random(seed, *shape):
    return wl.normal_tensor(shape, torch.bfloat16, "cuda", seed)


@pytest.mark.parametrize("hq,hkv,t_q", [(32, 8, 5), (28, 4, 24), (32, 8, 64), (7, 1, 33), (64, 8, 128), (16, 16, 100)])
@pytest.mark.parametrize("n_ctx", [0, 1, 63, 250, 830, 1700, 3300])
def test_probe_over_a_short_context(ad, oracle_mod, hq, hkv, t_q, n_ctx):
    w = dataclasses.replace(wl.WORKLOADS["tiny_fp32"], name=f"probe_{hq}_{hkv}", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, dtype="bf16",
                            rope_theta=5.0e5)
    ctx = ad.Context.for_workload(w, max_position=1 << 14)
    c = ad.Cache(ctx, max(n_ctx, 1), with_index=False)
    c.k.copy_(_random(3 + n_ctx, *c.k.shape))
    c.v.copy_(_random(4 + n_ctx, *c.v.shape))
    c.c.len = n_ctx
    q, ks, vs = _random(5, t_q, hq, 128), _random(6, t_q, hkv, 128), _random(7, t_q, hkv, 128)
    outs = [ctx.query_attn(c, 0, n_ctx, q, ks, vs, n_ctx + 3)]
    outs.append(ctx.query_attn(c, 0, n_ctx, q, ks, vs, n_ctx + 3))
    one = torch.empty_like(q)
    ctx.query_attn_batched([c], 0, [(0, n_ctx, q, ks, vs, n_ctx + 3, one)])  # a batch of one takes the same kernel
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    ref = oracle_mod.query_attn(H.to_storage(c.k[0]), H.to_storage(c.v[0]), "bf16", n_ctx, H.to_storage(q), H.to_storage(ks),
                                H.to_storage(vs), w.rope_theta, n_ctx + 3)
    H.check_attention(outs[0].float().cpu().numpy(), ref, **BAR)
    H.check_attention(one.float().cpu().numpy(), ref, **BAR)
