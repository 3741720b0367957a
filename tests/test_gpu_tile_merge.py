"""Splits of the tile kernel and their merge, which has a launch of its own: a merge inside the launch would have workgroups hold their
compute units while they wait for each other and merge alone what others have left, and calls on two streams then take turns.
Zero-copy calls whose row counts end inside a row tile, one split and the most, own tokens that take longer than a context split, several
calls one after the other; against the same call in a batch of two, and, as everywhere, the oracle's bar."""
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


# n_shots < 0: shots that fill -n_shots key tiles (64 slots each)
@pytest.mark.parametrize("hq,hkv,t_q,n_shots,splits", [(32, 8, 3, 3, 0), (32, 8, 16, 40, 0), (28, 4, 37, 60, 5), (28, 4, 73, 9, 0), (8, 8, 300, 4, 0),
                                                       (4, 1, 65, 90, 63), (32, 8, 128, 64, 1), (9, 1, 29, 70, 0), (4, 1, 65, -63, 63), (4, 1, 65, -64, 64)])
def test_a_call_by_tiles_is_merged_by_a_launch_of_its_own(ad, oracle_mod, hq, hkv, t_q, n_shots, splits):
    w = dataclasses.replace(wl.WORKLOADS["tiny_fp32"], name=f"merge_{hq}_{hkv}", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, dtype="bf16",
                            rope_theta=5.0e5, n_shots=96, len_lo=30, len_hi=120)
    off = wl.shot_offsets(w).copy()
    if n_shots < 0:
        end = -64 * n_shots - 5
        n_shots = int((off < end).sum())
        off[n_shots] = end
    k_pool, v_pool = _random(1, 1, int(off[-1]), hkv, 128), _random(2, 1, int(off[-1]), hkv, 128)
    ctx = ad.Context.for_workload(w, n_layers=1, max_position=1 << 15)
    ctx.pool_register(k_pool, v_pool, off)
    ids = list(range(n_shots))
    n = int(off[n_shots] - off[0])
    q, ks, vs = _random(5, t_q, hq, 128), _random(6, t_q, hkv, 128), _random(7, t_q, hkv, 128)
    ctx.set_attn_splits(splits)
    ctx.profile_enable(True)
    outs = [ctx.query_attn_pool(0, ids, None, q, ks, vs, n) for _ in range(3)]
    torch.cuda.synchronize()
    assert ctx.profile_read()["attn_combine"][1] == 3
    ctx.profile_enable(False)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    two = [torch.empty_like(q), torch.empty_like(q)]
    ctx.query_attn_pool_batched(0, ([ids], None), [(0, n, q, ks, vs, n, two[0]), (0, n, q, ks, vs, n, two[1])])
    c = ad.Cache(ctx, n, with_index=False)
    ctx.assemble(c, ids)
    torch.cuda.synchronize()
    if splits:   # the same split length: the same partials, added in the same order
        assert torch.equal(outs[0], two[0])
    assert torch.equal(two[0], two[1])
    ref = oracle_mod.query_attn(H.to_storage(c.k[0]), H.to_storage(c.v[0]), "bf16", n, H.to_storage(q), H.to_storage(ks), H.to_storage(vs),
                                w.rope_theta, n)
    for o in (outs[0], two[0]):
        H.check_attention(o.float().cpu().numpy(), ref, **BAR)
