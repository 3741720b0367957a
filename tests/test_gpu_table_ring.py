"""Calls whose kernels read tables in pinned host memory, many more in flight than there are buffers: every call's tables
have to stay as they are until its kernel has read them."""
import numpy as np
import pytest
import torch

from paper_2605_03644_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("profiled", [False, True])
def test_tables_of_calls_in_flight(profiled):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding as ad
    ad.load_library()
    ctx = ad.Context(1, 4, 2, 128, 1.0e4, ad.BF16, max_position=1 << 15)
    rng = np.random.default_rng(5)
    lens = rng.integers(20, 200, 400).astype(np.int64)
    offsets = np.concatenate([[0], np.cumsum(lens)])
    tokens = int(offsets[-1])
    k = wl.normal_tensor((1, tokens, 2, 128), torch.bfloat16, "cuda", 1)
    v = wl.normal_tensor((1, tokens, 2, 128), torch.bfloat16, "cuda", 2)
    ctx.pool_register(k, v, offsets)
    calls = []
    for i in range(20):
        lists = [rng.permutation(400)[:n].astype(np.int32) for n in (40 + i, 30)]
        calls.append(([ad.Cache(ctx, int(lens[s].sum()) + 1) for s in lists], lists))
    ctx.profile_enable(profiled)
    for rep in range(2):  # the second time all buffers are there
        for caches, lists in calls:
            for c in caches:
                c.c.len = 0
            ctx.assemble_batched(caches, lists)
    torch.cuda.synchronize()
    for caches, lists in calls:
        for c, shots in zip(caches, lists):
            n = int(lens[shots].sum())
            assert c.len == n
            src = np.concatenate([np.arange(offsets[s], offsets[s + 1]) for s in shots])
            assert torch.equal(c.v[0, :n], v[0, torch.from_numpy(src).cuda()])
            assert np.array_equal(c.slot_shot[:n].cpu().numpy(), np.repeat(shots, lens[shots]))
    # the tables of batched attention: outputs of calls in flight against each call alone
    q = wl.normal_tensor((len(calls), 2, 24, 4, 128), torch.bfloat16, "cuda", 3)
    ks = wl.normal_tensor((24, 2, 128), torch.bfloat16, "cuda", 4)
    outs = []
    for wait in (False, True):
        out = torch.empty_like(q)
        for i, (caches, _) in enumerate(calls):
            ctx.query_attn_batched(caches, 0, [(b, c.len, q[i, b], ks, ks, c.len, out[i, b]) for b, c in enumerate(caches)])
            if wait:
                torch.cuda.synchronize()
        torch.cuda.synchronize()
        outs.append(out)
    assert torch.equal(outs[0], outs[1])
    ctx.close()
