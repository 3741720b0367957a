"""Calls whose kernels read tables in pinned host memory, many more in flight than there are buffers: every call's tables
have to stay as they are until its kernel has read them."""
import numpy as np
import pytest
import torch

from paper_2605_03644_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ad():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding
    binding.load_library()
    return binding


def _busy():
    """Tens of milliseconds of work ahead on the stream: what is called next piles up behind it."""
    x = torch.ones(4096, 4096, device="cuda")
    for _ in range(30):
        x = x @ x * 2.0 ** -12
    return x


def _by_tiles(n_caches, n_shots, tokens, token_bytes):
    """Whether an assembly keeps its descriptors in pinned memory: more shots than the kernel arguments hold, too little written for a
    list in device memory."""
    args = n_shots <= H.constant("kAssembleShots") if n_caches == 1 else (
        n_caches <= H.constant("kAssembleFewCaches") and n_shots <= H.constant("kAssembleFewShots"))
    return not args and 2 * tokens * token_bytes <= H.constant("kAssembleStreamBytes")


@pytest.mark.parametrize("profiled", [False, True])
def test_tables_of_calls_in_flight(ad, profiled):
    ctx = ad.Context(1, 4, 2, 128, 1.0e4, ad.BF16, max_position=1 << 16)
    rng = np.random.default_rng(5)
    lens = rng.integers(20, 200, 400).astype(np.int64)
    offsets = np.concatenate([[0], np.cumsum(lens)])
    tokens = int(offsets[-1])
    k = wl.normal_tensor((1, tokens, 2, 128), torch.bfloat16, "cuda", 1)
    v = wl.normal_tensor((1, tokens, 2, 128), torch.bfloat16, "cuda", 2)
    ctx.pool_register(k, v, offsets)
    calls = []
    for i in range(20):
        lists = [rng.permutation(400)[:n].astype(np.int32) for n in (160 + i, 120)]
        assert _by_tiles(2, sum(len(s) for s in lists), sum(int(lens[s].sum()) for s in lists), 2 * 128 * 2)
        calls.append(([ad.Cache(ctx, int(lens[s].sum()) + 1) for s in lists], lists))
    ctx.profile_enable(profiled)
    for rep in range(2):  # the second time all buffers are there
        for caches, lists in calls:
            for c in caches:
                c.c.len = 0
        torch.cuda.synchronize()
        _busy()
        for caches, lists in calls:
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
    per_cache = 17
    assert 2 * per_cache > H.constant("kBatchArgItems")  # rows enough for the tile kernel, items too many for the kernel arguments
    q = wl.normal_tensor((len(calls), 2, per_cache, 24, 4, 128), torch.bfloat16, "cuda", 3)
    ks = wl.normal_tensor((24, 2, 128), torch.bfloat16, "cuda", 4)
    outs = []
    for wait in (False, True):
        out = torch.empty_like(q)
        if not wait:
            _busy()
        for i, (caches, _) in enumerate(calls):
            ctx.query_attn_batched(caches, 0, [(b, c.len - 64 * j, q[i, b, j], ks, ks, c.len, out[i, b, j])
                                               for b, c in enumerate(caches) for j in range(per_cache)])
            if wait:
                torch.cuda.synchronize()
        torch.cuda.synchronize()
        outs.append(out)
    assert torch.equal(outs[0], outs[1])
    ctx.close()


@pytest.mark.parametrize("profiled", [False, True])
def test_lists_of_calls_in_flight(ad, profiled):
    """Assemblies by lists in device memory, one piece of it for every pinned buffer, that have to be made larger while earlier calls still
    read them, and between them assemblies by tiles (cut by the host: 8 layers), which take buffers of the same ring."""
    layers, hkv, d = 8, 8, 128
    ctx = ad.Context(layers, 8, hkv, d, 1.0e4, ad.BF16, max_position=1 << 17)
    rng = np.random.default_rng(6)
    n_pool = 6000
    lens = rng.integers(0, 41, n_pool).astype(np.int64)
    offsets = np.concatenate([[0], np.cumsum(lens)])
    k, v = (wl.normal_tensor((layers, int(offsets[-1]), hkv, d), torch.bfloat16, "cuda", s) for s in (1, 2))
    ctx.pool_register(k, v, offsets)
    token_bytes = layers * hkv * d * 2
    assert layers >= H.constant("kAssemblePieceLayers")
    wg_tok = 16384 // (hkv * d * 2)
    calls, sizes = [], []
    for m in (900, 950, 900, 2200, 1000, 900, 900, 4400, 950, 1200, 900, 900, 900):
        shots = rng.permutation(n_pool)[:m].astype(np.int32)
        n = int(lens[shots].sum())
        assert m > H.constant("kAssembleShots") and 2 * n * token_bytes > 2 * H.constant("kAssembleStreamBytes")
        sizes.append(16 * (int((lens[shots] > 0).sum()) + -(-n // wg_tok)))
        calls.append(([ad.Cache(ctx, n + 3)], [shots]))
        lists = [rng.permutation(n_pool)[:170].astype(np.int32) for _ in range(2)]
        assert _by_tiles(2, sum(int((lens[s] > 0).sum()) for s in lists), sum(int(lens[s].sum()) for s in lists), token_bytes)
        calls.append(([ad.Cache(ctx, int(lens[s].sum())) for s in lists], lists))
    # (the pieces start at 64 KiB and double: they grow twice, each time with calls in flight)
    assert sizes[0] < 65536 < sizes[3] < 131072 < sizes[7]
    ctx.profile_enable(profiled)
    torch.cuda.synchronize()
    _busy()
    for caches, lists in calls:
        ctx.assemble_batched(caches, lists)
    torch.cuda.synchronize()
    if profiled:  # a list is a launch of its own
        assert ctx.profile_read()["assemble_reencode"][1] == 2 * len(sizes) + len(sizes)
    for caches, lists in calls:
        for c, shots in zip(caches, lists):
            n = int(lens[shots].sum())
            assert c.len == n
            src = np.concatenate([np.arange(offsets[s], offsets[s + 1]) for s in shots])
            assert torch.equal(c.v[:, :n], v[:, torch.from_numpy(src).cuda()])
            assert np.array_equal(c.slot_shot[:n].cpu().numpy(), np.repeat(shots, lens[shots]))
            want = ad.Cache(ctx, n)
            for a in range(0, len(shots), 300):  # (lists in the kernel arguments)
                ctx.assemble(want, shots[a:a + 300])
            assert torch.equal(c.k[:, :n], want.k) and torch.equal(c.slot_pos[:n], want.slot_pos)
            torch.cuda.synchronize()
    ctx.close()
