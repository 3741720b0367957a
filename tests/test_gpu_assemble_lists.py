"""Assembly of batches and of long shot lists (lists in the kernel arguments of up to 8 caches, tiles, lists in device memory, more caches
than a launch takes) against the same shots assembled cache by cache, 300 at a time: the same bits and index arrays."""
import numpy as np
import pytest
import torch

from paper_2605_03644_amd import workloads as wl

pytestmark = pytest.mark.gpu


# one cache: lists in two parts, tiles; 2 x 136: the longest list in the arguments, 2 x 137 and 9 x 3: tiles; 49: two launches
@pytest.mark.parametrize("n_caches,m", [(1, 321), (2, 136), (2, 137), (8, 34), (9, 3), (48, 30), (49, 7)])
@pytest.mark.parametrize("lens_hi,local,index", [(1, 0, True), (12, 1, True), (70, 0, False)])
def test_small_batches(n_caches, m, lens_hi, local, index):
    _check(2, 1, 64, "bf16", n_caches, m, lens_hi, local, index)


# more than 256 MB written: workgroups of 32, 8 and 2 slots, runs of empty shots between the others
@pytest.mark.parametrize("layers,hkv,d,dtype,n_caches,m,lens_hi,local", [
    (28, 1, 256, "bf16", 1, 4200, 4, 1), (28, 1, 256, "bf16", 48, 34, 12, 0), (28, 1, 256, "bf16", 49, 34, 12, 1),
    (2, 8, 128, "bf16", 1, 1100, 70, 1), (2, 8, 128, "bf16", 3, 380, 70, 0), (2, 16, 128, "f32", 9, 40, 70, 0), (1, 8, 128, "bf16", 8, 400, 55, 0)])
def test_lists_in_device_memory(layers, hkv, d, dtype, n_caches, m, lens_hi, local):
    written = _check(layers, hkv, d, dtype, n_caches, m, lens_hi, local, True, 2 if n_caches <= 48 else 3)  # (a 49th cache: a launch of its own)
    assert written > 256 << 20


# arguments: one launch; tiles: one; a list in device memory: the launch that writes it, and the assembly
@pytest.mark.parametrize("n_caches,m,layers,launches", [(1, 300, 2, 1), (2, 200, 2, 1), (1, 1100, 2, 2), (49, 30, 2, 3)])
def test_every_launch_is_recorded(n_caches, m, layers, launches):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding as ad
    ctx = ad.Context(layers, 8, 8, 128, 1.0e4, ad.BF16, max_position=1 << 19)
    off = (35 * np.arange(1201)).astype(np.int64)
    k, v = (wl.normal_tensor((layers, int(off[-1]), 8, 128), torch.bfloat16, "cuda", s) for s in (1, 2))
    ctx.pool_register(k, v, off)
    caches = [ad.Cache(ctx, 35 * m, with_index=False) for _ in range(n_caches)]
    ctx.profile_enable(True)
    ctx.assemble_batched(caches, [np.arange(m, dtype=np.int32)] * n_caches)
    ms, n = ctx.profile_read()["assemble_reencode"]
    assert n == launches and ms > 0
    ctx.close()


# the same rows by tiles: more than 256 MB of long shots in pieces cut by the host, fp32 shots of more than a tile
@pytest.mark.parametrize("layers,hkv,d,dtype,n_caches,m,lens_hi,local", [(8, 8, 128, "bf16", 9, 40, 70, 0), (2, 8, 128, "f32", 3, 130, 120, 1)])
def test_tiles_past_the_cache(layers, hkv, d, dtype, n_caches, m, lens_hi, local):
    written = _check(layers, hkv, d, dtype, n_caches, m, lens_hi, local, True, 1)
    assert 256 << 20 < written <= 512 << 20


def _check(layers, hkv, d, dtype, n_caches, m, lens_hi, local, index, launches=None):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding as ad
    ad.load_library()
    rng = np.random.default_rng([n_caches, m, lens_hi])
    n_pool = 6000
    lens = rng.integers(1, lens_hi, size=n_pool, endpoint=True)
    lens[rng.integers(0, n_pool, size=300)] = 0
    off = np.concatenate([[3], 3 + np.cumsum(lens)]).astype(np.int64)
    torch_dtype = torch.float32 if dtype == "f32" else torch.bfloat16
    k, v = (wl.normal_tensor((layers, int(off[-1]), hkv, d), torch_dtype, "cuda", s) for s in (1, 2))
    ctx = ad.Context(layers, hkv, hkv, d, 1.0e4, ad.F32 if dtype == "f32" else ad.BF16, key_state=local, max_position=1 << 19)
    ctx.pool_register(k, v, off)
    ids = [rng.permutation(n_pool)[:m].astype(np.int32) for _ in range(n_caches)]
    totals = [int(lens[i].sum()) for i in ids]
    got, want = ([ad.Cache(ctx, 5 + t + 2, with_index=index) for t in totals] for _ in range(2))
    for c in got + want:
        c.c.len = 5
    ctx.profile_enable(launches is not None)
    ctx.assemble_batched(got, ids, [None] * n_caches, pos0=9)
    if launches is not None:  # the route: a list is a launch of its own
        assert ctx.profile_read()["assemble_reencode"][1] == launches
        ctx.profile_enable(False)
    for c, i in zip(want, ids):
        for a in range(0, m, 300):
            ctx.assemble(c, i[a:a + 300], None, pos0=9)
    torch.cuda.synchronize()
    for a, b, i, t in zip(got, want, ids, totals):
        assert a.len == b.len == 5 + t
        src = np.concatenate([np.arange(off[s], off[s + 1]) for s in i])
        assert torch.equal(a.v[:, 5:5 + t], v[:, torch.from_numpy(src).cuda()])
        assert torch.equal(a.k, b.k) and torch.equal(a.v, b.v)
        if index:
            assert torch.equal(a.slot_shot, b.slot_shot) and torch.equal(a.slot_tok, b.slot_tok) and torch.equal(a.slot_pos, b.slot_pos)
    ctx.close()
    return 2 * sum(totals) * layers * hkv * d * k.element_size()
