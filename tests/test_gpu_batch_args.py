"""Batches of the tile kernel on either side of the borders between tables in the kernel arguments and tables in device memory (items,
entries of work): the same items, cut into the same splits, give the same bits either way, the next layer of a kept batch included."""
import numpy as np
import pytest
import torch

from paper_2605_03644_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _entries(items, hq, hkv, splits):
    """Entries of work of a batch cut into `splits` splits of its longest context: row tiles times context splits and the own tokens'."""
    tiles = [-(-n // 64) for _, n in items]
    st = -(-max(max(tiles), 1) // splits)
    return sum(-(-t * (hq // hkv) // 256) * (-(-x // st) + 1) for (t, _), x in zip(items, tiles))


# (query tokens, context slots) of the items: as many splits as there are, and the borders of both limits
FULL, LONG = (17, 1280), (3, 4096)
BORDERS = {
    "32 items, 352 entries": ([FULL] * 32, 10, 352),
    "32 items, 353 entries": ([FULL] * 31 + [(100, 640)], 10, 353),
    "64 splits, 352 entries": ([LONG] * 5 + [(1, 0)] * 27, 64, 352),
    "64 splits, 353 entries": ([LONG] * 5 + [(1, 0)] * 26 + [(1, 64)], 64, 353),
    "33 items, 33 entries": ([(17, 0)] * 33, 1, 33),
    "9 row tiles": ([(576, 200), (9, 130)], 2, 9 * 3 + 3),
}


@pytest.mark.parametrize("form", ["cache", "pool"])
@pytest.mark.parametrize("name", BORDERS)
def test_either_side_of_a_border(name, form):
    sizes, splits, entries = BORDERS[name]
    hq, hkv = 8, 2
    assert _entries(sizes, hq, hkv, splits) == entries
    assert H.constant("kBatchArgItems") == 32 and H.constant("kBatchArgWork") == 352
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding as ad
    ctx = ad.Context(1, hq, hkv, 128, 1.0e4, ad.BF16, max_position=1 << 15)
    off = np.arange(0, 5001, 50).astype(np.int64)
    kp, vp = (wl.normal_tensor((1, 5000, hkv, 128), torch.bfloat16, "cuda", 1 + i) for i in range(2))
    ctx.pool_register(kp, vp, off)
    lists = [np.random.default_rng(3).permutation(100).astype(np.int32)]
    caches = [ad.Cache(ctx, 5000, with_index=False)]
    ctx.assemble_batched(caches, lists)
    items = []
    for i, (t, n) in enumerate(sizes):
        q, ks, vs = (wl.normal_tensor((t, h, 128), torch.bfloat16, "cuda", 10 + 3 * i + k) for k, h in enumerate((hq, hkv, hkv)))
        items.append((0, n, q, ks, vs, 6000 + i))
    ctx.set_attn_splits(splits)

    def run(its):
        outs = [torch.full_like(it[2], float("nan")) for it in its]
        packed = [it + (o,) for it, o in zip(its, outs)]
        if form == "cache":
            ctx.query_attn_batched(caches, 0, packed)
        else:
            ctx.query_attn_pool_batched(0, (lists, None), packed)
        return outs

    got = run(items)
    tables = run(items + [items[-1]] * 40)
    longest = max(items, key=lambda it: it[1])  # twice beside every item: splits as long as in the batch, a context that two of them read
    args = [run([longest, longest, it])[2] for it in items]
    for a, b, c in zip(got, tables, args):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b) and torch.equal(a, c)
    ctx.close()


# (33 items: tables in both of its runs)
@pytest.mark.parametrize("form", ["cache", "pool"])
@pytest.mark.parametrize("hq,hkv,n_items,splits", [(8, 2, 32, 3), (8, 2, 33, 3), (4, 4, 7, 1), (2, 1, 6, 64), (7, 1, 32, 5)])
def test_batches_in_arguments_and_in_tables(hq, hkv, n_items, splits, form):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_03644_amd import binding as ad
    ctx = ad.Context(2, hq, hkv, 128, 1.0e4, ad.BF16, max_position=1 << 15)
    rng = np.random.default_rng(n_items)
    off = np.arange(0, 5001, 50).astype(np.int64)
    kp, vp = (wl.normal_tensor((2, 5000, hkv, 128), torch.bfloat16, "cuda", 1 + i) for i in range(2))
    ctx.pool_register(kp, vp, off)
    lists = [rng.permutation(100)[:n].astype(np.int32) for n in (100, 20, 3)]
    caches = [ad.Cache(ctx, 50 * len(x), with_index=False) for x in lists]
    ctx.assemble_batched(caches, lists)
    items = []
    for i in range(n_items):
        li, t = i % 3, int(rng.choice([1, 17, 70, 300]))  # up to several row tiles
        n = int(rng.choice([0, 1, 64, 65, 50 * len(lists[li])]))
        q, ks, vs = (wl.normal_tensor((t, h, 128), torch.bfloat16, "cuda", 10 + 3 * i + k) for k, h in enumerate((hq, hkv, hkv)))
        items.append((li, n, q, ks, vs, 6000 + i))
    ctx.set_attn_splits(splits)

    def run(its, layer):
        outs = [torch.full_like(it[2], float("nan")) for it in its]
        packed = [it + (o,) for it, o in zip(its, outs)]
        if form == "cache":
            ctx.query_attn_batched(caches, layer, packed)
        else:
            ctx.query_attn_pool_batched(layer, (lists, None), packed)
        return outs, packed

    # all of them; each batch again with enough copies of its first item to leave the arguments
    for layer in (0, 1):
        small, packed = run(items, layer)
        large, _ = run(items + [items[0]] * 40, layer)
        assert all(torch.equal(a, b) and torch.isfinite(a.float()).all() for a, b in zip(small, large))
        # the same call for the other layer (a kept batch names its layer at the launch), then this one again
        call = (lambda l: ctx.query_attn_batched(caches, l, packed)) if form == "cache" else (lambda l: ctx.query_attn_pool_batched(l, (lists, None), packed))  # noqa: E731
        call(layer)
        call(1 - layer)
        assert any(not torch.equal(a, b) for a, b in zip(small, large))  # the other layer has other keys
        call(layer)
        assert all(torch.equal(a, b) for a, b in zip(small, large))
    ctx.close()
