"""Assembly of one cache with its shot list in the kernel arguments, against the lists of a batch there and against the tiles of a batch
of more caches than the arguments hold: the same bits and the same index arrays, for shots shorter than a workgroup, empty ones,
lists up to and beyond the argument's length, caches that already hold tokens, both key states."""
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


def _lens(kind, n, rng):
    if kind == "empty":  # runs of empty shots, at both ends too
        lens = rng.integers(0, 3, size=n) * rng.integers(0, 40, size=n)
        lens[[0, 1, -1]] = 0
        return lens
    return rng.integers(*{"ones": (1, 2), "short": (1, 12), "mixed": (1, 130)}[kind], size=n)


@pytest.mark.parametrize("dtype,hq,hkv,d", [("bf16", 32, 8, 128), ("bf16", 4, 1, 64), ("bf16", 3, 3, 16), ("bf16", 2, 2, 256), ("f32", 4, 2, 64),
                                            ("f32", 8, 2, 128), ("f32", 1, 1, 8)])
@pytest.mark.parametrize("kind,m,have", [("ones", 320, 0), ("short", 65, 7), ("mixed", 1, 0), ("mixed", 64, 5), ("empty", 130, 1), ("short", 321, 3)])
@pytest.mark.parametrize("local", [0, 1])
def test_the_list_in_the_arguments_gives_what_descriptors_give(ad, dtype, hq, hkv, d, kind, m, have, local):
    layers, n_pool = 2, 400
    rng = np.random.default_rng([m, have, d])
    off = np.concatenate([[3], 3 + np.cumsum(_lens(kind, n_pool, rng))]).astype(np.int64)
    torch_dtype = torch.float32 if dtype == "f32" else torch.bfloat16
    k, v = (wl.normal_tensor((layers, int(off[-1]), hkv, d), torch_dtype, "cuda", s) for s in (1, 2))
    ctx = ad.Context(layers, hq, hkv, d, 1.0e4, ad.F32 if dtype == "f32" else ad.BF16, key_state=local, max_position=1 << 15)
    ctx.pool_register(k, v, off)
    ids, order = rng.permutation(n_pool)[:m].astype(np.int32), rng.permutation(m).astype(np.int32)
    total = int(np.sum(off[ids + 1] - off[ids]))
    first = np.flatnonzero(np.diff(off))[:1].astype(np.int32)  # a shot with tokens, for the other caches of the batches
    n_first = int(off[first[0] + 1] - off[first[0]])
    one, two, tiles = (ad.Cache(ctx, have + total + 2, with_index=True) for _ in range(3))
    others = [ad.Cache(ctx, have + n_first, with_index=False) for _ in range(H.constant("kAssembleFewCaches"))]
    assert 2 * (total + len(others) * n_first) * layers * hkv * d * k.element_size() <= H.constant("kAssembleStreamBytes")  # (no list in device memory)
    for c in [one, two, tiles] + others:
        c.c.len = have
    ctx.assemble(one, ids, order, pos0=11)
    ctx.assemble_batched([two, others[0]], [ids, first], [order, None], pos0=11)
    others[0].c.len = have
    ctx.assemble_batched([tiles] + others, [ids] + [first] * len(others), [order] + [None] * len(others), pos0=11)
    torch.cuda.synchronize()
    assert total > 0 and one.len == two.len == tiles.len == have + total
    for x in (two, tiles):
        for a, b in ((one.k, x.k), (one.v, x.v), (one.slot_shot, x.slot_shot), (one.slot_tok, x.slot_tok), (one.slot_pos, x.slot_pos)):
            assert torch.equal(a, b)
    for x in others:
        assert x.len == have + n_first and torch.equal(x.v[:, have:], v[:, off[first[0]]:off[first[0] + 1]])
    if total:
        assert int(one.slot_pos[have + total - 1]) == 11 + have + total - 1 and int(one.slot_pos[have + total]) == -1
