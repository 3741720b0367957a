"""The zero-copy form (adapshot_query_attn_pool): attention straight over the pool through a slot table, keys
re-encoded inside the key loop.  Checked against the oracle chain plan -> assemble -> attention (the oracle needs
no change: by R(a)R(b) = R(a+b) the result is that of the assembled cache), and against the two-pass GPU path."""
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


def _case(ad, oracle_mod, w, ids, order, t_q, pos0=0, q_pos0=None, layer=0, n_layers=1, pairs=None, splits=0):
    k_pool, v_pool, off = wl.make_pool(w, "cuda", n_layers=n_layers)
    ctx = ad.Context.for_workload(w, n_layers=n_layers)
    ctx.pool_register(k_pool, v_pool, off)
    seq = [int(ids[o]) for o in order] if order is not None else [int(i) for i in ids]
    total = int(sum(off[s + 1] - off[s] for s in seq))
    q_pos0 = pos0 + total if q_pos0 is None else q_pos0
    q, ks, vs = wl.make_query(w, "cuda", t_q=t_q, layer=layer)
    ctx.set_attn_splits(splits)
    out = ctx.query_attn_pool(layer, ids, order, q, ks, vs, q_pos0, pos0=pos0)
    # the two-pass path on the same inputs
    cache = ad.Cache(ctx, max(total, 1), with_index=False)
    ctx.assemble(cache, ids, order, pos0=pos0)
    two = ctx.query_attn(cache, layer, total, q, ks, vs, q_pos0)
    torch.cuda.synchronize()
    kp, vp = H.to_storage(k_pool[layer:layer + 1]), H.to_storage(v_pool[layer:layer + 1])
    pl = oracle_mod.plan(off, ids, order, slot0=0, pos0=pos0)
    ko, vo, _ = oracle_mod.assemble(kp, vp, w.dtype, w.rope_theta, 0, pl, 0, max(total, 1))
    ref = oracle_mod.query_attn(ko[0], vo[0], w.dtype, total, H.to_storage(q), H.to_storage(ks), H.to_storage(vs),
                                w.rope_theta, q_pos0, pairs=pairs)
    got, got2 = out.float().cpu().numpy(), two.float().cpu().numpy()
    assert np.isfinite(got).all()
    assert float(np.abs(got - got2).max()) <= 2.0 ** -6 * max(1.0, float(np.abs(got2).max()))   # both within rounding of one result
    if pairs is not None:
        got = np.stack([got[j, h] for j, h in pairs])
    bars = dict(max_abs=2e-2, rel_fro=1e-2) if w.dtype == "bf16" else dict(max_abs=1e-4, rel_fro=1e-5)
    res = H.check_attention(got, ref, **bars)
    ctx.close()
    return res


def test_zero_copy_llama8b_full_size(ad, oracle_mod):
    """Config 2 at full size: 256 shots in a seeded order (~27k tokens), 128 query tokens, every output."""
    w = wl.WORKLOADS["llama8b_1layer"]
    ids, order = wl.selection(w)
    err, fro = _case(ad, oracle_mod, w, ids, order, w.t_q)
    assert err < 2e-2


@pytest.mark.parametrize("n_sel,t_q,pos0,splits", [(1, 1, 0, 0), (3, 16, 0, 0), (9, 128, 11, 0), (5, 37, 100000, 1),
                                                   (40, 64, 777, 7), (17, 300, 64, 2), (2, 5, 1048576 - 400, 0)])
def test_zero_copy_small_cases(ad, oracle_mod, n_sel, t_q, pos0, splits):
    """Ragged contexts, one and several tiles, positions near the table's end, forced split counts, duplicates."""
    w = wl.WORKLOADS["llama8b_1layer"]
    ids, order = wl.selection(w, variant=n_sel)
    ids, order = ids[:n_sel].copy(), np.argsort(np.argsort(order[:n_sel])).astype(np.int32)
    if n_sel >= 3:
        ids[1] = ids[0]                                    # a shot selected twice
    _case(ad, oracle_mod, w, ids, order, t_q, pos0=pos0, splits=splits)


def test_zero_copy_other_shapes_layers_and_identity_order(ad, oracle_mod):
    """g = 7 rows per kv head (Qwen2 shape) on layer 1 of two, order = NULL; g = 8 (70B shape), sampled outputs."""
    w = wl.WORKLOADS["qwen7b_decode"]
    ids, _ = wl.selection(w)
    _case(ad, oracle_mod, w, ids[:30], None, 1, layer=1, n_layers=2)
    _case(ad, oracle_mod, w, ids[:30], None, 19, layer=1, n_layers=2)
    w = wl.WORKLOADS["llama70b_128k"]
    ids, order = wl.selection(w)
    ids, order = ids[:200], np.argsort(np.argsort(order[:200])).astype(np.int32)
    rng = np.random.default_rng(5)
    pairs = np.stack([rng.integers(0, 64, 300), rng.integers(0, w.n_q_heads, 300)], axis=1).astype(np.int32)
    _case(ad, oracle_mod, w, ids, order, 64, pairs=pairs)


def test_zero_copy_llama70b_128k_sampled(ad, oracle_mod):
    """Config 4's context on one layer: 1000 of 4000 shots (~127k tokens, 495 key tiles per context split, so the
    rings of table pieces and rotation rows wrap many times), 256 query tokens, 64 q / 8 kv heads; 400 sampled
    outputs against the oracle chain, every output against the two-pass path."""
    w = wl.WORKLOADS["llama70b_128k"]
    ids, order = wl.selection(w)
    rng = np.random.default_rng(8)
    pairs = np.stack([rng.integers(0, w.t_q, 400), rng.integers(0, w.n_q_heads, 400)], axis=1).astype(np.int32)
    pairs[0] = (0, 0); pairs[1] = (w.t_q - 1, w.n_q_heads - 1)
    err, fro = _case(ad, oracle_mod, w, ids, order, w.t_q, pairs=pairs)
    assert err < 2e-2


def test_zero_copy_generic_kernel_fp32(ad, oracle_mod):
    """The fp32 / head_dim 64 workload goes through the streaming kernel, which gathers and rotates the keys in registers: single calls (with an order, a position base, a duplicate) and a batch over two lists."""
    w = wl.WORKLOADS["tiny_fp32"]
    ids, order = wl.selection(w)
    _case(ad, oracle_mod, w, ids, order, w.t_q)
    ids2 = ids.copy()
    ids2[1] = ids2[0]
    _case(ad, oracle_mod, w, ids2, order, 5, pos0=77)
    _case(ad, oracle_mod, w, ids[:1], None, 1, pos0=(1 << 17) - 100)
    _batched_case(ad, oracle_mod, w, [(ids, order), (ids[:3], None), (ids[:0], None)],
                  [(0, None, 16), (0, 70, 3), (1, None, 1), (1, 0, 4), (2, 0, 2)], pos0=5)


def test_zero_copy_empty_context_and_errors(ad, oracle_mod):
    w = wl.WORKLOADS["llama8b_1layer"]
    k_pool, v_pool, off = wl.make_pool(w, "cuda", n_layers=1)
    ctx = ad.Context.for_workload(w, n_layers=1)
    q, ks, vs = wl.make_query(w, "cuda", t_q=9)
    out = torch.full_like(q, 3.0)
    with pytest.raises(ad.AdapshotError) as e:             # no pool yet
        ctx.query_attn_pool(0, [1, 2], None, q, ks, vs, 0, out=out)
    assert e.value.status == ad.ESTATE
    ctx.pool_register(k_pool, v_pool, off)
    for bad_ids, bad_order, status in (([1, w.n_shots], None, ad.ESHOT), ([1, 2], [0, 2], ad.ESHOT), ([-1], None, ad.ESHOT)):
        with pytest.raises(ad.AdapshotError) as e:
            ctx.query_attn_pool(0, bad_ids, bad_order, q, ks, vs, 0, out=out)
        assert e.value.status == status
    with pytest.raises(ad.AdapshotError) as e:             # positions beyond the tables
        ctx.query_attn_pool(0, [1, 2], None, q, ks, vs, 0, pos0=(1 << 20) - 10, out=out)
    assert e.value.status == ad.ECAPACITY
    with pytest.raises(ad.AdapshotError):
        ctx.query_attn_pool(1, [1, 2], None, q, ks, vs, 0, out=out)
    torch.cuda.synchronize()
    assert float(out.float().min()) == 3.0 and float(out.float().max()) == 3.0     # nothing was launched
    # no shots: the query attends to its own tokens only
    got = ctx.query_attn_pool(0, [], None, q, ks, vs, 0)
    ref = oracle_mod.query_attn(H.to_storage(k_pool[0]), H.to_storage(v_pool[0]), w.dtype, 0, H.to_storage(q),
                                H.to_storage(ks), H.to_storage(vs), w.rope_theta, 0)
    H.check_attention(got.float().cpu().numpy(), ref)
    ctx.close()
    # a pool whose keys were stored rotated is refused (the kernel re-encodes from position-free keys)
    ctx = ad.Context.for_workload(w, key_state=ad.KEYS_ROTATED_LOCAL, n_layers=1)
    ctx.pool_register(k_pool, v_pool, off)
    with pytest.raises(ad.AdapshotError) as e:
        ctx.query_attn_pool(0, [1, 2], None, q, ks, vs, 0, out=out)
    assert e.value.status == ad.ESTATE
    ctx.close()


# ---- adapshot_query_attn_pool_batched: prefixes of several shot lists in one call -------------------------------

def _batched_case(ad, oracle_mod, w, lists, item_specs, pos0=0, layer=0, n_layers=1, n_pairs=None, splits=0, seed=0):
    """lists: [(ids, order or None)]; item_specs: [(list index, n_ctx or None for the whole list, t_q)].  Every item
    is checked against the oracle chain over its own list, and against the two-pass batched GPU path."""
    k_pool, v_pool, off = wl.make_pool(w, "cuda", n_layers=n_layers)
    ctx = ad.Context.for_workload(w, n_layers=n_layers)
    ctx.pool_register(k_pool, v_pool, off)
    totals = []
    for ids, order in lists:
        seq = [int(ids[o]) for o in order] if order is not None else [int(i) for i in ids]
        totals.append(int(sum(off[s + 1] - off[s] for s in seq)))
    g = torch.Generator(device="cuda")
    g.manual_seed(1234 + seed)
    items = []
    dt = torch.bfloat16 if w.dtype == "bf16" else torch.float32
    for li, n_ctx, t_q in item_specs:
        n_ctx = totals[li] if n_ctx is None else n_ctx
        q = torch.randn(t_q, w.n_q_heads, w.head_dim, device="cuda", generator=g).to(dt)
        ks = torch.randn(t_q, w.n_kv_heads, w.head_dim, device="cuda", generator=g).to(dt)
        vs = torch.randn(t_q, w.n_kv_heads, w.head_dim, device="cuda", generator=g).to(dt)
        items.append((li, n_ctx, q, ks, vs, pos0 + n_ctx, torch.full_like(q, 7.0)))
    ctx.set_attn_splits(splits)
    ctx.query_attn_pool_batched(layer, ([l[0] for l in lists], [l[1] for l in lists]), items, pos0=pos0)
    torch.cuda.synchronize()
    got = [it[6].float().cpu().numpy().copy() for it in items]
    # the two-pass path: assemble every list, attend in one batched call
    caches = [ad.Cache(ctx, max(t, 1), with_index=False) for t in totals]
    ctx.assemble_batched(caches, [l[0] for l in lists], [l[1] for l in lists], pos0=pos0)
    two_items = [(li, n, q, ks, vs, qp, torch.empty_like(q)) for (li, n, q, ks, vs, qp, _) in items]
    ctx.query_attn_batched(caches, layer, two_items)
    torch.cuda.synchronize()
    kp, vp = H.to_storage(k_pool[layer:layer + 1]), H.to_storage(v_pool[layer:layer + 1])
    oc = {}
    rng = np.random.default_rng(77 + seed)
    worst = 0.0
    for i, (li, n_ctx, q, ks, vs, qp, _) in enumerate(items):
        assert np.isfinite(got[i]).all()
        two = two_items[i][6].float().cpu().numpy()
        assert float(np.abs(got[i] - two).max()) <= 2.0 ** -6 * max(1.0, float(np.abs(two).max())), i
        if li not in oc and totals[li] == 0:
            oc[li] = (kp, vp, None)                        # an empty list: no slot is ever read
        elif li not in oc:
            pl = oracle_mod.plan(off, lists[li][0], lists[li][1], slot0=0, pos0=pos0)
            oc[li] = oracle_mod.assemble(kp, vp, w.dtype, w.rope_theta, 0, pl, 0, totals[li])
        ko, vo, _ = oc[li]
        t_q = q.shape[0]
        pairs = None
        g_i = got[i]
        if n_pairs is not None and t_q * w.n_q_heads > n_pairs:
            flat = rng.choice(t_q * w.n_q_heads, n_pairs, replace=False)
            pairs = np.stack([flat // w.n_q_heads, flat % w.n_q_heads], axis=1).astype(np.int32)
            g_i = np.stack([got[i][j, h] for j, h in pairs])
        ref = oracle_mod.query_attn(ko[0], vo[0], w.dtype, n_ctx, H.to_storage(q), H.to_storage(ks), H.to_storage(vs),
                                    w.rope_theta, qp, pairs=pairs)
        bars = dict(max_abs=2e-2, rel_fro=1e-2) if w.dtype == "bf16" else dict(max_abs=1e-4, rel_fro=1e-5)
        err, _ = H.check_attention(g_i, ref, **bars)
        worst = max(worst, err)
    ctx.close()
    return worst


def test_zero_copy_batched_nested_prefixes_and_ragged_items(ad, oracle_mod):
    """Two lists (one with an order, one without, a shot picked twice); items over nested prefixes that end at shot
    boundaries and in the middle of a shot, an empty prefix, single-token and ragged row counts."""
    w = wl.WORKLOADS["llama8b_sweep"]
    off = wl.shot_offsets(w)
    ids0, order0 = wl.selection(w, query=0)
    ids0, order0 = ids0[:24].copy(), np.argsort(np.argsort(order0[:24])).astype(np.int32)
    ids0[3] = ids0[2]
    ids1, _ = wl.selection(w, query=1)
    ids1 = ids1[:9]
    seq0 = [int(ids0[o]) for o in order0]
    cum0 = np.cumsum([off[s + 1] - off[s] for s in seq0])
    specs = [(0, int(cum0[3]), 64), (0, int(cum0[7]), 64), (0, int(cum0[15]), 64), (0, None, 64),
             (0, int(cum0[5]) - 17, 5), (0, 0, 9), (1, None, 1), (1, 77, 33), (1, 64, 300)]
    for splits in (0, 1, 3):
        _batched_case(ad, oracle_mod, w, [(ids0, order0), (ids1, None)], specs, pos0=0 if splits else 129, splits=splits)


def test_zero_copy_batched_other_shapes(ad, oracle_mod):
    """g = 7 rows per kv head on layer 1 of two (decode-like single tokens), and g = 8 with an empty list beside a
    full one."""
    w = wl.WORKLOADS["qwen7b_decode"]
    ids, _ = wl.selection(w)
    _batched_case(ad, oracle_mod, w, [(ids[:20], None), (ids[20:50], None)], [(0, None, 1), (1, None, 1), (1, 100, 3)],
                  layer=1, n_layers=2)
    w = wl.WORKLOADS["llama70b_128k"]
    ids, order = wl.selection(w)
    _batched_case(ad, oracle_mod, w, [(ids[:0], None), (ids[:40], None)], [(0, 0, 16), (1, None, 40), (1, 1000, 40)],
                  n_pairs=200)


def test_zero_copy_batched_sweep_full_size_one_layer(ad, oracle_mod):
    """Config 3 on one layer at its full batch: 8 queries with their own 512-shot orderings, six nested prefixes
    each (16 .. 512 shots, up to ~53k tokens), 64 probe tokens per item; 25 sampled outputs per item (1200 in all)
    against the oracle chain, every output against the two-pass batched path."""
    w = wl.WORKLOADS["llama8b_sweep"]
    off = wl.shot_offsets(w)
    lists, specs = [], []
    for qi in range(w.n_queries):
        ids, order = wl.selection(w, query=qi)
        lists.append((ids, order))
        seq = [int(ids[o]) for o in order]
        cum = np.cumsum([off[s + 1] - off[s] for s in seq])
        for k in w.prefixes:
            specs.append((qi, int(cum[k - 1]), w.t_q))
    worst = _batched_case(ad, oracle_mod, w, lists, specs, n_pairs=25)
    assert worst < 2e-2


def test_zero_copy_batched_errors_write_nothing(ad):
    w = wl.WORKLOADS["llama8b_1layer"]
    k_pool, v_pool, off = wl.make_pool(w, "cuda", n_layers=1)
    ctx = ad.Context.for_workload(w, n_layers=1)
    q, ks, vs = wl.make_query(w, "cuda", t_q=9)
    out = torch.full_like(q, 3.0)
    lists = ([[1, 2, 3], [4]], None)
    total0 = int(sum(off[s + 1] - off[s] for s in (1, 2, 3)))
    good = (0, total0, q, ks, vs, total0, out)
    with pytest.raises(ad.AdapshotError) as e:             # no pool yet
        ctx.query_attn_pool_batched(0, lists, [good])
    assert e.value.status == ad.ESTATE
    ctx.pool_register(k_pool, v_pool, off)
    cases = [(lists, [good, (2, 1, q, ks, vs, 1, out)], ad.EINVAL),                     # list index out of range
             (lists, [good, (0, total0 + 1, q, ks, vs, 1, out)], ad.ESTATE),            # prefix longer than the list
             (([[1, w.n_shots]], None), [(0, 1, q, ks, vs, 1, out)], ad.ESHOT),         # shot id out of range
             (([[1, 2]], [[0, 2]]), [(0, 1, q, ks, vs, 1, out)], ad.ESHOT),             # order out of range
             (lists, [good, (1, 1, q, ks, vs, -1, out)], ad.EINVAL)]                    # negative position
    for ls, items, status in cases:
        with pytest.raises(ad.AdapshotError) as e:
            ctx.query_attn_pool_batched(0, ls, items)
        assert e.value.status == status, e.value
    with pytest.raises(ad.AdapshotError) as e:             # positions beyond the tables
        ctx.query_attn_pool_batched(0, lists, [good], pos0=(1 << 20) - 10)
    assert e.value.status == ad.ECAPACITY
    torch.cuda.synchronize()
    assert float(out.float().min()) == 3.0 and float(out.float().max()) == 3.0     # nothing was launched
    ctx.query_attn_pool_batched(0, lists, [])              # no items: nothing to do
    ctx.query_attn_pool_batched(0, ([], None), [])
    ctx.close()


def test_zero_copy_plan_kept_for_the_next_layer(ad):
    """A single zero-copy call over the same shots at the same positions as the previous one (the next layer) keeps
    the slot table: bit-identical to a fresh context's result for that layer; another list in between rebuilds it."""
    w = wl.WORKLOADS["llama8b_1layer"]
    L = 2
    k_pool, v_pool, off = wl.make_pool(w, "cuda", n_layers=L)
    ids, order = wl.selection(w)
    ids, order = ids[:40], np.argsort(np.argsort(order[:40])).astype(np.int32)
    total = int(sum(off[i + 1] - off[i] for i in ids))
    q, ks, vs = wl.make_query(w, "cuda", t_q=33)

    def fresh(layer, the_ids, the_order, n):
        c2 = ad.Context.for_workload(w, n_layers=L)
        c2.pool_register(k_pool, v_pool, off)
        o = c2.query_attn_pool(layer, the_ids, the_order, q, ks, vs, n)
        torch.cuda.synchronize()
        c2.close()
        return o

    ctx = ad.Context.for_workload(w, n_layers=L)
    ctx.pool_register(k_pool, v_pool, off)
    for layer in (0, 1, 1, 0):
        o = ctx.query_attn_pool(layer, ids, order, q, ks, vs, total)
        assert torch.equal(o.view(torch.int16), fresh(layer, ids, order, total).view(torch.int16)), layer
    other = ids[::-1].copy()
    n2 = int(sum(off[i + 1] - off[i] for i in other[:7]))
    o = ctx.query_attn_pool(1, other[:7], None, q, ks, vs, n2)
    assert torch.equal(o.view(torch.int16), fresh(1, other[:7], None, n2).view(torch.int16))
    o = ctx.query_attn_pool(1, ids, order, q, ks, vs, total)
    assert torch.equal(o.view(torch.int16), fresh(1, ids, order, total).view(torch.int16))
    o = ctx.query_attn_pool(0, ids, order, q, ks, vs, total + 3, pos0=3)      # same shots, other positions
    c2 = ad.Context.for_workload(w, n_layers=L)
    c2.pool_register(k_pool, v_pool, off)
    ref = c2.query_attn_pool(0, ids, order, q, ks, vs, total + 3, pos0=3)
    assert torch.equal(o.view(torch.int16), ref.view(torch.int16))
    c2.close()
    ctx.close()


@pytest.mark.parametrize("t_q", [1, 2])
def test_zero_copy_of_few_rows_is_cut_like_the_tile_kernel_wants_it(ad, t_q):
    """A few-row call over 160 shots gives the bits of the split count that a call of 16 rows per kv head over as many
    slots gets (the tile kernel's plan depends on the row tiles, not on the rows in them)."""
    w = wl.WORKLOADS["llama8b_1layer"]
    k_pool, v_pool, off = wl.make_pool(w, "cuda", n_layers=1)
    ids = wl.selection(w)[0][:160]
    total = int(np.sum(off[ids + 1] - off[ids]))
    ctx = ad.Context.for_workload(w, n_layers=1)
    ctx.pool_register(k_pool, v_pool, off)
    q, ks, vs = wl.make_query(w, "cuda", t_q=t_q)
    auto = ctx.query_attn_pool(0, ids, None, q, ks, vs, total)
    n_split, _ = ad.attn_split_plan(w.n_q_heads, w.n_kv_heads, 128, ad.BF16, torch.cuda.get_device_properties(0).multi_processor_count,
                                    4, total)
    ctx.set_attn_splits(n_split)
    assert torch.equal(auto, ctx.query_attn_pool(0, ids, None, q, ks, vs, total))
    ctx.set_attn_splits(n_split - 8)                   # another split count rounds elsewhere: the comparison sees it
    assert not torch.equal(auto, ctx.query_attn_pool(0, ids, None, q, ks, vs, total))
    ctx.close()
