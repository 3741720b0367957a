"""How attention calls are cut into workgroups (csrc/attn_plan.h): host logic over sizes, compiled here with the host compiler
and called directly.  No GPU, no HIP."""
import ctypes
import heapq
import math
import os
import random
import subprocess
import time

import pytest

from paper_2605_03644_amd import binding as ad

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "attn_plan.h"
using namespace adapshot;
extern "C" void single(const adapshot_model_desc* d, int64_t n_cu, int32_t t_q, int64_t n_ctx, int32_t zero_copy, int64_t* out) {
    out[0] = single_by_tiles(*d, t_q, n_ctx, zero_copy != 0);
    plan_single_attn(*d, n_cu, 0, t_q, n_ctx, zero_copy != 0, out + 1, out + 2);
}
extern "C" int64_t tile_splits(int64_t n_cu, int64_t units, int64_t key_tiles, int64_t self_tiles) {
    return plan_mfma_splits(n_cu, units, key_tiles, self_tiles);
}
extern "C" int32_t row_blocks(const adapshot_model_desc* d, int64_t n_cu, const int64_t* rows, const int64_t* tiles, int32_t n) {
    std::vector<StreamShape> s;
    for (int32_t i = 0; i < n; ++i) s.push_back(StreamShape{rows[i], tiles[i]});
    return stream_row_blocks(*d, n_cu, s.data(), n);
}
extern "C" void stream(const adapshot_model_desc* d, int64_t n_cu, int32_t force, const int64_t* rows, const int64_t* tiles,
                       int32_t n, int64_t* out) {
    std::vector<StreamShape> s;
    for (int32_t i = 0; i < n; ++i) s.push_back(StreamShape{rows[i], tiles[i]});
    const StreamPlan p = plan_stream(*d, n_cu, force, s.data(), n);
    out[0] = p.row_blocks, out[1] = p.units, out[2] = p.split_tiles, out[3] = p.n_split;
}
static std::vector<BatchShape> batch(const int64_t* shapes, int32_t n) {
    std::vector<BatchShape> s;
    for (int32_t i = 0; i < n; ++i) s.push_back(BatchShape{shapes[3 * i], shapes[3 * i + 1], shapes[3 * i + 2]});
    return s;
}
extern "C" int64_t balanced(int64_t n_cu, const int64_t* shapes, int32_t n) { return plan_balanced_split_tiles(n_cu, batch(shapes, n)); }
extern "C" int64_t equal_splits(int64_t n_cu, const int64_t* shapes, int32_t n) { return plan_batch_split_tiles(n_cu, batch(shapes, n), 0); }
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("plan") / "plan.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2605_03644_amd", "csrc"), "-x", "c++", "-", "-o", so], input=SHIM.encode(), check=True)
    lib = ctypes.CDLL(so)
    lib.tile_splits.restype = lib.balanced.restype = lib.equal_splits.restype = ctypes.c_int64
    return lib


def _desc(hq, hkv, d, dtype):
    return ad.ModelDesc(1, hq, hkv, d, 5.0e5, dtype, ad.KEYS_UNROTATED, 1 << 20)


def _single(plan, desc, t_q, n_ctx, zero_copy, n_cu=256):
    """(runs the tile kernel, splits, keys per split)"""
    out = (ctypes.c_int64 * 3)()
    plan.single(ctypes.byref(desc), ctypes.c_int64(n_cu), ctypes.c_int32(t_q), ctypes.c_int64(n_ctx), ctypes.c_int32(zero_copy), out)
    return tuple(out)


@pytest.mark.parametrize("hq,hkv", [(32, 8), (28, 4), (64, 8), (4, 4)])
@pytest.mark.parametrize("t_q", [1, 2, 4, 64])
@pytest.mark.parametrize("n_ctx", [64, 600, 2500, 16000, 26000, 60000])
def test_a_zero_copy_call_is_planned_for_the_kernel_it_runs(plan, hq, hkv, t_q, n_ctx):
    """bf16 / head_dim 128: the tile kernel, however few rows there are."""
    tiles, n_split, keys = _single(plan, _desc(hq, hkv, 128, ad.BF16), t_q, n_ctx, 1)
    assert tiles
    units, key_tiles = hkv * -(-t_q * (hq // hkv) // 256), -(-n_ctx // 64)
    want = plan.tile_splits(ctypes.c_int64(256), ctypes.c_int64(units), ctypes.c_int64(key_tiles), ctypes.c_int64(-(-t_q // 64)))
    assert keys == -(-key_tiles // want) * 64 and n_split == -(-n_ctx // keys)
    # other shapes have a gathered form of the streaming kernel, and are planned like a call over a cache
    for d, dtype in ((64, ad.BF16), (128, ad.F32)):
        assert _single(plan, _desc(hq, hkv, d, dtype), t_q, n_ctx, 1) == _single(plan, _desc(hq, hkv, d, dtype), t_q, n_ctx, 0)
        assert not _single(plan, _desc(hq, hkv, d, dtype), t_q, n_ctx, 1)[0]


def _row_blocks(plan, desc, rows, tiles, n_cu=256):
    arr = lambda x: (ctypes.c_int64 * len(x))(*x)  # noqa: E731
    return plan.row_blocks(ctypes.byref(desc), ctypes.c_int64(n_cu), arr(rows), arr(tiles), ctypes.c_int32(len(rows)))


@pytest.mark.parametrize("dtype", [ad.BF16, ad.F32])
def test_two_row_blocks_only_where_the_problems_fill_them(plan, dtype):
    """Many problems of one 16-row block each are many rows, but no workgroup of two blocks would have a second one."""
    d = _desc(32, 8, 64, dtype)
    for n in (1, 16, 32):
        for rows in (1, 4, 16):
            assert _row_blocks(plan, d, [rows] * n, [63] * n) == 1
    assert _row_blocks(plan, d, [16] * 31 + [32], [63] * 32) == 1
    assert _row_blocks(plan, d, [32] * 32, [63] * 32) == 2
    assert _row_blocks(plan, d, [48] * 32, [63] * 32) == 2
    assert _row_blocks(plan, _desc(128, 128, 64, dtype), [16], [63]) == 1
    # what one problem alone gets: two blocks from half a workgroup (fp32: two) per compute unit on
    assert _row_blocks(plan, d, [256], [63]) == (2 if dtype == ad.BF16 else 1)
    assert _row_blocks(plan, d, [240], [63]) == 1
    assert _row_blocks(plan, d, [1024], [2]) == 2
    assert _row_blocks(plan, _desc(32, 8, 128, ad.F32), [1024], [63]) == 1


def _stream(plan, desc, rows, tiles, force=0, n_cu=256):
    """(row blocks, units, tiles per split, splits of the longest problem)"""
    arr = lambda x: (ctypes.c_int64 * len(x))(*x)  # noqa: E731
    out = (ctypes.c_int64 * 4)()
    plan.stream(ctypes.byref(desc), ctypes.c_int64(n_cu), ctypes.c_int32(force), arr(rows), arr(tiles), ctypes.c_int32(len(rows)), out)
    return tuple(out)


@pytest.mark.parametrize("hq,hkv,d,dtype", [(32, 8, 64, ad.F32), (32, 8, 64, ad.BF16), (8, 8, 128, ad.F32), (28, 4, 128, ad.BF16)])
def test_the_public_plan_is_the_launch_s_plan(plan, hq, hkv, d, dtype):
    """adapshot_attn_split_plan names the splits that the launch makes, also beyond 4096 units, where it makes none."""
    desc, g = _desc(hq, hkv, d, dtype), hq // hkv
    beyond = 0
    for t_q in (1, 2, 100, 2048, 4130, 9000):
        for n_ctx in (1, 64, 700, 6400, 40000):
            if dtype == ad.BF16 and d == 128 and t_q > 1:     # the tile kernel
                continue
            n_split, keys = ad.attn_split_plan(hq, hkv, d, dtype, 256, t_q, n_ctx)
            _, units, tiles, splits = _stream(plan, desc, [t_q * g], [-(-n_ctx // 64)])
            assert (n_split, keys) == (splits, tiles * 64)
            assert splits == 1 or units <= 4096
            assert splits <= 64 and splits * keys >= n_ctx > (splits - 1) * keys
            beyond += units > 4096
            forced = _stream(plan, desc, [t_q * g], [-(-n_ctx // 64)], force=100)
            assert forced[3] <= (64 if units <= 4096 else 1)
    assert beyond or (dtype == ad.BF16 and d == 128)
    assert ad.attn_split_plan(hq, hkv, d, dtype, 256, 1, 0) == (0, 64)
    assert _stream(plan, desc, [g], [0])[2:] == (1, 1)


def _batch(f, shapes, n_cu=256):
    flat = [x for s in shapes for x in s]
    return f(ctypes.c_int64(n_cu), (ctypes.c_int64 * len(flat))(*flat), ctypes.c_int32(len(shapes)))


def _balanced_by_dealing(shapes, n_cu):
    """The rule of plan_balanced_split_tiles, every workgroup dealt by itself."""
    longest, total = max([1] + [t for _, t, _ in shapes]), sum(u * t for u, t, _ in shapes)
    cand = [-(-longest // n) for n in (1, 2, 3, 4, 6, 8)]
    cand += [math.ceil(total * f / (k * n_cu)) for k in (1, 2, 3, 4) for f in (1.02, 1.05, 1.1)]
    best, best_t = longest, math.inf
    for st in sorted({min(longest, max(min(8, longest), c)) for c in cand}, reverse=True):
        wgs = []
        for units, tiles, own in shapes:
            wgs += ([st + 2.5] * (tiles // st) + [tiles % st + 2.5] * (tiles % st > 0) + [own + 2.5]) * units
        if len(wgs) > 64 * n_cu:
            continue
        busy, end = [0.0] * n_cu, 0.0
        for w in sorted(wgs, reverse=True):
            t = heapq.heappop(busy) + w
            heapq.heappush(busy, t)
            end = max(end, t)
        if end + 0.13 * len(wgs) < best_t:
            best, best_t = st, end + 0.13 * len(wgs)
    return best


def test_balanced_split_length(plan):
    rng = random.Random(3)
    for _ in range(60):
        hkv = rng.choice([1, 2, 3, 4, 5, 7, 8])
        shapes = [(hkv * rng.randint(1, 2), rng.randint(0, 500), rng.randint(1, 2)) for _ in range(rng.randint(1, 20))]
        n_cu = rng.choice([64, 104, 256])
        if sum(u * t for u, t, _ in shapes) < 32 * n_cu:
            assert _batch(plan.balanced, shapes, n_cu) == _batch(plan.equal_splits, shapes, n_cu)
        else:
            assert _batch(plan.balanced, shapes, n_cu) == _balanced_by_dealing(shapes, n_cu)


@pytest.mark.parametrize("hkv", [1, 3, 4, 5, 7, 8])
def test_balanced_split_length_costs_what_the_items_cost(plan, hkv):
    """The host's time for a plan follows the items, not the workgroups: a few times that of the equal splits' plan, whatever
    the number of KV heads (dealt one by one, 64 items of 5 or 7 KV heads took 13 to 16 times as long)."""
    rng = random.Random(hkv)
    shapes = [(hkv, rng.randint(100, 700), 1) for _ in range(64)]

    def best(f):
        t = math.inf
        for _ in range(15):
            t0 = time.perf_counter()
            for _ in range(4):
                _batch(f, shapes)
            t = min(t, time.perf_counter() - t0)
        return t

    assert best(plan.balanced) < 7 * best(plan.equal_splits)
