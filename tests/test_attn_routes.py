"""Which kernel an attention call of a bf16 / head_dim 128 model runs (csrc/attn_plan.h), compiled here with the host compiler.  No GPU."""
import ctypes
import os
import subprocess

import pytest

from paper_2605_03644_amd import binding as ad

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "attn_plan.h"
using namespace adapshot;
extern "C" int32_t by_tiles(const adapshot_model_desc* d, int32_t t_q, int64_t n_ctx) { return single_by_tiles(*d, t_q, n_ctx, false, 256); }
extern "C" int32_t by_stream(const adapshot_model_desc* d, const adapshot_attn_item* items, int32_t n) { return batch_by_stream(*d, items, n, 256); }
extern "C" int64_t workgroups(const adapshot_model_desc* d, const int64_t* rows, const int64_t* tiles, int32_t n) {
    std::vector<StreamShape> s;
    for (int32_t i = 0; i < n; ++i) s.push_back(StreamShape{rows[i], tiles[i]});
    const StreamPlan p = plan_stream(*d, 256, 0, s.data(), n);
    int64_t wgs = 0;
    for (const StreamShape& x : s) wgs += stream_units(*d, x, p.row_blocks) * stream_splits(x, p.split_tiles);
    return wgs;
}
"""
MODELS = [(32, 8), (28, 4), (64, 8), (16, 16), (8, 1), (4, 4), (200, 200)]
SLOTS = [0, 1, 63, 250, 1000, 1024, 1025, 1700, 2400, 4000, 9000, 12261, 16000, 24461, 30000, 48828, 48829, 97656, 97657, 200000, 400000]


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("routes") / "routes.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2605_03644_amd", "csrc"), "-x", "c++", "-", "-o", so], input=SHIM.encode(), check=True)
    lib = ctypes.CDLL(so)
    lib.workgroups.restype = ctypes.c_int64
    return lib


def _desc(hq, hkv):
    return ad.ModelDesc(1, hq, hkv, 128, 5.0e5, ad.BF16, ad.KEYS_UNROTATED, 1 << 20)


def _bytes(hkv, slots):
    return slots * hkv * 512


def _by_stream(plan, d, t_q, slots, caches=None):
    its = (ad.AttnItem * len(slots))()
    for i, n in enumerate(slots):
        its[i].t_q, its[i].n_ctx, its[i].cache_index = t_q, n, i if caches is None else caches[i]
    return bool(plan.by_stream(ctypes.byref(d), its, ctypes.c_int32(len(slots))))


@pytest.mark.parametrize("hq,hkv", MODELS)
def test_calls_of_few_rows_keep_their_fp32_partials(plan, hq, hkv):
    """The streaming kernel's partials are fp32, the tile kernel's 16-bit rows.  Up to 8 rows, and up to 16 over 1024 slots, a single call
    takes the streaming kernel as far as the context is 200 MB, a batch of one up to 16 rows, however cheap the tile kernel would be."""
    d, g, seen = _desc(hq, hkv), hq // hkv, set()
    for t_q in range(1, 16 // g + 1):
        for n in SLOTS:
            few = _bytes(hkv, n) <= 200000000
            single = not plan.by_tiles(ctypes.byref(d), ctypes.c_int32(t_q), ctypes.c_int64(n))
            if few and (t_q * g <= 8 or n <= 1024):
                assert single, (t_q, n)
            assert few or not single
            assert _by_stream(plan, d, t_q, [n]) == few, (t_q, n)
            seen.add(few)
    assert seen == {True, False}


@pytest.mark.parametrize("hq,hkv", MODELS)
def test_a_batch_of_one_streams_where_the_single_call_does(plan, hq, hkv):
    d, g = _desc(hq, hkv), hq // hkv
    for t_q in (1, 3, 8, 17, 32, 64, 128, 600, 5000):
        for n in SLOTS:
            single = not plan.by_tiles(ctypes.byref(d), ctypes.c_int32(t_q), ctypes.c_int64(n))
            assert _by_stream(plan, d, t_q, [n]) == (single or (t_q * g <= 16 and _bytes(hkv, n) <= 200000000))


@pytest.mark.parametrize("hq,hkv", [(32, 8), (28, 4)])
def test_batches_of_decode_steps(plan, hq, hkv):
    """Up to 300 MB of contexts of their own; beyond that the tile kernel draws more from the memory than the rest of it costs."""
    d = _desc(hq, hkv)
    for nq in (2, 7, 32, 48):
        at = 300000000 // (hkv * 512 * nq)
        assert _by_stream(plan, d, 1, [at] * nq) and not _by_stream(plan, d, 1, [at] * (nq - 1) + [at + 200])
        assert _by_stream(plan, d, 16 * hkv // hq, [at] * nq)
        assert not _by_stream(plan, d, 16 * hkv // hq + 1, [64] * nq)
        assert not _by_stream(plan, d, 1, [64] * nq, [0] * nq) and _by_stream(plan, d, 1, [0] * nq, [0] * nq)


@pytest.mark.parametrize("hq,hkv", [(32, 8), (28, 4), (8, 2)])
@pytest.mark.parametrize("nq", [1, 2, 3, 4, 6, 8])
@pytest.mark.parametrize("n", [1000, 2000, 4000, 8000, 16000])
def test_a_few_decode_steps_fill_the_chip_at_most_once(plan, hq, hkv, nq, n):
    """A workgroup takes a compute unit: a 257th one starts when the first has ended."""
    lens = [int(n * (0.9 + 0.2 * ((7 * i) % 11) / 11)) for i in range(nq)]
    arr = lambda x: (ctypes.c_int64 * len(x))(*x)  # noqa: E731
    wgs = plan.workgroups(ctypes.byref(_desc(hq, hkv)), arr([hq // hkv] * nq), arr([-(-x // 64) for x in lens]), ctypes.c_int32(nq))
    assert min(28, hkv * nq * (n // 64)) <= wgs <= 256


@pytest.mark.parametrize("hq,hkv,d,dtype", [(8, 2, 128, ad.F32), (4, 2, 64, ad.F32), (32, 8, 64, ad.BF16), (28, 4, 128, ad.BF16), (8, 4, 256, ad.BF16)])
def test_a_launch_makes_the_splits_of_the_public_plan(plan, hq, hkv, d, dtype):
    """Also where the query's own tokens would give the last split another step (they were a split of their own there, which the public
    plan did not name)."""
    desc, g = ad.ModelDesc(1, hq, hkv, d, 5.0e5, dtype, ad.KEYS_UNROTATED, 1 << 20), hq // hkv
    arr = lambda x: (ctypes.c_int64 * 1)(x)  # noqa: E731
    for t_q in (1, 2, 16, 64):
        for n in (1, 63, 64, 256, 2300, 3315, 8100, 30000):
            if dtype == ad.BF16 and d == 128 and t_q * g > 8:
                continue
            n_split, _ = ad.attn_split_plan(hq, hkv, d, dtype, 256, t_q, n)
            wgs = plan.workgroups(ctypes.byref(desc), arr(t_q * g), arr(-(-n // 64)), ctypes.c_int32(1))
            units = hkv * -(-t_q * g // 16)
            assert wgs in (n_split * units, n_split * hkv * -(-t_q * g // 32))   # one or two row blocks a workgroup
