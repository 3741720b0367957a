"""How the shots of an assembly reach its kernel (csrc/assemble_plan.h), compiled here with the host compiler.  No GPU."""
import ctypes
import os
import subprocess

import pytest

from paper_2605_03644_amd import binding as ad
from tests import helpers as H

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "assemble_plan.h"
extern "C" int32_t route(const adapshot_model_desc* d, int64_t caches, int64_t runs, int64_t tok, int64_t blocks, int64_t tiles) {
    return adapshot::assemble_route(*d, caches, runs, tok, blocks, tiles);
}
"""
ONE, FEW, LIST, TILES = range(4)


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("routes") / "routes.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2605_03644_amd", "csrc"), "-x", "c++", "-", "-o", so], input=SHIM.encode(), check=True)
    lib = ctypes.CDLL(so)

    def call(layers, hkv, d, dtype, caches, runs, tok, tiles=None):
        row = hkv * d * (4 if dtype == ad.F32 else 2)
        wg = H.constant("kTileTok")
        while wg > 1 and wg * row > 16384:
            wg //= 2
        blocks = -(-tok // wg)
        tiles = -(-tok // (wg if layers >= H.constant("kAssemblePieceLayers") else 32)) if tiles is None else tiles
        desc = ad.ModelDesc(layers, hkv, hkv, d, 1.0e4, dtype, ad.KEYS_UNROTATED, 1 << 20)
        return lib.route(ctypes.byref(desc), *(ctypes.c_int64(x) for x in (caches, runs, tok, blocks, tiles)))
    return call


def _at(layers, hkv, d, dtype, mb=256):
    """The most tokens that write no more than so many MB."""
    return (mb << 20) // (2 * layers * hkv * d * (4 if dtype == ad.F32 else 2))


def _long(layers, hkv, d, dtype):
    """The same for lists of long shots, which stay with the tiles up to 512 MB in fp32 models and from 8 layers on, but for rows below 256 bytes."""
    e = 4 if dtype == ad.F32 else 2
    return _at(layers, hkv, d, dtype, 256 if hkv * d * e < 256 or (layers < 8 and dtype == ad.BF16) else 512)


@pytest.mark.parametrize("layers,hkv,d,dtype", [(1, 8, 128, ad.BF16), (28, 4, 128, ad.BF16), (80, 8, 128, ad.BF16), (2, 2, 64, ad.F32), (32, 2, 128, ad.BF16),
                                                (28, 1, 16, ad.BF16), (1, 1, 8, ad.F32)])
def test_one_cache_by_its_number_of_shots(route, layers, hkv, d, dtype):
    for tok in (1, 400, 10 ** 7):
        assert route(layers, hkv, d, dtype, 1, 1, tok) == route(layers, hkv, d, dtype, 1, 320, tok) == ONE
    assert route(layers, hkv, d, dtype, 1, 321, _long(layers, hkv, d, dtype)) == TILES
    assert route(layers, hkv, d, dtype, 1, 321, _long(layers, hkv, d, dtype) + 1) == LIST


@pytest.mark.parametrize("layers,hkv,d,dtype", [(1, 8, 128, ad.BF16), (28, 4, 128, ad.BF16), (80, 8, 128, ad.BF16), (2, 2, 64, ad.F32), (32, 2, 128, ad.BF16)])
def test_batches_by_caches_and_shots(route, layers, hkv, d, dtype):
    at = _long(layers, hkv, d, dtype)
    for tok in (8, at, at + 1, 10 ** 7):
        assert route(layers, hkv, d, dtype, 2, 272, tok) == route(layers, hkv, d, dtype, 8, 8, tok) == FEW
    for caches, runs in ((2, 273), (8, 273), (9, 9), (48, 300)):
        assert route(layers, hkv, d, dtype, caches, runs, at) == TILES and route(layers, hkv, d, dtype, caches, runs, at + 1) == LIST


@pytest.mark.parametrize("hkv,d,dtype", [(1, 16, ad.BF16), (1, 8, ad.F32), (1, 64, ad.BF16), (2, 64, ad.BF16), (3, 80, ad.BF16), (1, 96, ad.F32)])
def test_batches_of_narrow_rows(route, hkv, d, dtype):
    """Rows of less than 512 bytes: no batch of a launch of 16 layers and more, or of more than 4096 workgroups an operand, in the arguments."""
    for layers in (1, 2, 4, 8, 15):
        tok = 32 * (4096 // layers)
        assert route(layers, hkv, d, dtype, 2, 20, tok) == FEW
        assert route(layers, hkv, d, dtype, 2, 20, tok + 1) == (TILES if tok < _long(layers, hkv, d, dtype) else LIST)
    for layers in (16, 28, 80):
        assert route(layers, hkv, d, dtype, 2, 2, 40) == route(layers, hkv, d, dtype, 8, 272, _long(layers, hkv, d, dtype)) == TILES
        assert route(layers, hkv, d, dtype, 8, 272, _long(layers, hkv, d, dtype) + 1) == LIST


def test_lists_between_256_and_512_mb(route):
    """Short shots leave tiles of 32 tokens half empty, and pieces of a workgroup's size from a quarter of it on."""
    at = _at(2, 8, 128, ad.F32)
    assert route(2, 8, 128, ad.F32, 9, at // 48 + 1, at + 1) == LIST and route(2, 8, 128, ad.F32, 9, (at + 1) // 48, at + 1) == TILES
    assert route(2, 8, 128, ad.F32, 9, at, at) == TILES
    at = _at(28, 4, 128, ad.BF16)  # 16 slots a workgroup
    blocks = -(-(at + 1) // 16)
    assert route(28, 4, 128, ad.BF16, 9, 400, at + 1, 4 * blocks) == LIST and route(28, 4, 128, ad.BF16, 9, 400, at + 1, 4 * blocks - 1) == TILES
    assert route(28, 4, 128, ad.BF16, 9, 400, at, 4 * blocks) == TILES
