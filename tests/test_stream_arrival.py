"""Who merges the partials of a unit (csrc/arrival.h): every order in which the workgroups of a unit can arrive, look, leave and
finish, walked through with the kernel's steps on the header's functions.  No GPU, no HIP."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "arrival.h"
using namespace adapshot;
extern "C" unsigned left() { return kArrivalLeft; }
extern "C" int all(unsigned word, int n) { return arrived_all(word, n); }
extern "C" int role(unsigned word, int n, int last, int waits) { return merge_role(word, n, last != 0, waits != 0); }
"""
NOTHING, SHARE, ALL = 0, 1, 2


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("arrival") / "arrival.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2605_03644_amd", "csrc"), "-x", "c++",
                    "-", "-o", so], input=SHIM.encode(), check=True)
    so = ctypes.CDLL(so)
    so.left.restype = ctypes.c_uint
    return so


@pytest.mark.parametrize("n", [2, 3, 4])
@pytest.mark.parametrize("waits", [0, 1])
def test_every_order_merges_each_row_once_and_leaves_the_counter_at_zero(lib, n, waits):
    left = lib.left()
    # a workgroup: (state, word it saw, arrived last, role); the unit: (counter, exits, resets)
    start = (0, 0, 0, (("new", 0, 0, None),) * n)
    seen, todo, ends = {start}, [start], 0
    while todo:
        word, exits, resets, wgs = todo.pop()
        nexts = []

        def step(i, wg, word=word, exits=exits, resets=resets):
            nexts.append((word, exits, resets, wgs[:i] + (wg,) + wgs[i + 1:]))

        for i, (state, saw, last, role) in enumerate(wgs):
            if state == "new":                                   # fetch_add on the counter
                w = word + 1
                is_last = lib.all(w, n)
                if waits:
                    step(i, ("look", w, is_last, None), word=w)
                else:
                    r = lib.role(w, n, is_last, 0)
                    step(i, ("done", w, is_last, r), word=0 if is_last else w, resets=resets + is_last)
            elif state == "look" and not lib.all(saw, n):
                if saw != word:
                    step(i, ("look", word, last, None))          # the load, or an exchange that failed
                else:
                    step(i, ("leave", word + left, last, None), word=word + left)  # the exchange
            elif state in ("look", "leave"):                     # fetch_add on the exits, then the role
                r = lib.role(saw, n, last, 1) if state == "look" else lib.role(saw, n, last, 1)
                step(i, ("reset" if exits + 1 == n else "done", saw, last, r), exits=exits + 1)
            elif state == "reset":
                step(i, ("done", saw, last, role), word=0, exits=0, resets=resets + 1)
        if not nexts:
            assert all(w[0] == "done" for w in wgs) and (word, exits, resets) == (0, 0, 1)
            roles = sorted(w[3] for w in wgs)
            assert roles in ([SHARE] * n, [NOTHING] * (n - 1) + [ALL])
            assert waits or roles[-1] == ALL
            ends += 1
        for s in nexts:
            # nobody touches the counter after it was put back to zero
            assert s[2] == 0 or all(w[0] in ("done", "reset") for w in s[3]) or not waits
            if s not in seen:
                seen.add(s)
                todo.append(s)
    assert ends >= (2 if waits else 1)
