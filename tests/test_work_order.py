"""The order in which attention work is dealt to the eight XCDs (csrc/fp_order.hpp), compiled for the host: every (KV head, row) is
served once, and a launch on sparse lists does not depend on how densely each KV head keeps its blocks."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2603_06199_amd import build as hip_build

SHIM = """
#define __host__
#define __device__
#include "fp_order.hpp"
extern "C" int order_of(int sparse, int d, int parts, int m, int hkv, int g, long long kv) { return fp::attn_order(sparse, d, parts, m, hkv, g, kv); }
extern "C" int two_groups(int d, int block, int lists, int wg, int n_max) { return fp::search_two_groups(d, block, lists, wg, n_max); }
extern "C" int turns_of(int order, int m, int hkv) { return fp::attn_turns(order, m, hkv); }
extern "C" void items(int order, int m, int hkv, int *out) {   // [xcd][turn][2], -1 where there is none
    const int turns = fp::attn_turns(order, m, hkv);
    for (int x = 0; x < 8; ++x)
        for (int t = 0; t < turns; ++t) {
            int *o = out + 2 * (x * turns + t), hk = -1, rank = -1;
            const bool there = fp::attn_item<true>(order, x, t, m, hkv, hk, rank);
            o[0] = there ? hk : -1;
            o[1] = there ? rank : -1;
        }
}
"""
DEALT, BY_HEAD, ROUNDS = 0, 1, 2


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("order")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", hip_build.CSRC, "-o", str(d / "shim.so"), str(d / "shim.cpp")],
                   check=True, capture_output=True)
    so = ctypes.CDLL(os.fspath(d / "shim.so"))
    so.order_of.argtypes = [ctypes.c_int] * 6 + [ctypes.c_longlong]
    return so


def _items(lib, order, m, hkv):
    """Per XCD its (KV head, rank) in turn."""
    out = np.empty((8, lib.turns_of(order, m, hkv), 2), np.int32)
    lib.items(order, m, hkv, out.ctypes.data_as(ctypes.c_void_p))
    return [[tuple(int(v) for v in p) for p in x if p[0] >= 0] for x in out]


@pytest.mark.parametrize("hkv", (1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 16, 24, 32))
def test_every_item_once(lib, hkv):
    for m in list(range(1, 70)) + [127, 128, 129, 1000]:
        for order in (DEALT, ROUNDS) + ((BY_HEAD,) if 8 % hkv == 0 or hkv % 8 == 0 else ()):
            got = sorted(sum(_items(lib, order, m, hkv), []))
            assert got == [(h, r) for h in range(hkv) for r in range(m)], (order, m)


# a last round of fewer than eight rows falls to other XCDs for each head
@pytest.mark.parametrize("hkv", (1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 16, 24, 32))
def test_items_per_xcd(lib, hkv):
    for m in range(1, 70):
        for order in (DEALT, ROUNDS):
            assert max(len(x) for x in _items(lib, order, m, hkv)) <= -(-m * hkv // 8), (order, m)


# Weights fall with the rank.  Of eight consecutive ranks of a head an XCD takes one, which weighs no more than the mean of the eight
# before: over the whole head it gets at most its eighth and the heaviest row.  In the dealt order a head may begin within a turn:
# one more row.
@pytest.mark.parametrize("head_dim", (64, 128, 256))
@pytest.mark.parametrize("hq,hkv", ((32, 1), (32, 2), (24, 3), (32, 4), (28, 4), (32, 8), (16, 16), (48, 24)))
def test_share_of_every_head(lib, hq, hkv, head_dim):
    g = hq // hkv
    for m in (9, 12, 31, 32, 64, 65, 128, 200, 512):
        for parts in (1, 2):
            if m * hq * parts <= 256:      # one workgroup per CU at most: no shares
                continue
            order = lib.order_of(1, head_dim, parts, m, hkv, g, 512 * m * hkv)
            weight = np.arange(m, 0, -1)
            for x in _items(lib, order, m, hkv):
                mine = np.zeros(hkv)
                for hk, rank in x:
                    mine[hk] += weight[rank]
                assert (mine <= weight.sum() / 8 + (2 if order == DEALT else 1) * weight[0]).all(), (m, parts, order)


def test_rule(lib):
    small, large = 8 << 20, (128 << 20) + 1
    for hq, hkv in ((32, 4), (32, 8), (24, 3), (4, 1)):
        g = hq // hkv
        for d, most in ((64, 96), (128, 64), (256, 64)):
            for m in (1, 8, 9, 64, 65, 96, 97, 1000):
                assert lib.order_of(0, d, 1, m, hkv, g, small) == (DEALT if hkv == 3 else BY_HEAD)   # full attention: heads are alike
                assert lib.order_of(0, d, 1, m, hkv, g, large) == lib.order_of(1, d, 1, m, hkv, g, large) == DEALT
                want = (DEALT if hkv == 3 else BY_HEAD) if m * hq <= 256 else ROUNDS if m <= most else DEALT
                assert lib.order_of(1, d, 1, m, hkv, g, small) == want
        # a launch that the pair kernel takes (q-blocks for half the CUs at most) never asks for rounds
        assert all(lib.order_of(s, d, 1, m, hkv, g, small) != ROUNDS for s in (0, 1) for d in (64, 128) for m in range(1, 128 // hq + 1))
        assert lib.order_of(1, 128, 2, 32, hkv, 64 // hkv, small) == ROUNDS and lib.order_of(1, 128, 2, 33, hkv, 64 // hkv, small) == DEALT


# (head dimension, block, lists in one pass): the longest rows on which a second group of waves was measured to lose, the shortest on
# which it gains
@pytest.mark.parametrize("form,loses,gains", (((64, 128, 0), 80, 128), ((64, 128, 1), 80, 160), ((128, 128, 0), 160, 256), ((128, 128, 1), 320, 416),
                                              ((128, 64, 0), 160, 256), ((128, 64, 1), 192, 256), ((128, 256, 0), 192, 288), ((128, 256, 1), 192, 288),
                                              ((256, 128, 0), 320, 448), ((256, 128, 1), 384, 448)))
def test_second_group_of_the_search(lib, form, loses, gains):
    assert not any(lib.two_groups(*form, wg, n) for wg in (1, 100, 256) for n in range(1, loses + 1))
    assert all(lib.two_groups(*form, wg, n) for wg in (1, 100, 256) for n in range(gains, 4097))
    assert not any(lib.two_groups(*form, 257, n) for n in range(1, 4097))
