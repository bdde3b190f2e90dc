"""How a wave of the persistent launch goes through its workgroup's share (csrc/mq_share_walk.h), compiled for the CPU: every tile once, in its row block, from
the slot it was fetched into, and a stored piece is counted only when the wait before it covers its stores, whatever the compiler adds."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#define __device__
#define __host__
#define __forceinline__ inline
#include "mq_share_walk.h"
using namespace mq;
// One wave's transfers in order of issue: `issued` so many, the piece's store the `store`-th.  loads: of a tile.  What is wrong: a line of the source.
template <int D, int NW> static int wave(int G, int begin, int end, int w, int loads, bool &partial_wait) {
    ShareWalk walk(G, begin, end);
    StoredPiece head;
    const int tail_rb = (end - 1) / G, tail_gb = end - tail_rb * G;
    const bool has_tail = tail_gb < G && tail_rb * G >= begin;
    int slots[D + 1], next = begin + w, bad = 0, at = begin;
    long issued = 0, store = -1;
    auto check = [&](bool ok, int line) { if (!ok && !bad) bad = line; };
    for (int &s : slots) s = -1;
    walk.template run<D, NW>(
        w, head,
        [&](auto slot, int u, int g) {
            check(u >= begin && u < end && g == u % G, __LINE__);
            slots[slot] = u;
            issued += loads;
        },
        [&](auto slot) {
            check(slots[slot] == next && next < end && next / G == walk.rb && next < walk.seg_end, __LINE__);
            next += NW;
        },
        [&](int gb) {
            check(walk.rb * G + walk.ga == at && walk.seg_end == walk.rb * G + gb && gb <= G, __LINE__);
            check(next >= walk.seg_end, __LINE__);
            at = walk.seg_end;
            const bool tail = has_tail && walk.seg_end == end;
            if (head.to_count()) {
                const long in_flight = head.template behind_loads<D>() ? (long)D * loads : 0;
                partial_wait |= in_flight > 0;
                check(store <= issued - in_flight, __LINE__);
                head.counted = true;
            }
            if (!(walk.ga == 0 && gb == G) && !tail) {
                check(head.n == 0, __LINE__);
                store = ++issued;
                head.stored(walk.rb, gb - walk.ga);
            }
        },
        [] {},
        [&] { for (int j = 0; j < D; ++j) slots[j] = slots[j + 1]; });
    check(at == end && next >= end, __LINE__);
    return bad;
}
template <int D, int NW> static int all(int *partial) {
    bool p = false;
    for (int G : {1, 2, 3, 5, 8, 9, 17, 40, 133})
        for (int begin = 0; begin < G; begin += G > 20 ? 7 : 1)
            for (int len = 1; len < 6 * NW + 2 * G; len += len > 4 * NW ? 5 : 1)
                for (int w = 0; w < NW; ++w)
                    for (int loads : {1, 7})
                        if (const int bad = wave<D, NW>(G, begin, begin + len, w, loads, p)) return bad;
    *partial = p;
    return 0;
}
extern "C" int walk(int D, int NW, int *partial) {
    if (NW == 8) return D == 1 ? all<1, 8>(partial) : D == 2 ? all<2, 8>(partial) : D == 3 ? all<3, 8>(partial) : all<4, 8>(partial);
    return D == 1 ? all<1, 16>(partial) : D == 2 ? all<2, 16>(partial) : D == 3 ? all<3, 16>(partial) : all<4, 16>(partial);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("walk")
    (d / "w.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC",
                           "-I", os.path.join(ROOT, "paper_2602_03537_amd", "csrc"), str(d / "w.cpp"), "-o", str(d / "w.so")])
    return ctypes.CDLL(str(d / "w.so"))


@pytest.mark.parametrize("waves", [8, 16])
@pytest.mark.parametrize("depth", [1, 2, 3, 4])
def test_every_tile_once_and_pieces_counted_behind_their_stores(lib, depth, waves):
    partial = ctypes.c_int(0)
    assert lib.walk(depth, waves, ctypes.byref(partial)) == 0   # otherwise the line of the source that was not met
    assert partial.value                                        # waits that leave loads in flight are among the cases
