"""Who owns a share of the persistent launch (csrc/mq_routes.h), compiled for the CPU: measured stacks and single layers on the faster side, and the calls by which
the GPU tests reach either kernel."""
import ctypes
import os
import subprocess

import pytest

from test_gpu_shares import LONG, MANY, SMALL, WHOLE, few_shares, stack_of
from test_gpu_wave_shares import SINGLES, STACKS, _shapes

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "mq_routes.h"
using namespace mq;
extern "C" int waves(int n, const int *RB, const int *G, const int *r, int64_t M) {
    return wave_shares(n, M, [&](int i) { return RowLayer{RB[i], G[i], r[i]}; });
}
extern "C" int waves_single(int r, int64_t M) { return wave_shares_single(r, M); }
extern "C" int low_latency(int64_t RB, int64_t G, int r, int64_t M) { return low_latency_call(RB, G, r, M, (size_t)1 << 24); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("shares")
    (d / "s.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC",
                           "-I", os.path.join(ROOT, "paper_2602_03537_amd", "csrc"), str(d / "s.cpp"), "-o", str(d / "s.so")])
    return ctypes.CDLL(str(d / "s.so"))


def _waves(lib, shapes, widths, M):
    n = len(shapes)
    ints = ctypes.c_int * n
    return bool(lib.waves(n, ints(*[-(-N // 64) for N, _ in shapes]), ints(*[K // 128 for _, K in shapes]), ints(*widths), ctypes.c_int64(M)))


def _block(hidden, kv, ffn):
    return [(hidden, hidden), (kv, hidden), (kv, hidden), (hidden, hidden), (ffn, hidden), (ffn, hidden), (hidden, ffn)]


# a block's layers, blocks, widths in turn, M: us, shares of workgroups and of waves
@pytest.mark.parametrize("block,blocks,widths,M,workgroups,waves", [
    ((4096, 4096, 11008), 32, (2,), 1, 382.2, 313.0), ((4096, 4096, 11008), 32, (3,), 1, 432.9, 412.3), ((4096, 4096, 11008), 32, (4,), 1, 516.5, 546.4),
    ((4096, 4096, 11008), 32, (8,), 1, 975.2, 996.3), ((4096, 4096, 11008), 32, (2, 3, 4, 6, 8), 1, 614.8, 693.4), ((4096, 4096, 11008), 32, (2, 2, 2, 2, 8), 1, 468.3, 520.3),
    ((8192, 1024, 28672), 4, (2,), 1, 191.5, 162.3), ((8192, 1024, 28672), 4, (3,), 1, 224.7, 215.3), ((8192, 1024, 28672), 4, (4,), 1, 268.9, 273.8),
    ((2048, 512, 5632), 22, (2,), 1, 74.7, 58.3), ((2048, 512, 5632), 22, (3,), 1, 91.6, 72.9), ((2048, 512, 5632), 22, (8,), 1, 157.2, 161.2),
    ((4096, 4096, 11008), 32, (2,), 2, 379.0, 322.0), ((4096, 4096, 11008), 32, (4,), 3, 535.3, 572.0), ((4096, 4096, 11008), 32, (2,), 4, 408.3, 372.1),
    ((1280, 1152, 4608), 26, (3, 4), 4, 78.6, 58.2), ((1280, 1152, 4608), 26, (3, 4), 8, 89.9, 59.0), ((4096, 4096, 11008), 32, (8,), 5, 1030.5, 1116.2),
    ((8064, 2304, 1280), 9, (3, 4), 1, 170.4, 140.7), ((4096, 3840, 1152), 6, (2, 8), 9, 90.4, 78.4), ((6016, 832, 1280), 14, (3, 4), 4, 161.5, 128.5), ((1408, 384, 7808), 15, (6,), 5, 103.1, 90.7), ((1664, 576, 1280), 40, (6,), 8, 102.5, 91.4),
    ((512, 256, 16512), 40, (4,), 16, 200.9, 155.2), ((6784, 1216, 1408), 10, (4,), 16, 186.8, 170.6), ((128, 3136, 13568), 40, (3,), 12, 165.7, 48.3),
    ((128, 960, 10112), 40, (2, 8), 9, 155.2, 42.5), ((1280, 1152, 4608), 26, (3, 4), 16, 106.2, 86.0), ((2048, 512, 5632), 22, (2,), 16, 119.6, 100.0),
    ((4096, 4096, 11008), 32, (2,), 16, 564.4, 511.0), ((4096, 4096, 11008), 32, (4,), 16, 732.7, 716.6), ((4096, 4096, 11008), 32, (8,), 16, 1139.3, 1148.0),
    ((4096, 4096, 11008), 32, (2, 3, 4, 6, 8), 16, 809.9, 860.8), ((8192, 1024, 28672), 4, (3,), 16, 344.7, 335.1),
    ((8192, 1024, 28672), 4, (2, 4, 8), 16, 412.3, 428.1), ((8192, 1024, 28672), 4, (8,), 16, 569.6, 586.4)])
def test_stacks_take_the_faster_shares(lib, block, blocks, widths, M, workgroups, waves):
    shapes = _block(*block) * blocks
    assert _waves(lib, shapes, [widths[i % len(widths)] for i in range(len(shapes))], M) == (waves < workgroups)


@pytest.mark.parametrize("r,M,workgroups,waves", [(2, 1, 49.6, 52.0), (2, 4, 27.2, 25.4), (2, 3, 35.5, 33.4), (3, 4, 54.7, 61.4), (6, 8, 46.7, 52.4)])
def test_single_layers_take_the_faster_shares(lib, r, M, workgroups, waves):
    assert bool(lib.waves_single(r, ctypes.c_int64(M))) == (waves < workgroups)


def test_calls_by_which_the_gpu_tests_reach_shares_of_waves(lib):
    for name, (_, widths) in STACKS.items():
        shapes = _shapes(name)
        for M in (1, 2, 3, 4, 5, 8, 9, 16):
            assert _waves(lib, shapes, [widths[i % len(widths)] for i in range(17)], M), (name, M)
        if name in ("few_groups", "one_group", "short", "eight_groups"):
            assert _waves(lib, shapes, [8] * 17, 4), name
    for N, K in SINGLES:
        for M in (2, 3, 4):
            assert not lib.low_latency(ctypes.c_int64(-(-N // 64)), ctypes.c_int64(K // 128), 2, ctypes.c_int64(M)) and lib.waves_single(2, ctypes.c_int64(M))


def test_calls_by_which_the_gpu_tests_reach_shares_of_workgroups(lib):
    for shape in (LONG, MANY, SMALL, WHOLE):
        for M in (1, 2, 4, 5, 8, 9, 16):
            assert not _waves(lib, *stack_of(shape, M), M), (shape, M)
    for tiles in (238, 240):
        shapes = few_shares(tiles)
        assert sum(-(-N // 64) * (K // 128) for N, K in shapes) == tiles
        for M in (1, 3, 8, 16):
            assert not _waves(lib, shapes, [8] * 17, M), (tiles, M)
