"""The rules that choose a launch shape from sizes (csrc/mq_routes.h), compiled for the CPU: measured calls go to the faster side, and
every shape that a rule hands out is one that its kernel can run."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "mq_routes.h"
using namespace mq;
extern "C" void shares(int C, int64_t tiles, int64_t G, int resident, int *out) {
    const WideShares s = wide_shares(C, tiles, G, resident);
    out[0] = s.workers;
    out[1] = s.finish_apart;
}
extern "C" int single_rows(int64_t row_blocks, int64_t G, int64_t M, size_t part_bytes) { return row_kernels_single(row_blocks, G, M, part_bytes); }
extern "C" int single_low_latency(int64_t row_blocks, int64_t G, int r, int64_t M) { return low_latency_call(row_blocks, G, r, M, (size_t)1 << 24); }
extern "C" int single_low_latency_in(int64_t row_blocks, int64_t G, int64_t M, size_t part_bytes) { return low_latency_call(row_blocks, G, 4, M, part_bytes); }
extern "C" int stack_rows(int64_t M) { return row_kernels_stack(M); }
extern "C" int stack_low_latency(int n, const int *RB, const int *G, int64_t M, size_t part_bytes) {
    return low_latency_stack(n, M, part_bytes, [&](int i) { return RowLayer{RB[i], G[i], 4}; });
}
extern "C" int tile_cost(int r, int M, int by_wave) { return valu_tile_cost(r, M, by_wave); }
extern "C" void single_shape(int RB, int G, int M, int *out) {
    out[0] = pick_k_slices(RB, G, M);
    out[1] = quad_wave_tiles(G, out[0]);
}
extern "C" void stack_shape(int n, const int *RB, const int *G, int M, int resident, int *out) {
    const RowStackShape s = row_stack_shape(n, M, false, [&](int i) { return RowLayer{RB[i], G[i], 4}; }, [&](int) { return resident; });
    out[0] = s.blocks;
    out[1] = s.waves;
    out[2] = s.ks_cap;
    out[3] = s.all_resident;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("routes")
    (d / "r.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC",
                           "-I", os.path.join(ROOT, "paper_2602_03537_amd", "csrc"), str(d / "r.cpp"), "-o", str(d / "r.so")])
    return ctypes.CDLL(str(d / "r.so"))


def _passes(M):
    chunks = -(-M // 32)
    passes = -(-chunks // 4)
    return passes, -(-chunks // passes)


def _wide(lib, N, K, M, resident=256):
    passes, C = _passes(M)
    out = (ctypes.c_int * 2)()
    lib.shares(C, ctypes.c_int64(passes * -(-N // 256) * (K // 128)), ctypes.c_int64(K // 128), resident, out)
    return out[0], bool(out[1])


# (N, K, M) with the times of a call, us, r = 4: row blocks finished by their last contributor, and apart
@pytest.mark.parametrize("N,K,M,inside,apart", [
    (28672, 1024, 96, 26.2, 29.1), (28672, 1024, 128, 29.2, 32.0), (20000, 1024, 160, 26.7, 33.2), (20000, 1024, 256, 30.1, 36.5),
    (24000, 1024, 160, 26.7, 35.2), (17000, 1024, 256, 29.4, 36.8), (13003, 1024, 160, 26.0, 28.3), (28672, 8192, 24, 48.7, 49.3),
    (28672, 8192, 64, 60.5, 61.7), (20000, 2048, 32, 22.1, 23.4), (20000, 3072, 32, 23.9, 24.1),
    (13003, 1536, 256, 40.4, 34.3), (28672, 1536, 96, 34.9, 31.9), (4096, 1024, 128, 27.2, 22.7), (6000, 1024, 96, 24.2, 22.3),
    (8192, 512, 128, 31.6, 21.1), (28672, 512, 96, 28.7, 20.1), (4096, 11008, 128, 59.4, 35.5), (8192, 28672, 61, 63.9, 58.4),
    (20000, 4096, 48, 36.0, 33.5), (8192, 1536, 24, 22.3, 18.2), (20000, 1152, 128, 38.7, 32.0),
    (18975, 2048, 68, 31.4, 33.5), (9371, 2048, 166, 32.8, 35.2), (17043, 2048, 102, 38.4, 40.9), (11122, 2048, 176, 31.6, 33.2),
    (13464, 2048, 190, 37.4, 35.8), (12866, 2048, 252, 44.9, 42.6), (7848, 2048, 239, 35.7, 32.3), (7609, 2048, 133, 29.0, 26.8)])
def test_wide_row_blocks_are_finished_on_the_faster_side(lib, N, K, M, inside, apart):
    assert _wide(lib, N, K, M)[1] == (apart < inside)


def test_wide_shares_fit_the_device_and_own_a_tile_each(lib):
    rng = np.random.default_rng(701)
    for resident in (1, 8, 104, 256, 512):
        for _ in range(2000):
            N, K, M = int(np.exp(rng.uniform(0, 11))), 128 * int(np.exp(rng.uniform(0, 6))), int(rng.integers(17, 257))
            workers, _ = _wide(lib, N, K, M, resident)
            assert 1 <= workers <= resident
            assert workers <= _passes(M)[0] * -(-N // 256) * (K // 128)


PARTS = {16: 256 * 2 * 8 * 64 * 16 * 4, 32: 512 * 2 * 4 * 32 * 64 * 4, 64: 512 * 2 * 8 * 32 * 64 * 4, 96: 256 * 2 * 12 * 32 * 64 * 4, 128: 256 * 2 * 16 * 32 * 64 * 4}


def _part(M):
    """Bytes of partial sums in the workspace of a batch of M."""
    return PARTS[min(k for k in PARTS if M <= k)]


def _blocks(N):
    return -(-N // 64)


# (N, K, M) with the times of a call, us, r = 4, when the line was drawn, by 4x4x4 instructions: row kernel, and the wide kernel.  (By 16x16x32 instructions
# the row kernel is the faster one in all of these, csrc/mq_routes.h; the line has not been moved.)
@pytest.mark.parametrize("N,K,M,rows,other", [
    (13003, 2048, 32, 16.6, 21.0), (4096, 4096, 64, 18.5, 22.5), (6000, 1536, 112, 21.3, 26.6), (8192, 1024, 128, 21.1, 24.1),
    (20000, 768, 48, 20.1, 31.1), (8192, 768, 128, 19.9, 25.4),
    (4096, 8192, 64, 29.6, 23.5), (6000, 8192, 32, 29.8, 23.6), (2048, 14336, 96, 42.7, 28.4),
    (2048, 14336, 128, 44.9, 31.3), (1024, 28672, 128, 43.9, 34.9), (1500, 14336, 128, 43.0, 29.1), (2048, 28672, 48, 38.1, 29.8),
    (20000, 2048, 32, 25.8, 23.4), (17000, 2048, 32, 25.4, 21.6), (28672, 1024, 32, 21.0, 18.8), (28672, 1024, 48, 29.4, 22.7), (20000, 1024, 64, 25.7, 22.2)])
def test_single_layers_go_to_the_faster_kernel(lib, N, K, M, rows, other):
    assert bool(lib.single_rows(ctypes.c_int64(_blocks(N)), ctypes.c_int64(K // 128), ctypes.c_int64(M), ctypes.c_size_t(_part(M)))) == (rows < other)


# (N, K, M) with the times of a call, us, r = 4: low-latency, and persistent; what differs by less than 2 % may go either way
@pytest.mark.parametrize("N,K,M,low,persistent", [
    (4096, 4096, 16, 11.5, 9.6), (28672, 1024, 16, 10.4, 12.0), (12288, 8192, 9, 20.9, 18.6), (28672, 8192, 16, 31.4, 30.5), (8192, 28672, 16, 30.8, 28.5),
    (20000, 2048, 16, 13.0, 14.5), (8192, 8192, 16, 15.8, 14.3)])
def test_single_layers_of_9_to_16_rows_take_the_faster_launch(lib, N, K, M, low, persistent):
    assert bool(lib.single_low_latency(ctypes.c_int64(_blocks(N)), ctypes.c_int64(K // 128), 4, ctypes.c_int64(M))) == (low < persistent)


@pytest.mark.parametrize("M", (1, 4, 5, 8, 9, 16))
@pytest.mark.parametrize("N,K", [(1, 128), (1000, 28672), (12288, 8192), (13003, 5120), (28672, 27264), (448 * 64, 140 * 128), (28672, 28672)])
def test_calls_of_up_to_16_rows_go_to_the_row_kernels(lib, N, K, M):
    assert lib.single_rows(ctypes.c_int64(_blocks(N)), ctypes.c_int64(K // 128), ctypes.c_int64(M), ctypes.c_size_t(0)) and lib.stack_rows(ctypes.c_int64(M))


@pytest.mark.parametrize("M", (17, 32, 128, 256))
def test_stacks_of_more_go_to_the_wide_kernel(lib, M):
    assert not lib.stack_rows(ctypes.c_int64(M))


GATE_UP, QKV, QKV_70B = [(11008, 4096)] * 2, [(4096, 4096)] * 3, [(8192, 8192), (1024, 8192), (1024, 8192)]
UNEVEN = [(2048, 2048), (512, 2048), (512, 2048), (2048, 2048), (5504, 2048), (5504, 2048), (2048, 5504)]


def _arrays(layers):
    n = len(layers)
    return n, (ctypes.c_int * n)(*[_blocks(N) for N, _ in layers]), (ctypes.c_int * n)(*[K // 128 for _, K in layers])


# times of a launch, us, r = 2, M = 12: low-latency, and persistent
@pytest.mark.parametrize("layers,low,persistent", [
    (QKV, 12.8, 14.5), ([(11008, 4096)], 13.5, 13.6), ([(5504, 2048)] * 2, 10.4, 11.5), ([(1024, 1024)] * 2, 8.7, 9.1), (UNEVEN, 17.0, 15.4)],
    ids=["qkv", "one", "two", "one_k", "uneven"])
def test_small_stacks_of_9_to_16_rows_take_the_faster_launch(lib, layers, low, persistent):
    for M in (9, 12, 16):
        assert bool(lib.stack_low_latency(*_arrays(layers), ctypes.c_int64(M), ctypes.c_size_t(_part(16)))) == (low < persistent)


# gate and up of Llama-2-7B (eight tiles a wave): r = 2, M = 12 16.2 / 16.3, r = 4, M = 16 19.9 / 19.3; one 13824 x 5120 (five) 15.6 / 15.3, 17.7 / 18.2
def test_small_stacks_of_9_to_16_rows_where_the_launches_are_level(lib):
    for M in (9, 12, 16):
        assert not lib.stack_low_latency(*_arrays(GATE_UP), ctypes.c_int64(M), ctypes.c_size_t(_part(16)))
        assert lib.stack_low_latency(*_arrays([(13824, 5120)]), ctypes.c_int64(M), ctypes.c_size_t(_part(16)))


# tiles of 2 .. 8 bits beyond the low-latency launch: the persistent one, whoever owns its shares
@pytest.mark.parametrize("tiles", [13, 69, 134, 184])
def test_large_stacks_of_5_to_8_rows_take_the_persistent_launch(lib, tiles):
    n, RB, G = 1, (ctypes.c_int * 1)(tiles * 10), (ctypes.c_int * 1)(100)
    for M in (5, 8):
        assert not lib.stack_low_latency(n, RB, G, ctypes.c_int64(M), ctypes.c_size_t(1 << 30))


def _seven(hidden, kv, ffn):
    return [(hidden, hidden), (kv, hidden), (kv, hidden), (hidden, hidden), (ffn, hidden), (ffn, hidden), (hidden, ffn)]


# the layers of one block: times of a launch, us, r = 4, M = 8: low-latency, and persistent
@pytest.mark.parametrize("layers,low,persistent", [
    (_seven(1920, 3520, 7808), 25.2, 17.7), (_seven(1792, 2880, 7424), 24.1, 16.7), (_seven(1664, 3200, 7168), 22.9, 17.0),
    (_seven(2432, 3456, 7680), 24.8, 19.0), (_seven(1920, 1792, 11520), 23.2, 19.6), (_seven(1152, 960, 6528), 10.6, 17.4),
    (_seven(1920, 896, 2816), 10.6, 15.1), (_seven(1280, 2496, 7168), 12.8, 16.2), (_seven(1664, 1088, 3456), 11.4, 14.2)])
def test_small_stacks_of_5_to_8_rows_take_the_faster_launch(lib, layers, low, persistent):
    for M in (5, 8):
        assert bool(lib.stack_low_latency(*_arrays(layers), ctypes.c_int64(M), ctypes.c_size_t(_part(16)))) == (low < persistent)
    assert lib.stack_low_latency(*_arrays(layers), ctypes.c_int64(4), ctypes.c_size_t(_part(16)))


# Two layers of 92.9 million weights, 2 and 8 bits: with costs 3 times as large at 8 bits M = 2 and 3 took 31.6 us, where 1.6 to 2 times took 29.4;
# at M = 1 the costs are near the bytes, 3.4 times as many
@pytest.mark.parametrize("M,least,most", [(1, 2.5, 3.4), (2, 1.5, 2.1), (3, 1.5, 2.1)])
def test_cost_of_wide_tiles_in_mixed_stacks(lib, M, least, most):
    for by_wave in (0, 1):
        assert least <= lib.tile_cost(8, M, by_wave) / lib.tile_cost(2, M, by_wave) <= most
        costs = [lib.tile_cost(r, M, by_wave) for r in (2, 3, 6, 8)]
        assert costs == sorted(costs)


# shares of waves, three rows: 1.6 times as long at 8 bits, not 2.1
def test_cost_of_wide_tiles_in_shares_of_waves_of_three_rows(lib):
    assert lib.tile_cost(8, 3, 1) <= 1.7 * lib.tile_cost(2, 3, 1)
    for M in (1, 2, 4, 5, 8, 9, 16):
        assert all(lib.tile_cost(r, M, 1) == lib.tile_cost(r, M, 0) for r in (2, 3, 4, 6, 8))


def test_row_shapes_hold_to_their_bounds(lib):
    """At most eight slices of at least four groups (one of fewer), slots for all of them, at most four bits of a counter."""
    rng = np.random.default_rng(702)
    out = (ctypes.c_int * 4)()
    for _ in range(20000):
        RB, G, M = int(np.exp(rng.uniform(0, 9))), int(np.exp(rng.uniform(0, 6))), int(rng.integers(1, 129))
        lib.single_shape(RB, G, M, out)
        ks, tiles = out[0], out[1]
        assert 1 <= ks <= 8 and (ks == 1 or G // ks >= 4)
        chunks = -(-M // 16)
        if M > 8:
            assert ks == 1 or RB * ks * chunks <= 512
            part = int(np.exp(rng.uniform(10, 18)))
            if lib.single_low_latency_in(ctypes.c_int64(RB), ctypes.c_int64(G), ctypes.c_int64(M), ctypes.c_size_t(part)):
                assert RB * ks * chunks * 16 * 64 * 4 <= part and tiles <= 7 and chunks <= 8
        else:
            assert lib.single_rows(ctypes.c_int64(RB), ctypes.c_int64(G), ctypes.c_int64(M), ctypes.c_size_t(0))
    assert not lib.single_rows(ctypes.c_int64(1), ctypes.c_int64(1), ctypes.c_int64(129), ctypes.c_size_t(1 << 30))


def test_small_stack_shapes_are_resident_or_uncut(lib):
    rng = np.random.default_rng(703)
    out = (ctypes.c_int * 4)()
    for _ in range(5000):
        layers = [(64 * int(np.exp(rng.uniform(0, 5.5))), 128 * int(np.exp(rng.uniform(0, 5)))) for _ in range(int(rng.integers(1, 17)))]
        M, resident = int(rng.integers(1, 17)), int(rng.choice([64, 256, 512, 1024]))
        n, RB, G = _arrays(layers)
        lib.stack_shape(n, RB, G, M, resident, out)
        blocks, waves, cap, fits = out
        assert waves in (4, 8, 16) and cap in (0, 1, 2, 4) and bool(fits) == (blocks <= resident)
        assert fits or (waves == 4 and cap == 1)
        assert sum(RB) <= blocks <= 8 * sum(RB) and (cap == 0 or blocks <= cap * sum(RB))
    for n in (16, 17):   # more layers than a launch has arguments for
        assert bool(lib.stack_low_latency(*_arrays([(64, 128)] * n), ctypes.c_int64(16), ctypes.c_size_t(_part(16)))) == (n == 16)


def test_shapes_by_which_the_gpu_tests_reach_the_persistent_launch_and_the_wide_kernel(lib):
    def rows(N, K, M):
        return bool(lib.single_rows(ctypes.c_int64(_blocks(N)), ctypes.c_int64(K // 128), ctypes.c_int64(M), ctypes.c_size_t(_part(M))))
    def low_latency(N, K, M, r=3):
        return bool(lib.single_low_latency(ctypes.c_int64(_blocks(N)), ctypes.c_int64(K // 128), r, ctypes.c_int64(M)))
    for M in (9, 16):
        assert not low_latency(200, 233 * 128, M) and not low_latency(321, 233 * 128, M)
        assert not low_latency(12401, 8192, M) and not low_latency(8192, 28672, M)
    for M in (17, 64, 65, 128):
        assert not rows(200, 233 * 128, M) and _wide(lib, 200, 233 * 128, M)[1]     # finished by a launch of its own
    for M, N in ((20, 33000), (64, 16500), (65, 16500), (128, 16500)):
        assert not rows(N, 1152, M) and _wide(lib, N, 1152, M)[1] == (M > 64)
    for M in (20, 64):
        assert not rows(4200, 12672, M) and _wide(lib, 4200, 12672, M)[1]
    assert all(low_latency(12401, 8192, M, r) for M in (2, 3, 4, 5, 8) for r in (2, 3, 4, 6, 8))
    for M in (17, 33, 100, 128):
        assert all(rows(N, K, M) for N, K in ((1, 128), (65, 128), (200, 1152), (1000, 2176), (4100, 640)))
    assert not lib.stack_low_latency(*_arrays([(64, 128)] * 17), ctypes.c_int64(9), ctypes.c_size_t(_part(16)))
    for M, N in ((68, 17000), (128, 17000), (130, 8500)):
        assert (M > 128 or not rows(N, 2048, M)) and not _wide(lib, N, 2048, M)[1]    # finished by the last contributor
    assert not low_latency(28672, 17920, 5, 2)
    assert not lib.stack_low_latency(*_arrays([(49600, 128), (100, 3200)]), ctypes.c_int64(5), ctypes.c_size_t(_part(16)))
