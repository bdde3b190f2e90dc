"""Launch shapes of single layers of up to 8 rows and the launch a single layer takes (csrc/mq_routes.h), compiled for the CPU: what the kernels and
the workspaces can hold, and measured calls on the faster side."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "mq_routes.h"
using namespace mq;
extern "C" void shape(int RB, int G, int r, int M, int *out) {
    const RowShape s = single_row_shape(RB, G, r, M);
    out[0] = s.KS;
    out[1] = s.W;
}
extern "C" void stack(int n, int RB, int G, int r, int M, int *out) {
    const RowStackShape s = row_stack_shape(n, M, false, [&](int) { return RowLayer{RB, G, r}; }, [](int waves) { return waves > 8 ? 256 : 512; });
    out[0] = s.ks_cap;
    out[1] = s.waves;
}
extern "C" void uneven(int n, const int *RB, int G, const int *r, int M, int *out) {
    const RowStackShape s = row_stack_shape(n, M, false, [&](int i) { return RowLayer{RB[i], G, r[i]}; }, [](int waves) { return waves > 8 ? 256 : 512; });
    out[0] = s.ks_cap;
    out[1] = s.waves;
}
extern "C" int low_latency(int64_t RB, int64_t G, int r, int64_t M) { return low_latency_call(RB, G, r, M, (size_t)1 << 24); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("shapes")
    (d / "s.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC",
                           "-I", os.path.join(ROOT, "paper_2602_03537_amd", "csrc"), str(d / "s.cpp"), "-o", str(d / "s.so")])
    return ctypes.CDLL(str(d / "s.so"))


def test_shapes_hold_to_their_bounds(lib):
    rng = np.random.default_rng(801)
    out = (ctypes.c_int * 2)()
    for _ in range(20000):
        RB, G, M, r = int(np.exp(rng.uniform(0, 9))), int(np.exp(rng.uniform(0, 6))), int(rng.integers(1, 17)), int(rng.choice([2, 3, 4, 6, 8]))
        lib.shape(RB, G, r, M, out)
        assert 1 <= out[0] <= 8 and (out[0] == 1 or G // out[0] >= 4)          # slots and groups of a slice
        assert out[1] in ((4, 8, 16) if M <= 4 else (4, 8) if M <= 8 else (4,))  # waves the kernels are built for
        # 5 .. 8 rows: a compute unit holds all workgroups of a shape that is cut for it (registers: four waves a SIMD up to 4 bits, three beyond)
        if 4 < M <= 8 and RB <= 256 and out[0] > 1:
            assert -(-RB * out[0] // 256) * out[1] <= (16 if r <= 4 else 12), (RB, G, r, M, list(out))


# row blocks, groups, r, M: K slices and waves measured faster than the slices of pick_k_slices (us: those / these)
@pytest.mark.parametrize("RB,G,r,M,shape", [
    (204, 40, 6, 3, (1, 16)), (157, 64, 4, 2, (3, 8)), (157, 64, 4, 1, (3, 16)), (204, 64, 4, 4, (1, 16)), (448, 16, 4, 2, (1, 8)), (64, 32, 4, 8, (4, 4)),
    (172, 32, 4, 8, (4, 4)), (64, 32, 4, 1, (4, 8)), (392, 13, 3, 1, (1, 16)), (37, 54, 4, 1, (7, 8)), (133, 27, 8, 1, (1, 16)), (133, 27, 8, 3, (1, 16)),
    (13, 195, 6, 6, (8, 8)), (11, 206, 4, 5, (8, 8)), (16, 139, 6, 7, (8, 8))],
    ids=["16.9/12.2", "14.9/11.7", "12.6/10.5", "17.4/14.8", "9.4/8.4", "8.3/7.6", "11.4/9.9", "kept_a", "kept_b", "7.0/6.7", "9.4/8.8", "10.0/9.7", "14.4/12.8", "13.4/11.6", "12.8/12.3"])
def test_measured_shapes(lib, RB, G, r, M, shape):
    out = (ctypes.c_int * 2)()
    lib.shape(RB, G, r, M, out)
    assert (out[0], out[1]) == shape


# (N, K, r, M): us, low-latency and persistent
@pytest.mark.parametrize("N,K,r,M,low,persistent", [
    (15680, 14208, 4, 3, 23.7, 25.8), (28672, 8192, 4, 2, 24.0, 24.4), (28672, 8192, 3, 1, 19.7, 21.0), (28672, 12288, 2, 1, 22.4, 23.8),
    (28672, 12288, 4, 2, 34.5, 32.7), (28672, 20480, 3, 1, 43.2, 41.8), (28672, 8192, 8, 1, 43.0, 40.8),
    (13003, 8192, 4, 6, 16.2, 17.9), (18900, 8192, 6, 6, 29.5, 25.8), (5150, 17024, 6, 6, 22.1, 18.3),
    (4096, 8192, 4, 6, 10.2, 9.3), (4096, 4096, 4, 6, 7.7, 8.0), (4096, 4096, 4, 16, 10.5, 8.9), (13003, 5120, 4, 16, 15.9, 16.5),
    (20000, 2048, 4, 16, 12.5, 13.2), (8192, 8192, 4, 16, 15.3, 14.2)])
def test_single_layers_take_the_faster_launch(lib, N, K, r, M, low, persistent):
    assert bool(lib.low_latency(ctypes.c_int64(-(-N // 64)), ctypes.c_int64(K // 128), r, ctypes.c_int64(M))) == (low < persistent)


# layers, row blocks of each, groups, r, M: most slices and waves on the faster side (None: cut is faster)
@pytest.mark.parametrize("n,RB,G,r,M,shape", [
    (3, 64, 32, 4, 1, (1, 16)), (2, 88, 16, 4, 1, (1, 16)), (2, 64, 40, 4, 1, (2, 16)), (2, 96, 40, 4, 1, (1, 16)), (2, 48, 32, 6, 1, (2, 16)), (2, 4, 8, 8, 3, (1, 8)),
    (2, 24, 32, 4, 1, (4, 8)), (2, 56, 32, 8, 1, (2, 16)), (2, 24, 8, 4, 6, (1, 4)), (2, 112, 16, 4, 16, (1, 4)), (2, 80, 32, 4, 6, None), (2, 112, 32, 4, 6, (1, 8)),
    (2, 112, 32, 4, 16, None)],
    ids=["9.7/8.4", "7.5/5.8", "9.1/9.4", "11.2/10.2", "9.1/9.1", "5.2/5.2", "6.3/6.0", "10.6/9.5", "7.1/6.7", "12.3/11.3", "11.6/12.5", "14.2/13.1", "16.5/17.1"])
def test_measured_stack_shapes(lib, n, RB, G, r, M, shape):
    out = (ctypes.c_int * 2)()
    lib.stack(n, RB, G, r, M, out)
    assert (out[0], out[1]) == shape if shape else out[0] != 1


# row blocks, groups, widths, M: most slices (times in the ids, cut as each layer would be alone / in two / in four)
@pytest.mark.parametrize("RB,G,r,M,cap", [
    ((52, 21, 21), 26, (4, 3, 8), 1, 4), ((60, 15, 15), 30, (4, 6, 3), 1, 4), ((62, 3, 3), 31, (2, 4, 8), 4, 4), ((56, 4, 4), 28, (2, 2, 6), 1, 4),
    ((60, 4, 4), 30, (2, 4, 6), 4, 4), ((88, 15, 15), 44, (8, 4, 4), 4, 2)],
    ids=["1/1.11/0.99", "1/1.11/0.99", "1/1.06/0.96", "1/1.05/0.92", "1/1.08/0.97", "1/0.84/0.94"])
def test_stacks_of_uneven_layers(lib, RB, G, r, M, cap):
    out = (ctypes.c_int * 2)()
    ints = ctypes.c_int * 3
    lib.uneven(3, ints(*RB), G, ints(*r), M, out)
    assert out[0] == cap


def test_six_bits_stay_cut_up_to_160_row_blocks(lib):
    out = (ctypes.c_int * 2)()
    ints = ctypes.c_int * 3
    lib.uneven(3, ints(54, 48, 48), 27, ints(4, 2, 6), 4, out)      # cut / uncut 1 / 1.06
    assert out[0] != 1
    lib.uneven(3, ints(54, 53, 53), 27, ints(4, 2, 6), 4, out)
    assert out[0] == 1
