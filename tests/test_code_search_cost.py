"""What the candidate search of Algorithm 1 (csrc/mq_code_search.h) costs where it leaves its common path, in residuals evaluated
per weight, counted on the CPU: it has to stay far below the 256 candidates x widths that it replaces."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "mq_code_search.h"
using namespace mq;
static long count;
extern "C" void __attribute__((no_instrument_function)) __cyg_profile_func_enter(void *f, void *) {
    count += f == (void *)&code_residual_f;
}
extern "C" void __attribute__((no_instrument_function)) __cyg_profile_func_exit(void *, void *) {}
template <uint32_t M> static void run(long n, const float *w, const float *s, const float *z, const QuantLambda &l, uint8_t *q, int *c) {
    for (long i = 0; i < n; ++i) {
        float one[1] = {w[i]};
        uint32_t out[1];
        count = 0;
        code_search<M, 1>(one, s[i], z[i], l, out);
        c[i] = (int)count;
        q[i] = (uint8_t)out[0];
    }
}
extern "C" void search(long n, const float *w, const float *s, const float *z, const float *lam, uint8_t *q, int *c) {
    QuantLambda l;
    uint32_t need = 0;
    for (int i = 0; i < 8; ++i) { l.v[i] = lam[i]; if (lam[i] != 0.f) need |= 1u << i; }
    switch (quant_variant_mask(need)) {
        case 0x80u: return run<0x80u>(n, w, s, z, l, q, c);
        case 0x8Cu: return run<0x8Cu>(n, w, s, z, l, q, c);
        case 0xAEu: return run<0xAEu>(n, w, s, z, l, q, c);
    }
    run<0xFFu>(n, w, s, z, l, q, c);
}
"""


@pytest.fixture(scope="module")
def search(tmp_path_factory):
    d = tmp_path_factory.mktemp("code_search_cost")
    (d / "s.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O0", "-fno-inline", "-finstrument-functions", "-ffp-contract=off",
                           "-Wno-unknown-pragmas", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-I", os.path.join(ROOT, "paper_2602_03537_amd", "csrc"),
                           str(d / "s.cpp"), "-o", str(d / "s.so")])
    fn = ctypes.CDLL(str(d / "s.so")).search
    fn.restype = None

    def call(w, s, z, widths, lam):
        """codes and evaluated residuals per weight, after a comparison with the brute force"""
        lam8 = np.zeros(8, np.float32)
        lam8[[r - 1 for r in widths]] = lam
        n = w.size
        w, s, z = (np.ascontiguousarray(np.broadcast_to(a, n), np.float16 if a is not w else np.float32) for a in (w, s, z))
        out, cost = np.empty(n, np.uint8), np.empty(n, np.int32)
        p = [np.ascontiguousarray(a, np.float32) for a in (w, s, z, lam8)]
        fn(ctypes.c_long(n), *[ctypes.c_void_p(a.ctypes.data) for a in p], ctypes.c_void_p(out.ctypes.data),
           ctypes.c_void_p(cost.ctypes.data))
        with np.errstate(all="ignore"):
            E = oracle.quant_errors(w[:, None], s[:, None], z[:, None], 8, widths, lam, 1, np.float32)[:, :, 0]
        ref = np.argmin(np.where(np.isnan(E), np.inf, E), axis=0)   # a sum that is no number is never smaller
        bad = np.flatnonzero(out != ref)
        assert bad.size == 0, (widths, lam, w[bad[:3]], s[bad[:3]], z[bad[:3]], out[bad[:3]], ref[bad[:3]])
        return cost
    return call


def _residuals(widths):
    """of the common path: two slices and the candidate's own per width below 8, the residual of width 8 at every candidate,
    and one for the code below the winner; the built variant's widths count"""
    built = 1 if widths == (8,) else 3 if set(widths) <= {3, 4, 8} else 5 if set(widths) <= {2, 3, 4, 6, 8} else 8
    return 2 + 4 * (built - 1) + 1


SETS = [(8,), (3, 4, 8), (2, 3, 4, 6, 8), (1, 2, 5, 7, 8), (1, 2, 3, 4, 5, 6, 7, 8)]


@pytest.mark.parametrize("widths", SETS)
@pytest.mark.parametrize("scale", [0.0, -0.0, -0.0011, -2.0 ** -6, np.inf, np.nan])
def test_zero_negative_and_odd_scales_cost_no_sweep_of_the_codes(search, widths, scale):
    rng = np.random.default_rng([301, len(widths)])
    w = np.concatenate([np.zeros(8), rng.normal(0, 0.1, 300)]).astype(np.float32)
    z = np.where(np.arange(w.size) % 2, 128.0, rng.uniform(-50, 300, w.size)).astype(np.float16)
    cost = search(w, np.full(w.size, scale, np.float16), z, widths, [1.0] * len(widths))
    assert cost.max() <= 3 * _residuals(widths) + 8


@pytest.mark.parametrize("widths", SETS)
def test_weights_beyond_every_step_cost_no_sweep_of_the_codes(search, widths):
    # from 2^58 on no de-quantised value changes the weight, whatever the fp16 grid; infinities and NaN have no smallest error
    w = np.array([2.0 ** 58, -2.0 ** 58, 2.0 ** 60 * 1.3, 1e30, -1e38, np.inf, -np.inf, np.nan], np.float32).repeat(6)
    s = np.tile(np.array([65504, -65504, 1e-3, 6e-8, 1, 0], np.float16), 8)
    z = np.tile(np.array([65504, -65504, 0, 128, 300, np.nan], np.float16), 8)
    cost = search(w, s, z, widths, [1.0] * len(widths))
    assert cost.max() <= 3 * _residuals(widths) + 8
    # just below it a step can show
    w = np.array([np.nextafter(np.float32(2.0 ** 58), np.float32(0))] * 2, np.float32)
    search(w, np.array([65504, -65504], np.float16), np.array([-65504, 65504], np.float16), widths, [1.0] * len(widths))


@pytest.mark.parametrize("widths", [s for s in SETS if len(s) > 1] + [(3, 4), (4,), (1,)])
@pytest.mark.parametrize("fade", [0, 12, 24, 60, 90])
def test_codes_with_the_same_error_cost_no_walk(search, widths, fade):
    # each width's lambda 2^-fade of the one before (up to a range of 2^100): the sums absorb the finer terms, and long runs of codes
    # have the same error; so have most or all codes for weights that few of the steps show in
    rng = np.random.default_rng([302, len(widths), fade])
    fade = min(fade, 100 / max(1, len(widths) - 1))
    lam = [2.0 ** -int(fade * i) for i in range(len(widths))]
    w = np.concatenate([rng.normal(0, 0.1, 300), 10.0 ** rng.uniform(0, 17, 300) * rng.choice([-1, 1], 300)]).astype(np.float32)
    s = np.where(rng.random(w.size) < 0.1, 6e-8, rng.uniform(2e-4, 2e-3, w.size)).astype(np.float16)
    z = rng.integers(0, 256, w.size).astype(np.float16)
    cost = search(w, s, z, widths, lam)
    built = 3 if set(widths) <= {3, 4, 8} else 5 if set(widths) <= {2, 3, 4, 6, 8} else 8
    assert cost.max() <= 2 * _residuals(widths) + 16 + 16 * built   # the list twice, U found anew, the run's start
