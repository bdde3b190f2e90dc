"""The candidate search of Algorithm 1 (csrc/mq_code_search.h), compiled for the CPU, against the oracle's brute force over
all 256 candidates: bit for bit, for every set of target widths, on weights where a shortcut would go wrong."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "mq_code_search.h"
using namespace mq;
template <uint32_t M> static void run(long n, const float *w, const float *s, const float *z, const QuantLambda &l, uint8_t *q) {
    for (long i = 0; i < n; ++i) {
        const float one[1] = {w[i]};
        uint32_t out[1];
        code_search<M, 1>(one, s[i], z[i], l, out);
        q[i] = (uint8_t)out[0];
    }
}
extern "C" void search(long n, const float *w, const float *s, const float *z, const float *lam, uint8_t *q) {
    QuantLambda l;
    uint32_t need = 0;
    for (int i = 0; i < 8; ++i) { l.v[i] = lam[i]; if (lam[i] != 0.f) need |= 1u << i; }
    switch (quant_variant_mask(need)) {
        case 0x80u: return run<0x80u>(n, w, s, z, l, q);
        case 0x8Cu: return run<0x8Cu>(n, w, s, z, l, q);
        case 0xAEu: return run<0xAEu>(n, w, s, z, l, q);
    }
    run<0xFFu>(n, w, s, z, l, q);
}
"""


@pytest.fixture(scope="module")
def search(tmp_path_factory):
    d = tmp_path_factory.mktemp("code_search")
    (d / "s.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wno-unknown-pragmas", "-shared", "-fPIC",
                           "-I", os.path.join(ROOT, "paper_2602_03537_amd", "csrc"), str(d / "s.cpp"), "-o", str(d / "s.so")])
    fn = ctypes.CDLL(str(d / "s.so")).search
    fn.restype = None

    def call(w, s, z, lam8):
        out = np.empty(w.size, np.uint8)
        p = [np.ascontiguousarray(a, np.float32) for a in (w, s, z, lam8)]
        fn(ctypes.c_long(w.size), *[ctypes.c_void_p(a.ctypes.data) for a in p], ctypes.c_void_p(out.ctypes.data))
        return out
    return call


def _weights(rng, n):
    """(w, s, z), one group per weight: on, between and far outside the codes; scales down to 0 and below; huge weights."""
    s = np.where(rng.random(n) < 0.2, np.exp2(-rng.integers(0, 24, n)), rng.uniform(2e-4, 2e-3, n)).astype(np.float16)
    z = np.where(rng.random(n) < 0.5, rng.integers(0, 256, n), rng.uniform(-50, 400, n)).astype(np.float16)
    u = rng.uniform(-40, 300, n)
    kind = rng.integers(0, 8, n)
    u = np.where(kind == 0, np.rint(u), np.where(kind == 1, np.floor(u) + 0.5, np.where(kind == 2, 8 * np.rint(u / 8), u)))
    u = np.where(kind == 3, u * rng.choice([1e2, 1e5, 1e9], n), u)
    odd = rng.random(n)
    s = np.where(odd < 0.01, 0, np.where(odd < 0.02, -s, s)).astype(np.float16)
    w = ((u - z.astype(np.float64)) * s.astype(np.float64)).astype(np.float32)
    w = np.where(odd > 0.995, w * np.float32(1e20), w).astype(np.float32)
    return w, s, z


EVERY_SET = [c for k in range(1, 9) for c in itertools.combinations(range(1, 9), k)]


@pytest.mark.parametrize("first", range(0, len(EVERY_SET), 32))
def test_search_is_the_brute_force_for_every_set_of_widths(search, first):
    for i, widths in enumerate(EVERY_SET[first:first + 32], first):
        rng = np.random.default_rng([91, i])
        lam = [[1.0] * len(widths), list(rng.uniform(0.01, 3, len(widths)).astype(np.float32)),
               list(np.exp2(rng.integers(-30, 30, len(widths))))][i % 3]
        w, s, z = _weights(rng, 1500)
        lam8 = np.zeros(8, np.float32)
        lam8[[r - 1 for r in widths]] = lam
        with np.errstate(over="ignore", invalid="ignore"):
            ref = oracle.quant_matgptq(w[:, None], s[:, None], z[:, None], 8, widths, lam, 1, np.float32)[:, 0]
        got = search(w, s.astype(np.float32), z.astype(np.float32), lam8)
        bad = np.flatnonzero(got != ref)
        assert bad.size == 0, (widths, lam, w[bad[:3]], s[bad[:3]], z[bad[:3]], got[bad[:3]], ref[bad[:3]])
