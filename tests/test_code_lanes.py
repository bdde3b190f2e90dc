"""The column loop's decision, spread over the 16 lanes of a row (csrc/mq_code_lanes.h), emulated lane by lane on the CPU: the code
against the oracle's brute force and the propagated error against the IEEE divisions of the definition, bit for bit."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "mq_code_lanes.h"
using namespace mq;
// as the kernel has it, the lanes one after the other
template <uint32_t M, bool ALL>
static uint32_t decide(float w, float s, float z, const QuantLambda &l, float nw, float u, float &err, int &kind) {
    const float sign = code_sign(s);
    w *= sign; s *= sign;
    const int U = code_estimate(w, 1.f / s, z + 1.f);
    uint32_t bits = ~0u, key = ~0u;
    for (int part = 0; part < kRowLanes; ++part) {
        const LaneDecision d = lane_decision<M, ALL>(lane_candidate<M>(part), U, w, s, z, l, !ALL && l.v[7] == 0.f,
                                                     code_grid_normal(s, z) & divisor_plain(u), nw, 1.f / nw, u, 1.f / u);
        const uint32_t b = d.bad ? 0 : d.bits, k = d.bad ? kLaneBad : d.key;
        if (b < bits || (b == bits && k < key)) { bits = b; key = k; err = d.err; }
    }
    int q = key >> 2;
    kind = key & (kLaneBad | kLaneLook);
    if (kind) {
        if (key & kLaneBad) q = code_search_closely<M>(U, w, s, z, l);
        else
            for (int step = kRowLanes; step; step /= kRowLanes) {
                int n = 0;
                for (int part = 0; part < kRowLanes; ++part) n += code_same<M>(q - step * (part + 1), bits, w, s, z, l);
                q -= step * n;
            }
        float E = 0, acc = 0, e8;
        bool any = false;
        code_terms<M, ALL>(q, w, s, z, l, E, acc, any, e8);
        err = (acc / nw) / u;
    }
    err *= sign;
    return q;
}
extern "C" void lanes(long n, const float *w, const float *s, const float *z, const float *u, const float *lam, uint8_t *q, float *err, uint8_t *kind) {
    QuantLambda l;
    uint32_t need = 0;
    for (int i = 0; i < 8; ++i) { l.v[i] = lam[i]; if (lam[i] != 0.f) need |= 1u << i; }
    const float nw = popc8(need);
    for (long i = 0; i < n; ++i) {
        int k = 0;
        switch (quant_variant_mask(need)) {
            case 0x80u: q[i] = decide<0x80u, true>(w[i], s[i], z[i], l, nw, u[i], err[i], k); break;
            case 0x8Cu: q[i] = need == 0x8Cu ? decide<0x8Cu, true>(w[i], s[i], z[i], l, nw, u[i], err[i], k)
                                             : decide<0x8Cu, false>(w[i], s[i], z[i], l, nw, u[i], err[i], k); break;
            case 0xAEu: q[i] = decide<0xAEu, false>(w[i], s[i], z[i], l, nw, u[i], err[i], k); break;
            default: q[i] = decide<0xFFu, false>(w[i], s[i], z[i], l, nw, u[i], err[i], k);
        }
        kind[i] = k;
    }
}
extern "C" void divide(long n, const float *a, const float *b, float *fast, uint8_t *plain) {
    for (long i = 0; i < n; ++i) {
        fast[i] = divide_by(a[i], b[i], 1.f / b[i]);
        plain[i] = divides_plainly(a[i]) & divisor_plain(b[i]);
    }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("code_lanes")
    (d / "s.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wno-unknown-pragmas", "-shared", "-fPIC",
                           "-I", os.path.join(ROOT, "paper_2602_03537_amd", "csrc"), str(d / "s.cpp"), "-o", str(d / "s.so")])
    return ctypes.CDLL(str(d / "s.so"))


def _p(a):
    return ctypes.c_void_p(a.ctypes.data)


def _decide(lib, w, s, z, u, widths, lam):
    lam8 = np.zeros(8, np.float32)
    lam8[[r - 1 for r in widths]] = lam
    f = [np.ascontiguousarray(a, np.float32) for a in (w, s, z, u, lam8)]
    q, err, kind = np.empty(w.size, np.uint8), np.empty(w.size, np.float32), np.empty(w.size, np.uint8)
    lib.lanes(ctypes.c_long(w.size), *[_p(a) for a in f], _p(q), _p(err), _p(kind))
    return q, err, kind


def _definition(w, s, z, u, widths, lam):
    w, s, z, u = (a.astype(np.float32) for a in (w, s, z, u))
    with np.errstate(all="ignore"):
        E = oracle.quant_errors(w[:, None], s[:, None], z[:, None], 8, widths, lam, 1, np.float32)[:, :, 0]
        q = np.argmin(np.where(np.isnan(E), np.inf, E), axis=0).astype(np.uint8)
        acc = None
        for r in sorted(widths):
            d = w - s * (oracle.slice_codes(q, 8, r).astype(np.float32) - z)
            acc = d if acc is None else acc + d
        return q, (acc / np.float32(len(widths))) / u


def _weights(rng, n):
    """on, between, next to and far outside the codes; zero, negative, subnormal scales; weights that no step shows in"""
    s = np.where(rng.random(n) < 0.2, np.exp2(-rng.integers(0, 24, n)), rng.uniform(2e-4, 2e-3, n)).astype(np.float16)
    z = np.where(rng.random(n) < 0.5, rng.integers(0, 256, n), rng.uniform(-50, 400, n)).astype(np.float16)
    g = rng.uniform(-40, 300, n)
    kind = rng.integers(0, 8, n)
    g = np.where(kind == 0, np.rint(g), np.where(kind == 1, np.floor(g) + 0.5, np.where(kind == 2, 8 * np.rint(g / 8), g)))
    g = np.where(kind == 3, g * rng.choice([1e2, 1e5, 1e9, 1e14], n), g)
    odd = rng.random(n)
    s = np.where(odd < 0.02, 0, np.where(odd < 0.06, -s, s)).astype(np.float16)
    w = ((g - z.astype(np.float64)) * s.astype(np.float64)).astype(np.float32)
    w = np.where(odd > 0.99, w * np.float32(1e20), w)
    w = np.nextafter(w, np.where(rng.random(n) < 0.5, -np.inf, np.inf).astype(np.float32), where=rng.random(n) < 0.2, out=w.copy())
    w[odd < 0.005] = 0
    tiny = (odd > 0.5) & (odd < 0.53)   # so small that dividing by a reciprocal would underflow on the way; at the grid's own zero
    z = np.where(tiny, np.rint(z), z).astype(np.float16)
    w = np.where(tiny, 10.0 ** rng.uniform(-44, -30, n), w)
    return w.astype(np.float32), s, z


EVERY_SET = [c for k in range(1, 9) for c in itertools.combinations(range(1, 9), k)]


@pytest.mark.parametrize("spread", ["equal", "uniform", "2^30", "2^90"])
@pytest.mark.parametrize("first", range(0, len(EVERY_SET), 51))
def test_lanes_decide_as_the_brute_force(lib, first, spread):
    looked = 0
    for i, widths in enumerate(EVERY_SET[first:first + 51], first):
        rng = np.random.default_rng([501, i])
        k = len(widths)
        lam = {"equal": np.ones(k), "uniform": rng.uniform(0.01, 3, k), "2^30": np.exp2(rng.integers(-30, 31, k)),
               "2^90": np.exp2(rng.integers(-90, 91, k))}[spread].astype(np.float32)
        w, s, z = _weights(rng, 600)
        u = (rng.choice([-1.0, 1.0], w.size) * np.exp2(rng.uniform(-3, 3, w.size))).astype(np.float32)
        u[::50] = np.exp2(rng.uniform(-70, 70, u[::50].size))
        q, err, kind = _decide(lib, w, s, z, u, widths, [float(x) for x in lam])
        ref_q, ref_err = _definition(w, s, z, u, widths, [float(x) for x in lam])
        bad = np.flatnonzero(q != ref_q)
        assert bad.size == 0, (widths, lam, w[bad[:3]], s[bad[:3]], z[bad[:3]], q[bad[:3]], ref_q[bad[:3]])
        bad = np.flatnonzero(~((err == ref_err) | (np.isnan(err) & np.isnan(ref_err))))   # (the sign of a zero error is not kept)
        assert bad.size == 0, (widths, w[bad[:3]], u[bad[:3]], err[bad[:3]], ref_err[bad[:3]])
        looked += np.count_nonzero(kind)
    assert looked > 0   # both ways to a decision were taken


def _divisors():
    """1 .. 8 (the numbers of widths), mantissas near all ones and all zeros, random ones, at every exponent that counts as plain"""
    ones = np.array([0x3F800000, 0x3F800001, 0x3F800002, 0x3FFFFFFF, 0x3FFFFFFE, 0x3FFFFFFD, 0x3FC00000, 0x3FBFFFFF, 0x3FB504F3], np.uint32)
    rng = np.random.default_rng(502)
    m = np.concatenate([ones.view(np.float32), (1 + rng.random(40)).astype(np.float32)])
    b = np.concatenate([np.float32(2.0) ** e * m for e in range(-50, 50)])
    return np.concatenate([np.arange(1, 9, dtype=np.float32), b, -b])


def test_division_by_a_reciprocal_is_correctly_rounded(lib):
    rng = np.random.default_rng(503)
    for e in (-49, -48, -20, -1, 0, 1, 20, 45, 48):
        for near in range(3):
            b = _divisors()
            a = {0: (1 + rng.random(b.size)) * 2.0 ** e,                                  # random
                 1: (2 - 2.0 ** -23 * rng.integers(1, 4, b.size)) * 2.0 ** e,             # mantissas near all ones
                 2: np.abs(b.astype(np.float64)) * (rng.integers(1, 1 << 12, b.size) + 0.5) * 2.0 ** (e - 12)}[near]  # quotients halfway
            a = np.where(rng.random(b.size) < 0.5, -a, a).astype(np.float32)
            a = np.concatenate([a, np.zeros(1, np.float32)])
            b = np.concatenate([b, np.ones(1, np.float32)])
            fast, plain = np.empty_like(a), np.empty(a.size, np.uint8)
            lib.divide(ctypes.c_long(a.size), _p(a), _p(b), _p(fast), _p(plain))
            assert plain[-1] and plain.mean() > 0.4
            ok = (plain != 0) & (np.abs(a) < 2.0 ** 50)   # weights that count as normal: below 2^46, eight widths
            with np.errstate(all="ignore"):
                bad = np.flatnonzero(ok & (fast != a / b))
            assert bad.size == 0, (e, near, a[bad[:3]], b[bad[:3]], fast[bad[:3]])
