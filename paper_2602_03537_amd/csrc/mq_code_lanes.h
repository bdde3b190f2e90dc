// One decision of Algorithm 1 spread over the lanes that share a row of weights (the column loop), with the error it propagates:
// what a lane evaluates, and what it says about it.  The lexicographic minimum of (bits, key) over the lanes decides.
#pragma once
#include "mq_code_search.h"

namespace mq {

constexpr int kRowLanes = 16;  // lanes that share a row: one DPP row

// Entries of the candidate list (mq_code_search.h), two lanes each: U (its second lane: width 7's candidate, where
// the variant has it), U - 1, and one per coarser width; the second lane of an entry evaluates the code below, so that
// the minimum also shows whether a smaller code has the same E.
constexpr int lanes_coarse(uint32_t mask) { return popc8(mask & 0x3Fu); }  // widths 1 .. 6
constexpr int lanes_used(uint32_t mask) {  // lanes that hold different entries: a power of two, 4 .. 16
    const int need = 2 * (2 + lanes_coarse(mask));
    return need <= 4 ? 4 : need <= 8 ? 8 : 16;
}
// What a lane evaluates, given U:  T - (T < U ? left : 0) - second, T = roundup(U, step) - half
struct LaneCandidate {
    int step, half, left, second;
    bool seven;  // width 7's candidate: reported as a second one where it is below U (its own lower neighbour is not listed)
};
template <uint32_t MASK> MQ_HD LaneCandidate lane_candidate(int part) {
    const int e = (part & (lanes_used(MASK) - 1)) >> 1, second = part & 1;
    LaneCandidate c{1, 0, 0, 0, false};  // U
    if (e == 0 && second && (MASK & 0x40u)) c = {2, 1, 1, 0, true};
    if (e == 1) c = {1, 1, 0, second, false};  // U - 1
    int k = 2;
#pragma unroll
    for (int r = 1; r <= 6; ++r) {
        if (!((MASK >> (r - 1)) & 1)) continue;
        const int step = 1 << (kCodeBits - r);
        if (e == k) c = {step, step / 2, 1, second, false};
        ++k;
    }
    return c;
}

// E(q), the sum (w - D_r1) + (w - D_r2) + ... over the widths with lambda_r != 0 (r ascending), and the residual of
// width 8.  ALL: every width of MASK has lambda_r != 0.
template <uint32_t MASK, bool ALL, int R = 1>
MQ_HD void code_terms(uint32_t q, float w, float s, float z, const QuantLambda &lam, float &E, float &acc, bool &any, float &e) {
#pragma clang fp contract(off)
    if constexpr (R <= kCodeBits) {
        if constexpr ((MASK >> (R - 1)) & 1) {
            constexpr bool first = (MASK & ((1u << (R - 1)) - 1)) == 0;
            e = code_residual(slice_of<R>(q), w, s, z);
            const float p = e * e;
            const float term = lam.v[R - 1] * p;
            E = first ? term : E + term;
            if constexpr (ALL) {
                acc = first ? e : acc + e;
            } else if (lam.v[R - 1] != 0.f) {
                acc = any ? acc + e : e;
                any = true;
            }
        }
        code_terms<MASK, ALL, R + 1>(q, w, s, z, lam, E, acc, any, e);
    }
}

// a / b, correctly rounded, y = RN(1 / b): the first correction brings a * y (off by up to two units in the last place) to
// within one unit, from where one more exact remainder rounds correctly (Markstein's theorem; no over- or underflow on the
// way while |a| and |b| are within 2^-60 .. 2^60, or a = 0, whose sign may be lost).  Half as long a chain as the general division.
MQ_HD float divide_by(float a, float b, float y) {
    const float q0 = a * y;
    const float q1 = __builtin_fmaf(__builtin_fmaf(-b, q0, a), y, q0);
    return __builtin_fmaf(__builtin_fmaf(-b, q1, a), y, q1);
}
MQ_HD bool divides_plainly(float a) {  // from below; normal weights are small enough
    return (a == 0.f) | (__builtin_fabsf(a) > 0x1p-50f);
}
MQ_HD bool divisor_plain(float b) { return (__builtin_fabsf(b) > 0x1p-50f) & (__builtin_fabsf(b) < 0x1p50f); }

// A lane's code in units of 4, and below it: the search does not hold here (such a lane wins, with E = 0); look closer if this one wins
constexpr uint32_t kLaneBad = 2, kLaneLook = 1;
struct LaneDecision {
    uint32_t bits, key;  // of E; the code and whether to look closer
    float err;           // (mean of the residuals over the widths) / u
    bool bad;
};
// U: an estimate; nw: |R|, u: the diagonal of the factor, with their reciprocals; runs: lambda_8 = 0; plain: the grid is normal and u plain
template <uint32_t MASK, bool ALL>
MQ_HD LaneDecision lane_decision(const LaneCandidate &lc, int U, float w, float s, float z, const QuantLambda &lam, bool runs, bool plain,
                                 float nw, float inv_nw, float u, float inv_u) {
#pragma clang fp contract(off)
    const int T = ((U + lc.step - 1) & -lc.step) - lc.half;
    int q = T - (T < U ? lc.left : 0);
    int second = lc.second;
    if constexpr (!ALL) {
        if (runs) q = code_run_start(code_clamp(q), lam);
        if (lc.seven) second = T < U ? 1 : 0;
        q = code_clamp(lc.seven ? q : q - second);
    } else {
        q = code_clamp(q - second);
    }
    float E = 0.f, acc = 0.f, e8 = 0.f;
    bool any = false;
    code_terms<MASK, ALL>((uint32_t)q, w, s, z, lam, E, acc, any, e8);
    LaneDecision d;
    d.err = divide_by(divide_by(acc, nw, inv_nw), u, inv_u);
    d.bad = !(plain & code_weight_normal(w) & code_side_ok(q, U, e8));
    d.bits = code_bits(E);
    d.key = 4u * (uint32_t)q + (((second != 0) | !divides_plainly(acc)) ? kLaneLook : 0u);
    return d;
}

}  // namespace mq
