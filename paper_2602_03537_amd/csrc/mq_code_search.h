// Algorithm 1 of the paper from the |R| + 1 of its 256 candidates that can win.
//
// For one weight w the code wanted is the smallest q in 0 .. 255 that minimises
//     E(q) = sum_r lambda_r * (w - scale * (S(q, r) - zero))^2          (r ascending, S = Eq. 1)
// in binary32, every operation rounded on its own:  t = S - zero;  D = scale * t;  e = w - D;
// p = e * e;  E = E + lambda_r * p.  The paper evaluates all 256 candidates; so does the definition.
//
// Why a handful is enough, bit for bit (scale >= 0, nothing overflows: code_grid_normal, code_weight_normal).  Rounding is
// monotone, so D is a non-decreasing function of the slice value S, e_r(q) never rises with q, and every
// term of E is a non-decreasing function of |e_r|.  Let U be the smallest slice value with D(U) > w (256: none)
// and T_r the smallest q with S(q, r) >= U: below T_r width r's error is >= 0 and falls towards it, from T_r on it
// is < 0 and its square grows.  Slice values of width r are multiples of step_r = 2^(8-r), so with
// c = U rounded up to a multiple of step_r, T_r = c - step_r / 2 (the half-up rounding of Eq. 1), and T_8 = U.
// Take the coarsest width r1.  T_r1 is a multiple of every finer step, so all finer T lie on the side of T_r1
// that U lies on (T_r1 >= U: below it; else above it).  On the other side all errors have one sign and E grows
// away from T_r1: its best code is the one next to T_r1.  On U's side S(q, r1) is constant around the finer T's and
// E is monotone beyond them, so the same argument applies to the remaining widths there.  By induction the minimum
// is attained at one of
//     U - 1,  U,  and for every width r < 8:  T_r if T_r >= U, else T_r - 1
// (clamped to 0 .. 255): |R| + 1 candidates instead of 256, and more candidates do no harm.
// The smallest minimiser: E is monotone (not strictly: a rounded sum can absorb a difference) on the way from any
// other minimiser to a candidate, so the codes with the same E below the smallest winning candidate are a run that ends
// at it (code_lowest_equal).  Where lambda_8 = 0 E is constant on whole runs of codes;
// code_run_start takes the step down to the start of a run at once.
//
// U itself is estimated with a reciprocal and then checked in the arithmetic above (D(U-1) <= w < D(U)), and found in it
// where the check fails.
// What lies outside the argument needs no search.  Scale 0, a weight so large that no D shows in it, an infinity or a NaN
// anywhere (code_flat): E is the same for every code, or infinite or NaN for every code, and the answer is code 0.  A negative scale:
// negating w and scale together negates every D and e and changes no E, so the callers do that first (code_sign).
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define MQ_HD __host__ __device__ __forceinline__
#else
#define MQ_HD inline
#endif

namespace mq {

constexpr int kCodeBits = 8;  // width of the parent code

struct QuantLambda {
    float v[kCodeBits];  // lambda of width r at v[r - 1]; 0 = not a target width
};

constexpr int popc8(uint32_t m) { int c = 0; for (int i = 0; i < 8; ++i) c += (m >> i) & 1; return c; }

template <int R> struct CodeWidth {
    static constexpr int r = R;
};

// Eq. 1 on a code 0 .. 255, in 8-bit units
template <int r> MQ_HD uint32_t slice_of(uint32_t q) {
    constexpr uint32_t step = 1u << (kCodeBits - r);
    if constexpr (step == 1) return q;
    else {
        const uint32_t top = 255u - step / 2;  // codes above it would round to 256: the clamp of Eq. 1
        const uint32_t v = q < top ? q : top;
        return (v + step / 2) & ~(step - 1);
    }
}
// w - scale * (S - zero)
MQ_HD float code_residual_f(float S, float w, float s, float z) {
#pragma clang fp contract(off)
    const float t = S - z;
    const float D = s * t;
    return w - D;
}
MQ_HD float code_residual(uint32_t S, float w, float s, float z) { return code_residual_f((float)S, w, s, z); }
// E(q) and the residual of width 8; MASK: bit r-1 set = the term of width r is evaluated (widths outside MASK have
// lambda 0; 8 is always in)
template <uint32_t MASK, int R = 1>
MQ_HD float code_error(uint32_t q, float w, float s, float z, const QuantLambda &lam, float &e8, float E = 0.f) {
#pragma clang fp contract(off)
    static_assert(MASK & 0x80u, "every variant evaluates width 8");
    if constexpr (R > kCodeBits) return E;
    else if constexpr (!((MASK >> (R - 1)) & 1)) return code_error<MASK, R + 1>(q, w, s, z, lam, e8, E);
    else {
        e8 = code_residual(slice_of<R>(q), w, s, z);
        const float p = e8 * e8;
        const float term = lam.v[R - 1] * p;
        const bool first = (MASK & ((1u << (R - 1)) - 1)) == 0;
        return code_error<MASK, R + 1>(q, w, s, z, lam, e8, first ? term : E + term);
    }
}

// The fast search applies: monotone in S, no overflow in e * e, no NaN.  (scale and zero are fp16 values.)
MQ_HD bool code_grid_normal(float s, float z) { return (s >= 0.f) & (s < 1e6f) & (__builtin_fabsf(z) < 1e6f); }
MQ_HD bool code_weight_normal(float w) { return __builtin_fabsf(w) < 0x1p46f; }
// Every code has the same E, or none has one that is a number (scale not negative): w - D falls with the slice value, so where it is
// the same at the two ends it is the same throughout.  (Finite w and grid: |D| < 2^33, no more than half the distance of
// neighbours at 2^58, so from there on every weight is one of these.)
MQ_HD bool code_flat(float w, float s, float z) {
    return !(code_grid_normal(s, z) & (code_residual_f(0.f, w, s, z) > code_residual_f(255.f, w, s, z)));
}
// The factor that scale and weights of a group are multiplied by before a search: exact, and E stays the same
MQ_HD float code_sign(float s) { return s < 0.f ? -1.f : 1.f; }
// Estimate of U from 1 / scale and zero + 1, in 0 .. 256.  It is right if and only if the residual of width 8 is
// negative exactly for the codes from it on, which the candidates on its two sides show (code_side_ok).
MQ_HD int code_estimate(float w, float inv_s, float z1) {
    const float u = w * inv_s + z1;
#if defined(__HIP_DEVICE_COMPILE__)
    return (int)__builtin_amdgcn_fmed3f(u, 0.f, 256.f);
#else
    return (int)(u > 0.f ? (u < 256.f ? u : 256.f) : 0.f);  // NaN -> 0
#endif
}
MQ_HD bool code_side_ok(int q, int U, float e8) { return (e8 < 0.f) == (q >= U); }
// The smallest x in 0 .. hi from which on `holds` is true (it is true from some x on; hi itself is not asked), looked for from
// `at` (< hi) outwards in steps that double, then by halves: few evaluations where it is near, 2 log2(hi) at most.
template <class F> MQ_HD int code_first(int at, int hi, F &&holds) {
    int lo = 0, step = 1;
    bool above = false, below = false;  // of an answer already tried
#pragma unroll 1
    while (lo < hi) {
        if (holds(at)) {
            hi = at;
            above = true;
        } else {
            lo = at + 1;
            below = true;
        }
        const int down = hi - step > 0 ? hi - step : 0, up = lo + step < hi ? lo + step - 1 : hi - 1;
        at = (above && below) ? (lo + hi) >> 1 : above ? down : up;
        step *= 2;
    }
    return hi;
}
// U from an estimate: off by one nearly always, which four residuals side by side settle
MQ_HD int code_first_above(int U, float w, float s, float z) {
    auto above = [&](int q) { return (q > 255) | ((q >= 0) & (code_residual_f((float)q, w, s, z) < 0.f)); };
    const bool a = above(U - 2), b = above(U - 1), c = above(U), d = above(U + 1);
    if (!a & d) return U + 1 - b - c;
    return code_first(U < 255 ? U : 255, 256, above);
}
MQ_HD int code_clamp(int q) { return q < 0 ? 0 : q > 255 ? 255 : q; }
// E as a number that sorts like it (E >= 0)
MQ_HD uint32_t code_bits(float E) { return __builtin_bit_cast(uint32_t, E); }

// start of the run of codes around q on which no slice of a target width changes (q itself where 8 is one)
template <int R = 1> MQ_HD int code_run_start(int q, const QuantLambda &lam, int start = 0) {
    if constexpr (R > kCodeBits) return start;
    else {
        const int S = (int)slice_of<R>((uint32_t)q);
        constexpr int half = (1 << (kCodeBits - R)) / 2;
        const int b = S - half;  // first code of S's run (S = 0: below 0)
        return code_run_start<R + 1>(q, lam, lam.v[R - 1] != 0.f && b > start ? b : start);
    }
}

// E(q) has these bits (q from -255 on; below 0 there is none)
template <uint32_t MASK> MQ_HD bool code_same(int q, uint32_t bits, float w, float s, float z, const QuantLambda &lam) {
    float e8;
    return (q >= 0) & (code_bits(code_error<MASK>((uint32_t)q & 255u, w, s, z, lam, e8)) == bits);
}
// The smallest code with E's bits, q being one and the codes above it of no interest
template <uint32_t MASK>
MQ_HD int code_lowest_equal(int q, uint32_t bits, float w, float s, float z, const QuantLambda &lam) {
    if (lam.v[kCodeBits - 1] == 0.f) q = code_run_start(q, lam);
    if (q == 0) return 0;
    return code_first(q - 1, q, [&](int p) { return code_same<MASK>(p, bits, w, s, z, lam); });
}

// ---- one weight per lane.  All in fp32 (codes and slice values are exact there, and fp32 operations issue faster than
// integer ones), and every slice a candidate needs is known without rounding its code.  Width r's slice is
//   near_r on U's side of T_r, far_r on the other side; at another width's candidate T_r' (or T_r' - 1), r' coarser: T_r' itself
// (a multiple of r's step; T_r' - 1 rounds up to it), r' finer: near_r, as that candidate is on U's side of T_r.
struct CoarseTerm {
    float T, near_term, far_term;  // T_r (not below 0), lambda_r * residual^2 at near_r and at far_r
    bool right;                    // T_r >= U
};
template <uint32_t MASK> struct CoarseTerms {
    CoarseTerm t[kCodeBits];
};
template <int R> MQ_HD CoarseTerm coarse_term(float U, float w, float s, float z, const QuantLambda &lam) {
#pragma clang fp contract(off)
    constexpr float step = (float)(1 << (kCodeBits - R));
    const float c = __builtin_ceilf(U * (1.f / step)) * step;
    CoarseTerm k;
    k.T = c - step / 2;
    k.right = k.T >= U;
    const float up = c < 256.f - step ? c : 256.f - step;      // the clamp of Eq. 1
    const float down = c - step > 0.f ? c - step : 0.f;
    k.T = k.T > 0.f ? k.T : 0.f;
    const float en = code_residual_f(k.right ? down : up, w, s, z), ef = code_residual_f(k.right ? up : down, w, s, z);
    const float pn = en * en, pf = ef * ef;
    k.near_term = lam.v[R - 1] * pn;
    k.far_term = lam.v[R - 1] * pf;
    return k;
}
// E's part below width 8 at a candidate: C = the coarse width whose candidate it is (0: U - 1, kCodeBits: U)
template <uint32_t MASK, int C, int R = 1>
MQ_HD float coarse_sum(const CoarseTerms<MASK> &k, float U, float p_at_T, const QuantLambda &lam, float E = 0.f) {
#pragma clang fp contract(off)
    if constexpr (R == kCodeBits) return E;
    else if constexpr (!((MASK >> (R - 1)) & 1)) return coarse_sum<MASK, C, R + 1>(k, U, p_at_T, lam, E);
    else {
        const CoarseTerm &t = k.t[R - 1];
        float term;
        if constexpr (C == 0) term = t.near_term;
        else if constexpr (C == kCodeBits) term = t.T == U ? t.far_term : t.near_term;
        else if constexpr (R < C) term = t.near_term;
        else if constexpr (R == C) term = t.far_term;
        else term = lam.v[R - 1] * p_at_T;
        const bool first = (MASK & ((1u << (R - 1)) - 1)) == 0;
        return coarse_sum<MASK, C, R + 1>(k, U, p_at_T, lam, first ? term : E + term);
    }
}
template <uint32_t MASK, int R, class F> MQ_HD void each_coarse(F &&f) {  // R, R - 1, .. 1
    if constexpr (R >= 1) {
        if constexpr ((MASK >> (R - 1)) & 1) f(CodeWidth<R>{});
        each_coarse<MASK, R - 1>(f);
    }
}

// The best of the candidates, whether the search holds for this weight, and whether a smaller code might have the same E.
struct CodeBest {
    float q;
    uint32_t bits;  // of E
    bool ok, tie;
};
template <uint32_t MASK>
MQ_HD CodeBest code_best(int U_estimate, float w, float s, float z, const QuantLambda &lam) {
#pragma clang fp contract(off)
    constexpr bool plain = MASK == 0x80u;
    const float U = (float)U_estimate;
    CoarseTerms<MASK> k;
    each_coarse<MASK, kCodeBits - 1>([&](auto rc) { k.t[decltype(rc)::r - 1] = coarse_term<decltype(rc)::r>(U, w, s, z, lam); });
    const float lam8 = lam.v[kCodeBits - 1];
    // sum of the widths below 8, E, and the residual of width 8 at code q
    auto finish = [&](float q, float sum, float &e8) {
#pragma clang fp contract(off)
        e8 = code_residual_f(q, w, s, z);
        const float p = e8 * e8;
        const float term = lam8 * p;
        return plain ? term : sum + term;
    };
    float e8;
    float q = U - 1.f > 0.f ? U - 1.f : 0.f;
    float sum = coarse_sum<MASK, 0>(k, U, 0.f, lam);
    uint32_t best = code_bits(finish(q, sum, e8));
    bool ok = code_weight_normal(w) & ((e8 < 0.f) == (q >= U));
    auto consider = [&](float cq, float csum, float E, uint32_t tie_wins) {
        const bool take = code_bits(E) < best + tie_wins;
        best = take ? code_bits(E) : best;
        q = take ? cq : q;
        sum = take ? csum : sum;
    };
    {
        const float cq = U < 255.f ? U : 255.f;
        const float csum = coarse_sum<MASK, kCodeBits>(k, U, 0.f, lam);
        const float E = finish(cq, csum, e8);
        ok = ok & ((e8 < 0.f) == (cq >= U));
        consider(cq, csum, E, 0u);
    }
    // from the finest width to the coarsest: a candidate below U is smaller than all before it and wins a tie, one
    // above is larger and does not
    each_coarse<MASK, kCodeBits - 1>([&](auto rc) {
#pragma clang fp contract(off)
        constexpr int r = decltype(rc)::r;
        const CoarseTerm &t = k.t[r - 1];
        const float left = t.T - 1.f > 0.f ? t.T - 1.f : 0.f;
        const float cq = t.right ? t.T : left;
        const float eT = code_residual_f(t.T, w, s, z);
        const float csum = coarse_sum<MASK, r>(k, U, eT * eT, lam);
        consider(cq, csum, finish(cq, csum, e8), t.right ? 0u : 1u);
    });
    // Only a winner below U can have a smaller code with the same E (a winner above it would have lost the tie to a candidate),
    // and only if the width-8 term of the code below, added to no more than that code's own sum, does not show.
    const float below = finish(q - 1.f, sum, e8);
    const bool tie = (q < U) & (q > 0.f) & (code_bits(below) <= best);
    return {q, best, ok, tie};
}

// The decision for one weight, whatever it is (U: an estimate; scale not negative).  With width 8 in R it is
// seldom needed: 4e-5 of Gaussian weights have an estimate that is off by one, fewer have a smaller code with the same E.  Without it
// E is constant on runs of codes, and nearly every weight comes here for the start of its run (4096 x 4096, one call at a time: R = {3,4}
// 127 us, {6,7} 276, {3,4,8} 55; with all 256 candidates 594, 784 and 611).
template <uint32_t MASK> MQ_HD uint32_t code_search_closely(int U, float w, float s, float z, const QuantLambda &lam) {
    if (code_flat(w, s, z)) return 0;  // (|w| < 2^58 from here on)
    const CodeBest b = code_best<MASK>(code_first_above(U, w, s, z), w, s, z, lam);
    const int q = (int)b.q;
    return (uint32_t)(b.tie ? code_lowest_equal<MASK>(q, b.bits, w, s, z, lam) : q);
}

// The decision for VEC weights that share scale and zero
template <uint32_t MASK, int VEC>
MQ_HD void code_search(const float (&w_in)[VEC], float s_in, float z, const QuantLambda &lam, uint32_t (&out)[VEC]) {
    float s = s_in, w[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) w[v] = w_in[v];
    if (__builtin_expect(s < 0.f, 0)) {  // a branch: multiplied by code_sign throughout, R = {2,3,4,6,8} took 113 us instead of 82 (4096 x 4096)
        s = -s;
#pragma unroll
        for (int v = 0; v < VEC; ++v) w[v] = -w[v];
    }
    const float inv_s = 1.f / s, z1 = z + 1.f;
    const bool grid_ok = code_grid_normal(s, z);
    bool rare = !grid_ok;
    CodeBest b[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        b[v] = code_best<MASK>(code_estimate(w[v], inv_s, z1), w[v], s, z, lam);
        out[v] = (uint32_t)b[v].q;
        rare = rare | b[v].tie | !b[v].ok;
    }
    if (!rare) return;
#pragma unroll
    for (int v = 0; v < VEC; ++v)
        if (b[v].tie | !(grid_ok & b[v].ok)) out[v] = code_search_closely<MASK>(code_estimate(w[v], inv_s, z1), w[v], s, z, lam);
}

// Built variants: {8} (plain rounding to the nearest code), {3,4,8} (the paper's experiments),
// {2,3,4,6,8} (the widths this library packs), and all eight widths for anything else.
inline uint32_t quant_variant_mask(uint32_t need) {
    if (!(need & ~0x80u)) return 0x80u;
    if (!(need & ~0x8Cu)) return 0x8Cu;
    if (!(need & ~0xAEu)) return 0xAEu;
    return 0xFFu;
}

}  // namespace mq
