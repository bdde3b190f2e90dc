// Sliced, group-dequantised linear layer  y = x * W_D^T  (Section 4 of the paper)
// for small batches: one row of x on the vector ALUs, 2 .. 4 by 4x4x4 and 5 .. 16 by 16x16x32 matrix
// instructions (larger batches in chunks of 16), and the mixed-precision stack of such layers (Section 3.3), as ONE persistent kernel.  Schedule: mq_device.h.
//
// Arithmetic per tile and lane (one row, one group g):
//   D   = sum_k x[k] * t[k]            t = r-bit code, via fp16-subnormal fields
//   y  += scale * (2^(8-r) * D - zero * X_g),   X_g = sum_{k in g} x[k]
// which is  sum_k x[k] * scale * (S[k] - zero)  with S = t * 2^(8-r)  (Eq. 1's
// rescale), the zero-offset and scale applied once per group instead of per weight.
#include "mq_dma.h"
#include "mq_share_walk.h"

namespace mq {

// How a wave gets the 64 activation pairs of a group (they are the same for every lane): each lane fetches ONE pair together with
// the tile (one tile ahead, like the weights), drops it into the wave's 256 bytes of LDS per batch row and all lanes read the
// pairs back with ds_read_b128.
// A batch of 2 .. 4 is multiplied by the matrix core (tile_math_mfma), whose result has four rows per lane, ...
template <int M> constexpr bool kQuadRows = M >= 2 && M <= 4;
template <int M> constexpr bool kColRows = M > 4;                        // ... and from 5 rows on by tile_math_cols, 16 batch rows at a time
template <int M> constexpr int kAcc = kColRows<M> ? 16 : kQuadRows<M> ? 4 : 1;  // fp32 running sums per lane
// The persistent launch: waves of a workgroup, one workgroup per compute unit
constexpr int kWgWaves = 8;
template <int M> constexpr int kRbWaves = M > 8 ? 4 : M > 4 ? 8 : 16;                 // most waves of a low-latency workgroup (registers)
// Waves of it that a SIMD has to have room for.  One row of x and up to four bits need 59 - 67 registers as they come, and two workgroups of 16
// waves a compute unit end at 64 (13003 x 5120, r = 3: 67 registers 11.4 us, 64 9.3)
// More than 8 rows: two workgroups of four waves, which their launch shape counts on (kQuadResident)
template <int R, int M> constexpr int kRbPerSimd = M == 1 && R <= 4 ? 8 : M > 8 ? 2 : kRbWaves<M> / 4;
// Dwords from batch row to batch row in LDS: the four rows that a quad of lanes reads at one time lie in different banks (64 dwords
// apart they shared them: 28672 x 8192, r = 4, eight rows by 4x4x4 instructions 37.0 us, 30.8 so)
template <int M> constexpr int kRowDwords = M > 1 ? 68 : 64;
// M of a kernel is 1 .. 4, 8 or 16 (vector_rows): in the last two the rows of x that do not exist are read as the last one and not stored
template <int M> __device__ __forceinline__ int row_count(const LayerDesc &L) { return M > 4 ? L.M : M; }
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));  // four fp16 at any address of one
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));  // eight at any address of a pair
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// Four registers as a 4 x 4 matrix of quarters of the wave, transposed: afterwards register t holds, in quarter h, what register h held in quarter t
__device__ __forceinline__ void quarter_transpose(uint32_t &a, uint32_t &b, uint32_t &c, uint32_t &d) {
    auto swap32 = [](uint32_t &p, uint32_t &q) {
        const auto v = __builtin_amdgcn_permlane32_swap(p, q, false, false);
        p = v[0];
        q = v[1];
    };
    auto swap16 = [](uint32_t &p, uint32_t &q) {
        const auto v = __builtin_amdgcn_permlane16_swap(p, q, false, false);
        p = v[0];
        q = v[1];
    };
    swap32(a, c);
    swap32(b, d);
    swap16(a, b);
    swap16(c, d);
}

template <int R, int M> struct TileRegs {
    uint32_t w[4 * R];
    std::conditional_t<kQuadRows<M>, half4_t, _Float16> s, z;  // of the lane's rows
    uint32_t xl[M];  // lane l's pair (x[2l], x[2l+1]) of the group per batch row; from 5 rows on see load_tile_x
};

// v in a vector register (an address made from it gives a load whose result stays in one: for a scalar register it would be waited for at once)
__device__ __forceinline__ int own_register(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
// weights, scale and zero-offset of tile u
template <int R, int M>
__device__ __forceinline__ void load_tile_w(TileRegs<R, M> &t, const LayerDesc &L, int u, int lane) {
    // Weights, scales and zeros are read exactly once per call: non-temporal loads (streaming hint) keep them from
    // displacing anything in the caches and, measured with a plain read kernel on this chip, stream at 7.0 TB/s where
    // ordinary loads reach 6.2.  The activations below are shared by every wave and stay ordinary loads.
    const u32x4 MQ_GLOBAL *src = gl(reinterpret_cast<const u32x4 *>(L.Wp) + (size_t)u * (R * 64) + lane);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const u32x4 v = __builtin_nontemporal_load(src + i * 64);
        t.w[4 * i] = v.x; t.w[4 * i + 1] = v.y; t.w[4 * i + 2] = v.z; t.w[4 * i + 3] = v.w;
    }
    const size_t su = (size_t)u * 64, zu = (size_t)(u & L.zmask) * 64;
    if constexpr (kQuadRows<M>) {
        t.s = __builtin_bit_cast(half4_t, (u32x2)__builtin_nontemporal_load(reinterpret_cast<const u32x2_any MQ_GLOBAL *>(gl(L.st) + su + (lane & ~3))));
    } else {
        t.s = __builtin_nontemporal_load(gl(L.st) + su + lane);
    }
    // A symmetric layer has no zero-offset array: its zt is a few lines of 64 x 128.0 inside the library and zmask
    // folds every tile onto them (cache hits, no HBM traffic).  The load is neither branched around nor selected -- either
    // costs the ALU-bound 2-bit tiles and the mixed Llama-3-70B stack 3-9 % -- and an asymmetric layer pays one scalar AND.
    if constexpr (kQuadRows<M>) {
        t.z = __builtin_bit_cast(half4_t, (u32x2)__builtin_nontemporal_load(reinterpret_cast<const u32x2_any MQ_GLOBAL *>(gl(L.zt) + zu + (lane & ~3))));
    } else {
        t.z = __builtin_nontemporal_load(gl(L.zt) + zu + lane);
    }
}
// the lane's activation pair of group g, per batch row.  fresh: x was written by other workgroups of this very launch
// (a chained stack): the loads go to where the whole device sees memory, past whatever this compute die's caches hold.
template <int R, int M>
__device__ __forceinline__ void load_tile_x(TileRegs<R, M> &t, const LayerDesc &L, int g, int lane, bool fresh = false) {
    if constexpr (kColRows<M>) {
        // A load takes 128 bytes of 8 rows (16 rows' 64 bytes, as the matrix core wants them, cost 2.5 us of 28672 x 8192, r = 4, M = 16), its
        // 16-byte pieces in an order that depends on the row, so that reading them back by columns meets no bank twice.  Rows that do not
        // exist repeat the last one, and their sums are not stored.
        static_for<M / 8>([&](auto b) {
            const int row = 8 * b + (lane >> 3) < L.M ? 8 * b + (lane >> 3) : L.M - 1;
            const u32x4_any MQ_GLOBAL *src = gl(reinterpret_cast<const u32x4_any *>(L.x + (size_t)row * L.K + (size_t)g * kGroup)) + ((lane & 7) ^ (lane >> 3));
            static_for<2>([&](auto c) {
                const u32x4 v = src[8 * c];
                constexpr int i = 8 * b + 4 * c;
                t.xl[i] = v.x; t.xl[i + 1] = v.y; t.xl[i + 2] = v.z; t.xl[i + 3] = v.w;
            });
        });
    } else {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const uint32_t MQ_GLOBAL *src = gl(reinterpret_cast<const uint32_t *>(L.x + (size_t)m * L.K + (size_t)g * kGroup)) + lane;
            t.xl[m] = fresh ? __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *src;
        }
    }
}
template <int R, int M>
__device__ __forceinline__ void load_tile(TileRegs<R, M> &t, const LayerDesc &L, int u, int g, int lane) {
    load_tile_w<R, M>(t, L, u, lane);
    load_tile_x<R, M>(t, L, g, lane);
}

// Eq. 1 on the two 8-bit codes of a masked pair (one per 16-bit half), in 8-bit units:
//   S = min((q + 2^(sh-1)) & ~(2^sh - 1), 256 - 2^sh),  sh = 8 - rs
// (rounding half up; q + 2^(sh-1) < 256 + 2^sh, so the only value above the top code is 256 itself).
struct SliceConst {
    uint32_t half2, keep2;
    u16x2 cap2;
};
__device__ __forceinline__ SliceConst slice_const(int rs) {
    const uint32_t low = (1u << (kC - rs)) - 1;  // the bits Eq. 1 drops
    const uint16_t cap = (uint16_t)(255u - low);
    return {((low + 1) >> 1) * 0x10001u, (0x1FFu & ~low) * 0x10001u, {cap, cap}};
}
__device__ __forceinline__ uint32_t slice_pair(uint32_t v, const SliceConst &c) {
    const u16x2 t = __builtin_bit_cast(u16x2, (v + c.half2) & c.keep2);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(t, c.cap2));
}

// A batch of 2 .. 4 on the matrix core: v_mfma_f32_4x4x4_16b_f16 takes, from every lane, four weights of its row (two masked
// dwords) and four activations of batch row lane % 4, and gives lane 4 b + m the sums of rows 4 b .. 4 b + 3 for batch row m.  The
// operand layout is the tile's own, so a quad of activations is read from LDS once for four batch rows (by v_dot2 it was once for
// each, which is what bound these kernels) and the multiplications leave the vector ALUs.  Two fields with one key make an operand;
// Steps<R> lists them.  Lanes of batch rows that do not exist read some other row's and their sums are dropped.
// By v_dot2 / now, us: 28672 x 8192 M = 4: r = 2 35.8 / 20.6, r = 4 35.4 / 27.3, r = 8 48 / 44.9; 4096 x 4096 r = 4 M = 2, 3, 4 7.3 / 6.9,
// 7.9 / 7.2, 8.4 / 7.3; a decode step of four Llama-2-7B blocks 179 / 159, 205 / 169, 244 / 175; a mixed stack of 12 Llama-3-70B blocks
// 968 / 948, 1179 / 923.
// X_g per batch row: partial sums of the four rows change places over DPP steps until lane l holds those of row l % 4.
template <int M> __device__ __forceinline__ float quad_sums(const uint32_t (&x)[M], int lane) {
    float s[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) s[m] = m < M ? dot2(x[m < M ? m : 0], 0x3C003C00u, 0.f) : 0.f;  // (1.0, 1.0)
    auto swap1 = [](float v) { return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xf, 0xf, true)); };
    auto swap2 = [](float v) { return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xf, 0xf, true)); };
    const bool odd = lane & 1, high = lane & 2;
    const float a = (odd ? s[1] : s[0]) + swap1(odd ? s[0] : s[1]);
    float t;
    if constexpr (M > 2) {
        const float b = (odd ? s[3] : s[2]) + swap1(odd ? s[2] : s[3]);
        t = (high ? b : a) + swap2(high ? a : b);
    } else {
        t = a + swap2(a);
    }
    t = dpp_add<0x124>(t);  // row_ror:4
    t = dpp_add<0x128>(t);  // row_ror:8
    t += __shfl_xor(t, 16);
    t += __shfl_xor(t, 32);
    return t;
}
template <int R, int M, bool SL, bool XB>
__device__ __forceinline__ void tile_math_mfma(const TileRegs<R, M> &t, const LayerDesc &L, int lane, uint32_t *xlds, float (&yacc)[kAcc<M>]) {
    using T = Layout<R>;
    using S = Steps<R>;
    const SliceConst sc = slice_const(SL ? L.rs : kC);
    uint32_t xl[M];
    const int pos = (lane & ~15) | (int)((step_table<R>() >> (4 * (lane & 15))) & 15);
#pragma unroll
    for (int m = 0; m < M; ++m) {
        xl[m] = XB ? bf16_pair_to_f16_pair(t.xl[m]) : t.xl[m];
        xlds[m * kRowDwords<M> + pos] = xl[m];
    }
    const float xg = quad_sums<M>(xl, lane);
    const int m = lane & 3;
    f32x4 acc[T::NKEYS];
#pragma unroll
    for (int k = 0; k < T::NKEYS; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    const u32x4 *xq = reinterpret_cast<const u32x4 *>(xlds + (m < M ? m : 0) * kRowDwords<M>);
    static_for<64 / S::BP>([&](auto bl) {
        u32x4 x[S::BP / 4];
#pragma unroll
        for (int i = 0; i < S::BP / 4; ++i) x[i] = xq[bl * (S::BP / 4) + i];
        static_for<S::N>([&](auto si) {
            constexpr Step st = S::at(si);
            auto field = [&](auto uc, auto oc) {
                constexpr Op o = T::op(oc);
                uint32_t v = t.w[(bl * (S::BP / T::PPU) + uc) * T::UD + o.dw];
                if constexpr (o.sh != 0) v >>= o.sh;
                v &= (uint32_t)o.mask * 0x10001u;
                if constexpr (SL) v = slice_pair(v, sc);
                return v;
            };
            const u32x2 a = {field(IntC<st.ua>{}, IntC<st.oa>{}), field(IntC<st.ub>{}, IntC<st.ob>{})};
            constexpr int key = key_index<R>(st.oa);
            const u32x2 b = {x[st.pa / 4][st.pa % 4], x[st.pb / 4][st.pb % 4]};
            acc[key] = __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(half4_t, a), __builtin_bit_cast(half4_t, b), acc[key], 0, 0, 0);
        });
    });
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float d = 0.f;
        // field value = digit * 2^(key-24); back to code units, then Eq. 1's rescale 2^(8-r)
        static_for<T::NKEYS>([&](auto k) { d = fmaf(acc[k][i], __builtin_ldexpf(1.f, 24 - T::key(k) + kC - R), d); });
        yacc[i] = fmaf((float)t.s[i], fmaf(-(float)t.z[i], xg, d), yacc[i]);
    }
}

// 5 and more rows, 16 at a time: v_mfma_f32_16x16x32_f16, activations (batch row lane % 16) times weights (row lane % 16 of a quarter of
// the tile), the four quarters of a wave holding the four quarters of 32 columns.  In the tile a quarter of the wave holds all columns of ITS
// 16 rows, so four lane dwords at a time change places like the entries of a 4 x 4 matrix (a v_permlane32_swap and a v_permlane16_swap
// for every two): afterwards dword t of the four holds rows 16 t .. 16 t + 15, and quarter h of the wave the columns of what was dword h.  All codes
// come to one place of their half, so that one accumulator serves the tile, and the matrix core adds the activations up as well (times 1.0).
// The place: this instruction adds its products after aligning them as if a subnormal weight began at 2^-14, so codes stand as high in the
// mantissa as they can without an exponent (the two lowest widths lower by what one mask or shift allows).  Largest error of one group against 64 bits, units of 2^-24 of the magnitudes
// added up, one activation 100 times the others, with the codes at bit 0 / here: r = 6 36.9 / 1.9, r = 8 9.6 / 2.8 (4x4x4 instructions 1.9 and 6.9); relative error of 8192 x 28672,
// r = 2, M = 16 2.44e-4 / 2.07e-4.  At bit 0 6 and 8 bits take an instruction less per pair: 4096 x 4096 r = 6 M = 8 9.1 us, here 9.2; 11008 x 4096 r = 8 M = 16 18.6 / 19.2.
//   The activations turn from rows to columns in the wave's own LDS (4 or 8 transfers of 1 KB a tile); no wave waits for another.  A tile is
// 20 matrix and 226 .. 319 vector instructions (counted, hand-overs included: r = 2, 3, 4, 6, 8, M = 16 256, 278, 260, 319, 297), the matrix pipe is busy 9 .. 24 % of the time; memory bounds it from 4 bits on,
// instruction issue with two waves a SIMD below.  us, what this took the place of (4x4x4 instructions, which read all
// activations from LDS for every four rows of x, or a kernel with an activation launch of its own and a barrier a tile) / now, r = 4: 28672 x 8192 M = 8 31.1 /
// 27.1, M = 16 41.6 / 30.4; 8192 x 28672 M = 16 40.2 / 29.1; 4096 x 4096 M = 8 8.6 / 7.6, M = 16 12.1 / 8.9; r = 8 28672 x 8192 M = 16 61.8 / 44.2; mixed stacks, every layer its own x: four
// Llama-3-70B blocks M = 8 356 / 325, M = 16 379 / 362, 32 Llama-2-7B blocks M = 8 647 / 633, M = 16 704 / 711.
template <int R> constexpr int kCodeBit = R == 2 ? 8 : R == 3 ? 6 : R == 8 ? 2 : 4;
template <int R, bool XB, int M>
__device__ __forceinline__ void tile_math_cols(const TileRegs<R, M> &t, int lane, uint32_t *xlds, float (&yacc)[kAcc<M>]) {
    using T = Layout<R>;
    using C = ColSteps<R>;
    static_for<M / 4>([&](auto i) {
        u32x4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = XB ? bf16_pair_to_f16_pair(t.xl[4 * i + k]) : t.xl[4 * i + k];
        reinterpret_cast<u32x4 *>(xlds)[i * 64 + lane] = v;
    });
    half8_t x[4];
    static_for<4>([&](auto q) {
        const int c = C::chunk(q, lane >> 4), row = lane & (M - 1) & 15;  // (8 rows: the other half of the lanes repeats them)
        x[q] = __builtin_bit_cast(half8_t, reinterpret_cast<const u32x4 *>(xlds)[((row >> 3) * 2 + (c >> 3)) * 64 + (row & 7) * 8 + ((c ^ row) & 7)]);
    });
    uint32_t w[4 * R];
#pragma unroll
    for (int i = 0; i < 4 * R; ++i) w[i] = t.w[i];
    static_for<4 * R>([&](auto b) {
        if constexpr (b / C::S % 4 == 0) quarter_transpose(w[b], w[b + C::S], w[b + 2 * C::S], w[b + 3 * C::S]);
    });
    // scale and zero-offset of the rows l % 16 of each quarter
    uint32_t sz[4];
    sz[0] = (uint32_t)__builtin_bit_cast(uint16_t, t.s) | (uint32_t)__builtin_bit_cast(uint16_t, t.z) << 16;
#pragma unroll
    for (int i = 1; i < 4; ++i) {
        sz[i] = sz[0];
        asm volatile("" : "+v"(sz[i]));  // four registers, not one value: the swaps change both of theirs
    }
    quarter_transpose(sz[0], sz[1], sz[2], sz[3]);
    constexpr int P = kCodeBit<R>;
    const _Float16 one = (_Float16)1.f;
    const half8_t ones = {one, one, one, one, one, one, one, one};
    f32x4 acc[4], xg = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    static_for<4>([&](auto q) {
        xg = __builtin_amdgcn_mfma_f32_16x16x32_f16(x[q], ones, xg, 0, 0, 0);
        static_for<4>([&](auto tc) {
            u32x4 b;
            static_for<4>([&](auto i) {
                constexpr int pair = 4 * C::chunk(q, 0) + i, unit = pair / T::PPU;
                uint32_t code = 0;
                static_for<T::NOPS>([&](auto oc) {
                    constexpr Op o = T::op(oc);
                    if constexpr (o.pair == pair % T::PPU) {
                        constexpr int pos = ctz16(o.mask) + o.sh, bits = popc16(o.mask), to = P + o.d;
                        const uint32_t v = w[unit * T::UD + o.dw + tc * C::S];
                        if constexpr (pos + bits == 16 && to == 0)  // the top of its half, down to bit 0: no mask
                            code |= __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, v) >> (uint16_t)pos);
                        else
                            code |= (pos >= to ? v >> (pos - to) : v << (to - pos)) & ((uint32_t)(((1 << bits) - 1) << to) * 0x10001u);
                    }
                });
                b[(int)i] = code;
            });
            acc[tc] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x[q], __builtin_bit_cast(half8_t, b), acc[tc], 0, 0, 0);
        });
    });
    // scale * (2^(32-r-P) * acc - zero * X_g): the power of two goes to scale and zero, once for four batch rows
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const half2_t h = __builtin_bit_cast(half2_t, sz[i]);
        const float s = (float)h.x * __builtin_ldexpf(1.f, 24 + kC - R - P), z = (float)h.y * -__builtin_ldexpf(1.f, P + R - kC - 24);
#pragma unroll
        for (int v = 0; v < 4; ++v) yacc[4 * i + v] = fmaf(s, fmaf(z, xg[v], acc[i][v]), yacc[4 * i + v]);
    }
}

// xlds: this wave's M rows of LDS
// SL (R == 8 only): the tile holds the unsliced parent; its codes are sliced to L.rs bits first.
// XB: the activations are bf16 and are converted here
template <int R, int M, bool SL = false, bool XB = false>
__device__ __forceinline__ void tile_math(const TileRegs<R, M> &t, const LayerDesc &L, int lane, uint32_t *xlds, float (&yacc)[kAcc<M>]) {
    using T = Layout<R>;
    static_assert(!SL || R == kC, "slicing in registers starts from the 8-bit parent");
    if constexpr (kColRows<M>) {
        static_assert(!SL, "from the parent: up to 4 rows");
        tile_math_cols<R, XB, M>(t, lane, xlds, yacc);
    } else if constexpr (kQuadRows<M>) {
        tile_math_mfma<R, M, SL, XB>(t, L, lane, xlds, yacc);
    } else {
        constexpr int NU = 4 * R / T::UD;
        const SliceConst sc = slice_const(SL ? L.rs : kC);
        const uint32_t xl = XB ? bf16_pair_to_f16_pair(t.xl[0]) : t.xl[0];
        const float xg = wave_sum(dot2(xl, 0x3C003C00u, 0.f));  // (1.0, 1.0)
        xlds[lane] = xl;
        float acc[T::NKEYS];
#pragma unroll
        for (int k = 0; k < T::NKEYS; ++k) acc[k] = 0.f;
        // quad by quad of activation pairs: one broadcast 16-byte LDS read serves four pairs
        static_for<16>([&](auto qi) {
            const u32x4 xq = reinterpret_cast<const u32x4 *>(xlds)[qi];
            static_for<NU>([&](auto un) {
                static_for<T::NOPS>([&](auto oi) {
                    constexpr Op o = T::op(oi);
                    constexpr int pidx = un * T::PPU + o.pair;
                    if constexpr (pidx / 4 == qi) {
                        constexpr int key = key_index<R>(oi);
                        uint32_t v = t.w[un * T::UD + o.dw];
                        if constexpr (o.sh != 0) v >>= o.sh;
                        v &= (uint32_t)o.mask * 0x10001u;
                        if constexpr (SL) v = slice_pair(v, sc);
                        acc[key] = dot2(v, xq[pidx % 4], acc[key]);
                    }
                });
            });
        });
        float d = 0.f;
        static_for<T::NKEYS>([&](auto k) {
            // field value = digit * 2^(key-24); back to code units, then Eq. 1's rescale 2^(8-r)
            d = fmaf(acc[k], __builtin_ldexpf(1.f, 24 - T::key(k) + kC - R), d);
        });
        yacc[0] = fmaf((float)t.s, fmaf(-(float)t.z, xg, d), yacc[0]);
    }
}

// a wave's sums as one row per lane, in M rows of LDS of its own
template <int M> __device__ __forceinline__ void put_rows(const float (&yacc)[kAcc<M>], uint32_t *room, int lane) {
    if constexpr (kColRows<M>) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int m = 4 * (lane >> 4) + v;  // quarter i of the tile, row lane % 16 of it: register 4 i + v
            if (m < M) {
#pragma unroll
                for (int i = 0; i < 4; ++i) room[m * kRowDwords<M> + 16 * i + (lane & 15)] = __builtin_bit_cast(uint32_t, yacc[4 * i + v]);
            }
        }
    } else if constexpr (kQuadRows<M>) {
        const f32x4 v = {yacc[0], yacc[1], yacc[2], yacc[3]};
        const int m = lane & 3;
        if (m < M) *reinterpret_cast<u32x4 *>(room + m * kRowDwords<M> + (lane & ~3)) = __builtin_bit_cast(u32x4, v);
    } else {
        room[lane] = __builtin_bit_cast(uint32_t, yacc[0]);
    }
}
template <int M> __device__ __forceinline__ void rows_of(const float (&yacc)[kAcc<M>], uint32_t *xlds, int lane, float (&rows)[M]) {
    if constexpr (M >= 2) {
        put_rows<M>(yacc, xlds, lane);
#pragma unroll
        for (int m = 0; m < M; ++m) rows[m] = __builtin_bit_cast(float, xlds[m * kRowDwords<M> + lane]);
    } else {
        rows[0] = yacc[0];
    }
}

// Tiles a wave keeps in flight ahead of the one it is working on.  A wave with one small tile
// in flight cannot pull more than tile_bytes / memory_latency (1.3 GB/s at r = 2), less than
// its fair share of HBM once wider layers free bandwidth, so narrow tiles are fetched deeper:
// about 8 KB per wave in flight at every width.
template <int R, int M> struct PrefetchDepth {
    static constexpr int value = M > 4 ? (R <= 4 ? 2 : 1) : R <= 2 ? 4 : R == 3 ? 3 : R <= 6 ? 2 : 1;
};

// Workgroup i of a launch runs on die i % 8, each with an L2 of its own: neighbouring shares, which read the same activations as a rule, go to one die (grids of a multiple of eight).  Above
// four rows a tile has as many bytes of activations as of weights: 32 Llama-2-7B blocks, mixed widths of 3.5 bits, every layer its own x, M = 16 746 / 696 us, shares of waves 758 / 709;
// four Llama-3-70B blocks 371 / 358; M = 8 611 / 607 and 322 / 321.
__device__ __forceinline__ unsigned die_order() {
    return gridDim.x % 8 == 0 ? blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8 : blockIdx.x;
}

// Shares of waves.  End of a run inside a row block: groups [ga, gb) are in acc[NV] (per lane).
// Complete row block -> final(acc).  Otherwise publish the partial sums; the last
// contributor sums all slots in wave order and calls final(total).
//   cnt     : the row block's counter
//   a       : cost position of the row block's first tile
// Partial sums travel through agent-scope atomic stores/loads (write-through, cache
// bypassing), so no whole-L2 write-back or invalidate is needed to publish them.
template <int NV, class Final>
__device__ __forceinline__ void finish_row_block(const LayerDesc &L, const StackParams &p, int32_t *cnt, uint64_t a,
                                                 int ga, int gb, float (&acc)[NV], int worker, int lane, Final &&final) {
    if (ga == 0 && gb == L.G) {
        final(acc);
        return;
    }
    const int slot = ga == 0 ? 1 : 0;  // the wave holding a row block's first tile uses slot 1
    const size_t slot_floats = (size_t)p.slot_floats;
    float MQ_GLOBAL *mine = gl(p.part + (size_t)(worker * 2 + slot) * slot_floats + lane);
#pragma unroll
    for (int v = 0; v < NV; ++v) __hip_atomic_store(mine + v * 64, acc[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the write-through stores must have been acknowledged before the counter moves
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(gl(cnt), gb - ga, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    old = __builtin_amdgcn_readfirstlane(old);
    if (old + (gb - ga) != L.G) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const int w_lo = wave_of(a, p.nworkers, p.cost_total);
    const int w_hi = wave_of(a + (uint64_t)(L.G - 1) * L.cost, p.nworkers, p.cost_total);
    // Fixed summation order (w_lo's slot 1, then slot 0 of w_lo+1 .. w_hi); loads are issued
    // in batches so that their round trips overlap.
    constexpr int kBatch = NV >= 16 ? 4 : NV >= 8 ? 8 : 16;  // slots fetched per round trip (NV * kBatch registers)
    float tot[NV];
    const float MQ_GLOBAL *first = gl(p.part + (size_t)(w_lo * 2 + 1) * slot_floats + lane);
#pragma unroll
    for (int v = 0; v < NV; ++v) tot[v] = __hip_atomic_load(first + v * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int w0 = w_lo + 1; w0 <= w_hi; w0 += kBatch) {
        float t[kBatch][NV];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int w = w0 + j <= w_hi ? w0 + j : w_hi;
            const float MQ_GLOBAL *src = gl(p.part + (size_t)(w * 2) * slot_floats + lane);
#pragma unroll
            for (int v = 0; v < NV; ++v)
                t[j][v] = __hip_atomic_load(src + v * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (w0 + j <= w_hi) {
#pragma unroll
                for (int v = 0; v < NV; ++v) tot[v] += t[j][v];
            }
    }
    final(tot);
    if (lane == 0) __hip_atomic_store(gl(cnt), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Tiles [u_begin, u_end) of one layer, owned by share `wave`.
template <int R, int M, bool SL = false>
__device__ __forceinline__ void run_units(const LayerDesc &L, const StackParams &p, int u_begin, int u_end, int wave,
                                          int lane, uint32_t *xlds) {
    constexpr int D = PrefetchDepth<R, M>::value, NB = D + 1;
    int rb = u_begin / L.G;
    int g = u_begin - rb * L.G;
    int ga = g;
    float yacc[kAcc<M>];
#pragma unroll
    for (int i = 0; i < kAcc<M>; ++i) yacc[i] = 0.f;

    // ring of NB tile buffers with compile-time indices (no register copies, which would wait
    // for the loads); past the end of the run the last tile is fetched again instead of
    // branching around the loads
    TileRegs<R, M> buf[NB];
    int u_pf = u_begin, g_pf = g;
    auto prefetch = [&](TileRegs<R, M> &t) {
        load_tile<R, M>(t, L, u_pf, g_pf, lane);
        if (u_pf + 1 < u_end) {
            ++u_pf;
            g_pf = g_pf + 1 == L.G ? 0 : g_pf + 1;
        }
    };
    static_for<D>([&](auto j) { prefetch(buf[j]); });
    int u = u_begin;
    while (u < u_end) {
        static_for<NB>([&](auto j) {
            if (u >= u_end) return;
            prefetch(buf[(j + D) % NB]);
            tile_math<R, M, SL>(buf[j], L, lane, xlds, yacc);
            ++g;
            ++u;
            if (g == L.G || u == u_end) {
                const int row = rb * kRowBlock + lane;
                float rows[M];
                rows_of<M>(yacc, xlds, lane, rows);
                finish_row_block<M>(L, p, p.cnt + L.cnt_off + rb, L.cost_start + (uint64_t)rb * L.G * L.cost, ga, g,
                                    rows, wave, lane, [&](const float(&tot)[M]) {
#pragma unroll
                                        for (int m = 0; m < M; ++m)
                                            if (row < L.N && m < row_count<M>(L)) store_y(L.y, (size_t)m * L.N + row, tot[m], L.flags);
                                    });
                ++rb;
                g = 0;
                ga = 0;
#pragma unroll
                for (int i = 0; i < kAcc<M>; ++i) yacc[i] = 0.f;
            }
        });
    }
}

// Shares of waves (wave_shares in mq_routes.h says for which stacks): no barrier and no sums of other waves at the end of a row block, and as many waves as registers allow
// (143 registers and 12 waves a compute unit at one row, 244 and 8 at 16), for which every share hands its two ends over.  32 Llama-2-7B blocks, r = 2, one row 313 us (5.8 TB/s; 382 by shares of
// workgroups), 40 blocks of 128 / 3136 / 13568, r = 3, M = 12 48 (166).  One row is bound by the vector ALUs at 2 bits, by memory from 4 bits on.
template <int M, bool SL = false> __global__ __launch_bounds__(256, M > 4 ? 2 : 1) void stack_wave_kernel(const StackParams p) {
    __shared__ __attribute__((aligned(16))) uint32_t xlds_all[4 * M * kRowDwords<M>];
    uint32_t *xlds = xlds_all + (threadIdx.x >> 6) * M * kRowDwords<M>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)((die_order() * blockDim.x + threadIdx.x) >> 6));
    if (wave >= p.nwaves) return;
    for (int worker = wave; worker < p.nworkers; worker += p.nwaves) {
        walk_tiles(p, worker, [&](const LayerDesc &L, int u_begin, int u_end) {
            if constexpr (SL) {
                run_units<8, M, true>(L, p, u_begin, u_end, worker, lane, xlds);
            } else {
                switch (L.r) {
                    case 2: run_units<2, M>(L, p, u_begin, u_end, worker, lane, xlds); break;
                    case 3: run_units<3, M>(L, p, u_begin, u_end, worker, lane, xlds); break;
                    case 4: run_units<4, M>(L, p, u_begin, u_end, worker, lane, xlds); break;
                    case 6: run_units<6, M>(L, p, u_begin, u_end, worker, lane, xlds); break;
                    default: run_units<8, M>(L, p, u_begin, u_end, worker, lane, xlds); break;
                }
            }
        });
    }
}

// Shares of workgroups: the waves take the groups of a row block in turn and add their sums up through
// LDS where the row block ends, so that what a share hands over to others is one set of sums for each of its two ends.  (A share per wave handed over eight
// times as much: 28672 x 8192, r = 4, M = 16 37.3 us, 33.1 so, M = 4 26.9 / 25.3, before what follows and the launch's order.)
//   The first of them (the end of a row block that earlier shares began) is stored as soon as it is known and counted when the next
// row block ends.  The last one is kept in registers: the counter, read while the last tiles are multiplied, shows as a rule that all others
// have been counted, and then the share adds their sums to its own and is done.  Otherwise it stores and counts its own, too, and
// whoever completes the count adds the slots up, in the same order.  (All pieces stored and counted at the end: 33.1 us, 31.9 so.)
// Tiles [u_begin, u_end) of one layer.
template <int R, int M, bool SL>
__device__ __forceinline__ void run_share(const LayerDesc &L, const StackParams &p, int u_begin, int u_end, int worker, int w, int lane,
                                          uint32_t *xlds, uint32_t (*red)[kWgWaves][M][kRowDwords<M>], int32_t *flags, int &parity) {
    constexpr int D = PrefetchDepth<R, M>::value, NB = D + 1, NW = kWgWaves;
    constexpr int MR = (M + NW - 1) / NW;  // rows of x that a wave adds up
    constexpr int kTileLoads = R + 2 + (kColRows<M> ? M / 4 : M);
    const int G = L.G, rows = row_count<M>(L);
    int32_t MQ_GLOBAL *cnt = gl(p.cnt + L.cnt_off);
    ShareWalk walk(G, u_begin, u_end);
    float yacc[kAcc<M>];
#pragma unroll
    for (int i = 0; i < kAcc<M>; ++i) yacc[i] = 0.f;
    TileRegs<R, M> buf[NB];  // a ring with compile-time indices: copies of registers would wait for the loads

    auto store_row = [&](int b, int m, float v) {
        const int row = b * kRowBlock + lane;
        if (row < L.N && m < rows) store_y(L.y, (size_t)m * L.N + row, v, L.flags);
    };
    auto slot_of = [&](int wk, int slot, int m) { return gl(p.part + (size_t)(wk * 2 + slot) * (size_t)(64 * M) + (m * 64 + lane)); };
    // slots of the shares w_lo .. w_hi that worked on row block b, added up in share order (the first one's is slot 1)
    auto add_slots = [&](int w_lo, int w_hi, int first, float (&tot)[MR]) {
        constexpr int kBatch = 4;
        for (int w0 = w_lo; w0 <= w_hi; w0 += kBatch) {
            float t[kBatch][MR];
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
#pragma unroll
                for (int i = 0; i < MR; ++i) {
                    const int wk = w0 + j <= w_hi ? w0 + j : w_hi, m = w + NW * i;
                    t[j][i] = __hip_atomic_load(slot_of(wk, wk == first ? 1 : 0, m < M ? m : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (w0 + j <= w_hi) {
#pragma unroll
                    for (int i = 0; i < MR; ++i) tot[i] += t[j][i];
                }
        }
    };
    auto first_share = [&](int b) { return wave_of(L.cost_start + (uint64_t)b * G * L.cost, p.nworkers, p.cost_total); };
    auto last_share = [&](int b) { return wave_of(L.cost_start + ((uint64_t)b * G + (G - 1)) * L.cost, p.nworkers, p.cost_total); };
    StoredPiece head;
    int tail_n = 0;  // groups of the last piece once it is stored
    const int tail_rb = (u_end - 1) / G, tail_gb = u_end - tail_rb * G;
    const bool has_tail = tail_gb < G && tail_rb * G >= u_begin;
    int32_t others = -1;  // wave 0: groups of the last row block that others have stored
    // flags: 0 this share completes the first row block, 1 the last, 2 + parity the last one's other pieces are there
    auto count_head = [&]() {
        if (w == 0 && lane == 0) flags[0] = __hip_atomic_fetch_add(cnt + head.rb, head.n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + head.n == G;
        head.counted = true;
    };
    // the end of a row block, or of the share: wave w adds up rows w, w + 8, ... of x
    auto finish = [&](int gb) {
        const int rb = walk.rb, ga = walk.ga;
        const bool tail = has_tail && walk.seg_end == u_end;
        if (tail && w == 0 && lane == 0) flags[2 + parity] = others + gb == G;
        put_rows<M>(yacc, &red[parity][w][0][0], lane);
#pragma unroll
        for (int i = 0; i < kAcc<M>; ++i) yacc[i] = 0.f;
        const bool count = head.to_count();
        if (count) {  // every wave's write-through stores must have been acknowledged before the counter moves
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            if (head.behind_loads<D>()) wait_transfers<D * kTileLoads>();
            else wait_transfers<0>();
        }
        lds_barrier();
        if (count) count_head();
        float t[MR];
#pragma unroll
        for (int i = 0; i < MR; ++i) {
            const int m = w + NW * i < M ? w + NW * i : 0;
            t[i] = __builtin_bit_cast(float, red[parity][0][m][lane]);
#pragma unroll
            for (int k = 1; k < NW; ++k) t[i] += __builtin_bit_cast(float, red[parity][k][m][lane]);
        }
        const bool all_there = tail && __builtin_amdgcn_readfirstlane(flags[2 + parity]);
        parity ^= 1;  // (whoever writes here next has passed the next row block's barrier, and so has everyone who reads now)
        if ((ga == 0 && gb == G) || all_there) {
            if (all_there) {
                const int lo = first_share(rb);
                add_slots(lo + 1, last_share(rb), -1, t);
                if (w == 0 && lane == 0) __hip_atomic_store(cnt + rb, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int i = 0; i < MR; ++i)
                if (w + NW * i < M) store_row(rb, w + NW * i, t[i]);
        } else {
#pragma unroll
            for (int i = 0; i < MR; ++i)
                if (w + NW * i < M)
                    __hip_atomic_store(slot_of(worker, ga == 0 ? 1 : 0, w + NW * i), t[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (tail) tail_n = gb;
            else head.stored(rb, gb - ga);
        }
    };

    walk.run<D, NW>(
        w, head, [&](auto slot, int u, int g) { load_tile<R, M>(buf[slot], L, u, g, lane); },
        [&](auto slot) { tile_math<R, M, SL>(buf[slot], L, lane, xlds, yacc); }, finish,
        [&]() {
            if (has_tail && w == 0) others = __hip_atomic_load(cnt + tail_rb + own_register(0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        },
        [&]() { static_for<NB - 1>([&](auto j) { buf[j] = buf[j + 1]; }); });
    if (head.n == 0 && tail_n == 0) return;
    if (tail_n != 0 || !head.counted) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        wait_transfers<0>();
        lds_barrier();
        if (head.to_count()) count_head();
        if (tail_n != 0 && w == 0 && lane == 0)
            flags[1] = __hip_atomic_fetch_add(cnt + tail_rb, tail_n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + tail_n == G;
    }
    lds_barrier();
    auto complete = [&](int b) {
        float tot[MR];
#pragma unroll
        for (int i = 0; i < MR; ++i) tot[i] = 0.f;
        const int lo = first_share(b);
        add_slots(lo, last_share(b), lo, tot);
#pragma unroll
        for (int i = 0; i < MR; ++i)
            if (w + NW * i < M) store_row(b, w + NW * i, tot[i]);
        if (w == 0 && lane == 0) __hip_atomic_store(cnt + b, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (head.n != 0 && __builtin_amdgcn_readfirstlane(flags[0])) complete(head.rb);
    if (tail_n != 0 && __builtin_amdgcn_readfirstlane(flags[1])) complete(tail_rb);
}

// SL: every layer of the stack is computed from its resident 8-bit parent (LayerDesc::rs).
template <int M, bool SL = false> __global__ __launch_bounds__(64 * kWgWaves, kWgWaves / 4) void stack_kernel(const StackParams p) {
    __shared__ __attribute__((aligned(16))) uint32_t xlds_all[kWgWaves * M * kRowDwords<M>];
    __shared__ __attribute__((aligned(16))) uint32_t red[2][kWgWaves][M][kRowDwords<M>];
    __shared__ int32_t flags[4];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t *xlds = xlds_all + w * M * kRowDwords<M>;
    int parity = 0;
    for (int worker = die_order(); worker < p.nworkers; worker += p.nwaves) {
        walk_tiles(p, worker, [&](const LayerDesc &L, int u_begin, int u_end) {
            if constexpr (SL) {
                run_share<8, M, true>(L, p, u_begin, u_end, worker, w, lane, xlds, red, flags, parity);
            } else {
                switch (L.r) {
                    case 2: run_share<2, M, false>(L, p, u_begin, u_end, worker, w, lane, xlds, red, flags, parity); break;
                    case 3: run_share<3, M, false>(L, p, u_begin, u_end, worker, w, lane, xlds, red, flags, parity); break;
                    case 4: run_share<4, M, false>(L, p, u_begin, u_end, worker, w, lane, xlds, red, flags, parity); break;
                    case 6: run_share<6, M, false>(L, p, u_begin, u_end, worker, w, lane, xlds, red, flags, parity); break;
                    default: run_share<8, M, false>(L, p, u_begin, u_end, worker, w, lane, xlds, red, flags, parity); break;
                }
            }
        });
    }
}

// ------------------------------------------------------------------ one layer, low latency
// mq_linear on a single layer is latency- rather than bandwidth-bound for Llama-sized
// matrices (a 4096 x 4096 layer at r = 4 is 8 MB: one microsecond of HBM time), so the
// single-layer entry point uses a launch shaped for the shortest dependency chain instead of
// the streaming schedule above: one workgroup per (row block, K slice); its W waves take the
// slice's groups round-robin (all their loads are in flight at once), add their lane sums up
// through LDS in wave order, and -- only if K is cut into KS > 1 slices -- hand over to the
// last-arriving slice through KS slots (same deterministic protocol as the stack kernel, with
// KS <= 8 contributors instead of up to G).
// Body shared by the single-layer kernel and the small-stack kernel below.  blk = index of this workgroup among the
// layer's RB * KS workgroups, slot0 = index of the layer's first partial-sum slot, cnt = the layer's row-block counters.
// A layer of a chained small stack that reads what earlier layers of the same launch write (LayerDesc::chain): its
// workgroups fetch their first weights, wait until the finished-row-block counters of all earlier stages have reached
// their totals, and only then read activations.  Nobody can wait for ever: the launch shape keeps every workgroup of
// the stack resident at one time (checked when the stack is planned), so the workgroups waited for are running, and
// they wait for strictly earlier layers only; the number of polls is bounded on top of that (a wait that runs out goes
// on with whatever x holds).  Visibility follows the split-K hand-over's protocol: in a chained stack every y is stored
// through to device-wide memory and acknowledged before its row block is counted, and a layer that has waited reads
// its activations with device-scope loads -- no cache-wide write-back or invalidation anywhere (one per row block and
// one per waiting wave made the chained launch 2.6 times slower than the launches it replaces).
constexpr int kChainPolls = 1 << 20;
// What a workgroup of a chained small stack needs besides its descriptor (all of it uniform over the launch and held
// in scalar registers): the counters, the totals of the stages before the layer's own, and the launch's total.
struct ChainCtl {
    int32_t *counters;         // kChainCounters of them; nullptr: the stack is not chained
    const int32_t *stage_rb;   // row blocks per stage (kernel arguments)
    int32_t total;
};
__device__ __forceinline__ void chain_wait(const ChainCtl &c, int stage) {
    for (int s = 0; s < stage; ++s) {
        const int32_t MQ_GLOBAL *ctr = gl(c.counters + s);
        const int want = c.stage_rb[s];
        for (int polls = 0; polls < kChainPolls; ++polls) {
            if (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= want) break;
            __builtin_amdgcn_s_sleep(2);
        }
    }
}
// by the wave that has just stored a row block of y
__device__ __forceinline__ void chain_announce(const ChainCtl &c, int stage, int lane) {
    // the write-through stores of y must have been acknowledged before the counters move
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane != 0) return;
    int32_t MQ_GLOBAL *ctr = gl(c.counters);
    __hip_atomic_fetch_add(ctr + stage, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // every row block of the launch is counted once more in the last counter; whoever completes it is the last to
    // touch the counters (each waiter has contributed to a row block counted here, after its wait) and zeroes them
    const int old = __hip_atomic_fetch_add(ctr + kSmallStackLayers, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old + 1 == c.total)
        for (int i = 0; i < kChainCounters; ++i) __hip_atomic_store(ctr + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// CH: the launch is a chained small stack (`chain` is live); the plain variants carry none of its code
template <int R, int M, bool SL, bool CH = false, bool XB = false>
__device__ __forceinline__ void linear_rb_body(const LayerDesc &L, const int KS, const int blk, const int slot0,
                                               float *part, int32_t *cnt, uint32_t (*red)[M][kRowDwords<M>], uint32_t *xlds_all,
                                               const ChainCtl chain = ChainCtl{nullptr, nullptr, 0}, const int chunk = 0) {
    uint32_t *xlds = xlds_all + (threadIdx.x >> 6) * M * kRowDwords<M>;
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6, W = blockDim.x >> 6;
    const int rb = blk / KS, ks = blk - rb * KS;
    const int g_lo = (int)((int64_t)ks * L.G / KS), g_hi = (int)((int64_t)(ks + 1) * L.G / KS);
    float yacc[kAcc<M>];
#pragma unroll
    for (int i = 0; i < kAcc<M>; ++i) yacc[i] = 0.f;
    int g = g_lo + w;
    const bool waits = CH && (L.chain & kChainWaits);
    TileRegs<R, M> cur, nxt;
    if (g < g_hi) load_tile_w<R, M>(cur, L, rb * L.G + g, lane);
    bool have_nxt = false;  // a waiting layer has the weights of its second tile on their way, too, before it waits
    if constexpr (CH) {
        if (waits) {  // uniform over the workgroup
            if (g + W < g_hi) {
                load_tile_w<R, M>(nxt, L, rb * L.G + g + W, lane);
                have_nxt = true;
            }
            if (w == 0) chain_wait(chain, L.chain & 0xFF);
            __syncthreads();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        }
    }
    if (g < g_hi) {
        load_tile_x<R, M>(cur, L, g, lane, waits);
        while (true) {
            const int g2 = g + W;
            if (g2 < g_hi) {
                if (!have_nxt) load_tile_w<R, M>(nxt, L, rb * L.G + g2, lane);
                have_nxt = false;
                load_tile_x<R, M>(nxt, L, g2, lane, waits);
            }
            tile_math<R, M, SL, XB>(cur, L, lane, xlds, yacc);
            if (g2 >= g_hi) break;
            cur = nxt;
            g = g2;
        }
    }
    put_rows<M>(yacc, &red[w][0][0], lane);
    __syncthreads();
    if (w != 0) return;
    float tot[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        tot[m] = __builtin_bit_cast(float, red[0][m][lane]);
        for (int i = 1; i < W; ++i) tot[m] += __builtin_bit_cast(float, red[i][m][lane]);
    }
    const int row = rb * kRowBlock + lane;
    if (KS > 1) {
        float MQ_GLOBAL *mine = gl(part + ((size_t)(slot0 + blk) * M) * 64 + lane);
#pragma unroll
        for (int m = 0; m < M; ++m) __hip_atomic_store(mine + m * 64, tot[m], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // the write-through stores must have been acknowledged before the counter moves
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        int old = 0;
        // (a counter serves up to eight chunks of batch rows, four bits each)
        const int shift = M > 8 ? 4 * chunk : 0;
        if (lane == 0) old = __hip_atomic_fetch_add(gl(cnt + rb), (int)(1u << shift), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        old = __builtin_amdgcn_readfirstlane(old);
        if ((M > 8 ? (int)((uint32_t)old >> shift & 15u) : old) != KS - 1) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        const float MQ_GLOBAL *src = gl(part + ((size_t)(slot0 + rb * KS) * M) * 64 + lane);
        float v[8][M];
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int m = 0; m < M; ++m)
                v[i][m] = __hip_atomic_load(src + ((size_t)(i < KS ? i : KS - 1) * M + m) * 64, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            tot[m] = v[0][m];
#pragma unroll
            for (int i = 1; i < 8; ++i)
                if (i < KS) tot[m] += v[i][m];
        }
        if (lane == 0) {
            if constexpr (M > 8) __hip_atomic_fetch_add(gl(cnt + rb), (int)-((uint32_t)KS << shift), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else __hip_atomic_store(gl(cnt + rb), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if constexpr (CH) {
#pragma unroll
        for (int m = 0; m < M; ++m)
            if (row < L.N)
                __hip_atomic_store(gl(reinterpret_cast<uint16_t *>(L.y)) + (size_t)m * L.N + row, y_bits(tot[m], L.flags),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        chain_announce(chain, L.chain & 0xFF, lane);
        return;
    }
#pragma unroll
    for (int m = 0; m < M; ++m)
        if (row < L.N && m < row_count<M>(L)) store_y(L.y, (size_t)m * L.N + row, tot[m], L.flags);
}

// XB: L.x holds bf16 activations.  One variant per kind, because this launch is short: converting ahead of it costs a launch of
// its own (13003 x 5120, r = 6, M = 3: 22.4 us with it, 20.3 without), while in the tile loop it is four operations per lane,
// row and tile.
template <int R, int M, bool SL = false, bool XB = false>
__global__ __launch_bounds__(64 * kRbWaves<M>, (kRbPerSimd<R, M>)) void linear_rb_kernel(const LayerDesc L, const int KS, float *part, int32_t *cnt) {
    __shared__ __attribute__((aligned(16))) uint32_t red[kRbWaves<M>][M][kRowDwords<M>];
    __shared__ __attribute__((aligned(16))) uint32_t xlds_all[kRbWaves<M> * M * kRowDwords<M>];
    if constexpr (M <= 8) {
        linear_rb_body<R, M, SL, false, XB>(L, KS, (int)blockIdx.x, 0, part, cnt, red, xlds_all);
    } else {
        // 16 batch rows per workgroup; the workgroups that share a tile's weights have numbers 8 apart: one compute die's, one L2's
        const int nc = (L.M + 15) / 16, units = L.RB * KS;
        const int t = (int)blockIdx.x / (8 * nc), v = (int)blockIdx.x % (8 * nc), chunk = v / 8, blk = 8 * t + v % 8;
        if (blk >= units) return;
        LayerDesc C = L;
        C.x += (size_t)(16 * chunk) * L.K;
        C.y += (size_t)(16 * chunk) * L.N;
        C.M = L.M - 16 * chunk < 16 ? L.M - 16 * chunk : 16;
        linear_rb_body<R, M, SL, false, XB>(C, KS, blk, chunk * units, part, cnt, red, xlds_all, ChainCtl{nullptr, nullptr, 0}, chunk);
    }
}

template <int R, int M, bool SL = false>
static hipError_t launch_linear_rb_rm(const LayerDesc &L, float *part, int32_t *cnt, hipStream_t s) {
    const RowShape shape = single_row_shape(L.RB, L.G, L.r, L.M);
    const int KS = shape.KS, W = shape.W;
    const unsigned blocks = M > 8 ? (unsigned)((L.RB * KS + 7) / 8 * 8 * ((L.M + 15) / 16)) : (unsigned)(L.RB * KS);
    if constexpr (!SL) {  // a single from-parent call takes fp16 activations
        if (L.x_bf16) {
            LayerDesc B = L;
            B.x = static_cast<const _Float16 *>(L.x_bf16);
            return launch((linear_rb_kernel<R, M, false, true>), dim3(blocks), dim3(64 * W), 0, s, B, KS, part,
                          cnt);
        }
    }
    return launch((linear_rb_kernel<R, M, SL>), dim3(blocks), dim3(64 * W), 0, s, L, KS, part,
                       cnt);
}
template <int M> static hipError_t launch_linear_rb_m(const LayerDesc &L, float *part, int32_t *cnt, hipStream_t s) {
    if constexpr (M <= kValuMaxM) {
        if (L.rs) return launch_linear_rb_rm<8, M, true>(L, part, cnt, s);
    }
    switch (L.r) {
        case 2: return launch_linear_rb_rm<2, M>(L, part, cnt, s);
        case 3: return launch_linear_rb_rm<3, M>(L, part, cnt, s);
        case 4: return launch_linear_rb_rm<4, M>(L, part, cnt, s);
        case 6: return launch_linear_rb_rm<6, M>(L, part, cnt, s);
        case 8: return launch_linear_rb_rm<8, M>(L, part, cnt, s);
    }
    return hipErrorInvalidValue;
}
hipError_t launch_linear_rb(const LayerDesc &L, float *part, int32_t *cnt, hipStream_t s) {
    switch (L.M) {
        case 1: return launch_linear_rb_m<1>(L, part, cnt, s);
        case 2: return launch_linear_rb_m<2>(L, part, cnt, s);
        case 3: return launch_linear_rb_m<3>(L, part, cnt, s);
        case 4: return launch_linear_rb_m<4>(L, part, cnt, s);
        default: return L.M <= 8 ? launch_linear_rb_m<8>(L, part, cnt, s) : L.M <= kQuadMaxM ? launch_linear_rb_m<16>(L, part, cnt, s) : hipErrorInvalidValue;
    }
}

// The same shape for a SMALL stack (the linears of a decoder block that share their input, say): the workgroups of all
// layers in one launch; a workgroup finds its layer and its descriptor in the kernel arguments (at most 16 layers).
// MAXR: the widest layer it serves.  One row and up to four bits keep to 64 registers, as alone, so that two workgroups of 16 waves share a compute unit (at
// 100, for all widths, one): two 11008 x 4096 layers, r = 2 11.0 -> 9.8 us, r = 3 12.8 -> 11.6, r = 4 14.2 -> 13.4.  All widths at 64 registers spill.
template <int M, bool SL, bool CH = false, int MAXR = 8>
__global__ __launch_bounds__(64 * kRbWaves<M>, (kRbPerSimd<MAXR, M>)) void linear_rb_stack_kernel(const StackParams p, const SmallTable t) {
    __shared__ __attribute__((aligned(16))) uint32_t red[kRbWaves<M>][M][kRowDwords<M>];
    __shared__ __attribute__((aligned(16))) uint32_t xlds_all[kRbWaves<M> * M * kRowDwords<M>];
    // the grid holds exactly sum(RB * KS) workgroups; each layer's first one and the descriptors come with the kernel
    // arguments, so a workgroup reads nothing from device memory before its tiles (a walk along the table there was a
    // chain of dependent loads, 0.5 us each and 1.2 us for the first)
    int li = 0;
#pragma unroll
    for (int i = 1; i < 16; ++i)
        if (i < p.n_layers && (int)blockIdx.x >= p.ll_start[i]) li = i;
    const int slot0 = p.ll_start[li], blk = (int)blockIdx.x - slot0;
    const LayerDesc L = t.d[li];
    const int KS = stack_k_slices(L.RB, L.G, M, p.ks_cap);
    int32_t *cnt = p.cnt + L.cnt_off;
    const ChainCtl chain{CH ? p.cnt + p.chain_off : nullptr, p.stage_rb, p.chain_total};
    if constexpr (SL) {
        linear_rb_body<8, M, true, CH>(L, KS, blk, slot0, p.part, cnt, red, xlds_all, chain);
    } else {
        switch (L.r) {
            case 2: linear_rb_body<2, M, false, CH>(L, KS, blk, slot0, p.part, cnt, red, xlds_all, chain); break;
            case 3: linear_rb_body<3, M, false, CH>(L, KS, blk, slot0, p.part, cnt, red, xlds_all, chain); break;
            case 4: linear_rb_body<4, M, false, CH>(L, KS, blk, slot0, p.part, cnt, red, xlds_all, chain); break;
            case 6:
                if constexpr (MAXR >= 6) linear_rb_body<6, M, false, CH>(L, KS, blk, slot0, p.part, cnt, red, xlds_all, chain);
                break;
            case 8:
                if constexpr (MAXR >= 8) linear_rb_body<8, M, false, CH>(L, KS, blk, slot0, p.part, cnt, red, xlds_all, chain);
                break;
        }
    }
}

// The stacks of the kernel with MAXR = 4
template <class Layer> static bool rb_stack_low_widths(int n_layers, int M, bool from_parent, bool chained, Layer &&layer) {
    if (M != 1 || from_parent || chained) return false;
    for (int i = 0; i < n_layers; ++i)
        if (layer(i).r > 4) return false;
    return true;
}
// workgroups of `waves` waves of the small-stack kernel that the device holds at one time
template <int M, bool SL, bool CH = false, int MAXR = 8> static int rb_stack_resident(int waves) {
    static int cached[3] = {0, 0, 0};
    const int slot = waves == 16 ? 0 : waves == 8 ? 1 : 2;
    if (cached[slot]) return cached[slot];
    int dev = 0, cus = 0, b = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, (linear_rb_stack_kernel<M, SL, CH, MAXR>), 64 * waves, 0) != hipSuccess)
        return 0;
    cached[slot] = cus * (b < 1 ? 1 : b);
    return cached[slot];
}
template <int M> static int rb_stack_resident_v(bool from_parent, bool chained, int waves) {
    if constexpr (M <= kChainMaxM) {
        if (chained) return from_parent ? rb_stack_resident<M, true, true>(waves) : rb_stack_resident<M, false, true>(waves);
    }
    return from_parent ? rb_stack_resident<M, true>(waves) : rb_stack_resident<M, false>(waves);
}
// chained: the variant of the kernel whose layers may wait for each other (it is the one whose residency matters then)
static int rb_stack_resident_m(int M, bool from_parent, bool chained, bool low_widths, int waves) {
    switch (M) {
        case 1:
            if (low_widths) return rb_stack_resident<1, false, false, 4>(waves);
            return rb_stack_resident_v<1>(from_parent, chained, waves);
        case 2: return rb_stack_resident_v<2>(from_parent, chained, waves);
        case 3: return rb_stack_resident_v<3>(from_parent, chained, waves);
        case 4: return rb_stack_resident_v<4>(from_parent, false, waves);
        default: return M <= 8 ? rb_stack_resident<8, false>(waves) : rb_stack_resident<16, false>(waves);
    }
}

bool linear_rb_stack_shape(const LayerDesc *table, int n_layers, size_t part_bytes, bool from_parent, bool chained,
                           int *blocks, int *waves, int *ks_cap, int32_t *ll_start, bool *all_resident) {
    const int M = table[0].M;
    auto layer = [&](int i) { return RowLayer{table[i].RB, table[i].G, table[i].r}; };
    if (!low_latency_stack(n_layers, M, part_bytes, layer)) return false;
    const bool low_widths = rb_stack_low_widths(n_layers, M, from_parent, chained, layer);
    // A chained stack is a chain of dependent steps: what counts is the length of one step, and a row block that is
    // not cut along K needs no hand-over through device memory (three round trips) before its y can be announced.
    const RowStackShape s = row_stack_shape(n_layers, M, chained, layer,
                                            [&](int W) { return rb_stack_resident_m(M, from_parent, chained, low_widths, W); });
    *blocks = s.blocks;
    *waves = s.waves;
    *ks_cap = s.ks_cap;
    *all_resident = s.all_resident;
    int start = 0;
    for (int i = 0; i < 16; ++i) {
        ll_start[i] = start;
        if (i < n_layers) start += table[i].RB * stack_k_slices(table[i].RB, table[i].G, M, s.ks_cap);
    }
    return true;
}

template <int M> static hipError_t launch_linear_rb_stack_m(const StackParams &p, const SmallTable &t, int blocks, int waves,
                                                            bool from_parent, hipStream_t s) {
    if constexpr (M <= kChainMaxM) {
        if (p.chain_total) {
            if (from_parent)
                return launch((linear_rb_stack_kernel<M, true, true>), dim3((unsigned)blocks), dim3(64 * waves), 0, s, p, t);
            return launch((linear_rb_stack_kernel<M, false, true>), dim3((unsigned)blocks), dim3(64 * waves), 0, s, p, t);
        }
    }
    if (p.chain_total) return hipErrorInvalidValue;  // refused when the stack was planned
    if constexpr (M == 1) {
        if (rb_stack_low_widths(p.n_layers, M, from_parent, false, [&](int i) { return RowLayer{t.d[i].RB, t.d[i].G, t.d[i].r}; }))
            return launch((linear_rb_stack_kernel<M, false, false, 4>), dim3((unsigned)blocks), dim3(64 * waves), 0, s, p, t);
    }
    if constexpr (M <= kValuMaxM) {
        if (from_parent)
            return launch((linear_rb_stack_kernel<M, true>), dim3((unsigned)blocks), dim3(64 * waves), 0, s, p, t);
    }
    return launch((linear_rb_stack_kernel<M, false>), dim3((unsigned)blocks), dim3(64 * waves), 0, s, p, t);
}
hipError_t launch_linear_rb_stack(const StackParams &p, const SmallTable &t, int blocks, int waves, bool from_parent,
                                  hipStream_t s) {
    switch (p.M) {
        case 1: return launch_linear_rb_stack_m<1>(p, t, blocks, waves, from_parent, s);
        case 2: return launch_linear_rb_stack_m<2>(p, t, blocks, waves, from_parent, s);
        case 3: return launch_linear_rb_stack_m<3>(p, t, blocks, waves, from_parent, s);
        case 4: return launch_linear_rb_stack_m<4>(p, t, blocks, waves, from_parent, s);
        default:
            if (p.M > 16 || from_parent) return hipErrorInvalidValue;
            return p.M <= 8 ? launch_linear_rb_stack_m<8>(p, t, blocks, waves, false, s) : launch_linear_rb_stack_m<16>(p, t, blocks, waves, false, s);
    }
}

// workgroups of the persistent launch: one per compute unit
static int stack_workgroups() {
    static int cached = 0;
    if (!cached) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        cached = cus;
    }
    return cached;
}

template <int M, bool SL> static hipError_t launch_stack_mx(StackParams p, int max_cost, hipStream_t s) {
    const int hw = stack_workgroups();
    if (!hw) return hipErrorUnknown;
    const uint64_t most = (uint64_t)(p.worker_cap ? p.worker_cap : max_workers_valu(M));
    // every share must be at least one tile long, so that each share between the first
    // and last contributor of a row block really owns a tile of it
    uint64_t cap = p.cost_total / (uint64_t)max_cost;
    if (cap > most) cap = most;
    if (cap < 1) cap = 1;
    p.nwaves = (int)(cap < (uint64_t)hw ? cap : (uint64_t)hw);
    // Several interleaved shares per workgroup where they stay long (128 tiles a wave): they even out what the costs miss (12 Llama-3-70B blocks, M = 16, 1343 us with
    // one share a workgroup, 1148 so), and shorter ones cost more in hand-overs (three small blocks, M = 1 38 us, two shares a workgroup 41).
    uint64_t spw = p.cost_total / ((uint64_t)max_cost * (128 * kWgWaves) * (uint64_t)p.nwaves);  // whole shares per workgroup
    if (spw > (uint64_t)kSharesPerWave) spw = kSharesPerWave;
    while (spw > 1 && spw * (uint64_t)p.nwaves > most) --spw;
    if (spw < 1) spw = 1;
    p.nworkers = (int)(spw * (uint64_t)p.nwaves);
    return launch((stack_kernel<M, SL>), dim3((unsigned)p.nwaves), dim3(64 * kWgWaves), 0, s, p);
}
// waves that the device keeps resident of the kernel whose shares belong to waves, in workgroups of four
template <int M, bool SL> static int wave_resident() {
    static int cached = 0;
    if (!cached) {
        int dev = 0, cus = 0, b = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, (stack_wave_kernel<M, SL>), 256, 0) != hipSuccess) return 0;
        const int waves = cus * (b < 1 ? 1 : b) * 4;
        cached = waves < kMaxWaves ? waves : kMaxWaves;
    }
    return cached;
}

template <int M, bool SL> static hipError_t launch_stack_waves(StackParams p, int max_cost, hipStream_t s) {
    const int hw = wave_resident<M, SL>();
    if (!hw) return hipErrorUnknown;
    const uint64_t most = (uint64_t)(p.worker_cap ? p.worker_cap : max_workers_valu(M));
    uint64_t cap = p.cost_total / (uint64_t)max_cost;  // (as above)
    if (cap > most) cap = most;
    if (cap < 1) cap = 1;
    p.nwaves = (int)(cap < (uint64_t)hw ? cap : (uint64_t)hw);
    // A single big layer is over in 25-50 us: with every resident wave a share is only a few tiles
    // long and each row block is handed over many times.  2048 waves still saturate HBM for that
    // long (each keeps its 8 KB in flight) and take 10-25 % off the call (measured on the Llama-3-70B MLP shapes).
    if (!p.table && p.nwaves > 2048) p.nwaves = 2048;
    // Several interleaved shares per wave even out layers of different width (a wave serves
    // shares w, w + nwaves, ...), but every share ends with up to two hand-overs of a few
    // microseconds, so shares stay at least ~128 tiles long (measured: Llama-2-7B stacks are
    // best with one share per wave, Llama-3-70B stacks gain 15 % from eight).
    uint64_t spw = p.cost_total / ((uint64_t)max_cost * 128 * (uint64_t)p.nwaves);  // whole shares per wave
    if (spw > (uint64_t)kSharesPerWave) spw = kSharesPerWave;
    while (spw > 1 && spw * (uint64_t)p.nwaves > most) --spw;
    if (spw < 1) spw = 1;
    p.nworkers = (int)(spw * (uint64_t)p.nwaves);
    return launch((stack_wave_kernel<M, SL>), dim3((unsigned)((p.nwaves + 3) / 4)), dim3(256), 0, s, p);
}
template <int M, bool SL> static hipError_t launch_stack_x(const StackParams &p, int max_cost, hipStream_t s) {
    return p.by_wave ? launch_stack_waves<M, SL>(p, max_cost, s) : launch_stack_mx<M, SL>(p, max_cost, s);
}
template <int M> static hipError_t launch_stack_m(const StackParams &p, int max_cost, bool from_parent, hipStream_t s) {
    return from_parent ? launch_stack_x<M, true>(p, max_cost, s) : launch_stack_x<M, false>(p, max_cost, s);
}

hipError_t launch_stack(StackParams p, int max_cost, bool from_parent, hipStream_t s) {
    switch (p.M) {
        case 1: return launch_stack_m<1>(p, max_cost, from_parent, s);
        case 2: return launch_stack_m<2>(p, max_cost, from_parent, s);
        case 3: return launch_stack_m<3>(p, max_cost, from_parent, s);
        case 4: return launch_stack_m<4>(p, max_cost, from_parent, s);
        default:
            if (p.M > 16 || from_parent) return hipErrorInvalidValue;
            return p.M <= 8 ? launch_stack_x<8, false>(p, max_cost, s) : launch_stack_x<16, false>(p, max_cost, s);
    }
}

// ------------------------------------------------------------------ bf16 activations for the kernels above
// One small launch ahead of a row kernel whose layers (some of them) take bf16 activations (but for a single packed
// layer in the low-latency shape, which converts them itself): those layers'
// activations (LayerDesc::x_bf16) go, as fp16, to the room the workspace keeps for them, which is where LayerDesc::x of
// such a layer points: the kernels above never see the difference.  32 workgroups per layer; layers without the flag
// return at once.
constexpr int kXcvtBlocks = 32;
__global__ __launch_bounds__(256) void xcvt_kernel(const StackParams p) {
    const int li = (int)(blockIdx.x / kXcvtBlocks), bx = (int)(blockIdx.x % kXcvtBlocks);
    const LayerDesc L = p.table ? load_desc(p.table + li) : p.single;
    if (!(L.flags & kFlagXBf16)) return;
    const uint32_t MQ_GLOBAL *src = gl(reinterpret_cast<const uint32_t *>(L.x_bf16));
    uint32_t MQ_GLOBAL *dst = gl(reinterpret_cast<uint32_t *>(const_cast<_Float16 *>(L.x)));
    const int64_t pairs = (int64_t)L.M * L.K / 2;
    for (int64_t i = (int64_t)bx * 256 + threadIdx.x; i < pairs; i += (int64_t)kXcvtBlocks * 256)
        dst[i] = bf16_pair_to_f16_pair(src[i]);
}
hipError_t launch_xcvt(const StackParams &p, hipStream_t s) {
    return launch(xcvt_kernel, dim3((unsigned)(p.n_layers * kXcvtBlocks)), dim3(256), 0, s, p);
}

}  // namespace mq
