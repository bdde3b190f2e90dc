// Packed weight layout shared by the pack/unpack kernels and the linear kernels.
//
// W [N,K] is cut into tiles of 64 rows x 128 columns (one quantisation group).
// Tile (rb, g) lives at uint4 index ((rb*G + g)*R + i)*64 + lane, i = 0..R-1:
// a wavefront fetches it with R coalesced 16-byte loads and lane l then holds
// the whole group of row rb*64+l in 4R dwords ("lane dwords").
//
// Lane dwords are split into units of UD dwords.  Each 16-bit half of a dword
// is an independent container: the low half carries even columns, the high
// half the following odd column, so that one masked dword is an fp16 pair that
// meets the activation pair (x[2p], x[2p+1]).  A unit carries PPU such pairs.
// A code is stored as one or more bit-fields ("ops").  Every field sits, after
// an optional right shift of the whole dword, inside mantissa bits 0..9 of its
// half, so  (dword >> sh) & (mask * 0x10001)  is a pair of fp16 SUBNORMALS with
// value  digit * 2^(p-24)  where p = ctz(mask) and digit are `bits` bits of the
// code starting at bit d.  gfx950's v_dot2_f32_f16 and f16 MFMA take fp16
// subnormals at full rate and exactly, so no int->float conversion is issued.
// Fields with equal (p - d) share one fp32 accumulator ("key"); the group total
// is  sum_key acc[key] * 2^(24 - (p-d))  in units of the r-bit code.
//
// Section 4 of the paper splits 2..4-bit codes over three buffers (2+1+1 bits)
// so that widths share storage; here every width has its own dense layout and
// exactly r bits per weight are streamed.
#pragma once
#include <stdint.h>

namespace mq {

constexpr int kRowBlock = 64;   // rows per tile == lanes per wavefront
constexpr int kGroup = 128;     // columns per tile == quantisation group
constexpr int kC = 8;           // master bit-width of the parent

struct Op {
    int dw;    // dword inside the unit
    int sh;    // right shift applied to the dword before masking (0 = none)
    int mask;  // 16-bit mask after the shift (replicated to both halves)
    int d;     // first bit of the code this field carries
    int pair;  // activation pair inside the unit
};

constexpr int ctz16(int m) { int p = 0; while (!((m >> p) & 1)) ++p; return p; }
constexpr int popc16(int m) { int c = 0; for (int i = 0; i < 16; ++i) c += (m >> i) & 1; return c; }

template <int R> struct Layout;

// r = 2: eight codes per half.  Bits 0..9 hold five, bits 10..15 three more (one shift).
template <> struct Layout<2> {
    static constexpr int UD = 1, PPU = 8, NOPS = 8, NKEYS = 5;
    static constexpr Op op(int i) {
        constexpr Op t[NOPS] = {{0, 0, 0x0003, 0, 0},  {0, 0, 0x000C, 0, 1},  {0, 0, 0x0030, 0, 2},
                                {0, 0, 0x00C0, 0, 3},  {0, 0, 0x0300, 0, 4},  {0, 10, 0x0003, 0, 5},
                                {0, 10, 0x000C, 0, 6}, {0, 10, 0x0030, 0, 7}};
        return t[i];
    }
    static constexpr int key(int k) { constexpr int t[NKEYS] = {0, 2, 4, 6, 8}; return t[k]; }
};

// r = 3: a unit of three dwords holds 16 pairs.  Each half: five codes (15 bits)
// plus one bit of the 16th code (bit 15 of halves A, B, C = bits 0, 1, 2).
template <> struct Layout<3> {
    static constexpr int UD = 3, PPU = 16, NOPS = 18, NKEYS = 5;
    static constexpr Op op(int i) {
        constexpr Op t[NOPS] = {
            {0, 0, 0x0007, 0, 0},  {0, 0, 0x0038, 0, 1},  {0, 0, 0x01C0, 0, 2},  {0, 9, 0x0007, 0, 3},  {0, 9, 0x0038, 0, 4},
            {1, 0, 0x0007, 0, 5},  {1, 0, 0x0038, 0, 6},  {1, 0, 0x01C0, 0, 7},  {1, 9, 0x0007, 0, 8},  {1, 9, 0x0038, 0, 9},
            {2, 0, 0x0007, 0, 10}, {2, 0, 0x0038, 0, 11}, {2, 0, 0x01C0, 0, 12}, {2, 9, 0x0007, 0, 13}, {2, 9, 0x0038, 0, 14},
            {0, 9, 0x0040, 0, 15}, {1, 9, 0x0040, 1, 15}, {2, 9, 0x0040, 2, 15}};
        return t[i];
    }
    static constexpr int key(int k) { constexpr int t[NKEYS] = {0, 3, 6, 5, 4}; return t[k]; }
};

// r = 4: four codes per half; the upper two after a shift by 8.
template <> struct Layout<4> {
    static constexpr int UD = 1, PPU = 4, NOPS = 4, NKEYS = 2;
    static constexpr Op op(int i) {
        constexpr Op t[NOPS] = {{0, 0, 0x000F, 0, 0}, {0, 0, 0x00F0, 0, 1}, {0, 8, 0x000F, 0, 2}, {0, 8, 0x00F0, 0, 3}};
        return t[i];
    }
    static constexpr int key(int k) { constexpr int t[NKEYS] = {0, 4}; return t[k]; }
};

// r = 6: a unit of three dwords holds 8 pairs.  Each half: two whole codes
// (bits 0..5 and 6..11) and four spare bits; pair 6 = B[12:13] + 4*A[12:15],
// pair 7 = C[12:15] + 16*B[14:15], chosen so that only three keys occur.
template <> struct Layout<6> {
    static constexpr int UD = 3, PPU = 8, NOPS = 10, NKEYS = 3;
    static constexpr Op op(int i) {
        constexpr Op t[NOPS] = {{0, 0, 0x003F, 0, 0}, {0, 6, 0x003F, 0, 1}, {1, 0, 0x003F, 0, 2}, {1, 6, 0x003F, 0, 3},
                                {2, 0, 0x003F, 0, 4}, {2, 6, 0x003F, 0, 5}, {1, 6, 0x00C0, 0, 6}, {0, 6, 0x03C0, 2, 6},
                                {2, 6, 0x03C0, 0, 7}, {1, 6, 0x0300, 4, 7}};
        return t[i];
    }
    static constexpr int key(int k) { constexpr int t[NKEYS] = {0, 6, 4}; return t[k]; }
};

// r = 8: two codes per half, the upper after a shift by 8.
template <> struct Layout<8> {
    static constexpr int UD = 1, PPU = 2, NOPS = 2, NKEYS = 1;
    static constexpr Op op(int i) {
        constexpr Op t[NOPS] = {{0, 0, 0x00FF, 0, 0}, {0, 8, 0x00FF, 0, 1}};
        return t[i];
    }
    static constexpr int key(int k) { constexpr int t[NKEYS] = {0}; return t[k]; }
};

// accumulator index of an op: position of (p - d) in the key list
template <int R> constexpr int key_index(int i) {
    const Op o = Layout<R>::op(i);
    const int kd = ctz16(o.mask) - o.d;
    for (int k = 0; k < Layout<R>::NKEYS; ++k)
        if (Layout<R>::key(k) == kd) return k;
    return -1;
}

// Compile-time self-check of a layout: every op maps to a key, the fields of a
// unit tile its UD*32 bits exactly once, and each pair's fields cover bits 0..R-1 once.
template <int R> constexpr bool layout_ok() {
    using T = Layout<R>;
    if ((4 * R) % T::UD) return false;
    if (T::PPU * 2 * R != T::UD * 32) return false;
    unsigned used[4] = {0, 0, 0, 0};
    for (int i = 0; i < T::NOPS; ++i) {
        const Op o = T::op(i);
        if (key_index<R>(i) < 0) return false;
        if (o.mask & ~0x03FF) return false;  // must stay inside the fp16 mantissa
        const unsigned field = ((unsigned)o.mask << o.sh) & 0xFFFFu;
        if (popc16((int)field) != popc16(o.mask)) return false;  // shifted out of the half
        if (used[o.dw] & field) return false;
        used[o.dw] |= field;
    }
    for (int dw = 0; dw < T::UD; ++dw)
        if (used[dw] != 0xFFFFu) return false;
    for (int p = 0; p < T::PPU; ++p) {
        unsigned bits = 0;
        for (int i = 0; i < T::NOPS; ++i) {
            const Op o = T::op(i);
            if (o.pair != p) continue;
            const unsigned f = (unsigned)(o.mask >> ctz16(o.mask)) << o.d;
            if (bits & f) return false;
            bits |= f;
        }
        if (bits != (1u << R) - 1u) return false;
    }
    return true;
}
// Two fields with one key meet two activation pairs in a v_mfma_f32_4x4x4_16b_f16 (the row kernels from 2 rows on).  The list of such steps
// for a block of BP pairs: fields (unit, op) a and b, and where in the block their pairs stand once activation pair p of 16 has been
// moved to position pos(p), chosen so that the two are neighbours (but for the third bit of the 3-bit unit's last code).
struct Step {
    int ua, oa, ub, ob;  // unit within the block, op
    int pa, pb;          // position of their pairs within the block
};
template <int R> struct Steps;
template <> struct Steps<2> {
    static constexpr int BP = 16, N = 8;
    static constexpr Step at(int i) {
        constexpr Step t[N] = {{0, 0, 0, 5, 0, 1}, {0, 1, 0, 6, 2, 3}, {1, 0, 1, 5, 4, 5}, {1, 1, 1, 6, 6, 7},
                               {0, 2, 0, 7, 8, 9}, {1, 2, 1, 7, 10, 11}, {0, 3, 1, 3, 12, 13}, {0, 4, 1, 4, 14, 15}};
        return t[i];
    }
};
template <> struct Steps<3> {
    static constexpr int BP = 32, N = 18;
    static constexpr Step at(int i) {
        constexpr Step t[N] = {{0, 0, 0, 3, 0, 1}, {0, 1, 0, 4, 2, 3}, {0, 5, 0, 8, 4, 5}, {0, 6, 0, 9, 6, 7},
                               {0, 10, 0, 13, 8, 9}, {0, 11, 0, 14, 10, 11}, {0, 2, 0, 7, 12, 13}, {0, 12, 0, 15, 14, 15},
                               {1, 0, 1, 3, 16, 17}, {1, 1, 1, 4, 18, 19}, {1, 5, 1, 8, 20, 21}, {1, 6, 1, 9, 22, 23},
                               {1, 10, 1, 13, 24, 25}, {1, 11, 1, 14, 26, 27}, {1, 2, 1, 7, 28, 29}, {1, 12, 1, 15, 30, 31},
                               {0, 16, 1, 16, 15, 31}, {0, 17, 1, 17, 15, 31}};
        return t[i];
    }
};
template <> struct Steps<4> {
    static constexpr int BP = 16, N = 8;
    static constexpr Step at(int i) { return {i / 2, i % 2, i / 2, i % 2 + 2, 2 * i, 2 * i + 1}; }
};
template <> struct Steps<6> {
    static constexpr int BP = 16, N = 10;
    static constexpr Step at(int i) {
        const int u = i / 5, p = 8 * u;
        constexpr int oa[5] = {0, 2, 4, 6, 7}, ob[5] = {1, 3, 5, 8, 9}, at[5] = {0, 2, 4, 6, 6};
        return {u, oa[i % 5], u, ob[i % 5], p + at[i % 5], p + at[i % 5] + 1};
    }
};
template <> struct Steps<8> {
    static constexpr int BP = 16, N = 8;
    static constexpr Step at(int i) { return {i, 0, i, 1, 2 * i, 2 * i + 1}; }
};
// position of pair p of a block of 16, from the list
template <int R> constexpr int step_pos(int p) {
    using T = Layout<R>;
    for (int i = 0; i < Steps<R>::N; ++i) {
        const Step s = Steps<R>::at(i);
        if (s.ua * T::PPU + T::op(s.oa).pair == p) return s.pa;
        if (s.ub * T::PPU + T::op(s.ob).pair == p) return s.pb;
    }
    return -1;
}
// ... of all 16, four bits each
template <int R> constexpr uint64_t step_table() {
    uint64_t t = 0;
    for (int p = 0; p < 16; ++p) t |= (uint64_t)step_pos<R>(p) << (4 * p);
    return t;
}
template <int R> constexpr bool steps_ok() {
    using T = Layout<R>;
    using S = Steps<R>;
    constexpr int units = S::BP / T::PPU;
    int used[8][18] = {};
    for (int i = 0; i < S::N; ++i) {
        const Step s = S::at(i);
        if (s.ua >= units || s.ub >= units || key_index<R>(s.oa) != key_index<R>(s.ob)) return false;
        ++used[s.ua][s.oa];
        ++used[s.ub][s.ob];
        // every field meets its own pair
        if (s.pa != step_pos<R>(s.ua * T::PPU + T::op(s.oa).pair) || s.pb != step_pos<R>(s.ub * T::PPU + T::op(s.ob).pair)) return false;
    }
    for (int u = 0; u < units; ++u)
        for (int o = 0; o < T::NOPS; ++o)
            if (used[u][o] != 1) return false;  // every field once
    int seen[32] = {};
    for (int p = 0; p < S::BP; ++p) {
        const int q = step_pos<R>(p);
        if (q < 0 || q >= S::BP || seen[q]++) return false;          // a permutation ...
        if (q != step_pos<R>(p % 16) + p / 16 * 16) return false;  // ... the same in every 16
    }
    return true;
}
// The same weights in v_mfma_f32_16x16x32_f16 (the row kernels from 5 rows on): multiplication q of four takes activation pairs
// 4 chunk(q, h) .. + 3 in quarter h of the wave.  The dwords that hold their codes in the four quarters are S apart, so that a transpose of
// dwords b, b + S, b + 2 S, b + 3 S serves them all.
template <int R> struct ColSteps {
    using T = Layout<R>;
    static constexpr int S = T::UD == 3 ? 3 : T::PPU == 2 ? 2 : 1;
    static constexpr int chunk(int q, int h) { return T::PPU == 16 ? q + 4 * h : T::PPU == 8 ? 8 * (q / 2) + q % 2 + 2 * h : 4 * q + h; }
};
template <int R> constexpr bool col_steps_ok() {
    using T = Layout<R>;
    using C = ColSteps<R>;
    int seen[64] = {};
    for (int q = 0; q < 4; ++q)
        for (int h = 0; h < 4; ++h)
            for (int i = 0; i < 4; ++i) {
                const int p0 = 4 * C::chunk(q, 0) + i, p = 4 * C::chunk(q, h) + i;
                if (C::chunk(q, h) != C::chunk(q, 0) + C::chunk(0, h) || p >= 64 || seen[p]++) return false;
                if (p % T::PPU != p0 % T::PPU) return false;                                          // the same field in every quarter
                if (p / T::PPU * T::UD != p0 / T::PPU * T::UD + h * C::S) return false;               // of dwords S apart
                for (int o = 0; o < T::NOPS; ++o)
                    if (T::op(o).pair == p0 % T::PPU && ((p0 / T::PPU * T::UD + T::op(o).dw) / C::S) % 4 != 0) return false;
            }
    return true;
}
static_assert(col_steps_ok<2>() && col_steps_ok<3>() && col_steps_ok<4>() && col_steps_ok<6>() && col_steps_ok<8>(), "inconsistent columns of the 16-row steps");
static_assert(steps_ok<2>() && steps_ok<3>() && steps_ok<4>() && steps_ok<6>() && steps_ok<8>(), "inconsistent list of matrix-core steps");
static_assert(layout_ok<2>() && layout_ok<3>() && layout_ok<4>() && layout_ok<6>() && layout_ok<8>(),
              "inconsistent packed layout table");

}  // namespace mq
