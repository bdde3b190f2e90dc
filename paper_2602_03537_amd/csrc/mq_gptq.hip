// The MatGPTQ column loop (Algorithm 2 of the paper's appendix), from the point where U, the
// upper-triangular Cholesky factor of the inverse Hessian, is given.  Rows of W are independent of
// each other; columns are strictly sequential (each column's code depends on every earlier
// column's error), so the work is cut as the listing cuts it:
//
//   gptq_block_kernel    : walks the B columns of a block for the rows of one workgroup: Algorithm 1
//                          on the current weight (mq_code_search.h), the error averaged over R and
//                          divided by U[j,j], rank-1 update of the block's remaining columns;
//   gptq_trailing_kernel : W[:, i+B:] -= E @ U[i:i+B, i+B:], eight rows x four columns per lane.
//
// Every rounding decides later codes, so the arithmetic is fixed: binary32, each operation
// rounded on its own (no contraction), the error sum over r ascending as ((w - D_r1) + (w - D_r2))
// + ..., then / |R|, then / U[j,j]; an update is w = w - (E * U[j,k]); the update of the rest is
// applied as the same rank-1 terms in ascending j, so results do not depend on B.
#include "mq_code_lanes.h"
#include "mq_internal.h"
#include "mq_static_for.h"

namespace mq {

constexpr int kGptqMaxBlock = 128;
constexpr int kTrailRows = 8;
constexpr int kGptqMaxWaves = 8;  // of a workgroup of the block kernel

template <int CTRL> __device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL> __device__ __forceinline__ float dpp_f(float v) {
    return __builtin_bit_cast(float, dpp_u<CTRL>(__builtin_bit_cast(uint32_t, v)));
}
// lexicographic minimum of (E's bits, key) with err carried along, over two lanes
template <int CTRL> __device__ __forceinline__ void argmin_step(uint32_t &E, uint32_t &key, float &err) {
    const float oerr = dpp_f<CTRL>(err);
    const uint32_t oE = dpp_u<CTRL>(E), okey = dpp_u<CTRL>(key);
    const bool take = (((uint64_t)oE << 32) | okey) < (((uint64_t)E << 32) | key);
    E = take ? oE : E;
    key = take ? okey : key;
    err = take ? oerr : err;
}

// The smallest code with E's bits, q being one (mq_code_search.h: they are a run that ends at q): the lanes of the row try every
// 16th code below it, then the 15 in between
template <uint32_t MASK>
__device__ __forceinline__ uint32_t row_lowest_equal(int q, uint32_t bits, float w, float s, float z, const QuantLambda &lam, int part) {
    const int row_bit = (threadIdx.x & 63) & ~(kRowLanes - 1);
#pragma unroll 1
    for (int step = kRowLanes; step; step /= kRowLanes) {
        const bool same = code_same<MASK>(q - step * (part + 1), bits, w, s, z, lam);
        q -= step * __builtin_popcount((uint32_t)(__ballot(same) >> row_bit) & 0xffffu);
    }
    return (uint32_t)q;
}
// The 128 columns of a block for the rows of one workgroup.  What bounds it is the serial chain of the column steps
// (a column's code decides the next column's weight), so a step is made short and everything else is kept off it:
//   * kRowLanes lanes share a row and evaluate the handful of candidates that can win (mq_code_search.h) side by side, each with
//     the error it would propagate (two correctly rounded divisions, beside the chain that compares the E); DPP steps pick the winner;
//   * the block's weights live in registers, column k = 16 c + part in register c of lane `part` (after 16 columns the
//     registers move up by one), so that a column's weight reaches its row in one DPP broadcast;
//   * the block of U lives in LDS; 16 steps are straight-line code, so that its values are read well ahead.
// 4096 rows x 4096 columns, R = {3,4,8}: 43 - 45 us a block = 0.34 us a step, of about 145 instructions of one wave per SIMD (160 us
// with all 256 candidates over 64 lanes and the weights in LDS); the whole loop 6.85 -> 2.95 ms.
template <uint32_t MASK, bool ALL>
__global__ __launch_bounds__(64 * kGptqMaxWaves, 4) void gptq_block_kernel(const float *__restrict__ W, int64_t ldw, int64_t N, int64_t i0,
                                                          int B, const float *__restrict__ U, int64_t ldu,
                                                          const _Float16 *__restrict__ scales,
                                                          const _Float16 *__restrict__ zeros, int64_t G,
                                                          const QuantLambda lam, float n_widths,
                                                          uint8_t *__restrict__ Q, int64_t ldq, float *__restrict__ E) {
#pragma clang fp contract(off)
    constexpr int NC = kGptqMaxBlock / kRowLanes;
    __shared__ float ul[kGptqMaxBlock * kGptqMaxBlock + kGptqMaxBlock];  // row j of the block at ul + 128 j; padding
    __shared__ float rd[kGptqMaxBlock];                  // 1 / U[j,j]
    const int tid = threadIdx.x;
    const int part = tid & (kRowLanes - 1);
    const int64_t n = (int64_t)blockIdx.x * (blockDim.x / kRowLanes) + tid / kRowLanes;
    const bool valid = n < N;
    const int64_t nr = valid ? n : N - 1;  // idle rows shadow the last one and store nothing
    // a block never straddles a group (B divides the group size and blocks start at multiples of B)
    const int64_t g = i0 / kGroup;
    const float s_in = (float)scales[nr * G + g];
    const float z = (float)zeros[nr * G + g];
    // a row with a negative scale is decided on its negative: every step of the loop is odd in (w, scale)
    const float sign = code_sign(s_in), s = s_in * sign;
    float wreg[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) wreg[c] = c * kRowLanes < B ? W[nr * ldw + i0 + c * kRowLanes + part] : 0.f;
    const float inv_s = 1.f / s, z1 = z + 1.f;
    const LaneCandidate lc = lane_candidate<MASK>(part);
    const bool grid_ok = code_grid_normal(s, z);
    const bool runs = !ALL && lam.v[kC - 1] == 0.f;  // uniform
    const float nw = ALL ? (float)popc8(MASK) : n_widths, inv_nw = 1.f / nw;
    {
        // the upper triangle, columns fastest (B is 16, 32, 64 or 128: a thread keeps its column), sixteen loads in flight
        // per thread; what lies below it is not read from U, and not used
        const int col = tid & (B - 1), row0 = tid / B, rows = blockDim.x / B;
        const float *src = U + i0 * ldu + i0 + col;
        for (int j0 = row0; j0 < B; j0 += 16 * rows) {
            float v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int j = j0 + i * rows;
                v[i] = src[(int64_t)(j < col ? j : col) * ldu];
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int j = j0 + i * rows;
                if (j < B) ul[j * kGptqMaxBlock + col] = v[i];
            }
        }
    }
    bool u_ok = true;
    if (tid < B) {
        const float ujj = U[(i0 + tid) * ldu + i0 + tid];
        rd[tid] = 1.f / ujj;
        u_ok = divisor_plain(ujj);
    }
    const bool fast_ok = grid_ok & (__syncthreads_and(u_ok) != 0);
    // (not where W is loaded: the loads of U would wait for it, 1.5 us a launch)
#pragma unroll
    for (int c = 0; c < NC; ++c) wreg[c] *= sign;
    for (int c0 = 0; c0 < B; c0 += kRowLanes) {
        // 16 columns, one of them per lane of a row in wreg[0]; register k holds this lane's column 16 k further on.
        // (Past the block's end the registers hold nothing of use, and the rows of U run into the padding.)
        const float *urows = ul + c0 * kGptqMaxBlock + c0;
        float keep_err = 0.f;
        uint32_t keep_q = 0;
        float ur[2][NC], ujj[2], rjj[2];  // row jj of these 16 columns and row jj + 1, on its way
        int u_off = part;
        auto fetch_u = [&](auto jc) {
            constexpr int jj = jc;
            // (opaque: else the rows of all 16 steps are read at once, into more registers than there are)
            asm volatile("" : "+v"(u_off));
            ujj[jj % 2] = urows[jj * kGptqMaxBlock + jj];
            rjj[jj % 2] = rd[c0 + jj];
#pragma unroll
            for (int k = 0; k < NC; ++k) ur[jj % 2][k] = urows[jj * kGptqMaxBlock + k * kRowLanes + u_off];
        };
        fetch_u(IntC<0>{});
        static_for<kRowLanes>([&](auto jc) {
#pragma clang fp contract(off)
            constexpr int jj = jc;
            if constexpr (jj + 1 < kRowLanes) fetch_u(IntC<jj + 1>{});
            const float w = dpp_f<0x150 + jj>(wreg[0]);  // row_newbcast: column jj's weight, to all lanes of the row
            const int Uc = code_estimate(w, inv_s, z1);
            const LaneDecision d = lane_decision<MASK, ALL>(lc, Uc, w, s, z, lam, runs, fast_ok, nw, inv_nw, ujj[jj % 2], rjj[jj % 2]);
            uint32_t Eb = d.bits, key = d.key;
            float err = d.err;
            const bool bad = d.bad;
            asm volatile("" : "+v"(Eb), "+v"(key));  // selects below, no branch
            Eb = bad ? 0u : Eb;
            key = bad ? kLaneBad : key;
            constexpr int NL = lanes_used(MASK);
            argmin_step<0xB1>(Eb, key, err);  // quad_perm [1,0,3,2]
            argmin_step<0x4E>(Eb, key, err);  // quad_perm [2,3,0,1]
            if constexpr (NL >= 8) argmin_step<0x141>(Eb, key, err);   // row_half_mirror: the quads of 8 lanes
            if constexpr (NL >= 16) argmin_step<0x140>(Eb, key, err);  // row_mirror: the halves of 16 lanes
            uint32_t qw = key >> 2;
            if (__builtin_expect((key & (kLaneBad | kLaneLook)) != 0, 0)) {  // rare; the lanes of a row take it together
                // the list's minimum is the least E there is unless the search did not hold: then all that is left is a smaller code with it
                if (key & kLaneBad) qw = code_search_closely<MASK>(Uc, w, s, z, lam);
                else qw = row_lowest_equal<MASK>((int)qw, Eb, w, s, z, lam, part);
                float e2 = 0.f, a2 = 0.f, e8_2;
                bool any2 = false;
                code_terms<MASK, ALL>(qw, w, s, z, lam, e2, a2, any2, e8_2);
                err = (a2 / nw) / ujj[jj % 2];
            }
            keep_q = part == jj ? qw : keep_q;
            keep_err = part == jj ? err : keep_err;
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                const float p = err * ur[jj % 2][k];
                wreg[k] = wreg[k] - p;
                asm volatile("" : "+v"(wreg[k]));  // here: put off to the end of the 16 steps it would hold their rows of U in registers
            }
        });
        if (valid) {
            Q[n * ldq + i0 + c0 + part] = (uint8_t)keep_q;
            E[n * B + c0 + part] = keep_err * sign;
        }
#pragma unroll
        for (int k = 0; k + 1 < NC; ++k) wreg[k] = wreg[k + 1];
    }
}

// W[n, c0 + k] -= sum_j E[n, j] * U[i0 + j, c0 + k], the terms subtracted one by one in ascending j.
// A wave owns kTrailRows rows x 256 columns (four consecutive columns per lane): per j one 16-byte
// load of U per lane, the E values are the same for the whole wave (scalar loads), and 2 x 4 x
// kTrailRows vector operations, so the kernel is bound by the vector ALUs, not by loads.
// VEC4 needs c0, ldw, ldu multiples of 4 and 16-byte aligned W and U; otherwise one column per lane.
template <bool VEC4>
__global__ __launch_bounds__(64) void gptq_trailing_kernel(float *__restrict__ W, int64_t ldw, int64_t N, int64_t c0,
                                                           int64_t ncols, const float *__restrict__ E, int B,
                                                           const float *__restrict__ U, int64_t ldu, int64_t i0,
                                                           int64_t kblocks) {
#pragma clang fp contract(off)
    constexpr int CPT = VEC4 ? 4 : 1;  // columns per lane
    const int64_t rb = blockIdx.x / kblocks;
    const int64_t k = ((blockIdx.x - rb * kblocks) * 64 + threadIdx.x) * CPT;
    const int64_t n0 = rb * kTrailRows;
    const bool in = k < ncols;  // ncols is a multiple of CPT on the VEC4 path
    const int64_t kc = in ? k : 0;
    float w[kTrailRows][CPT];
    int64_t row[kTrailRows];
#pragma unroll
    for (int i = 0; i < kTrailRows; ++i) {
        row[i] = n0 + i < N ? n0 + i : N - 1;  // uniform over the wave
        const float *src = W + row[i] * ldw + c0 + kc;
        if constexpr (VEC4) {
            const float4 v = *reinterpret_cast<const float4 *>(src);
            w[i][0] = v.x; w[i][1] = v.y; w[i][2] = v.z; w[i][3] = v.w;
        } else {
            w[i][0] = src[0];
        }
    }
    const float *u = U + i0 * ldu + c0 + kc;
    // eight terms at a time: their loads (one 16-byte piece of U per lane and term, eight consecutive E values
    // per row through the scalar unit) are all issued before the first of them is used
    constexpr int JC = 8;  // B is a multiple of 16
    for (int j0 = 0; j0 < B; j0 += JC) {
        float uv[JC][CPT];
#pragma unroll
        for (int jj = 0; jj < JC; ++jj) {
            if constexpr (VEC4) {
                const float4 v = *reinterpret_cast<const float4 *>(u + (int64_t)(j0 + jj) * ldu);
                uv[jj][0] = v.x; uv[jj][1] = v.y; uv[jj][2] = v.z; uv[jj][3] = v.w;
            } else {
                uv[jj][0] = u[(int64_t)(j0 + jj) * ldu];
            }
        }
        float ev[kTrailRows][JC];
#pragma unroll
        for (int i = 0; i < kTrailRows; ++i)
#pragma unroll
            for (int jj = 0; jj < JC; ++jj) ev[i][jj] = E[row[i] * B + j0 + jj];
#pragma unroll
        for (int jj = 0; jj < JC; ++jj)
#pragma unroll
            for (int i = 0; i < kTrailRows; ++i)
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    const float p = ev[i][jj] * uv[jj][c];
                    w[i][c] = w[i][c] - p;
                }
    }
    if (!in) return;
#pragma unroll
    for (int i = 0; i < kTrailRows; ++i) {
        if (n0 + i < N) {
            float *dst = W + (n0 + i) * ldw + c0 + k;
            if constexpr (VEC4)
                *reinterpret_cast<float4 *>(dst) = make_float4(w[i][0], w[i][1], w[i][2], w[i][3]);
            else
                dst[0] = w[i][0];
        }
    }
}

// Waves per workgroup (four rows each): four up to 8192 rows, which is two workgroups per compute unit, and all that a
// workgroup's 67 KB of LDS let in; eight beyond, so that twice the rows share a compute unit's LDS and are resident at one time
// (R = {3,4,8}, us a block: 16384 rows 97, with four waves 112; 20480 rows 132 and 141).  Sixteen would leave one workgroup per compute unit
// (at most 128 registers a lane: 16 waves), the same rows in coarser pieces: 20480 rows 162, 65536 rows 328 against 323, and {2,3,4,6,8} 233 against 176.
inline int gptq_block_waves(int64_t N) { return N <= 8192 ? 4 : kGptqMaxWaves; }

template <uint32_t MASK, bool ALL>
static hipError_t launch_gptq_mask(float *W, int64_t ldw, int64_t N, int64_t K, const float *U, int64_t ldu,
                                   const _Float16 *scales, const _Float16 *zeros, const QuantLambda &lam, float n_widths,
                                   int B, uint8_t *Q, int64_t ldq, float *E, hipStream_t s) {
    const int64_t G = K / kGroup;
    if (((K + 63) / 64) * ((N + kTrailRows - 1) / kTrailRows) > (int64_t)0x7fffffff) return hipErrorInvalidValue;
    const int waves = gptq_block_waves(N), rows = waves * (64 / kRowLanes);
    // B, K and the block starts are multiples of 16, so only the strides and base addresses decide
    const bool vec4 = ldw % 4 == 0 && ldu % 4 == 0 && (reinterpret_cast<uintptr_t>(W) & 15) == 0 &&
                      (reinterpret_cast<uintptr_t>(U) & 15) == 0;
    for (int64_t i0 = 0; i0 < K; i0 += B) {
        hipError_t e = launch((gptq_block_kernel<MASK, ALL>), dim3((unsigned)((N + rows - 1) / rows)), dim3(64 * waves), 0, s,
                              W, ldw, N, i0, B, U, ldu, scales, zeros, G, lam, n_widths, Q, ldq, E);
        if (e != hipSuccess) return e;
        const int64_t c0 = i0 + B, ncols = K - c0;
        if (ncols > 0) {
            const int64_t rblocks = (N + kTrailRows - 1) / kTrailRows;
            if (vec4) {
                const int64_t kblocks = (ncols + 255) / 256;
                e = launch(gptq_trailing_kernel<true>, dim3((unsigned)(kblocks * rblocks)), dim3(64), 0, s, W, ldw, N, c0,
                           ncols, E, B, U, ldu, i0, kblocks);
            } else {
                const int64_t kblocks = (ncols + 63) / 64;
                e = launch(gptq_trailing_kernel<false>, dim3((unsigned)(kblocks * rblocks)), dim3(64), 0, s, W, ldw, N, c0,
                           ncols, E, B, U, ldu, i0, kblocks);
            }
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

hipError_t launch_gptq(float *W, int64_t ldw, int64_t N, int64_t K, const float *U, int64_t ldu, const _Float16 *scales,
                       const _Float16 *zeros, const float *lambda, int B, uint8_t *Q, int64_t ldq, float *E,
                       hipStream_t s) {
    QuantLambda lam;
    uint32_t need = 0;
    int nw = 0;
    for (int i = 0; i < kC; ++i) {
        lam.v[i] = lambda[i];
        if (lambda[i] != 0.f) {
            need |= 1u << i;
            ++nw;
        }
    }
    const float n_widths = (float)nw;
    switch (quant_variant_mask(need)) {
        case 0x80u: return launch_gptq_mask<0x80u, true>(W, ldw, N, K, U, ldu, scales, zeros, lam, n_widths, B, Q, ldq, E, s);
        case 0x8Cu:
            if (need == 0x8Cu)
                return launch_gptq_mask<0x8Cu, true>(W, ldw, N, K, U, ldu, scales, zeros, lam, n_widths, B, Q, ldq, E, s);
            return launch_gptq_mask<0x8Cu, false>(W, ldw, N, K, U, ldu, scales, zeros, lam, n_widths, B, Q, ldq, E, s);
        case 0xAEu: return launch_gptq_mask<0xAEu, false>(W, ldw, N, K, U, ldu, scales, zeros, lam, n_widths, B, Q, ldq, E, s);
    }
    return launch_gptq_mask<0xFFu, false>(W, ldw, N, K, U, ldu, scales, zeros, lam, n_widths, B, Q, ldq, E, s);
}

}  // namespace mq
