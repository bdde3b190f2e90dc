// Internal declarations shared by the host API and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/mq.h"
#include "mq_layout.h"
#include "mq_routes.h"

namespace mq {

// Caps on the wavefronts / workgroups of a persistent launch.  They size the partial-sum slots of a workspace, which
// must be plain host arithmetic (callable without a device); every launcher asks the device for its compute units
// and the kernel's occupancy and launches min(what is resident there, the cap), so a smaller or larger part stays
// correct and only loses the slots it cannot use.  (8192 = 256 compute units x 32 waves, the MI355X; shares of workgroups use an eighth and less of them.)
constexpr int kMaxWaves = 8192;
// 5 .. 16 rows: what a workspace holds (callers see its size, which has room to spare): pairs of partial-sum slots, floats in one, and bytes
// for the activations of a group
constexpr int kMidSlots = 256, kMidSlotFloats = 8 * 64 * 16, kMidXBytes = 6 * 1024;
// Persistent row kernels: each wave or workgroup serves up to so many interleaved shares of the schedule, so that
// layers of different widths (different speed per byte) even out.
constexpr int kSharesPerWave = 8;
constexpr size_t kMaxSlotBytes = (size_t)32 << 20;
inline int max_workers_valu(int64_t M) {
    const size_t by_mem = kMaxSlotBytes / (2 * (size_t)M * 64 * sizeof(float));
    const size_t want = (size_t)kMaxWaves * kSharesPerWave;
    return (int)(by_mem < want ? by_mem : want);
}
constexpr int kCounterBytesAlign = 256;

constexpr int kWideXtBlockBytes = 8 * 1024;  // prepared activations of one (group, chunk of 32 columns)

// One layer as the persistent kernels see it.
struct LayerDesc {
    const uint4 *Wp;
    const _Float16 *st;
    const _Float16 *zt;
    const _Float16 *x;
    _Float16 *y;
    const uint4 *xt;        // wide kernel: activations re-ordered by the prep kernel
    const void *x_bf16;     // row kernels with kFlagXBf16: the caller's bf16 activations (x then points to their fp16 copy)
    int32_t N, K, G, RB;    // RB = row blocks = ceil(N/64); super row blocks of the wide kernel: ceil(N/256)
    int32_t r;
    int32_t cost;           // schedule cost of one (row block, group) tile
    int32_t cnt_off;        // index of this layer's first row-block counter (CB*RB counters)
    int32_t M;              // batch rows of x
    int32_t CB;             // column chunks: 1, or the wide kernel's passes
    int32_t job_start;      // prep kernel: sum of CB*G over the preceding layers
    int32_t rs;             // 0, or: Wp is the 8-bit parent (r == 8) and Eq. 1 to rs bits is applied in registers
    int32_t flags;          // kFlagXBf16: x holds bf16 values; kFlagYBf16: y is written as bf16
    int32_t zmask;          // -1; a symmetric layer: zt is zmask + 1 lines of 64 x 128.0, tile u reads line u & zmask
    int32_t chain;          // chained small stack: bits 0..7 the layer's stage; kChainWaits: x is read only after every earlier stage is complete
    uint64_t cost_start;    // sum of CB*RB*G*cost over the preceding layers
};

// The descriptors of a small stack (at most kSmallStackLayers layers), passed to its low-latency kernel with the kernel
// arguments: a workgroup reads its descriptor from there in 0.3 us, where a first read from the table in device memory
// took 1.2 us of a launch that lasts 8.
constexpr int kChainWaits = 0x100;
constexpr int kChainMaxM = 3;
constexpr int kChainCounters = kSmallStackLayers + 1;
struct SmallTable {
    LayerDesc d[kSmallStackLayers];
};
static_assert(sizeof(SmallTable) <= 2048, "kernel arguments are limited to 4 KiB");

struct StackParams {
    const LayerDesc *table;  // device table, or nullptr to use `single`
    int32_t n_layers;
    int32_t nwaves;          // row kernels: workgroups launched (by_wave: waves)
    int32_t nworkers;        // schedule shares ("workers"); workgroup or wave w serves workers w, w + nwaves, ...
    uint64_t cost_total;
    float *part;             // [nworkers][2][slot_floats] partial sums
    int32_t *cnt;            // row-block counters, zero between launches
    int32_t M;
    int32_t slot_floats;     // wide: floats per partial-sum slot (4 x chunks x 32*64)
    int32_t n_jobs;          // wide: jobs of the prep kernel
    int32_t finish_apart;    // wide, single layers: row blocks that several shares worked on are finished by a launch of its own
    int32_t by_wave;         // row kernels: shares of the persistent schedule belong to waves (wave_shares), else to workgroups
    int32_t worker_cap;      // 0, or: `part` holds slots for this many schedule shares only (a small workspace)
    int32_t ks_cap;          // low-latency launch of a small stack: most K slices per row block (0: as one layer would choose)
    int32_t ll_start[16];    // ... and the first workgroup of each layer (a workgroup finds its layer without reading the table)
    // Chained small stack (some layer reads what earlier layers of the same launch write): the layers form stages,
    // a new stage starting at every layer that waits.  Counter chain_off + s of `cnt` counts the finished row blocks
    // of stage s, counter chain_off + kSmallStackLayers all of them; the last row block of the launch zeroes them.
    int32_t chain_total;     // row blocks of all layers; 0: nothing is chained and nothing is counted
    int32_t chain_off;
    int32_t stage_rb[16];    // row blocks per stage
    LayerDesc single;
};

// Wide kernel: cost of a super-tile (256 rows x one group) per pass with C chunks of 32 columns, again the measured
// times of uniform stacks (12 Llama-3-70B blocks at M = 32, 64, 96, 128; units of 10 us; the first two rows with two
// workgroups per compute unit, as stacks run there).  The matrix-core work grows with C, the unpacking with r; bytes
// matter least.
inline int wide_tile_cost(int r, int C) {
    static const int t[4][5] = {{130, 141, 147, 178, 199}, {173, 186, 191, 222, 239},
                                {239, 252, 262, 306, 323}, {293, 308, 318, 358, 377}};
    const int ri = r == 2 ? 0 : r == 3 ? 1 : r == 4 ? 2 : r == 6 ? 3 : 4;
    return t[(C < 1 ? 1 : C > 4 ? 4 : C) - 1][ri];
}

// Enqueue a kernel and return the status of THIS launch.  The runtime's sticky "last error" is neither read nor
// cleared, so an error the caller's own earlier work left pending stays where the caller will find it.
template <class... KArgs, size_t... I>
inline hipError_t launch_impl(void (*kernel)(KArgs...), dim3 grid, dim3 block, unsigned lds_bytes, hipStream_t s,
                              std::tuple<std::decay_t<KArgs>...> &vals, std::index_sequence<I...>) {
    void *ptrs[sizeof...(KArgs) ? sizeof...(KArgs) : 1] = {static_cast<void *>(&std::get<I>(vals))...};
    return hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, ptrs, lds_bytes, s);
}
template <class... KArgs, class... Args>
inline hipError_t launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, unsigned lds_bytes, hipStream_t s, Args &&...args) {
    static_assert(sizeof...(KArgs) == sizeof...(Args), "argument count differs from the kernel's");
    std::tuple<std::decay_t<KArgs>...> vals{static_cast<std::decay_t<KArgs>>(std::forward<Args>(args))...};
    return launch_impl(kernel, grid, block, lds_bytes, s, vals, std::index_sequence_for<KArgs...>{});
}

inline int64_t pad_rows(int64_t N) { return (N + kRowBlock - 1) / kRowBlock * kRowBlock; }

// launchers (mq_pack.hip / mq_linear.hip); each returns the hipError of the launch
hipError_t launch_slice(const uint8_t *parent, int64_t n, int c, int r, uint8_t *out, hipStream_t s);
hipError_t launch_pack(const uint8_t *S, int64_t N, int64_t K, int r, uint4 *packed, hipStream_t s);
hipError_t launch_unpack(const uint4 *packed, int64_t N, int64_t K, int r, uint8_t *S, hipStream_t s);
hipError_t launch_slice_pack(const uint8_t *parent, int64_t N, int64_t K, int r, uint4 *packed, hipStream_t s);
hipError_t launch_reslice(const uint4 *parent8, int64_t N, int64_t K, int r, uint4 *packed, hipStream_t s);
// n layers in ceil(n / kResliceBatch) launches; all arrays are host arrays of n entries
constexpr int kResliceBatch = 16;
hipError_t launch_reslice_many(const uint4 *const *src, uint4 *const *dst, const int64_t *N, const int64_t *K,
                               const int *r, int n, hipStream_t s);
hipError_t launch_pack_meta(const _Float16 *sc, const _Float16 *zr, int64_t N, int64_t G, _Float16 *st,
                            _Float16 *zt, hipStream_t s);
hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s);
// xor of all 16-byte words of buf is xor-ed into *out (measurement aid); bytes is a multiple of 16
hipError_t launch_read_probe(const void *buf, size_t bytes, uint32_t *out, hipStream_t s);
// table: host, n descriptors -> dst: device.  ceil(n / 32) small launches; the host array is free again on return.
hipError_t launch_write_table(const LayerDesc *table, int n, LayerDesc *dst, hipStream_t s);
// Algorithm 2 column loop (mq_gptq.hip): K / 128 launches on s.
hipError_t launch_gptq(float *W, int64_t ldw, int64_t N, int64_t K, const float *U, int64_t ldu, const _Float16 *scales,
                       const _Float16 *zeros, const float *lambda, uint8_t *Q, int64_t ldq, hipStream_t s);
// Algorithm 1 (mq_quant.hip).  lambda: host, kC floats (width r at [r-1]); vec4: four columns per lane (alignment checked by the caller)
hipError_t launch_quant(const float *W, int64_t ldw, int64_t N, int64_t ncols, int64_t col0, const _Float16 *scales,
                        const _Float16 *zeros, int64_t G, const float *lambda, uint8_t *Q, int64_t ldq, bool vec4,
                        hipStream_t s);
// bf16 activations of the layers that carry kFlagXBf16 -> fp16 in their LayerDesc::xt (ahead of a launch of row kernels)
hipError_t launch_xcvt(const StackParams &p, hipStream_t s);
// Fills p.nwaves and launches (row kernels, M <= 16).  max_cost = largest tile cost in the stack.
// from_parent: every layer has rs != 0 (the kernel variant that slices in registers).
hipError_t launch_stack(StackParams p, int max_cost, bool from_parent, hipStream_t s);
// Single layer (low_latency_single): one workgroup per (row block, K slice, chunk of 16 rows); see mq_linear.hip.
hipError_t launch_linear_rb(const LayerDesc &L, float *part, int32_t *cnt, hipStream_t s);
// The same shape for a small stack (low_latency_stack): all layers' workgroups in one launch.  `table` is the host copy
// of the descriptors; false = the stack is too big for it.
// ks_cap: see StackParams.
// ll_start: see StackParams (16 entries).
// all_resident: the device holds every workgroup of that shape at one time (what a chained stack needs).
bool linear_rb_stack_shape(const LayerDesc *table, int n_layers, size_t part_bytes, bool from_parent, bool chained,
                           int *blocks, int *waves, int *ks_cap, int32_t *ll_start, bool *all_resident);
hipError_t launch_linear_rb_stack(const StackParams &p, const SmallTable &t, int blocks, int waves, bool from_parent,
                                  hipStream_t s);
// Wide: activation prep kernel + persistent kernel, one workgroup per share (single layers: + a finishing launch where p.finish_apart).
hipError_t launch_stack_wide(StackParams p, int max_cost, hipStream_t s);

}  // namespace mq
