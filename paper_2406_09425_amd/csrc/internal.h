// Internal declarations shared by the host and kernel translation units of
// libsgprs.  Nothing here is part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <atomic>
#include <hip/hip_ext.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <string>
#include <cstring>
#include <utility>
#include <mutex>
#include <vector>

#include "sgprs.h"

namespace sgprs {

// ---- error reporting -------------------------------------------------------
int fail(int status, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

#define SGPRS_HIP(call)                                                                   \
    do {                                                                                  \
        hipError_t e_ = (call);                                                           \
        if (e_ != hipSuccess)                                                             \
            return ::sgprs::fail(SGPRS_ERR_HIP, "%s failed: %s (%s:%d)", #call,           \
                                 hipGetErrorString(e_), __FILE__, __LINE__);              \
    } while (0)

// CU-masked streams are hardware queues, and the queues of a process take turns on four dispatch
// pipes, queue after queue.  Two queues of one pipe that are busy together slow each other down four
// times (measured on MI355X, batch-1 tasks on 32-CU partitions of a pool of eight: 290 us per
// inference on partitions (p, p + 4) for every p, 74 us on all 24 other pairs; 39.5 us on any four
// partitions that differ modulo 4, 145-156 us on four that do not).  Idle queues cost nothing.
constexpr int kDispatchPipes = 4;
constexpr int kMaxBusyQueues = kDispatchPipes;

// ---- pool ------------------------------------------------------------------
struct Partition {
    hipStream_t stream = nullptr;
    std::vector<uint32_t> mask;
    int cus = 0;       // in the mask
    int plan_cus = 0;  // that launches are planned for
};

}  // namespace sgprs

struct sgprs_pool {
    int device = 0;
    int total_cus = 0;
    int n_xcd = 1;
    int cus_per_partition = 0;  // 0 when created from explicit masks of mixed size
    std::vector<sgprs::Partition> parts;
};

namespace sgprs {

// CUs that launches are planned for on a partition with an interleaved mask (sgprs_build_cu_mask; other
// masks are planned for all their CUs).  Workgroups are dealt to the 8 dies in turn and, within a die,
// to its 4 shader engines in turn, and a workgroup waits for room in the engine whose turn it is:
// the engine with the fewest CUs sets the pace, so beyond 32 CUs a partition is worth a multiple of
// 32 (batch-8 inference on 192 / 200 / 216 / 224 CUs, planned for all of them: 167 / 207 / 195 / 146 us;
// batch 1 on 32 / 48 / 56 / 64: 135 / 135 / 160 / 108).
inline int planning_cus(int cus) { return cus < 1 ? 1 : cus < 32 ? cus : cus / 32 * 32; }

// validates pool/partition, returns the stream and the number of CUs in the mask
int resolve(sgprs_pool_t* pool, int partition, hipStream_t* stream, int* cus);
// the same for calls that launch planned work: the CU count is the one to plan for
int resolve_launch(sgprs_pool_t* pool, int partition, hipStream_t* stream, int* plan_cus);

// With L = ceil(log2 d) and mul = ceil(2^(31+L) / d) < 2^32, floor(m / d) = (m * mul) >> (31 + L) for
// every 0 <= m < 2^31: the upper half of 2 m * mul, shifted by L.
inline void div_constants(int d, unsigned* mul, int* sh)
{
    int L = 0;
    while ((1ll << L) < d) ++L;
    *mul = (unsigned)(((1ull << (31 + L)) + (unsigned)d - 1) / (unsigned)d);
    *sh = L;
}

inline size_t dtype_size(int dtype) { return dtype == SGPRS_BF16 ? 2 : 4; }
inline bool dtype_ok(int dtype) { return dtype == SGPRS_F32 || dtype == SGPRS_BF16; }

// Device side: two fp32 values to one dword of bf16 (round to nearest even, a single packed
// conversion), then the optional ReLU on the packed pair as a signed 16-bit maximum against
// `floor16x2`: 0 for a ReLU (negative values and -0 carry the sign bit, read as negative integers
// and become +0; rounding keeps the sign, so this equals clamping before the conversion),
// 0x80008000 for none (the smallest 16-bit integer twice: every pattern passes unchanged).
__device__ __forceinline__ unsigned pack_bf16x2_relu(float lo, float hi, unsigned floor16x2)
{
    typedef float pk_f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 pk_bf16x2 __attribute__((ext_vector_type(2)));
    typedef short pk_s16x2 __attribute__((ext_vector_type(2)));
    const pk_f32x2 f = {lo, hi};
    const pk_s16x2 b = __builtin_bit_cast(pk_s16x2, __builtin_convertvector(f, pk_bf16x2));
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(b, __builtin_bit_cast(pk_s16x2, floor16x2)));
}
constexpr unsigned kReluFloor = 0u, kNoReluFloor = 0x80008000u;

// host bf16 conversion, round to nearest even
inline uint16_t f32_to_bf16_bits(float f)
{
    uint32_t u;
    __builtin_memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);  // quiet NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
inline float bf16_bits_to_f32(uint16_t b)
{
    uint32_t u = (uint32_t)b << 16;
    float f;
    __builtin_memcpy(&f, &u, 4);
    return f;
}

// ---- convolution -----------------------------------------------------------
// Stem layout constants: 7 tap rows, each 7 taps x 4 channel slots (3 real
// channels + 1 zero) = 28 elements padded to 32.
constexpr int kStemTapRow = 32;
constexpr int kStemK = 7 * kStemTapRow;  // 224

inline bool is_stem(const sgprs_conv_desc_t& d)
{
    return d.cin == 3 && d.r == 7 && d.s == 7 && d.stride == 2 && d.pad == 3;
}
inline bool is_igemm(const sgprs_conv_desc_t& d)
{
    return d.cin % 32 == 0 && d.r == d.s && (d.r == 1 || d.r == 3) && (d.stride == 1 || d.stride == 2);
}
int check_conv_desc(const sgprs_conv_desc_t* d);
inline int out_dim(int in, int k, int stride, int pad) { return (in + 2 * pad - k) / stride + 1; }

// Small memo for launch planning: the same few shapes are planned again on every launch, and the
// geometry searches behind a plan walk all row tiles.  Keys are plain structs compared bytewise
// (fill them with memset first); the oldest entries are dropped.
template <class K, class V, int CAP = 128> struct PlanMemo {
    std::vector<std::pair<K, V>> items;
    const V* find(const K& k)
    {
        for (size_t i = 0; i < items.size(); ++i)
            if (!memcmp(&items[i].first, &k, sizeof(K))) {
                if (i >= 8) {  // entries in use drift to the front
                    std::swap(items[i], items[i / 2]);
                    i /= 2;
                }
                return &items[i].second;
            }
        return nullptr;
    }
    void put(const K& k, const V& v)
    {
        if ((int)items.size() >= CAP) items.erase(items.begin(), items.begin() + CAP / 2);
        items.emplace_back(k, v);
    }
};
// Two levels: a memo per thread, read without a lock, in front of one per process behind a mutex,
// so that a thread that has never planned (a launcher thread just created) copies what another
// thread worked out instead of searching again.
template <class K, class V, int CAP = 128> struct SharedPlanMemo {
    std::mutex mu;
    PlanMemo<K, V, CAP> shared;
    template <class F> V get(PlanMemo<K, V, CAP>& local, const K& k, F compute)
    {
        if (const V* hit = local.find(k)) return *hit;
        V v;
        {
            std::lock_guard<std::mutex> guard(mu);
            if (const V* hit = shared.find(k)) v = *hit;
            else {
                v = compute();
                shared.put(k, v);
            }
        }
        local.put(k, v);
        return v;
    }
};
extern std::atomic<int> g_plan_generation;  // bumped whenever a tuning override changes what the planners return

// Tile configuration of one implicit-GEMM launch.
struct ConvPlan {
    int kind = 0;      // 0: implicit GEMM, 1: LDS-patch 3x3 kernel, 2: its stride-2 variant, 3: row streaming,
                       // 4: implicit GEMM with K split over a workgroup's wavefronts,
                       // 5: weights from the L2 to registers (variant: wavefronts that share a tile),
                       // 6: K split over a workgroup's wavefronts, input patch in LDS,
                       // 7: fp32 by three bf16 planes of every operand,
                       // 8: stride-2 pair, weights from the L2 to registers (5, 7 and 8 only where the weights are there in fragment order)
    int variant = 0;   // index into the kernel's tile table (row streaming: output rows per stream and job)
    int bm = 0, bn = 0;
    int splits = 1;    // split-K factor (grid.z)
    int ktiles = 0;    // total k-tiles of 128 bytes
    int grid_m = 0, grid_n = 0;
};
// Chooses tile shape and split-K factor from the GEMM shape and the CU count of
// the partition the launch will run on.
// (has_residual: kernels without a residual input are left out; ksplit false: so is the kernel that
// splits K over a workgroup's wavefronts; fragments: the weights are there in fragment order too).
ConvPlan plan_conv(const sgprs_conv_desc_t& d, int partition_cus, bool has_residual = false, bool ksplit = true, bool fragments = false);
// The plan of d0 for a launch that also runs the block's shortcut d1 on the same input (same output shape).
ConvPlan plan_conv_pair(const sgprs_conv_desc_t& d0, const sgprs_conv_desc_t& d1, int partition_cus, bool fragments);
size_t conv_workspace_bytes(const sgprs_conv_desc_t& d, const ConvPlan& p);

struct KernelRecord {
    int kind = 0, variant = 0;
    double flops = 0, bytes = 0;
    hipEvent_t start = nullptr, stop = nullptr;
};
// Optional per-launch timing hook.  begin() appends a record and publishes its
// stop event in tl_stop; the next kernel launch (SGPRS_LAUNCH) attaches it to
// its own dispatch, so it carries the kernel's completion time.  A record's
// start is the stop event of the kernel queued just before it on the same
// stream (kernels of a run are queued back to back), or a plain event when
// there is none: separately recorded event packets would add microseconds of
// their own latency to every interval.
extern thread_local hipEvent_t tl_start, tl_stop;
// (Plain launches when no timing is attached: those are what stream capture records.)
#define SGPRS_LAUNCH(kernel, grid, block, lds, stream, ...)                                                             \
    do {                                                                                                                \
        if (::sgprs::tl_start || ::sgprs::tl_stop)                                                                      \
            hipExtLaunchKernelGGL(kernel, grid, block, lds, stream, ::sgprs::tl_start, ::sgprs::tl_stop, 0, __VA_ARGS__); \
        else                                                                                                            \
            hipLaunchKernelGGL(kernel, grid, block, lds, stream, __VA_ARGS__);                                          \
    } while (0)
struct Profiler {
    bool on = false;
    std::vector<KernelRecord> recs;      // records of the stage being run
    std::vector<hipEvent_t> event_pool;  // reused events
    size_t next_event = 0;
    hipEvent_t prev = nullptr;           // completion event of the previous kernel on this stream
    int begin(hipStream_t s, int kind, int variant, double flops, double bytes);
    int end(hipStream_t s);
    void reset(hipEvent_t prev_stop = nullptr) { recs.clear(); next_event = 0; prev = prev_stop; }
    ~Profiler();
};

enum KernelKind { kKindIgemm = 0, kKindStem = 1, kKindReduce = 2, kKindMaxpool = 3, kKindAvgpool = 4,
                  kKindFc = 5, kKindBnRelu = 6, kKindAdd = 7, kKindPatch = 8, kKindStemPool = 9,
                  kKindIgemmPair = 10, kKindS2Patch = 11, kKindRows = 12, kKindWtile = 13 };

// launchers (device pointers; validated by callers)
int launch_conv(const sgprs_conv_desc_t& d, const void* x, const void* w, const float* scale,
                const float* shift, const void* residual, void* y, void* ws, size_t ws_bytes,
                hipStream_t stream, int cus, Profiler* prof, const void* w_fragments = nullptr);
int launch_stem(const sgprs_conv_desc_t& d, const void* x, const void* w, const float* scale,
                const float* shift, void* y, hipStream_t stream, int cus, Profiler* prof);
int launch_maxpool(int dtype, int n, int h, int w, int c, const void* x, void* y, hipStream_t stream,
                   int cus, Profiler* prof);
int launch_bn_relu(int dtype, size_t pixels, int c, const void* x, const float* scale,
                   const float* shift, void* y, hipStream_t stream, int cus, Profiler* prof);
int launch_add_relu(int dtype, size_t count, const void* a, const void* b, void* y, int relu,
                    hipStream_t stream, int cus, Profiler* prof);
int launch_avgpool(int dtype, int n, int hw, int cin, const void* x, float* pooled, hipStream_t stream, Profiler* prof);
int launch_avgpool_fc(int dtype, int n, int hw, int cin, int cout, const void* x, const void* w,
                      const float* bias, float* logits, float* ws, hipStream_t stream, int cus,
                      Profiler* prof);
// FC of a batch on the matrix cores: v fp32 [n][cin], w [cout][cin] in dtype
bool fc_gemm_applicable(int n, int cin, int cout);
int launch_fc_gemm(int dtype, const float* v, const void* w, const float* bias, float* y, int n, int cin, int cout, hipStream_t stream, int cus);
// Device address of this GPU's static pooled-vector scratch (kStaticScratchFloats fp32), looked up
// on first use; nothing is allocated.
constexpr size_t kStaticScratchFloats = 64 * 2048;
constexpr int kMaxStaticScratchDevices = 16;
int static_scratch(int device, float** out);
int launch_probe(int n_blocks, int spin_cycles, uint32_t* out, hipStream_t stream);
int launch_mfma_probe(int cus, int steps, int random_data, unsigned long long* out, hipStream_t stream);
int launch_load_probe(int cus, const void* buf, size_t buf_bytes, unsigned region, int iters, unsigned* out, hipStream_t stream);
// fp32 stem on packed input rows, alone (pool false) or with the max-pool; no profiling record of its own
bool stem_f32_applicable(int n, int h, int w);
bool stem_f32_one_round(int n, int h, int w, int cus);  // with the pool: at most one tile per CU
int launch_stem_f32(int n, int h, int w, const void* x, const void* wts, const float* scale, const float* shift, void* y,
                    int relu, bool pool, hipStream_t stream, int cus);
// stage 0 fused: conv7x7/2 + BN + ReLU + max-pool 3x3/2
bool stem_pool_applicable(int dtype, int n, int h, int w, int cus);
// wts: the stem layout of sgprs_pack_conv_weights; wts_rows: bf16 fragments of pack_stem_rows, negated
// where scale is negative, and both tables (may be NULL: then the kernel that reads wts runs)
constexpr int kStemRowsElems = 44 * 512 + 256;
void pack_stem_rows(const float* oihw, const float* scale, const float* shift, uint16_t* out);
void stem_pool_force(int v);  // -1 automatic, 1: never the packed-row kernel
int launch_stem_pool(int dtype, int n, int h, int w, const void* x, const void* wts, const void* wts_rows,
                     const float* scale, const float* shift, void* y, hipStream_t stream, int cus, Profiler* prof);

// LDS-patch 3x3 kernel (bf16, stride 1)
bool plan_patch(const sgprs_conv_desc_t& d, int cus, int* variant, int* splits, double* cost_us);
void patch_force(int variant, int splits);
const char* patch_variant_name(int variant);
int launch_conv3x3_patch(const sgprs_conv_desc_t& d, int variant, int splits, const void* x, const void* w,
                         const float* scale, const float* shift, const void* residual, void* y, void* ws,
                         size_t ws_bytes, hipStream_t stream, int cus, Profiler* prof);
int launch_splitk_reduce(int dtype, const float* partial, int splits, size_t total, int cout, const float* scale,
                         const float* shift, const void* res, void* y, int relu, hipStream_t stream);
// LDS-patch 3x3 stride-2 kernel (bf16), alone or together with the block's 1x1 stride-2 shortcut
bool plan_s2patch(const sgprs_conv_desc_t& d, int cus, int* variant);
void s2patch_force(int v);
int s2patch_num_variants();
const char* s2patch_variant_name(int variant);
int launch_conv3x3s2_patch(const sgprs_conv_desc_t& d, int variant, const void* x, const void* w, const float* scale,
                           const float* shift, void* y, const sgprs_conv_desc_t* d2, const void* w2, const float* scale2,
                           const float* shift2, void* y2, hipStream_t stream, int cus, Profiler* prof);
// row-streaming 3x3 kernel (bf16, 64 -> 64 channels, 56-pixel rows)
bool plan_rows(const sgprs_conv_desc_t& d, int cus, int* rows_per_stream);
void rows_force_off(bool off);
int launch_conv3x3_rows(const sgprs_conv_desc_t& d, int rows_per_stream, const void* x, const void* w, const void* w_fragments, const float* scale,
                        const float* shift, const void* residual, void* y, hipStream_t stream, int cus, Profiler* prof);
// implicit GEMM with the K range split over the wavefronts of a workgroup (few output tiles)
bool plan_ksplit(const sgprs_conv_desc_t& d, int cus, int* variant, double* cost_us);
int ksplit_num_variants();
double ksplit_cost(const sgprs_conv_desc_t& d, int variant, int cus, const sgprs_conv_desc_t* d1);
const char* ksplit_variant_name(int v);
constexpr int kKsplitNames = 32;  // launches of this kernel are recorded as implicit GEMM (or pair), variant 32 + 16 * dtype + tile (+ 32: four accumulator sets)
bool ksplit_fits(const sgprs_conv_desc_t& d, int variant);
int launch_conv_ksplit(const sgprs_conv_desc_t& d, int variant, const void* x, const void* w, const float* scale, const float* shift,
                       const void* res, void* y, const sgprs_conv_desc_t* d1, const void* w1, const float* scale1,
                       const float* shift1, void* y1, hipStream_t stream, Profiler* prof);
// 3x3 stride-1 kernel with private patches and weights from the L2 to registers (bf16); its weights come in fragment order
bool fragment_order(const sgprs_conv_desc_t& d);
int repack_fragments(const sgprs_conv_desc_t& d, const void* src, void* dst, hipStream_t stream);
bool wtile_applicable(const sgprs_conv_desc_t& d);
bool plan_wtile(const sgprs_conv_desc_t& d, int cus, int* ks, double* cost_us);
int launch_conv3x3_wtile(const sgprs_conv_desc_t& d, int ks, const void* x, const void* w_fragments, const float* scale, const float* shift,
                         const void* res, void* y, hipStream_t stream, int cus, Profiler* prof);
// 3x3 stride-1 kernel with K split over a workgroup's wavefronts and the tile's input pixels in LDS once (bf16, at most one tile per CU)
bool kpatch_fits(const sgprs_conv_desc_t& d, int variant);
bool plan_kpatch(const sgprs_conv_desc_t& d, int cus, int* variant, double* cost_us);
constexpr int kKpatchNames = 96;  // recorded as implicit GEMM, variant 96 + tile
const char* kpatch_variant_name(int variant);
int launch_conv3x3_kpatch(const sgprs_conv_desc_t& d, int variant, const void* x, const void* w, const float* scale, const float* shift,
                          const void* res, void* y, hipStream_t stream, int cus, Profiler* prof);
// a block's 3x3 stride-2 convolution with its shortcut, weights from the L2 to registers (bf16); its weights come in fragment order
bool plan_s2tile(const sgprs_conv_desc_t& d, const sgprs_conv_desc_t& d1, int cus, int* variant, double* cost_us);
bool s2tile_fits(const sgprs_conv_desc_t& d, const sgprs_conv_desc_t& d1, int variant);
constexpr int kS2tileNames = 24;  // recorded as implicit-GEMM pair, variant 24 + tile
const char* s2tile_variant_name(int variant);
int launch_conv_s2tile(const sgprs_conv_desc_t& d, int variant, const void* x, const void* fragments0, const float* scale0, const float* shift0, void* y0,
                       const sgprs_conv_desc_t& d1, const void* fragments1, const float* scale1, const float* shift1, void* y1, hipStream_t stream,
                       int cus, Profiler* prof);
// fp32 by three bf16 planes of every operand, K range split like conv_ksplit's
bool split_fits(const sgprs_conv_desc_t& d, int variant);
bool plan_split(const sgprs_conv_desc_t& d, int cus, int* variant, double* cost_us);
int split_num_variants();
double split_cost(const sgprs_conv_desc_t& d, int variant, int cus, const sgprs_conv_desc_t* d1);
constexpr int kSplitNames = 104;  // recorded as implicit GEMM (or pair), variant 104 + tile
const char* split_variant_name(int variant);
size_t split_weight_bytes(const sgprs_conv_desc_t& d);  // of the planes and what belongs to them; 0: none for this shape
// sets *unfit (device memory) where the planes do not hold the weights
int split_weights(const sgprs_conv_desc_t& d, const void* src, const float* scale, void* dst, int* unfit, hipStream_t stream);
int launch_conv_split(const sgprs_conv_desc_t& d, int variant, const void* x, const void* w, const void* planes, const float* scale, const float* shift,
                      const void* res, void* y, const sgprs_conv_desc_t* d1, const void* w1, const void* planes1, const float* scale1,
                      const float* shift1, void* y1, hipStream_t stream, Profiler* prof);
// tuning override: kind -1 automatic, 0 implicit GEMM only, 1 force patch (variant, splits)
extern std::atomic<int> g_conv_force_kind;
extern std::atomic<int> g_igemm_force_variant, g_igemm_force_splits;

const char* igemm_variant_name(int v);
const char* igemm_pair_variant_name(int v);
int launch_conv_pair(const sgprs_conv_desc_t& d0, const void* w0, const float* scale0, const float* shift0, void* y0,
                     const sgprs_conv_desc_t& d1, const void* w1, const float* scale1, const float* shift1, void* y1,
                     const void* x, hipStream_t stream, int cus, Profiler* prof, bool* done, const void* fragments0 = nullptr,
                     const void* fragments1 = nullptr);
int igemm_num_variants();

}  // namespace sgprs
