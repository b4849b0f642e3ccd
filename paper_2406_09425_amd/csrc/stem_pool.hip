// Stage 0 in one kernel, bf16 (fp32: stem_f32.hip): conv 7x7/2 (3 -> 64) + folded BN + ReLU + max-pool 3x3/2.
//
// The stem's 64 x 112 x 112 output is the largest tensor of the network; written out and read back by a
// separate pooling kernel it costs more HBM traffic than everything else in the stage.  Two kernels:
// stem_pool_packed_kernel, further down, is what tasks run; stem_pool_kernel takes images whose rows are not
// whole 16-byte pieces, and is what the other one is compared with (a task runs it under the tuning override only).
//
// stem_pool_kernel: a workgroup owns 7 x 8 pooled pixels.  It computes the 15 x 17 conv pixels they depend on
// (255 rows of a 256-row MFMA tile; the overlap between neighbouring tiles is recomputed), keeps them in
// LDS, pools there and writes only the pooled 16-byte vectors.
//
// As in the stand-alone stem kernel the input patch is staged in LDS with 4
// channel slots per pixel and zero fill outside the image, and the weights sit
// in LDS in the matching 7 x 32 tap-row layout.  The MFMA operands are swapped
// (weights as the row operand, pixels as the column operand) so that a lane's
// accumulator registers hold 4 consecutive channels of one pixel, which go to
// the LDS staging area as one 8-byte write.
// Positions outside the conv output hold 0 in the staging area (the post-ReLU
// values are pooled as unsigned bit patterns), so padding never wins the maximum.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "internal.h"

namespace sgprs {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned short u16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

struct StemPoolArgs {
    const unsigned char* x;
    const unsigned char* w;
    unsigned char* y;
    const float* scale;
    const float* shift;
    int N, H, W;      // input
    int P, Q;         // conv output
    int PP, PQ;       // pooled output
    int tiles_p, tiles_q, ntiles;
};

constexpr int kPoolTP = 7, kPoolTQ = 8;           // pooled pixels per tile
constexpr int kConvR = 2 * kPoolTP + 1;           // 15 conv rows
constexpr int kConvC = 2 * kPoolTQ + 1;           // 17 conv columns
constexpr int kInR = 2 * kConvR + 5;              // 35 input rows
constexpr int kInC = 2 * kConvC + 6;              // 40 input columns (one spare for the padded 8th tap)

template <int DT>
__global__ __launch_bounds__(256) void stem_pool_kernel(const StemPoolArgs a)
{
    static_assert(DT == SGPRS_BF16, "fp32 has stem_f32_kernel");
    constexpr int ES = 2;
    constexpr int PIX = 4 * ES;                      // staged input pixel: 4 channel slots
    constexpr int WROW = kStemK * ES + 16;           // padded weight row
    constexpr int W_BYTES = 64 * WROW;
    constexpr int SROWB = 64 * ES + 16;              // staged conv pixel: 64 channels + pad
    constexpr int PATCH_BYTES = kInR * kInC * PIX;
    constexpr int STG_BYTES = 256 * SROWB;
    constexpr int BUF_BYTES = PATCH_BYTES > STG_BYTES ? PATCH_BYTES : STG_BYTES;

    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* Ws = smem;
    unsigned char* Ps = smem + W_BYTES;              // patch, later the conv staging area

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int frow = lane & 31, fhalf = lane >> 5;

    for (int i = tid; i < 64 * (kStemK * ES / 16); i += 256) {
        const int row = i / (kStemK * ES / 16), ch = i - row * (kStemK * ES / 16);
        *(u32x4_t*)(Ws + row * WROW + ch * 16) = *(const u32x4_t*)(a.w + (size_t)row * kStemK * ES + ch * 16);
    }

    // The next tile's input patch is fetched into registers while the current
    // tile computes: PF_IT pixels per thread, 3 channels each.
    constexpr int PF_IT = (kInR * kInC + 255) / 256;
    unsigned pf_lo[PF_IT], pf_hi[PF_IT];
    auto fetch_patch = [&](int tile) {
        const int n = tile / (a.tiles_p * a.tiles_q), t2 = tile - n * (a.tiles_p * a.tiles_q);
        const int pp0 = (t2 / a.tiles_q) * kPoolTP, pq0 = (t2 % a.tiles_q) * kPoolTQ;
        const int h_base = 2 * (2 * pp0 - 1) - 3, w_base = 2 * (2 * pq0 - 1) - 3;
#pragma unroll
        for (int it = 0; it < PF_IT; ++it) {
            const int i = it * 256 + tid;
            const int pr = i / kInC, pc = i - pr * kInC;
            const int ih = h_base + pr, iw = w_base + pc;
            const bool ok = i < kInR * kInC && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
            const size_t g = ((size_t)(n * a.H + (ok ? ih : 0)) * a.W + (ok ? iw : 0)) * 3;
            const unsigned short* xp = (const unsigned short*)a.x + g;
            // unconditional loads from a clamped (always valid) pixel, zeroed afterwards:
            // nothing waits on a branch, all loads of the patch are in flight together
            const unsigned v0 = xp[0], v1 = xp[1], v2 = xp[2];
            pf_lo[it] = ok ? v0 | (v1 << 16) : 0u;
            pf_hi[it] = ok ? v2 : 0u;
        }
    };
    auto store_patch = [&]() {
#pragma unroll
        for (int it = 0; it < PF_IT; ++it) {
            const int i = it * 256 + tid;
            if (i >= kInR * kInC) continue;
            u32x2_t o = {pf_lo[it], pf_hi[it]};
            *(u32x2_t*)(Ps + i * PIX) = o;
        }
    };

    // this lane's BN scale / shift: accumulator register 4g+u of channel tile i is channel 32i + 8g + 4*fhalf + u
    f32x4_t sc[2][4], sh[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            sc[i][g] = *(const f32x4_t*)(a.scale + 32 * i + 8 * g + 4 * fhalf);
            sh[i][g] = *(const f32x4_t*)(a.shift + 32 * i + 8 * g + 4 * fhalf);
        }

    if ((int)blockIdx.x < a.ntiles) fetch_patch(blockIdx.x);
    for (int tile = blockIdx.x; tile < a.ntiles; tile += gridDim.x) {
        const int n = tile / (a.tiles_p * a.tiles_q), t2 = tile - n * (a.tiles_p * a.tiles_q);
        const int pp0 = (t2 / a.tiles_q) * kPoolTP, pq0 = (t2 % a.tiles_q) * kPoolTQ;
        const int cr0 = 2 * pp0 - 1, cc0 = 2 * pq0 - 1;   // first conv row / column of the tile

        __syncthreads();  // the previous tile's pooling reads are done
        store_patch();
        __syncthreads();
        if (tile + (int)gridDim.x < a.ntiles) fetch_patch(tile + gridDim.x);

        // accumulators: [channel tile i][pixel tile j]; this wavefront owns conv
        // pixels 64*wave .. 64*wave+63 of the tile (pixel t = row*17 + column)
        f32x16_t acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

        int poff[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            int t = wave * 64 + j * 32 + frow;
            if (t >= kConvR * kConvC) t = 0;  // the one padding row of the 256-row tile: computed, never used
            const int cr = t / kConvC, cc = t - cr * kConvC;
            poff[j] = ((2 * cr) * kInC + 2 * cc) * PIX;
        }
        const unsigned char* wbase = Ws + frow * WROW;

#pragma unroll
        for (int r = 0; r < 7; ++r) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int chunk = 2 * ks + fhalf;
                u32x4_t pf[2], wf[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) pf[j] = *(const u32x4_t*)(Ps + poff[j] + r * kInC * PIX + chunk * 16);
#pragma unroll
                for (int i = 0; i < 2; ++i) wf[i] = *(const u32x4_t*)(wbase + i * 32 * WROW + r * kStemTapRow * ES + chunk * 16);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, wf[i]),
                                                                          __builtin_bit_cast(bf16x8_t, pf[j]), acc[i][j], 0, 0, 0);
            }
        }

        __syncthreads();  // every wavefront is done with the patch: reuse it as the staging area

        // accumulator register e: column lane%32 = pixel, row 8*(e/4) + 4*(lane/32) + e%4 = channel
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int t = wave * 64 + j * 32 + frow;
            const int cr = t / kConvC, cc = t - cr * kConvC;
            const int crow = cr0 + cr, ccol = cc0 + cc;
            const bool ok = t < kConvR * kConvC && (unsigned)crow < (unsigned)a.P && (unsigned)ccol < (unsigned)a.Q;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int c = 32 * i + 8 * g + 4 * fhalf;
                    float v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = fmaxf(acc[i][j][4 * g + u] * sc[i][g][u] + sh[i][g][u], 0.f);
                    // After the ReLU every value is >= 0, so pooling can compare bf16 bit
                    // patterns as unsigned integers and positions outside the conv output
                    // hold 0: each pooling window has a real pixel, so 0 never wins wrongly.
                    // The sign bit is cleared so that a -0 cannot compare as large.
                    const f32x2_t p0 = {v[0], v[1]}, p1 = {v[2], v[3]};
                    const unsigned keep = ok ? 0x7fff7fffu : 0u;
                    u32x2_t o = {__builtin_bit_cast(unsigned, __builtin_convertvector(p0, bf16x2_t)) & keep,
                                 __builtin_bit_cast(unsigned, __builtin_convertvector(p1, bf16x2_t)) & keep};
                    *(u32x2_t*)(Ps + t * SROWB + c * 2) = o;
                }
        }
        __syncthreads();

        // pooling: one item = (pooled pixel, 16-byte channel group)
        constexpr int GROUPS = 64 * ES / 16;
        for (int it = tid; it < kPoolTP * kPoolTQ * GROUPS; it += 256) {
            const int grp = it % GROUPS, px = it / GROUPS;
            const int lp = px / kPoolTQ, lq = px - lp * kPoolTQ;
            const int gp = pp0 + lp, gq = pq0 + lq;
            if (gp >= a.PP || gq >= a.PQ) continue;
            const unsigned char* base = Ps + ((2 * lp) * kConvC + 2 * lq) * SROWB + grp * 16;
            u32x4_t m = *(const u32x4_t*)base;
#pragma unroll
            for (int rs = 1; rs < 9; ++rs) {
                const u32x4_t t = *(const u32x4_t*)(base + ((rs / 3) * kConvC + rs % 3) * SROWB);
                // whole-vector form: eight unsigned 16-bit maxima per tap
                m = __builtin_bit_cast(u32x4_t, __builtin_elementwise_max(__builtin_bit_cast(u16x8_t, m),
                                                                          __builtin_bit_cast(u16x8_t, t)));
            }
            *(u32x4_t*)(a.y + (((size_t)(n * a.PP + gp) * a.PQ + gq) * 64) * ES + grp * 16) = m;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// bf16 variant with packed input rows.
//
//  * The input keeps the image's own 3-channel packing: rows are copied global -> LDS by the load unit itself
//    (zero fill outside the image comes from the buffer bounds check).  A pixel's K-run for tap row r is the 24
//    consecutive bf16 that start one element before its first tap (elements 0, 22, 23 meet zero weights), so
//    K = 7 x 24 = 168 (+8 zero) = 176.
//  * A wavefront goes its own way, one per SIMD: a strip of `rows` pooled rows x up to 30 pooled columns.  It computes the
//    strip's conv rows one by one, even and odd columns as two MFMA tiles of 32 pixels, so that lane l has the conv
//    columns 2q and 2q + 1 of pooled column q = q0 - 1 + l and gets 2q - 1 from the lane before: the maximum over
//    the window never leaves the registers.  No patch staging, no pooling reads, no barriers; one conv row per strip and
//    one column in 29 are computed twice.
//  * The maximum is taken of the sums; scale, shift and ReLU follow it, a quarter of the work (they are monotone: the weights of
//    channels with a negative scale are negated, which is exact, and rounding keeps the order).
//  * The weights of both tiles (176 registers) and the input fragments (44) are accumulation registers, read from LDS right into
//    them; sums, maxima, scale and shift are the other 256.  Two thirds of a K-run's groups are the same for an
//    odd column and the even one before it: 15 reads per conv row, not 22 (8-aligned reads give 73 bytes a cycle and CU, and with
//    scale and shift read from there as well they were the bound).
//  * A SIMD starts an MFMA every 32 cycles and up to six other instructions of the same wavefront are free behind it (measured;
//    eight: 43 cycles).  A conv row has 44 MFMAs and about 220 others, laid behind them five at a time.
//  * Groups of four input rows are loaded one or two row pairs ahead, as their latency asks for, not as soon as there is room: a wavefront
//    that requests more than the memory takes waits at the request (all 27 loads of a strip first: 5 us instead of 2 before the
//    first MFMA at batch 64).
// Bound: the MFMAs (22 GFLOP with padding and what is computed twice at batch 64) at the clock they leave: 2816 cycles of MFMAs in
// 3660 per row pair, at 1.7 GHz.  Measured (us per launch inside the network, this kernel / the one of 8x7 patches with two
// workgroups per CU before it): batch 64 23.2 / 37.0, batch 128 41.0 / 67.6, 13 images on 96 CUs 11.8 / 19.6, 16 images 9.8 / 14.2,
// one image 5.9 / 6.0, on 64 CUs 6.2 / 6.0, on 32 CUs 6.3 / 7.8.  (The first pass of a new task, one image, weights and code cold: 6.8 / 7.0,
// on 32 CUs 7.2 / 8.7.)
// The elements of a run beside its taps (0 / 22 / 23, of even columns the three before and none behind) are real neighbouring inputs
// multiplied by zero weights: the result equals the plain definition for finite inputs.  A pixel that is NaN or infinite also makes the sums of
// these columns NaN: odd ones whose window begins right of it (its channel 2) or ends left of it (channels 0 and 1), even ones whose window
// begins right of it.  (An infinite one in a window's last row, too, meets the zero weights of the last K group: at the right end of odd columns'
// windows, at the left end of even ones'.)  NaN sums count as 0 (the ReLU's result) in the maximum over a window, the others as they are.
constexpr int kStripCols = 30, kStripRows = 7;       // pooled columns and rows of a strip, at most
constexpr int kRowPitch = 24 * kStripCols + 48;      // bytes of an input row in LDS: 48 pieces of 16
constexpr int kGroupBytes = 4 * kRowPitch;           // rows are loaded by fours: three instructions
constexpr int kStripLds = (kStripRows + 2) * kGroupBytes;
constexpr int kAhead = 5;                            // groups of rows loaded before the first is used
constexpr int kFragments = 44;                       // [odd, even][K-step 0 .. 10][channel tile], 1024 bytes each; then scale and shift
constexpr int kFragmentLds = 48 * 1024;              // (what the wavefronts load of them, twelve instructions each)
constexpr int kOutPitch = 144;                       // a pixel of a finished row, where the fragments were
static_assert(kFragments * 512 + 256 == kStemRowsElems, "");
static_assert(4 * 32 * kOutPitch <= kFragmentLds, "");
constexpr int kPackedLds = kFragmentLds + 4 * kStripLds + 64;  // (the idle lanes of the last row read a little past it)

typedef unsigned int u32x4a8_t __attribute__((ext_vector_type(4), aligned(8)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

struct StemRowsArgs {
    const unsigned char* x;
    const unsigned char* w;
    unsigned char* y;
    int H, W, P, PP, PQ;              // input, rows of the conv output, pooled output
    int rows, cols;                   // of a strip
    int ahead;                        // groups of rows loaded ahead: kAhead, or fewer where a strip has no more
    int strips_q, strips, per_die;    // strips of a pooled row, all, of a die (each walks a contiguous eighth: workgroup b runs on die b % 8)
    unsigned q_mul, p_mul;
    int q_sh, p_sh, strips_p;
};

template <int N> __device__ __forceinline__ void stem_wait_vmcnt()
{
    static_assert(N <= 63, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// Maxima that leave NaN out, as the ReLU does that comes after them: a NaN sum counts as 0, the others of its window as they are.  (As assembly: the
// builtin would first quieten each operand that no instruction known to it has written, one more instruction apiece; in pairs, or with the
// neighbour's value as an operand, because the compiler keeps what reads a result of assembly an instruction away from it.)
__device__ __forceinline__ float max_of(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// b = max(a, b, v), a = max(a, v)
__device__ __forceinline__ void max_both(float& a, float& b, float v)
{
    asm("v_max_f32 %0, %0, %2\n\tv_max_f32 %1, %1, %0" : "+&v"(a), "+v"(b) : "v"(v));
}
// With the lane before: its value (0 for lane 0) and this one's.
__device__ __forceinline__ float max_neighbours(float v)
{
    float r;
    asm("v_max_f32_dpp %0, %1, %1 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1" : "=v"(r) : "v"(v));
    return r;
}
__device__ __forceinline__ float max_neighbours(float v, float a)
{
    float r;
    asm("v_max_f32_dpp %0, %1, %1 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\tv_max_f32 %0, %0, %2" : "=&v"(r) : "v"(v), "v"(a));
    return r;
}

__global__ __launch_bounds__(256, 1) void stem_pool_packed_kernel(const StemRowsArgs a)
{
#if __HIP_DEVICE_COMPILE__
    // LDS by address (0: the start of the workgroup's): what reads it is not held up for the rows still on their way.
    typedef const __attribute__((address_space(3))) u32x4a8_t* lds_a8_t;
    typedef const __attribute__((address_space(3))) u32x4_t* lds_a16_t;
    typedef __attribute__((address_space(3))) u32x4_t* lds_w16_t;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int frow = lane & 31, fhalf = lane >> 5;
    constexpr unsigned kOutside = 0x80000000u;
    const __amdgpu_buffer_rsrc_t w_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, kStemRowsElems * 2, 0x00020000);
    const unsigned staged = wave * 32 * kOutPitch, mine = kFragmentLds + wave * kStripLds;
    const int row_bytes = a.W * 6;

    struct Strip { int n, p0, q0; bool valid; };
    const int die = (int)blockIdx.x & 7, block = (int)blockIdx.x >> 3, step = (int)gridDim.x >> 3;
    const int end = min(a.strips, (die + 1) * a.per_die);
    auto div = [](int m, unsigned mul, int sh) { return (int)(__umulhi(2u * (unsigned)m, mul) >> sh); };
    auto decode = [&](int t) {
        Strip s;
        s.valid = t < end;
        const int u = min(t, a.strips - 1), rest = div(u, a.q_mul, a.q_sh);
        s.n = div(rest, a.p_mul, a.p_sh);
        s.p0 = (rest - s.n * a.strips_p) * a.rows;
        s.q0 = (u - rest * a.strips_q) * a.cols;
        return s;
    };
    // Row k of a strip is input row 4 p0 - 5 + k, from byte 24 q0 - 32 on, 48 pieces of 16 bytes.  Instruction i of a group of four
    // rows has pieces 64 i .. 64 i + 63.  The descriptor is the image's: rows above and below it are beyond the size (as are all
    // where there is no strip: the waits count every instruction), pieces beside it are given such an offset.
    struct Pieces { unsigned at[3]; };
    auto pieces = [&](const Strip& s) {
        Pieces p;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int u = lane + i * 64, row = (int)(__umul24((unsigned)u, 1366u) >> 16), b = 24 * s.q0 + (u - row * 48) * 16 - 32;
            p.at[i] = (unsigned)b < (unsigned)row_bytes ? (unsigned)((4 * s.p0 - 5 + row) * row_bytes + b) : kOutside;
        }
        return p;
    };
    auto load_group = [&](const Strip& s, const Pieces& p, int group) {
        const __amdgpu_buffer_rsrc_t x_rs = __builtin_amdgcn_make_buffer_rsrc((void*)(a.x + (long long)s.n * a.H * row_bytes), 0,
                                                                              s.valid ? a.H * row_bytes : 0, 0x00020000);
#pragma unroll
        for (int i = 0; i < 3; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rs, (lds_ptr_t)(unsigned long)(mine + group * kGroupBytes + i * 1024), 16,
                                                     p.at[i] + (unsigned)(4 * group * row_bytes), 0, 0, 0);
    };
#pragma unroll
    for (int k = 0; k < kFragmentLds / 4096; ++k) {
        int f = k * 4 + wave + block % 16 * 3;  // (not all in the same order: a die's CUs would meet at one channel of its L2)
        f -= f >= 48 ? 48 : 0;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rs, (lds_ptr_t)(unsigned long)(f * 1024), 16, f * 1024 + lane * 16, 0, 0, 0);
    }
    int t = die * a.per_die + block + wave * step;  // (few strips: one or two on a CU, whose loads are what they wait for)
    Strip cur = decode(t);
    Pieces cur_at = pieces(cur);
#pragma unroll
    for (int k = 0; k < 3; ++k) load_group(cur, cur_at, k);
    __builtin_amdgcn_sched_barrier(0);
    stem_wait_vmcnt<9>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    u32x4_t w[2][11][2];              // of the odd and of the even columns
    f32x4_t sc[8], sh[8];             // of channels 8 q + 4 fhalf + 0 .. 3
#pragma unroll
    for (int f = 0; f < kFragments; ++f) w[f / 22][f % 22 / 2][f % 2] = *(lds_a16_t)(unsigned long)(f * 1024 + lane * 16);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        sc[q] = __builtin_bit_cast(f32x4_t, *(lds_a16_t)(unsigned long)(kFragments * 1024 + q * 32 + fhalf * 16));
        sh[q] = __builtin_bit_cast(f32x4_t, *(lds_a16_t)(unsigned long)(kFragments * 1024 + 256 + q * 32 + fhalf * 16));
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int k = 3; k < a.ahead; ++k) load_group(cur, cur_at, k);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < kFragments; ++f) asm volatile("" : "+a"(w[f / 22][f % 22 / 2][f % 2]));
#pragma unroll
    for (int q = 0; q < 8; ++q) asm volatile("" : "+v"(sc[q]), "+v"(sh[q]));
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();     // finished rows go where the fragments were
    asm volatile("" ::: "memory");

    // Groups are loaded `ahead` of the first one of a conv row, one every two rows (more at once only wait in the wavefront's way):
    // the three that a strip's first row reads have landed when all but the last ahead - 3 have.  From the second row pair on the
    // stores of a finished row lie between the loads and count as well: what is left in flight is one group and three stores, so
    // that a group has one row pair to land, 2.2 us.
    auto wait_for_rows = [&] {
        __builtin_amdgcn_sched_barrier(0);
        if (a.ahead >= kAhead) stem_wait_vmcnt<3 * (kAhead - 3)>();
        else stem_wait_vmcnt<0>();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // A conv row is two multiplications of 22 MFMAs; behind each, up to six other instructions are free.  What is done with the sums of
    // the multiplication before is cut into N steps and spread over them.
    f32x16_t acc[2][2];               // of the odd and of the even columns
    float odd[2][16], m[2][16];       // maxima: over the odd columns of a window, over the rows of a window so far
    u32x4_t both[7], own[4];          // the row's K groups that odd and even columns share, those that they do not
    auto read = [&](unsigned base, int off) { return (u32x4_t) * ((lds_a8_t)(unsigned long)base + off / 16); };
    struct Bases { unsigned s0, s3, s6, h0, h4, l6; };  // of tap rows: 0, 3, 6 of the shared groups; 0, 4 (upper half-wave: the next one) and 6 of the others
    auto multiply = [&](auto even, const Bases& row, unsigned next, auto steps, auto work) {
        constexpr int E = decltype(even)::value, N = decltype(steps)::value, OWN = E ? 0 : 48;
#pragma unroll
        for (int ks = 0; ks < 11; ++ks) {
            if (!E && ks < 3) both[ks + 3] = read(row.s3, ks * kRowPitch);
            if (!E && ks == 3) both[6] = read(row.s6, 0);
            // the last step's upper group has zero weights: it re-reads the lower one
            if (ks >= 4 && ks < 8) own[ks - 4] = read(ks == 7 ? row.l6 : ks == 6 ? row.h4 : row.h0, OWN + (ks == 5 ? 2 * kRowPitch : 0));
            if (E && ks >= 8) both[ks - 8] = read(next, (ks - 8) * kRowPitch);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const u32x4_t b = ks < 7 ? both[ks] : own[ks - 7];
                // (as assembly: the builtin would put the sums where vector instructions cannot read them)
                if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc[E][i]) : "a"(w[E][ks][i]), "a"(b));
                else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc[E][i]) : "a"(w[E][ks][i]), "a"(b));
                const int s = 2 * ks + i - 1;    // sums are read from the second MFMA on
                __builtin_amdgcn_sched_barrier(0);
                if (s >= 0) {
#pragma unroll
                    for (int k = s * N / 21; k < (s + 1) * N / 21; ++k) work(k);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    for (; cur.valid; t += 4 * step) {
        const Strip nxt = decode(t + 4 * step);
        const Pieces nxt_at = pieces(nxt);
        // Of the first strip of a row, lane 0 has the column left of the image: it takes the first one instead, which changes no maximum.
        const unsigned run = mine + 24 * (cur.q0 == 0 && frow == 0 ? 1 : frow);
        unsigned shared = run + fhalf * 16, upper = run - 16 + fhalf * kRowPitch, lower = run - 16;
        asm volatile("" : "+v"(shared), "+v"(upper), "+v"(lower));
        // Likewise the conv rows above and below the image: the first and the last one.
        auto conv_row = [&](int r) { return (unsigned)(max(min(r, a.P - 2 * cur.p0), cur.p0 == 0 ? 1 : 0) * (2 * kRowPitch)); };
        auto bases = [&](unsigned r) {
            return Bases{shared + r, shared + (r + 3 * kRowPitch), shared + (r + 6 * kRowPitch), upper + r, upper + (r + 4 * kRowPitch), lower + (r + 6 * kRowPitch)};
        };
        // Accumulator register e: column lane%32 = pixel, row 8*(e/4) + 4*(lane/32) + e%4 = channel.  Registers of both channel tiles
        // one after the other: x = 16 i + e.
        // Odd rows of the conv output are the last of a pooled row and the first of the next one.
        auto last_odd = [&](int x) { odd[x >> 4][x & 15] = max_neighbours(acc[0][x >> 4][x & 15]); };  // 32
        auto last_even = [&](int k) {     // 66: m becomes the result, an element behind its maxima
            const int x = k / 2, y = x - 1;
            if (k % 2 == 0 && x < 32) max_both(odd[x >> 4][x & 15], m[x >> 4][x & 15], acc[1][x >> 4][x & 15]);
            if (k % 2 == 1 && y >= 0) m[y >> 4][y & 15] = m[y >> 4][y & 15] * sc[y >> 2][y & 3] + sh[y >> 2][y & 3];
        };
        // A finished row goes to LDS, pixel by pixel, and from there eight pixels a store (straight from the lanes that have them, 16 bytes of a
        // pixel each, a store took four times as long).
        unsigned o[4];
        auto pack = [&](int x) {
            o[(x >> 1) & 3] = pack_bf16x2_relu(m[x >> 4][x & 15], m[x >> 4][(x & 15) + 1], kReluFloor);
        };
        auto stage = [&](int x) {         // lanes 0 .. 31 take all eight channels of the first group of four registers, lanes 32 .. 63 those of the second
            const auto s0 = __builtin_amdgcn_permlane32_swap(o[0], o[2], false, false);
            const auto s1 = __builtin_amdgcn_permlane32_swap(o[1], o[3], false, false);
            *(lds_w16_t)(unsigned long)(staged + frow * kOutPitch + fhalf * 16 + x * 4) = u32x4_t{s0[0], s1[0], s0[1], s1[1]};
        };
        auto middle_odd = [&](int k) {    // 64: packs the result, then m is the maximum of the next pooled row
            const int x = k / 4 * 2, i = x >> 4, e = (x & 15) + (k & 1);
            if (k % 4 == 0) pack(x);
            if (k % 4 == 1 && x % 8 == 6) stage(x - 6);
            if (k % 4 >= 2) m[i][e] = max_neighbours(acc[0][i][e], odd[i][e]);
        };
        u32x4_t line[4];
        auto fetch = [&](int s) {         // lane l has 16 bytes of the pixels 8 s + l / 8; the first one of the strip is pixel 1
            line[s] = *(lds_a16_t)(unsigned long)(staged + ((lane >> 3) + 8 * s) * kOutPitch + (lane & 7) * 16);
        };
        const int row_out = a.PQ * 128, records = min(a.cols, a.PQ - cur.q0) * 128, live_rows = min(a.rows, a.PP - cur.p0);
        const unsigned char* out = a.y + (((long long)cur.n * a.PP + cur.p0) * a.PQ + cur.q0) * 128;
        auto store = [&](int s, const unsigned char* out, bool live) {
            const __amdgpu_buffer_rsrc_t y_rs = __builtin_amdgcn_make_buffer_rsrc((void*)out, 0, live ? records : 0, 0x00020000);
            __builtin_amdgcn_raw_buffer_store_b128(line[s], y_rs, s ? lane * 16 + 896 + (s - 1) * 1024 : lane * 16 - 128, 0, 0);
        };
        const auto nothing = [](int) {};
        constexpr std::integral_constant<int, 0> odds, n0;
        constexpr std::integral_constant<int, 1> evens;
        constexpr std::integral_constant<int, 32> n32;
        constexpr std::integral_constant<int, 40> n40;
        constexpr std::integral_constant<int, 64> n64;
        constexpr std::integral_constant<int, 66> n66;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) m[i][e] = 0.f;  // (of a row that is not there)
        // Conv row r reads input rows 2r .. 2r + 6: new groups of four are needed by rows 0 (three, where row 1 stands in for it), 3, 5, ...
        // (not by what is read ahead for them); those that rows 0 .. 2j + 2 have read make room for the next strip's.
        auto load_next = [&](int k) {     // the strip's groups and then the next one's
            const int g = k - (a.rows + 2);
            Strip s = cur;
            Pieces p = cur_at;
            if (g >= 0) { s = nxt; p = nxt_at; }
            load_group(s, p, g >= 0 ? g : k);
        };
        wait_for_rows();
        unsigned r1 = conv_row(1);
        const Bases b0 = bases(conv_row(0));
#pragma unroll
        for (int k = 0; k < 3; ++k) both[k] = read(b0.s0, k * kRowPitch);
        multiply(odds, b0, 0, n0, nothing);
        multiply(evens, b0, shared + r1, n32, last_odd);
        for (int j = 0; j < a.rows; ++j) {
            wait_for_rows();
            const Bases b1 = bases(r1), b2 = bases(conv_row(2 * j + 2));
            r1 = conv_row(2 * j + 3);
            multiply(odds, b1, 0, n66, last_even);
            multiply(evens, b1, b2.s0, n64, middle_odd);
            multiply(odds, b2, 0, n40, [&](int k) {
                if (k < 32) m[k >> 4][k & 15] = max_of(m[k >> 4][k & 15], acc[1][k >> 4][k & 15]);
                if (k % 8 == 1 && k < 32) fetch(k / 8);
                if (k >= 32 && k % 2) store((k - 32) / 2, out - row_out, j > 0 && j <= live_rows);
            });
            multiply(evens, b2, shared + r1, n32, last_odd);
            load_next(j + a.ahead);
            out += row_out;
        }
        load_next(a.rows + a.ahead);
        load_next(a.rows + 1 + a.ahead);
        // The hazard recogniser does not see into the assembly: what reads the last sums keeps its distance (elsewhere MFMAs lie between).
        asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc[1][0]), "+v"(acc[1][1]));
#pragma unroll
        for (int k = 0; k < 66; ++k) last_even(k);
#pragma unroll
        for (int x = 0; x < 32; x += 2) {
            pack(x);
            if (x % 8 == 6) stage(x - 6);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) fetch(s);
#pragma unroll
        for (int s = 0; s < 4; ++s) store(s, out - row_out, live_rows == a.rows);
        cur = nxt;
        cur_at = nxt_at;
    }
    __builtin_amdgcn_s_waitcnt(0);
#endif
}

bool stem_pool_applicable(int dtype, int n, int h, int w, int cus)
{
    const int P = out_dim(h, 7, 2, 3), Q = out_dim(w, 7, 2, 3);
    const int PP = (P - 1) / 2 + 1, PQ = (Q - 1) / 2 + 1;
    const long long tiles = (long long)n * ((PP + kPoolTP - 1) / kPoolTP) * ((PQ + kPoolTQ - 1) / kPoolTQ);
    // smaller launches keep the finer-grained two-kernel path; in bf16 the fused kernel wins down
    // to one image (5.9 us, the stem alone 8.5); the line for fp32 is where its times cross
    // (us, two kernels and the gap between them against one, 256 CUs: 3 images 20 / 21, 5 images 24 / 21,
    // 9 images 38 / 34), expressed in the 7x8 tiles counted here, not the 4x8 ones of its own kernel; and where
    // its own tiles all run at once (the whole fp32 network, one image on 256 CUs: 115.5 us with two kernels, 112.8 fused)
    return dtype == SGPRS_BF16 ? tiles >= 32 : (tiles >= cus || stem_f32_one_round(n, h, w, cus)) && stem_f32_applicable(n, h, w);
}

std::atomic<int> g_stem_pool_force{-1};
void stem_pool_force(int v) { g_stem_pool_force = v; }

void pack_stem_rows(const float* oihw, const float* scale, const float* shift, uint16_t* out)
{
    // Fragment [odd, even][K-step][channel tile] of 64 lanes x 8 elements: lane l has channel 32 tile + l % 32 of K group l / 32.
    // K groups (tap row, part of 8 elements): steps 0 .. 6 are parts 0 and 1 of tap row `step`; steps 7 .. 10 tap rows 2 (step - 7) and the
    // next one, part 2 for odd columns and part -1 for even ones.  Element e of an odd column's run is tap (e - 1) / 3, channel (e - 1) % 3;
    // the run of the even column before it starts 6 elements earlier.
    std::fill(out, out + kStemRowsElems, (uint16_t)0);
    for (int f = 0; f < kFragments; ++f)
        for (int l = 0; l < 64; ++l) {
            const int even = f / 22, ks = f % 22 / 2, k = 32 * (f % 2) + l % 32, half = l / 32;
            const int r = ks < 7 ? ks : 2 * (ks - 7) + half, part = ks < 7 ? half : even ? -1 : 2;
            if (r >= 7) continue;
            for (int v = 0; v < 8; ++v) {
                const int e = part * 8 + v + (even ? 6 : 0) - 1;
                if (e < 0 || e >= 21) continue;
                const uint16_t bits = f32_to_bf16_bits(oihw[((k * 3 + e % 3) * 7 + r) * 7 + e / 3]);
                out[(f * 64 + l) * 8 + v] = bits ^ (std::signbit(scale[k]) ? 0x8000 : 0);
            }
        }
    for (int k = 0; k < 64; ++k) {
        const float table[2] = {std::fabs(scale[k]), shift[k]};
        memcpy(out + kFragments * 512 + 2 * k, table, 4);
        memcpy(out + kFragments * 512 + 128 + 2 * k, table + 1, 4);
    }
}

int launch_stem_pool(int dtype, int n, int h, int w, const void* x, const void* wts, const void* wts_rows,
                     const float* scale, const float* shift, void* y, hipStream_t stream, int cus, Profiler* prof)
{
    StemPoolArgs a;
    a.x = (const unsigned char*)x; a.w = (const unsigned char*)wts; a.y = (unsigned char*)y;
    a.scale = scale; a.shift = shift;
    a.N = n; a.H = h; a.W = w;
    a.P = out_dim(h, 7, 2, 3); a.Q = out_dim(w, 7, 2, 3);
    a.PP = (a.P - 1) / 2 + 1; a.PQ = (a.Q - 1) / 2 + 1;
    a.tiles_p = (a.PP + kPoolTP - 1) / kPoolTP; a.tiles_q = (a.PQ + kPoolTQ - 1) / kPoolTQ;
    const long long nt = (long long)n * a.tiles_p * a.tiles_q;
    if (nt >= (1ll << 31)) return fail(SGPRS_ERR_UNSUPPORTED, "too many stem tiles");
    a.ntiles = (int)nt;
    const int es = (int)dtype_size(dtype);
    const double flops = 2.0 * n * a.P * a.Q * 64.0 * 147.0;
    const double bytes = ((double)n * h * w * 3 + 64.0 * 147 + (double)n * a.PP * a.PQ * 64) * es;
    int rc;
    static std::atomic<bool> raised[2] = {{false}, {false}};
    const long long x_bytes = (long long)n * h * w * 6;
    const bool packed = dtype == SGPRS_BF16 && wts_rows && w % 8 == 0 && ((uintptr_t)x & 15) == 0 && x_bytes < (1ll << 31) &&
                        g_stem_pool_force.load() != 1;
    if (prof && prof->on && (rc = prof->begin(stream, kKindStemPool, packed ? 2 : dtype, flops, bytes))) return rc;
    if (packed) {
        StemRowsArgs r;
        memset(&r, 0, sizeof(r));
        r.x = a.x; r.w = (const unsigned char*)wts_rows; r.y = a.y;
        r.H = h; r.W = w; r.P = a.P; r.PP = a.PP; r.PQ = a.PQ;
        r.strips_q = (a.PQ + kStripCols - 1) / kStripCols;
        r.cols = ((a.PQ + r.strips_q - 1) / r.strips_q + 1) & ~1;  // even: a strip's rows begin on 16 bytes
        // The fewest conv rows one after the other (a strip computes 2 * rows + 1 and costs about one more); of equal ones the lower strips.
        double best = 1e30;
        for (int rows = 1; rows <= kStripRows; ++rows) {
            const long long strips = (long long)n * r.strips_q * ((a.PP + rows - 1) / rows), rounds = (strips + 4ll * cus - 1) / (4ll * cus);
            const double cost = (double)rounds * (2 * rows + 2);
            if (cost < best) { best = cost; r.rows = rows; }
        }
        r.ahead = std::min(kAhead, r.rows + 2);
        r.strips_p = (a.PP + r.rows - 1) / r.rows;
        const long long strips = (long long)n * r.strips_p * r.strips_q;
        if (strips >= 1ll << 30) return fail(SGPRS_ERR_UNSUPPORTED, "too many stem strips");
        r.strips = (int)strips;
        r.per_die = (r.strips + 7) / 8;
        div_constants(r.strips_q, &r.q_mul, &r.q_sh);
        div_constants(r.strips_p, &r.p_mul, &r.p_sh);
        if (!raised[1]) {
            SGPRS_HIP(hipFuncSetAttribute((const void*)stem_pool_packed_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kPackedLds));
            raised[1] = true;
        }
        const int grid = 8 * std::max(1, std::min(cus / 8, r.per_die));  // a partition's CUs are a multiple of eight
        SGPRS_LAUNCH(stem_pool_packed_kernel, dim3(grid), dim3(256), kPackedLds, stream, r);
    } else if (dtype == SGPRS_BF16) {
        constexpr int patch = kInR * kInC * 4 * 2, stg = 256 * (64 * 2 + 16);
        constexpr int lds = 64 * (kStemK * 2 + 16) + (patch > stg ? patch : stg), occ = lds <= 80 * 1024 ? 2 : 1;
        const int grid = (int)std::min<long long>(nt, (long long)cus * occ);
        if (!raised[0]) {
            SGPRS_HIP(hipFuncSetAttribute((const void*)stem_pool_kernel<SGPRS_BF16>,
                                          hipFuncAttributeMaxDynamicSharedMemorySize, lds));
            raised[0] = true;
        }
        SGPRS_LAUNCH(stem_pool_kernel<SGPRS_BF16>, dim3(grid), dim3(256), lds, stream, a);
    } else if ((rc = launch_stem_f32(n, h, w, x, wts, scale, shift, y, 1, true, stream, cus))) {
        return rc;
    }
    SGPRS_HIP(hipGetLastError());
    if (prof && prof->on && (rc = prof->end(stream))) return rc;
    return SGPRS_OK;
}

}  // namespace sgprs
