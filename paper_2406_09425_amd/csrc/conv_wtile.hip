// 3x3 stride-1 pad-1 convolution, bf16: a wavefront's own tile, weights straight from the L2 to registers.
//
// What bounds the LDS-patch kernel on the deep layers is the LDS: weights and pixels pass through it (three
// 1 KiB fragment reads for two 32x32x16 MFMAs, 192 bytes a clock and CU beside what the loads write), and
// eight wavefronts meet at a barrier every 18 k-steps.  Here a wavefront owns 112 pixels x 64 channels (7 x 4
// MFMA tiles, 112 accumulator registers; one wavefront a SIMD) and meets nobody:
//   * its weights never see the LDS.  A task keeps them a second time in fragment order, so that a fragment is
//     one coalesced 1 KiB load to registers, requested six steps ahead;
//   * its input patch (64 channels at a time, two buffers) is its own, filled by loads that write LDS directly
//     and awaited by its own vmcnt: 7 fragment reads for 28 MFMAs, 64 bytes a clock and CU;
//   * tiles of 7 x 14 pixels (14 x 7 where two 7-pixel-high images share one) cut 56, 28, 14 and 7 pixel maps
//     without remainder, at the price of one MFMA in eight (98 of 112 rows are written): 64 images are one tile for every SIMD of 256 CUs on all three deep layers, KS = 1, 2
//     and 4 wavefronts of a workgroup sharing one by input channels (their sums meet in LDS, in a fixed order).
// A step (one tap, 32 channels) is 28 MFMAs of 16 cycles with 45 to 55 other instructions between them, at
// most two behind each where that was possible: 580 to 610 cycles instead of 448.  With every SIMD of the
// chip in it the clock drops to 1.6-1.7 GHz (2.4 with few), so a step takes 0.25 us on few CUs and 0.36 on all;
// leaving out instructions or loads there shortens the step in cycles and less in time.  Around the steps a
// launch spends 2.3 us until its first MFMA (74 KiB of patch and 64-96 KiB of weights a CU at 64 bytes a clock)
// and 1.9 us behind the last one.  64 images on 256 CUs, us per launch in a loop, LDS-patch kernel / this one:
// 7x7x512 23.8 / 16.8, 14x14x256 19.4 / 18.5, 28x28x128 20.3 / 21.1, 56x56x64 (row streaming) 24.1 / 24.1; 128
// images 35.1 / 28.6, 33.3 / 32.4, 40.4 / 36.0, 40.1 / 41.3.  Whole inferences with inputs that change: 64 images
// 399.7 -> 368.9, 128 images 622.6 -> 589.1, 48 images on 192 CUs 378.7 -> 345.4.
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace sgprs {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr int kWtTM = 7, kWtTN = 4;            // 16x16 MFMA tiles of a wavefront: 112 pixels x 64 channels
constexpr int kWtCap = 152;                    // patch pixels: instructions of eight
constexpr int kWtBuf = kWtCap * 128;           // bytes
constexpr int kWtTables = 8 * kWtBuf;          // LDS offset of the tables
constexpr int kWtLds = kWtTables + (kWtCap + 128) * 8;

// A tile is TH rows (of one image, or TH / H whole images) x TW columns of output pixels; its patch has a
// row above and below each image's rows and a column on either side.
struct WtileArgs {
    const unsigned char* x;
    const unsigned char* w;      // fragments, see repack_fragments_kernel
    unsigned char* y;
    const float* scale;
    const float* shift;
    const unsigned char* res;
    unsigned x_bytes, w_bytes, y_bytes;
    int H, W;
    int x_pitch, y_pitch;        // bytes of a pixel
    int chunks, chunks_per_wave; // of 64 input channels
    int TH, TW, PW, patch, images, image_rows;  // patch pixels; images of a tile; patch rows of one of them
    int tiles_image, cb;         // tiles of an image (or of a group of images), of a row of it
    unsigned pw_mul, tw_mul, rows_mul, h_mul;
    unsigned image_mul, cb_mul, nb_mul;
    int image_sh, cb_sh, nb_sh;
    int gm;                      // pixel tiles
    int die_cols, die_rows, die_col_sh;  // channel and pixel tiles of a die, dies side by side (log2)
    int relu;
};

__device__ __forceinline__ int wt_div(int m, unsigned mul, int sh) { return (int)(__umulhi(2u * (unsigned)m, mul) >> sh); }
__device__ __forceinline__ int wt_small_div(int m, unsigned mul) { return (int)((unsigned)__umul24((unsigned)m, mul) >> 22); }
template <int N> __device__ __forceinline__ void wt_wait_vmcnt()
{
    static_assert(N <= 63, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}
// Sum and minimum of 16-bit halves: row << 16 | column lies inside the image when its minimum with the
// last row and column is itself (one before the first is 65535).
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned wt_add16(unsigned a, unsigned b) { return __builtin_bit_cast(unsigned, __builtin_bit_cast(u16x2_t, a) + __builtin_bit_cast(u16x2_t, b)); }
__device__ __forceinline__ unsigned wt_min16(unsigned a, unsigned b)
{
    return __builtin_bit_cast(unsigned, __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b)));
}

// KS wavefronts share an item (a tile of pixels x 64 channels) and split its input channels.
template <int KS>
__global__ __launch_bounds__(256, 1) void conv3x3_wtile_kernel(const WtileArgs a)
{
#if __HIP_DEVICE_COMPILE__
    constexpr int TM = kWtTM, TN = kWtTN, STEPS = 18, AHEAD = 6, LOADS = kWtCap / 8;
    constexpr unsigned kOutside = 0x80000000u;
    typedef __attribute__((address_space(3))) u32x4_t lds_u32x4_t;
    typedef __attribute__((address_space(3))) u32x2_t lds_u32x2_t;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kpart = wave % KS, group = wave / KS;
    constexpr int GROUPS = 4 / KS;
    const int frow = lane & 15, fgrp = lane >> 4;
    unsigned char* mine = smem + wave * 2 * kWtBuf;

    const __amdgpu_buffer_rsrc_t x_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, (int)a.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t w_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, (int)a.w_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t y_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.y, 0, (int)a.y_bytes, 0x00020000);

    // Items: die blockIdx % 8 has a range of pixel tiles and one of channel tiles, its workgroups' groups in turn.
    struct Item { int x_base, y_base; unsigned origin, above_left; int nb; bool valid; };  // of the tile's first pixel; row and column of that and of the one above and left
    auto decode = [&](int t) {
        Item it;
        const int die = (int)(blockIdx.x & 7), row = wt_div(t, a.nb_mul, a.nb_sh);
        it.valid = row < a.die_rows && (die >> a.die_col_sh) * a.die_rows + row < a.gm;
        const int mt = it.valid ? (die >> a.die_col_sh) * a.die_rows + row : 0;
        it.nb = it.valid ? (die & ((1 << a.die_col_sh) - 1)) * a.die_cols + t - row * a.die_cols : 0;
        const int image = wt_div(mt, a.image_mul, a.image_sh), rem = mt - image * a.tiles_image;
        const int rb = wt_div(rem, a.cb_mul, a.cb_sh), p0 = rb * a.TH, q0 = (rem - rb * a.cb) * a.TW;
        const int pixel = (image * a.images * a.H + p0) * a.W + q0;
        it.x_base = pixel * a.x_pitch;
        it.y_base = pixel * a.y_pitch + it.nb * 128;
        it.origin = (unsigned)(p0 << 16 | q0);
        it.above_left = (unsigned)((p0 - 1) << 16) | ((unsigned)(q0 - 1) & 0xffffu);
        return it;
    };
    const int stride = (int)(gridDim.x >> 3) * GROUPS;
    int t = (int)(blockIdx.x >> 3) * GROUPS + group;
    Item cur = decode(t);
    const int c_begin = kpart * a.chunks_per_wave;
    // Without a shared item every wavefront goes its own way; the others meet at barriers and end together.
    const bool any = KS == 1 || decode(t - group).valid;

    // Weights: 4 KB a step (tap, half of the 64 channels), streamed in order.  Of a shared item's channels a
    // wavefront finishes a quarter or half; it keeps those in the first columns of its accumulators.
    constexpr int NJ = TN / KS;
    int w_voff[KS];  // columns 0 .. NJ - 1, NJ .. 2 NJ - 1, ...
#pragma unroll
    for (int q = 0; q < KS; ++q) w_voff[q] = lane * 16 + (q ^ kpart) * NJ * 1024;
    u32x4_t wf[AHEAD][TN];
    auto request_w = [&](int set, int j, int soff) { wf[set][j] = __builtin_amdgcn_raw_buffer_load_b128(w_rs, w_voff[j / NJ] + j % NJ * 1024, soff, 0); };
    const int chunk_w = STEPS * 4096;
    int w_off = (cur.nb * a.chunks + c_begin) * chunk_w;

    auto first_weights = [&](int s0, int s1) {
#pragma unroll
        for (int s = 0; s < AHEAD; ++s)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (s >= s0 && s < s1) request_w(s, j, w_off + s * 4096);
    };
    first_weights(0, 1);

    // Tables, the same for all tiles: byte offset from the tile's first pixel, and row and column, of every
    // patch pixel (rows and columns counted from one above and left of the image) and of every output pixel.
    if (threadIdx.x < kWtCap) {
        const int px = threadIdx.x, pr = wt_small_div(px, a.pw_mul), pc = px - pr * a.PW;
        const int image = wt_small_div(pr, a.rows_mul), hr = pr - image * a.image_rows;
        const unsigned rel = (unsigned)((((a.images > 1 ? image * a.H : 0) + hr - 1) * a.W + pc - 1) * a.x_pitch);
        *(u32x2_t*)(smem + kWtTables + px * 8) = u32x2_t{px < a.patch ? rel : kOutside, (unsigned)(hr << 16 | pc)};
    }
    if (threadIdx.x >= 128) {
        const int r = threadIdx.x - 128, ty = wt_small_div(r, a.tw_mul), tx = r - ty * a.TW;
        const int hr = a.images > 1 ? ty - wt_small_div(ty, a.h_mul) * a.H : ty;
        *(u32x2_t*)(smem + kWtTables + (kWtCap + r) * 8) = u32x2_t{ty < a.TH ? (unsigned)((ty * a.W + tx) * a.y_pitch) : kOutside, (unsigned)(hr << 16 | tx)};
    }
    __syncthreads();
    if (KS == 1 ? !cur.valid : !any) return;

    const unsigned limit = (unsigned)((a.H - 1) << 16 | (a.W - 1));
    // Patch of 64 channels: instruction k moves 8 pixels of 128 bytes; slot s of pixel p holds group
    // s ^ ((p >> 1) & 7), pixels counted from the first buffer on (the second one starts at an odd multiple of eight).
    const unsigned in_table = kWtTables + (lane >> 3) * 8;
    unsigned slot = (unsigned)(((lane & 7) ^ (lane >> 4)) << 4);  // pixel k * 8 + lane / 8: (p >> 1) & 7 = (4 * k + lane / 16) & 7
    u32x2_t entry;
    unsigned voff;
    auto patch_part = [&](const Item& it, bool live, int k, int part) {
        if (part == 0) entry = *(const lds_u32x2_t*)(unsigned long)(in_table + k * 64);
        if (part == 1) voff = entry[0] + (slot ^ ((k & 1) << 6)) + (unsigned)it.x_base;
        if (part == 2) entry[1] = wt_add16(entry[1], it.above_left);
        if (part == 3) entry[0] = wt_min16(entry[1], limit);
        if (part == 4) voff = (entry[0] == entry[1]) & live ? voff : kOutside;
    };
    auto patch_issue = [&](int chunk, int k, unsigned char* buf) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rs, (lds_ptr_t)(buf + k * 1024), 16, voff, chunk * 128, 0, 0);
    };
#pragma unroll
    for (int k = 0; k < LOADS; ++k) {
#pragma unroll
        for (int part = 0; part < 5; ++part) patch_part(cur, cur.valid, k, part);
        patch_issue(c_begin, k, mine);
    }

    // This lane's pixels: byte address of the first tap.
    unsigned pp[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int px = i * 16 + frow, ty = wt_small_div(px, a.tw_mul), tx = px - ty * a.TW;
        int pr = ty;
        if (a.images > 1) pr += 2 * wt_small_div(ty, a.h_mul);
        pp[i] = (unsigned)(ty < a.TH ? pr * a.PW + tx : 0) * 128u + (unsigned)(wave * 2 * kWtBuf);
    }
    // Epilogue: eight channels a lane.
    constexpr int LPP = 2 * NJ, PXP = 64 / LPP, PASSES = (16 * TM + PXP - 1) / PXP;
    const int c8 = kpart * (64 / KS) + (lane % LPP) * 8, rsub = lane / LPP;
    const unsigned out_table = kWtTables + (kWtCap + rsub) * 8;
    first_weights(1, AHEAD);
    wt_wait_vmcnt<(AHEAD - 1) * TN>();  // the patch has landed (what is outstanding are weights)
    __builtin_amdgcn_sched_barrier(0);
    unsigned buf_off = 0;  // of the buffer being multiplied
    for (;;) {
        f32x4_t acc[TM][TN];
        const Item nxt = decode(t + stride);
        u32x4_t rres[PASSES];
        unsigned out_off[PASSES];
        u32x2_t out_entry;
        auto out_part = [&](int pass, int part) {
            if (part == 0) out_entry = *(const lds_u32x2_t*)(unsigned long)(out_table + pass * PXP * 8);
            if (part == 1) out_off[pass] = out_entry[0] + (unsigned)(cur.y_base + c8 * 2);
            if (part == 2) out_entry[1] = wt_add16(out_entry[1], cur.origin);
            if (part == 3) out_entry[0] = wt_min16(out_entry[1], limit);
            if (part == 4) out_off[pass] = (out_entry[0] == out_entry[1]) & cur.valid ? out_off[pass] : kOutside;
        };
        auto chunk_of_item = [&](int c, auto first) {
            constexpr bool FIRST = decltype(first)::value;  // the accumulators start from zero
            const bool last = c + 1 == a.chunks_per_wave;
            Item tgt;
            tgt.x_base = last ? nxt.x_base : cur.x_base;
            tgt.above_left = last ? nxt.above_left : cur.above_left;
            const bool live = last ? nxt.valid : cur.valid;
            const int tgt_chunk = last ? c_begin : c_begin + c + 1;
            const int w_next = last ? (nxt.nb * a.chunks + c_begin) * chunk_w : w_off + chunk_w;
            const __amdgpu_buffer_rsrc_t res_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.res, 0, a.res && last ? (int)a.y_bytes : 0, 0x00020000);
            unsigned char* const other = mine + (buf_off ? 0 : kWtBuf);
            slot ^= 64;  // for the other buffer
            u32x4_t pf[2][TM];
            unsigned addr[TM], pre[TM];
            auto address = [&](int tap, int i, int part) {
                if (part == 0) {
                    addr[i] = pp[i] + ((unsigned)((tap / 3) * a.PW + tap % 3) * 128u + buf_off);
                    pre[i] = addr[i] >> 4;
                } else {
                    addr[i] += (pre[i] & 0x70u) ^ (unsigned)(fgrp << 4);
                }
            };
            auto read_px = [&](int st, int i) { pf[st & 1][i] = *(const lds_u32x4_t*)(unsigned long)(addr[i] ^ ((st & 1) << 6)); };
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                address(0, i, 0);
                address(0, i, 1);
                read_px(0, i);
            }
            // A step: 28 MFMAs of 16 cycles, behind each at most two or three other instructions, which is what
            // a wavefront can issue in that time: the next step's pixels are read, the weights of the step AHEAD
            // requested as soon as their registers are free, then the next patch and the residual requested.
#pragma unroll
            for (int st = 0; st < STEPS; ++st) {
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    // patch loads in steps 0 .. 12: one in an even step, two in an odd one; then the residual,
                    // three a step.  Their table entries are read one group of MFMAs ahead.
                    constexpr int PATCH_STEPS = 13;
                    static_assert(LOADS == 19, "patch loads of steps 0 .. 12");
                    auto patch_of = [](int st, int j) { return st >= PATCH_STEPS ? -1 : j == 1 ? st / 2 * 3 + st % 2 : j == 3 && st % 2 ? st / 2 * 3 + 2 : -1; };
                    auto pass_of = [](int st, int j) { return st >= PATCH_STEPS && j > 0 && (st - PATCH_STEPS) * 3 + j - 1 < PASSES ? (st - PATCH_STEPS) * 3 + j - 1 : -1; };
                    const int k = patch_of(st, j), table_k = j + 1 < TN ? patch_of(st, j + 1) : -1;
                    const int pass = pass_of(st, j), table_pass = j + 1 < TN ? pass_of(st, j + 1) : -1;
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        if (FIRST && st == 0)
                            asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc[i][j]) : "v"(wf[st % AHEAD][j]), "v"(pf[st & 1][i]));
                        else
                            asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(wf[st % AHEAD][j]), "v"(pf[st & 1][i]));
                        if (j == 0 && st + 1 < STEPS) read_px(st + 1, i);
                        if (j >= 2 && st % 2 == 0 && st + 2 < STEPS) address(st / 2 + 1, i, j - 2);
                        if (table_k >= 0 && i == 6) patch_part(tgt, live, table_k, 0);
                        if (k >= 0) {
                            if (i >= 1 && i < 5) patch_part(tgt, live, k, i);
                            if (i == 5) patch_issue(tgt_chunk, k, other);
                        }
                        if (table_pass >= 0 && i == 6) out_part(table_pass, 0);
                        if (pass >= 0) {
                            if (i >= 1 && i < 5) out_part(pass, i);
                            if (i == 5) rres[pass] = __builtin_amdgcn_raw_buffer_load_b128(res_rs, out_off[pass], 0, 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    request_w(st % AHEAD, j, st + AHEAD < STEPS ? w_off + (st + AHEAD) * 4096 : w_next + (st + AHEAD - STEPS) * 4096);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            wt_wait_vmcnt<20>();  // the next patch has landed: 23 weight fragments at least were requested after it
            __builtin_amdgcn_sched_barrier(0);
            w_off = w_next;
            buf_off ^= kWtBuf;
        };
        chunk_of_item(0, std::integral_constant<bool, true>());
        for (int c = 1; c < a.chunks_per_wave; ++c) chunk_of_item(c, std::integral_constant<bool, false>());
        // The hazard recogniser does not see into the assembly of the MFMAs: what reads their results keeps its distance.
        asm volatile("s_nop 15");
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));

        // The buffer just multiplied (the next patch is in the other one) takes the exchange and the transposition.
        unsigned char* const scratch = mine + (buf_off ? 0 : kWtBuf);
        const unsigned relu_floor = a.relu ? kReluFloor : kNoReluFloor;
        const f32x4_t sc0 = *(const f32x4_t*)(a.scale + cur.nb * 64 + c8), sc1 = *(const f32x4_t*)(a.scale + cur.nb * 64 + c8 + 4);
        const f32x4_t sh0 = *(const f32x4_t*)(a.shift + cur.nb * 64 + c8), sh1 = *(const f32x4_t*)(a.shift + cur.nb * 64 + c8 + 4);
        if constexpr (KS > 1) {
            // Partial sums change hands as whole accumulators: the second half of the columns, then (KS = 4) the second quarter.
            auto exchange = [&](auto first, int partner) {
                constexpr int J = decltype(first)::value;
                const unsigned char* from = smem + (wave ^ partner) * 2 * kWtBuf + (buf_off ? 0 : kWtBuf);  // all walk the same number of chunks
                __syncthreads();
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < J; ++j) *(f32x4_t*)(scratch + (i * J + j) * 1024 + lane * 16) = acc[i][J + j];
                __syncthreads();
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < J; ++j) acc[i][j] += *(const f32x4_t*)(from + (i * J + j) * 1024 + lane * 16);
            };
            exchange(std::integral_constant<int, 2>(), KS / 2);
            if constexpr (KS == 4) exchange(std::integral_constant<int, 1>(), 1);
            __syncthreads();
        }
        constexpr int SROW = NJ * 16 + 4, PT = PXP > 16 ? PXP / 16 : 1;  // floats of a staged pixel, pixel tiles staged at once
        constexpr int ROUNDS = (TM + PT - 1) / PT, HP = PT * 16 / PXP;   // staging rounds, passes of one
        constexpr int BUFS = 4;                                          // staging buffers
        static_assert(BUFS * PT * 16 * SROW * 4 <= kWtBuf, "staging fits the buffer");
        auto stage = [&](int q) {
#pragma unroll
            for (int i = q * PT; i < q * PT + PT && i < TM; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    *(f32x4_t*)((float*)scratch + (q % BUFS * PT * 16 + (i - q * PT) * 16 + frow) * SROW + j * 16 + fgrp * 4) = acc[i][j];
        };
        f32x4_t v[2][HP][2];
        auto fetch = [&](int q) {
#pragma unroll
            for (int h = 0; h < HP; ++h)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    v[q & 1][h][e] = *(const f32x4_t*)((float*)scratch + (q % BUFS * PT * 16 + h * PXP + rsub) * SROW + lane % LPP * 8 + e * 4);
        };
#pragma unroll
        for (int q = 0; q < BUFS && q < ROUNDS; ++q) stage(q);
        fetch(0);
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            if (q + 1 < ROUNDS) fetch(q + 1);
#pragma unroll
            for (int h = 0; h < HP; ++h) {
                const int pass = q * HP + h;
                const f32x4_t v0 = v[q & 1][h][0] * sc0 + sh0, v1 = v[q & 1][h][1] * sc1 + sh1;
                const float f[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                u32x4_t ov;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const unsigned rv = rres[pass][u];
                    ov[u] = pack_bf16x2_relu(f[2 * u] + __uint_as_float(rv << 16), f[2 * u + 1] + __uint_as_float(rv & 0xffff0000u), relu_floor);
                }
                __builtin_amdgcn_raw_buffer_store_b128(ov, y_rs, out_off[pass], 0, 0);
            }
            if (q + BUFS < ROUNDS) stage(q + BUFS);
        }
        if (KS == 1 ? !nxt.valid : !decode(t - group + stride).valid) break;
        t += stride;
        cur = nxt;
    }
    __builtin_amdgcn_s_waitcnt(0);
#endif
}

// ---- weights in fragment order -----------------------------------------------------
// From [cout][tap][cin] to [cout / 64][cin / 64][tap][half][16 channels of 64][lane][16 bytes]: lane l of a
// fragment holds channel l % 16 and the 16-byte group l / 16 of the half.
__global__ void repack_fragments_kernel(const u32x4_t* src, u32x4_t* dst, int taps, int chunks, int units)
{
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= units) return;
    const int lane = u & 63, j = (u >> 6) & 3, ks = (u >> 8) & 1, rest = u >> 9;
    const int tap = rest % taps, chunk = rest / taps % chunks, nb = rest / taps / chunks;
    const int row = nb * 64 + j * 16 + (lane & 15);
    dst[u] = src[((size_t)row * taps + tap) * (chunks * 8) + chunk * 8 + ks * 4 + (lane >> 4)];
}

bool fragment_order(const sgprs_conv_desc_t& d)
{
    return is_igemm(d) && d.dtype == SGPRS_BF16 && d.cin % 64 == 0 && d.cout % 64 == 0 && (long long)d.cout * d.r * d.s * d.cin * 2 < (1ll << 31);
}

int repack_fragments(const sgprs_conv_desc_t& d, const void* src, void* dst, hipStream_t stream)
{
    if (!fragment_order(d)) return fail(SGPRS_ERR_INVALID_ARG, "internal: no fragment order for this shape");
    const int taps = d.r * d.s, units = d.cout * taps * (d.cin / 8);
    hipLaunchKernelGGL(repack_fragments_kernel, dim3((units + 255) / 256), dim3(256), 0, stream, (const u32x4_t*)src, (u32x4_t*)dst, taps, d.cin / 64, units);
    SGPRS_HIP(hipGetLastError());
    return SGPRS_OK;
}

// ---- host side ---------------------------------------------------------------------
struct WtileShape { int th, tw, pw, images, patch; long long gm; };
static constexpr unsigned wt_small_mul(int q) { return (unsigned)(((1 << 22) + q - 1) / q); }

static bool wtile_shape(const sgprs_conv_desc_t& d, WtileShape* best)
{
    best->gm = 0;
    for (int tw = 1; tw <= std::min(d.w, 16 * kWtTM); ++tw) {
        const int whole = tw == d.w;  // the zero column right of a row is the one left of the next
        const int pw = whole ? tw + 1 : tw + 2, cb = (d.w + tw - 1) / tw;
        for (int th = std::min(16 * kWtTM / tw, d.h); th >= 1; --th) {
            const int patch = (th + 2) * pw + whole;
            if (patch > kWtCap) continue;
            const long long gm = (long long)d.n * ((d.h + th - 1) / th) * cb;
            if (!best->gm || gm < best->gm) *best = WtileShape{th, tw, pw, 1, patch, gm};
            break;
        }
        for (int images = 2; images <= d.n && images * d.h * tw <= 16 * kWtTM; ++images) {
            const int patch = images * (d.h + 2) * pw + whole;
            if (patch > kWtCap) break;
            const long long gm = (long long)((d.n + images - 1) / images) * cb;
            if (!best->gm || gm < best->gm) *best = WtileShape{images * d.h, tw, pw, images, patch, gm};
        }
    }
    return best->gm > 0;
}

bool wtile_applicable(const sgprs_conv_desc_t& d)
{
    const long long xb = (long long)d.n * d.h * d.w * d.cin * 2, yb = (long long)d.n * d.h * d.w * d.cout * 2;
    return d.dtype == SGPRS_BF16 && d.r == 3 && d.s == 3 && d.stride == 1 && d.pad == 1 && d.cin % 64 == 0 && d.cout % 64 == 0 &&
           (long long)d.cout * 9 * d.cin * 2 < (1ll << 31) && xb < (1ll << 31) && yb < (1ll << 31) && d.h < (1 << 15) && d.w < (1 << 15);
}

// Best split of the input channels over KS wavefronts, and its time: launch, prologue and epilogue, 18 steps
// for every 64 input channels at the clock that the share of the chip in use leaves (20 launches of the
// network's layers on 24 to 256 CUs: within 10 %).  Whole inferences with this kernel and conv3x3_kpatch_kernel
// against those without, 1 to 96 images on 8 to 256 CUs: 0.87 to 1.006 of the time.
bool plan_wtile(const sgprs_conv_desc_t& d, int cus, int* ks, double* cost_us)
{
    WtileShape t;
    if (!wtile_applicable(d) || !wtile_shape(d, &t)) return false;
    const int chunks = d.cin / 64, wgs = std::max(1, cus / 8);
    *cost_us = 1e30;
    for (int k = 1; k <= 4; k *= 2) {
        if (chunks % k) continue;
        const long long items = t.gm * (d.cout / 64), per_die = (items + 7) / 8, rounds = (per_die + wgs * (4 / k) - 1) / (wgs * (4 / k));
        const double active = (double)std::min<long long>(items * k, cus * 4) / 1024;
        const double cost = 3.6 + rounds * (chunks / k * (4.4 + 2.0 * active) + 2.2 + (k > 1 ? 0.3 : 0.0));
        if (cost < *cost_us) { *cost_us = cost; *ks = k; }
    }
    return *cost_us < 1e30;
}

template <int KS> static int launch_wt(const WtileArgs& a, int grid, hipStream_t stream)
{
    static std::atomic<bool> raised{false};
    if (!raised) {
        SGPRS_HIP(hipFuncSetAttribute((const void*)conv3x3_wtile_kernel<KS>, hipFuncAttributeMaxDynamicSharedMemorySize, kWtLds));
        raised = true;
    }
    SGPRS_LAUNCH((conv3x3_wtile_kernel<KS>), dim3(grid), dim3(256), kWtLds, stream, a);
    SGPRS_HIP(hipGetLastError());
    return SGPRS_OK;
}

int launch_conv3x3_wtile(const sgprs_conv_desc_t& d, int ks, const void* x, const void* w_fragments, const float* scale, const float* shift,
                         const void* res, void* y, hipStream_t stream, int cus, Profiler* prof)
{
    WtileShape t;
    const int chunks = d.cin / 64;
    if (!wtile_applicable(d) || !wtile_shape(d, &t) || (ks != 1 && ks != 2 && ks != 4) || chunks % ks)
        return fail(SGPRS_ERR_INVALID_ARG, "internal: launch plan does not match the shape");
    WtileArgs a;
    memset(&a, 0, sizeof(a));
    a.x = (const unsigned char*)x; a.w = (const unsigned char*)w_fragments; a.y = (unsigned char*)y;
    a.scale = scale; a.shift = shift; a.res = (const unsigned char*)res;
    a.x_bytes = (unsigned)((long long)d.n * d.h * d.w * d.cin * 2);
    a.y_bytes = (unsigned)((long long)d.n * d.h * d.w * d.cout * 2);
    a.w_bytes = (unsigned)((long long)d.cout * 9 * d.cin * 2);
    a.H = d.h; a.W = d.w;
    a.x_pitch = d.cin * 2; a.y_pitch = d.cout * 2;
    a.chunks = chunks; a.chunks_per_wave = chunks / ks;
    a.TH = t.th; a.TW = t.tw; a.PW = t.pw; a.patch = t.patch; a.images = t.images;
    a.image_rows = t.images > 1 ? d.h + 2 : t.th + 2;
    a.cb = (d.w + t.tw - 1) / t.tw;
    a.tiles_image = t.images > 1 ? a.cb : (d.h + t.th - 1) / t.th * a.cb;
    a.pw_mul = wt_small_mul(t.pw); a.tw_mul = wt_small_mul(t.tw); a.rows_mul = wt_small_mul(a.image_rows); a.h_mul = wt_small_mul(d.h);
    const int gn = d.cout / 64;
    a.gm = (int)t.gm; a.relu = d.relu;
    // dies side by side along the channels: the split for which a die's weights and pixels are fewest
    double least = 1e30;
    for (int s = 0; s < 4; ++s) {
        if (gn % (1 << s)) continue;
        const double bytes = (double)a.w_bytes / (1 << s) + (double)a.x_bytes * (1 << s) / 8;
        if (bytes < least) { least = bytes; a.die_col_sh = s; }
    }
    a.die_cols = gn >> a.die_col_sh;
    const int die_row_count = 8 >> a.die_col_sh;
    a.die_rows = (a.gm + die_row_count - 1) / die_row_count;
    div_constants(a.tiles_image, &a.image_mul, &a.image_sh);
    div_constants(a.cb, &a.cb_mul, &a.cb_sh);
    div_constants(a.die_cols, &a.nb_mul, &a.nb_sh);
    const int groups = 4 / ks, per_die = (int)(((long long)a.die_rows * a.die_cols + groups - 1) / groups);
    const int grid = 8 * std::max(1, std::min(cus / 8, per_die));
    const double M = (double)d.n * d.h * d.w;
    int rc;
    if (prof && prof->on && (rc = prof->begin(stream, kKindWtile, ks, 2.0 * M * d.cout * 9 * d.cin, ((double)a.x_bytes + a.w_bytes + (double)a.y_bytes * (res ? 2 : 1)))))
        return rc;
    rc = ks == 1 ? launch_wt<1>(a, grid, stream) : ks == 2 ? launch_wt<2>(a, grid, stream) : launch_wt<4>(a, grid, stream);
    if (rc) return rc;
    if (prof && prof->on && (rc = prof->end(stream))) return rc;
    return SGPRS_OK;
}

}  // namespace sgprs
