// A down-sampling block's 3x3 stride-2 convolution and its 1x1 stride-2 shortcut, bf16, in one launch: a wavefront's
// own tile, weights straight from the L2 to registers.
//
// What bounds the paired implicit GEMM is its operands' way: tiles of 64 or 128 pixels fetch every input pixel
// 2.25 times and every weight once per tile through the LDS, with a barrier per k-tile, and inside a network the weights
// come cold (64 images on 256 CUs, 14x14x256 -> 512: 19 us in a loop, 28 with inputs that change).  Here
//   * a wavefront owns 98 (or up to 64) output pixels x 64 channels of both convolutions: 7 x 4 (4 x 4) MFMA tiles
//     each, in accumulator registers; the shortcut is one more step, on the centre tap's pixels, which are there;
//   * weights are one coalesced KiB per fragment from the L2 to registers, requested five steps ahead (two in the 4 x 1 variant,
//     whose two workgroups on a CU cover for each other and leave room for no more);
//   * two channel tiles share a patch of 32 input channels, fetched once, double buffered, the next one requested in the
//     first steps of the ten that this one takes: one barrier per 280 MFMAs of a wavefront (4 x 4 tiles: 160).  Four planes (rows
//     and columns even or odd) make consecutive output pixels read consecutive pixels; 64 bytes of each, groups permuted against conflicts;
//   * where pixels are few, two wavefronts share a tile by input channels (their sums meet in LDS).
// Timestamps, 64 images on 256 CUs, 56x56x64 -> 128, 7 x 1 tiles (us): 5.5 until the first patch is there (25.7 MB for the
// launch: the memory's rate), two stages of 3.5 (2.7 of MFMAs at the clock they leave), 3.5 for the stores.
// Inside networks whose inputs change, us per launch, paired implicit GEMM / this, the three blocks: 64 images on 256 CUs 22.8
// / 19.6, 20.8 / 17.8, 28.1 / 18.6; 128 images 39.0 / 37.8, 29.2 / 26.0, 33.0 / 25.9; 48 images on 192 CUs 21.7 / 17.8, 19.9 / 17.6,
// 27.4 / 17.9; 16 on 64 18.6 / 15.1, 16.2 / 16.5 (not chosen), 20.1 / 14.4; 68 on 256 23.3 / 24.8, 20.6 / 24.2, 28.4 / 24.0
// (not chosen, the last one for its few items).
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace sgprs {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr int kS2TN = 4, kS2Steps = 10;                           // channel tiles of a wavefront, steps of a stage
// Two workgroups a CU where registers allow it and there are no sums to exchange; steps that weights are requested ahead.
constexpr int s2_workgroups(int tm, int ks) { return tm == 4 && ks == 1 ? 2 : 1; }
constexpr int s2_ahead(int tm, int ks) { return s2_workgroups(tm, ks) == 2 ? 2 : 5; }
// patch pixels of a tile of 16 TM output pixels (instructions of 16, two wavefronts in turn)
constexpr int s2_cap(int tm) { return tm == 7 ? 480 : 256; }
// a buffer: two patches of 32 channels, or the sums that the wavefronts exchange
constexpr int s2_buffer(int tm) { return std::max(2 * s2_cap(tm) * 64, 4 * 2 * tm * 1024); }

constexpr int s2_lds(int tm) { return 2 * s2_buffer(tm) + (s2_cap(tm) + 16 * tm) * 8; }  // (tables behind the buffers)

// Output tiles are TH rows x TW columns of `images` images.  Their input pixels lie in LDS as four planes (row and
// column even or odd, counted from one above and left of the tile), a row of a plane PW = TW + 1 pixels, so
// that consecutive output pixels read consecutive pixels for every tap.
struct S2tileArgs {
    const unsigned char* x;
    const unsigned char* w[2];      // fragments, see repack_fragments_kernel: of the 3x3, of the shortcut
    unsigned char* y[2];
    const float* scale[2];
    const float* shift[2];
    unsigned x_bytes, y_bytes, w_bytes[2];
    int H, W, P, Q;
    int x_pitch, y_pitch;           // bytes of a pixel
    int chunks, stages;             // of 64 input channels; of 32, those of one wavefront
    int TH, TW, PW, images, image_slots, slots;  // TH rows of one image; patch pixels of an image and in all
    int tiles_image, cb, gm, gm_groups, gn;      // tiles of an image (or group), of a row of it, all; groups of a workgroup; pairs of channel tiles
    unsigned slots_mul, pw_mul, tw_mul, th_mul;
    unsigned image_mul, cb_mul, gn_mul;
    int image_sh, cb_sh, gn_sh;
    int relu[2];
};

__device__ __forceinline__ int s2_div(int m, unsigned mul, int sh) { return (int)(__umulhi(2u * (unsigned)m, mul) >> sh); }
__device__ __forceinline__ int s2_small_div(int m, unsigned mul) { return (int)((unsigned)__umul24((unsigned)m, mul) >> 22); }
template <int N> __device__ __forceinline__ void s2_wait_vmcnt()
{
    static_assert(N <= 63, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// Sum and minimum of 16-bit halves: row << 16 | column lies inside the image when its minimum with the
// last row and column is itself (one before the first is 65535).
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned s2_add16(unsigned a, unsigned b) { return __builtin_bit_cast(unsigned, __builtin_bit_cast(u16x2_t, a) + __builtin_bit_cast(u16x2_t, b)); }
__device__ __forceinline__ unsigned s2_min16(unsigned a, unsigned b)
{
    return __builtin_bit_cast(unsigned, __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b)));
}

// Four wavefronts: two tiles of pixels (KS = 1) or two halves of the input channels (KS = 2), times two channel tiles of 64.
template <int TM, int KS>
__global__ __launch_bounds__(256, s2_workgroups(TM, KS)) void conv_s2tile_kernel(const S2tileArgs a)
{
#if __HIP_DEVICE_COMPILE__
    constexpr int TN = kS2TN, AHEAD = s2_ahead(TM, KS), STEPS = kS2Steps, CAP = s2_cap(TM), PATCH = CAP * 64, BUF = s2_buffer(TM);
    constexpr int LOADS = CAP / 32;                   // of a wavefront
    constexpr int NJ = TN / KS;                       // channel tiles that a wavefront finishes
    constexpr unsigned kOutside = 0x80000000u;
    typedef __attribute__((address_space(3))) u32x4_t lds_u32x4_t;
    typedef __attribute__((address_space(3))) u32x2_t lds_u32x2_t;
    typedef __attribute__((address_space(3))) f32x4_t lds_f32x4_t;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = wave >> 1, cb = wave & 1;       // patch, channel tile
    const int kpart = KS == 2 ? group : 0;
    const int frow = lane & 15, fgrp = lane >> 4;

    const __amdgpu_buffer_rsrc_t x_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, (int)a.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t w_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.w[0], 0, (int)a.w_bytes[0], 0x00020000);
    const __amdgpu_buffer_rsrc_t w1_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.w[1], 0, (int)a.w_bytes[1], 0x00020000);

    // Items: consecutive channel pairs of a group of pixel tiles; die blockIdx % 8 has a contiguous eighth of them.
    struct Item { int image, p0, q0, nb; bool valid; };
    const int items = a.gm_groups * a.gn, per_die = (items + 7) >> 3, step = (int)(gridDim.x >> 3);
    const int die = (int)(blockIdx.x & 7), die_end = min(items, (die + 1) * per_die);
    auto decode = [&](int t) {
        Item it;
        const int row = s2_div(min(t, items - 1), a.gn_mul, a.gn_sh), mt = KS == 2 ? row : row * 2 + group;
        it.valid = t < die_end && mt < a.gm;
        const int m = min(mt, a.gm - 1), im = s2_div(m, a.image_mul, a.image_sh), rem = m - im * a.tiles_image;
        const int rb = s2_div(rem, a.cb_mul, a.cb_sh);
        it.image = im * a.images;
        it.p0 = rb * a.TH;
        it.q0 = (rem - rb * a.cb) * a.TW;
        it.nb = (min(t, items - 1) - row * a.gn) * 2 + cb;
        return it;
    };
    int t = die * per_die + (int)(blockIdx.x >> 3);
    if (t >= die_end) return;
    Item cur = decode(t);

    const int first_half = KS == 2 ? kpart * a.stages : 0;  // of the 32-channel halves
    // Weights: fragments of step s of a half; the steps are taps 0 .. 4, the shortcut, taps 5 .. 8.  Where two wavefronts share a
    // tile, the channel tiles that this one finishes come first.
    u32x4_t wf[AHEAD][TN];
    auto request_w = [&](int nb, int half, int s) {
        const int c = half >> 1, h = half & 1;
        const int block = nb * a.chunks + c;
        const int soff = s == 5 ? (block * 2 + h) * 4096 : (block * 18 + (s > 5 ? s - 1 : s) * 2 + h) * 4096;
#pragma unroll
        for (int j = 0; j < TN; ++j)
            wf[s % AHEAD][j] = __builtin_amdgcn_raw_buffer_load_b128(s == 5 ? w1_rs : w_rs, lane * 16 + (KS == 2 ? (j ^ (kpart * 2)) : j) * 1024, soff, 0);
    };
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) request_w(cur.nb, first_half, s);

    // Table: byte offset from the tile's first pixel's centre, and row and column (from one above and left of it), of every patch pixel.
    for (int s = threadIdx.x; s < CAP; s += 256) {
        const int im = s2_small_div(s, a.slots_mul), u = s - im * a.image_slots;
        const int v = s2_small_div(u, a.pw_mul), c = u - v * a.PW;
        const int even = a.TH + 1;                    // rows of the planes of even rows
        const bool odd_row = v >= 2 * even;
        const int v1 = odd_row ? v - 2 * even : v, n1 = odd_row ? a.TH : even;
        const bool odd_col = v1 >= n1;
        const int row = 2 * (v1 - (odd_col ? n1 : 0)) + odd_row, col = 2 * c + odd_col;
        const bool used = s < a.slots && (c < a.TW || !odd_col);
        *(lds_u32x2_t*)(unsigned long)(2 * BUF + s * 8) = u32x2_t{(unsigned)(((im * a.H + row - 1) * a.W + col - 1) * a.x_pitch), used ? (unsigned)(row << 16 | col) : 0x7fff7fffu};
    }
    if (threadIdx.x < 16 * TM) {                      // of every output pixel: the same, from the tile's first
        const int ty = s2_small_div(threadIdx.x, a.tw_mul), tx = threadIdx.x - ty * a.TW, im = s2_small_div(ty, a.th_mul), p = ty - im * a.TH;
        *(lds_u32x2_t*)(unsigned long)(2 * BUF + (CAP + threadIdx.x) * 8) = u32x2_t{(unsigned)(((im * a.P + p) * a.Q + tx) * a.y_pitch), im < a.images ? (unsigned)(p << 16 | tx) : 0x7fff7fffu};
    }
    __syncthreads();
    // Patch pixels of a wavefront's instruction k: 16, from (2 k + cb) * 16 on.  Position g of pixel s holds its 16-byte group g ^ ((s >> 2) & 3).
    const unsigned limit = (unsigned)((a.H - 1) << 16 | (a.W - 1)), lane_part = (unsigned)((((lane & 3) ^ (lane >> 4)) & 3) << 4);
    const lds_u32x2_t* const table = (const lds_u32x2_t*)(unsigned long)(2 * BUF) + cb * 16 + (lane >> 2);
    struct Origin { unsigned x_base, above_left; bool valid; };
    auto origin = [&](const Item& it) {
        return Origin{(unsigned)(((it.image * a.H + 2 * it.p0) * a.W + 2 * it.q0) * a.x_pitch), (unsigned)((2 * it.p0 - 1) << 16) | ((unsigned)(2 * it.q0 - 1) & 0xffffu), it.valid};
    };
    auto patch_issue = [&](const Origin& it, u32x2_t entry, int half, int k, unsigned buf) {
        const unsigned at = s2_add16(entry[1], it.above_left), off = entry[0] + (it.x_base + lane_part);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rs, (lds_ptr_t)(smem + buf + group * PATCH + (2 * k + cb) * 1024), 16,
                                                 (s2_min16(at, limit) == at) & it.valid ? off : kOutside, half * 64, 0, 0);
    };
#pragma unroll
    for (int k = 0; k < LOADS; ++k) {
        patch_issue(origin(cur), table[k * 32], first_half, k, 0);
    }

    // This lane's pixels: byte address of the first tap's pixel in the first buffer.
    unsigned pp[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int px = i * 16 + frow, ty = s2_small_div(px, a.tw_mul), tx = px - ty * a.TW;
        const int im = s2_small_div(ty, a.th_mul), r = ty - im * a.TH;
        pp[i] = (unsigned)(im < a.images ? im * a.image_slots + r * a.PW + tx : 0) * 64u + (unsigned)(group * PATCH);
    }
    const unsigned lane_group = (unsigned)(fgrp << 4);
    // pixel offset of tap (r, s): plane (r & 1, s & 1), row r >> 1, column s >> 1
    auto tap_offset = [&](int tap) {
        const int r = tap / 3, s = tap % 3, even = a.TH + 1;
        const int plane = (r & 1) * 2 * even + (s & 1) * ((r & 1) ? a.TH : even);
        return (unsigned)(((plane + (r >> 1)) * a.PW + (s >> 1)) * 64);
    };

    s2_wait_vmcnt<0>();                               // this wavefront's part of the patch has landed
    __syncthreads();
    unsigned buf = 0;                                 // of the stage being multiplied
    for (;;) {
        f32x4_t acc[2][TM][TN];
        const bool more = t + step < die_end;
        const Item nxt = decode(t + step);
        auto stage = [&](int half, bool last, auto first) {
            constexpr bool FIRST = decltype(first)::value;
            const unsigned other = buf ^ BUF;
            const int w_nb = last ? nxt.nb : cur.nb, next_half = last ? first_half : half + 1;
            u32x4_t pf[2][TM];
            unsigned addr[TM], pre[TM], tap_base;
            auto address = [&](int tap, int i, int part) {
                if (part == 0) {
                    if (i == 0) {
                        tap_base = tap_offset(tap) + buf;
                        asm volatile("" : "+s"(tap_base));  // else the sums without buf are kept in registers for all taps
                    }
                    addr[i] = pp[i] + tap_base;
                    pre[i] = (addr[i] >> 4) & 0x30u;
                } else {
                    addr[i] += pre[i] ^ lane_group;
                }
            };
            auto read_px = [&](int tap, int i) { pf[tap & 1][i] = *(const lds_u32x4_t*)(unsigned long)addr[i]; };
            const Origin from = last ? origin(nxt) : origin(cur);
            u32x2_t entry[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                address(0, i, 0);
                address(0, i, 1);
                read_px(0, i);
            }
            // A step: TM * TN MFMAs, behind each at most a few other instructions: the next tap's addresses and pixels, the
            // next patch in the first steps, the weights of the step AHEAD as their registers become free.
#pragma unroll
            for (int st = 0; st < STEPS; ++st) {
                const int tap = st > 5 ? st - 1 : st == 5 ? 4 : st, set = st == 5;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        if (FIRST && (st == 0 || st == 5))
                            asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc[set][i][j]) : "v"(wf[st % AHEAD][j]), "v"(pf[tap & 1][i]));
                        else
                            asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[set][i][j]) : "v"(wf[st % AHEAD][j]), "v"(pf[tap & 1][i]));
                        if (st != 4 && tap < 8) {  // (step 5 multiplies the pixels of step 4 again)
                            if (j < 2) address(tap + 1, i, j);
                            if (j == 2) read_px(tap + 1, i);
                        }
                        constexpr int PER_STEP = (LOADS + AHEAD - 1) / AHEAD;
                        static_assert(PER_STEP <= TM, "one behind each MFMA of a column");
                        const int k = st * PER_STEP + i;
                        if (st < AHEAD && i < PER_STEP && k < LOADS) {
                            if (j == 2) entry[i] = table[k * 32];
                            if (j == 3) patch_issue(from, entry[i], next_half, k, other);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                request_w(st + AHEAD < STEPS ? cur.nb : w_nb, st + AHEAD < STEPS ? half : next_half, (st + AHEAD) % STEPS);
                __builtin_amdgcn_sched_barrier(0);
            }
            s2_wait_vmcnt<AHEAD * TN>();              // the next patch has landed: only the weights of AHEAD steps were requested after it
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();                          // for every wavefront, and this one has been read
            buf = other;
        };
        stage(first_half, a.stages == 1, std::integral_constant<bool, true>());
        for (int s = 1; s < a.stages; ++s) stage(first_half + s, s + 1 == a.stages, std::integral_constant<bool, false>());
        const int ch0 = cur.nb * 64 + kpart * 32;
        // The hazard recogniser does not see into the assembly of the MFMAs: what reads their results keeps its distance.
        asm volatile("s_nop 15");
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[e][i][j]));

        // The buffer just multiplied (the next patch is in the other one) takes the exchange and the transposition.
        unsigned char* const scratch = smem + (buf ^ BUF);
        if constexpr (KS == 2) {
            unsigned char* const mine = scratch + wave * 2 * TM * 1024;
            const unsigned char* const theirs = scratch + (wave ^ 2) * 2 * TM * 1024;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) *(lds_f32x4_t*)(mine + (i * 2 + j) * 1024 + lane * 16) = acc[e][i][2 + j];
                __syncthreads();
#pragma unroll
                for (int i = 0; i < TM; ++i) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[e][i][j] += *(const lds_f32x4_t*)(theirs + (i * 2 + j) * 1024 + lane * 16);
                    if (i % 2) __builtin_amdgcn_sched_barrier(0);
                }
                __syncthreads();
            }
        }
        // Sixteen pixels at a time through LDS: a lane has four channels of one pixel and stores eight.
        constexpr int ROW = NJ * 32 + 16, LPP = 2 * NJ, PXP = 64 / LPP, BUFS = 2;
        unsigned char* const mine = scratch + wave * (BUFS * 16 * ROW);
        static_assert(4 * BUFS * 16 * ROW <= BUF, "staging fits the buffer");
        const unsigned y_base = (unsigned)(((cur.image * a.P + cur.p0) * a.Q + cur.q0) * a.y_pitch + (ch0 + lane % LPP * 8) * 2);
        const unsigned out_limit = (unsigned)((a.P - 1) << 16 | (a.Q - 1)), out_origin = (unsigned)(cur.p0 << 16 | cur.q0);
        const lds_u32x2_t* const out_table = (const lds_u32x2_t*)(unsigned long)(2 * BUF + CAP * 8) + lane / LPP;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const __amdgpu_buffer_rsrc_t y_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.y[e], 0, (int)a.y_bytes, 0x00020000);
            const unsigned relu_floor = a.relu[e] ? kReluFloor : kNoReluFloor;
            f32x4_t sc[NJ], sh[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                sc[j] = *(const f32x4_t*)(a.scale[e] + ch0 + j * 16 + fgrp * 4);
                sh[j] = *(const f32x4_t*)(a.shift[e] + ch0 + j * 16 + fgrp * 4);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                unsigned char* const rows = mine + i % BUFS * 16 * ROW;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const f32x4_t v = acc[e][i][j] * sc[j] + sh[j];
                    *(lds_u32x2_t*)(rows + frow * ROW + j * 32 + fgrp * 8) = u32x2_t{pack_bf16x2_relu(v[0], v[1], relu_floor), pack_bf16x2_relu(v[2], v[3], relu_floor)};
                }
#pragma unroll
                for (int h = 0; h < 16 / PXP; ++h) {
                    const u32x4_t v = *(const lds_u32x4_t*)(rows + (h * PXP + lane / LPP) * ROW + lane % LPP * 16);
                    const u32x2_t out = out_table[i * 16 + h * PXP];
                    const unsigned at = s2_add16(out[1], out_origin);
                    __builtin_amdgcn_raw_buffer_store_b128(v, y_rs, (s2_min16(at, out_limit) == at) & cur.valid ? out[0] + y_base : kOutside, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!more) break;
        t += step;
        cur = nxt;
        __syncthreads();                              // the scratch is the next stage's other buffer
    }
    __builtin_amdgcn_s_waitcnt(0);
#endif
}

// ---- host side ---------------------------------------------------------------------
struct S2tileShape { int th, tw, images, slots; long long gm; };
static constexpr unsigned s2_small_mul(int q) { return (unsigned)(((1 << 22) + q - 1) / q); }

// The tile of 16 * tm output pixels that cuts the maps into the fewest.
static bool s2tile_shape(const sgprs_conv_desc_t& d, int tm, S2tileShape* best)
{
    const int P = out_dim(d.h, 3, 2, 1), Q = out_dim(d.w, 3, 2, 1);
    best->gm = 0;
    auto offer = [&](int th, int tw, int images) {
        const int slots = images * (4 * th + 2) * (tw + 1);
        if (images * th * tw > 16 * tm || slots > s2_cap(tm)) return;
        const long long gm = (long long)((d.n + images - 1) / images) * ((P + th - 1) / th) * ((Q + tw - 1) / tw);
        if (!best->gm || gm < best->gm || (gm == best->gm && slots < best->slots)) *best = S2tileShape{th, tw, images, slots, gm};
    };
    for (int tw = 1; tw <= std::min(Q, 16 * tm); ++tw) {
        for (int th = 1; th <= std::min(P, 16 * tm / tw); ++th) offer(th, tw, 1);
        for (int images = 2; images <= d.n && images * P * tw <= 16 * tm; ++images) offer(P, tw, images);
    }
    return best->gm > 0;
}

// Variants: tiles of 7 or 4 MFMA tiles of pixels, the input channels in one or two parts.
constexpr int kS2tileVariants = 4;
static constexpr int s2_tm(int v) { return v < 2 ? 7 : 4; }
static constexpr int s2_ks(int v) { return 1 + v % 2; }

bool s2tile_fits(const sgprs_conv_desc_t& d, const sgprs_conv_desc_t& d1, int v)
{
    S2tileShape t;
    const long long xb = (long long)d.n * d.h * d.w * d.cin * 2, yb = (long long)d.n * out_dim(d.h, 3, 2, 1) * out_dim(d.w, 3, 2, 1) * d.cout * 2;
    return d.dtype == SGPRS_BF16 && d1.dtype == SGPRS_BF16 && d.r == 3 && d.s == 3 && d.stride == 2 && d.pad == 1 && d1.r == 1 && d1.s == 1 && d1.stride == 2 && d1.pad == 0 &&
           d1.n == d.n && d1.h == d.h && d1.w == d.w && d1.cin == d.cin && d1.cout == d.cout && d.cin % 64 == 0 && d.cout % 128 == 0 &&
           (long long)d.cout * 9 * d.cin * 2 < (1ll << 31) && xb < (1ll << 31) && yb < (1ll << 31) && d.h < (1 << 14) && d.w < (1 << 14) &&
           v >= 0 && v < kS2tileVariants && (d.cin / 64) % s2_ks(v) == 0 && s2tile_shape(d, s2_tm(v), &t);
}

// Estimated time (us) inside a network whose inputs change: a fixed part, what the busiest CU's items take (a part of their own and their
// stages, at the clock that the share of the chip in use leaves) and a part of the memory traffic.  Whole items on the busiest
// CU: one more than the others have takes as long as one on each (4 x 1 tiles, 56x56x64 -> 128 on 256 CUs: 64 images 19.6, 68 images 24.8).
// Two 4 x 1 items share a CU's matrix cores: 8.2 for the pair, 5.2 for one that is left.  Fitted to the three blocks, 1 to 512
// images on 8 to 256 CUs: 4 to 5 % off rms, 16 % at most.
bool plan_s2tile(const sgprs_conv_desc_t& d, const sgprs_conv_desc_t& d1, int cus, int* variant, double* cost_us)
{
    double best = 1e30;
    for (int v = 0; v < kS2tileVariants; ++v) {
        S2tileShape t;
        const int ks = s2_ks(v), tm = s2_tm(v), stages = d.cin / 32 / ks;
        // 4 x 1 tiles only where a wavefront has two stages: with four (28x28x128 -> 256) the other tiles or the implicit GEMM are as fast
        // or faster at 156 of 167 sizes (by 46 % at most) and slower by 6 % at most
        if (!s2tile_fits(d, d1, v) || !s2tile_shape(d, tm, &t) || (v == 2 && stages > 2)) continue;
        const double mb = 2e-6 * ((double)d.n * d.h * d.w * d.cin + 10.0 * d.cin * d.cout + 2.0 * d.n * out_dim(d.h, 3, 2, 1) * out_dim(d.w, 3, 2, 1) * d.cout);
        const long long items = (ks == 2 ? t.gm : (t.gm + 1) / 2) * (d.cout / 128), per_die = (items + 7) / 8;
        const int cus_die = std::max(1, cus / 8), busiest = (int)((per_die + cus_die - 1) / cus_die);
        const double active = (double)std::min<long long>(items, cus) / 256;
        const double cost = v == 0 ? 6.5 + busiest * (2.7 + stages * 2.85) + 0.11 * mb
                          : v == 1 ? 7.5 + busiest * (3.5 + stages * (2.25 + 0.7 * active)) + 0.063 * mb
                          : v == 2 ? 4.6 + busiest / 2 * 8.2 + busiest % 2 * 5.2 + (busiest == 1 ? 4.0 * active : 0.0) + 0.126 * mb
                                   : 4.9 + busiest * (2.4 + stages * (1.75 + 0.6 * active)) + 0.058 * mb;
        // With fewer items every CU waits for cold weights: 6 images on 96 CUs, 48 items, 13.6 us against 10.3.  One 4 x 1 item on a CU
        // has nothing that covers for it either, the less the more CUs ask for weights (whole networks with the implicit GEMM / with this:
        // 20 images on 256 CUs 198.5 / 201.5 us, 19 on 160 214.7 / 217.8, 10 on 96 198.5 / 199.8; 8 on 64 200.7 / 199.8).
        if (items * 5 < cus * (v == 2 && busiest == 1 ? 4 : 3)) continue;
        // Each of two workgroups on a CU fetches the weights, and on the whole chip the launches after this one pay for it (56x56x64 -> 128, 128
        // images on 256 CUs, 4 x 1 / 7 x 1 tiles: traced 35.7 / 37.8 us, whole network 551.1 / 548.5).
        const double rank = cost + (v == 2 ? 0.2 * busiest * active : 0.0);
        if (rank < best) { best = rank; *cost_us = cost; *variant = v; }
    }
    return best < 1e30;
}

// Name as a profiler prints it.
const char* s2tile_variant_name(int v)
{
    static char buf[kS2tileVariants][48];
    if (v < 0 || v >= kS2tileVariants) return "?";
    snprintf(buf[v], 48, "conv_s2tile_kernel<%d, %d>", s2_tm(v), s2_ks(v));
    return buf[v];
}

template <int TM, int KS> static int launch_s2(const S2tileArgs& a, int grid, hipStream_t stream)
{
    static std::atomic<bool> raised{false};
    if (!raised) {
        SGPRS_HIP(hipFuncSetAttribute((const void*)conv_s2tile_kernel<TM, KS>, hipFuncAttributeMaxDynamicSharedMemorySize, s2_lds(TM)));
        raised = true;
    }
    SGPRS_LAUNCH((conv_s2tile_kernel<TM, KS>), dim3(grid), dim3(256), s2_lds(TM), stream, a);
    SGPRS_HIP(hipGetLastError());
    return SGPRS_OK;
}

int launch_conv_s2tile(const sgprs_conv_desc_t& d, int variant, const void* x, const void* fragments0, const float* scale0, const float* shift0, void* y0,
                       const sgprs_conv_desc_t& d1, const void* fragments1, const float* scale1, const float* shift1, void* y1, hipStream_t stream,
                       int cus, Profiler* prof)
{
    S2tileShape t;
    if (!s2tile_fits(d, d1, variant) || !s2tile_shape(d, s2_tm(variant), &t))
        return fail(SGPRS_ERR_INVALID_ARG, "internal: launch plan does not match the shape");
    const int ks = s2_ks(variant);
    S2tileArgs a;
    memset(&a, 0, sizeof(a));
    a.x = (const unsigned char*)x;
    a.w[0] = (const unsigned char*)fragments0; a.w[1] = (const unsigned char*)fragments1;
    a.y[0] = (unsigned char*)y0; a.y[1] = (unsigned char*)y1;
    a.scale[0] = scale0; a.scale[1] = scale1; a.shift[0] = shift0; a.shift[1] = shift1;
    a.relu[0] = d.relu; a.relu[1] = d1.relu;
    a.H = d.h; a.W = d.w; a.P = out_dim(d.h, 3, 2, 1); a.Q = out_dim(d.w, 3, 2, 1);
    a.x_bytes = (unsigned)((long long)d.n * d.h * d.w * d.cin * 2);
    a.y_bytes = (unsigned)((long long)d.n * a.P * a.Q * d.cout * 2);
    a.w_bytes[0] = (unsigned)((long long)d.cout * 9 * d.cin * 2);
    a.w_bytes[1] = (unsigned)((long long)d.cout * d.cin * 2);
    a.x_pitch = d.cin * 2; a.y_pitch = d.cout * 2;
    a.chunks = d.cin / 64; a.stages = 2 * a.chunks / ks;
    a.TH = t.th; a.TW = t.tw; a.PW = t.tw + 1; a.images = t.images;
    a.image_slots = t.slots / t.images; a.slots = t.slots;
    a.cb = (a.Q + t.tw - 1) / t.tw;
    a.tiles_image = (a.P + t.th - 1) / t.th * a.cb;
    a.gm = (int)t.gm; a.gm_groups = ks == 2 ? a.gm : (a.gm + 1) / 2; a.gn = d.cout / 128;
    a.slots_mul = s2_small_mul(a.image_slots); a.pw_mul = s2_small_mul(a.PW); a.tw_mul = s2_small_mul(a.TW); a.th_mul = s2_small_mul(a.TH);
    div_constants(a.tiles_image, &a.image_mul, &a.image_sh);
    div_constants(a.cb, &a.cb_mul, &a.cb_sh);
    div_constants(a.gn, &a.gn_mul, &a.gn_sh);
    const int per_die = (a.gm_groups * a.gn + 7) / 8, grid = 8 * std::max(1, std::min(cus / 8 * s2_workgroups(s2_tm(variant), ks), per_die));
    const double M = (double)d.n * a.P * a.Q;
    int rc;
    if (prof && prof->on && (rc = prof->begin(stream, kKindIgemmPair, kS2tileNames + variant, 2.0 * M * d.cout * 10 * d.cin,
                                              (double)a.x_bytes + a.w_bytes[0] + a.w_bytes[1] + 2.0 * a.y_bytes)))
        return rc;
    switch (variant) {
        case 0: rc = launch_s2<7, 1>(a, grid, stream); break;
        case 1: rc = launch_s2<7, 2>(a, grid, stream); break;
        case 2: rc = launch_s2<4, 1>(a, grid, stream); break;
        default: rc = launch_s2<4, 2>(a, grid, stream); break;
    }
    if (rc) return rc;
    if (prof && prof->on && (rc = prof->end(stream))) return rc;
    return SGPRS_OK;
}

}  // namespace sgprs
