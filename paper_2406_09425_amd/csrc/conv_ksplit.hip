// Convolution for problems with few output tiles: implicit GEMM whose K range
// is split over the wavefronts of one workgroup.
//
// What bounds a one-image layer is latency, not arithmetic: a 14x14x256 layer
// is 0.23 GFLOP, 0.1 us of the chip's matrix rate, but it used to take two
// dependent launches (split-K over workgroups, then a pass that adds the
// slices).  Here a workgroup owns a small output tile and the whole K range:
//   * each wavefront owns a contiguous share of the k-tiles (128 bytes of one
//     filter tap per row) and a ring of NS stages in LDS of its own; it fills
//     the ring with loads that write LDS directly and waits on its own vmcnt,
//     so the k-loop has no barrier and up to 144 KB per compute unit are in
//     flight at once (144 KB arrive in 1.1 us from the L2; one wavefront
//     instruction moves 8 rows x 128 bytes, because fragment-shaped loads, a
//     row per lane, run at a quarter of that rate: 4.0 us);
//   * the weights are the row operand of the MFMA, so a lane ends up with four
//     consecutive channels of one pixel;
//   * the partial tiles meet in LDS and are added in wavefront order (bitwise
//     reproducible), then scale/shift, residual and ReLU in fp32.
// Measured in a chain of launches (us each, launch included; before: implicit GEMM with split-K
// over workgroups, or the LDS-patch kernel), bf16, one image on 256 CUs: 56x56x64 3.6 (5.8),
// 28x28x128 3.7 (7.4), 14x14x256 3.8 (9.9), 7x7x512 5.0 (11.3), 28x28x128 -> 256/2 3.4 (10.1); fp32
// with a residual 6.3 / 5.7 / 6.1 / 9.0 (10.2 / 11.4 / 13.1 / 14.8), and at 16 images 40 / 38 / 40 for the last three
// (50 with split-K; 27 at the fp32 matrix rate with the 12 % idle CUs of their tile counts).  An empty kernel in such a chain takes 1.8.
//
// Small tiles trade traffic for parallelism, so this kernel is for launches
// that cannot fill the partition with big tiles; see plan_ksplit for the line.
#include <algorithm>
#include <utility>

#include "internal.h"
#include "tap_mask.h"

namespace sgprs {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

// Pixel and channel tiles (of 16), ring stages.  The set covers the best of sixteen shapes (four and
// eight wavefronts among them) within 1 % over 171 measured launches (nine layers, 1..16 images,
// 8..256 CUs, both types): 16x16 and 16x32 for launches that leave CUs idle, 7-row tiles for fp32
// maps whose pixel count is a multiple of 7 * 16.
#define SGPRS_KSPLIT_VARIANTS(X) \
    X(0, 1, 1, 4) X(1, 1, 2, 3) X(2, 2, 2, 2) X(3, 4, 2, 2) X(4, 2, 4, 3) X(5, 4, 4, 2) X(6, 7, 1, 2) X(7, 7, 2, 2)
constexpr int kKsplitWaves = 4;
constexpr int kKsplitShape[][3] = {
#define X(v, tm, tn, ns) {tm, tn, ns},
    SGPRS_KSPLIT_VARIANTS(X)
#undef X
};
constexpr int kKsplitVariants = sizeof(kKsplitShape) / sizeof(kKsplitShape[0]);

// One convolution.  Divisions m / d of 0 <= m < 2^31 are umulhi(2 m, mul) >> sh (see div_constants).
struct KsplitArgs {
    const unsigned char* x;
    const unsigned char* w;
    unsigned char* y;
    const float* scale;
    const float* shift;
    const unsigned char* res;
    unsigned x_bytes, w_bytes;
    int H, W, Q, PQ, M, Cout;
    int taps, stride, pad;             // filter height and width
    int pixel_bytes, row_bytes, w_row_bytes;
    int ktiles, cin_tiles;
    unsigned pq_mul, q_mul, ct_mul, place_mul;
    int pq_sh, q_sh, ct_sh, place_sh;
    int gm, gn, die_cols, die_tiles;   // pixel tiles, channel tiles; see ks_place
    int relu, unused[3];
};
struct KsplitLaunch { KsplitArgs p[2]; };

__device__ __forceinline__ int ks_div(int m, unsigned mul, int sh) { return (int)(__umulhi(2u * (unsigned)m, mul) >> sh); }

// The pointers come out of the argument words as plain numbers: say that they are global addresses.
template <class T> __device__ __forceinline__ T load_global(const void* p) { return *(const __attribute__((address_space(1))) T*)p; }
template <class T> __device__ __forceinline__ void store_global(void* p, T v) { *(__attribute__((address_space(1))) T*)p = v; }

// At most N vector memory operations outstanding.
template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N <= 63, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
    __builtin_amdgcn_sched_barrier(0);
}
template <class F, int... I> __device__ __forceinline__ void for_each_stage(F f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>()), ...);
}

// One tile of 16*TM pixels x 16*TN channels: pixel tile mt, channel tile nt.
// SETS accumulator sets: the error of a sum grows with the square root of the length of its chains
// (each product is added and rounded in turn), so fp32 keeps the halves of a k-tile apart, and with
// SETS = 4 even and odd k-tiles too; the sets are added at the end (relative to 64 bits, one image,
// 14x14x256 and 7x7x512: 3.0e-7 each with 2 and 4 sets, 4.2e-7 and 5.8e-7 with one, 3.0e-7 and 3.1e-7
// for the implicit GEMM with K split over workgroups).
template <int DT, int TM, int TN, int NS, int SETS>
__device__ __forceinline__ void ksplit_tile(const KsplitArgs& a, int mt, int nt)
{
    constexpr int NW = kKsplitWaves;
    constexpr int ES = DT == SGPRS_BF16 ? 2 : 4;
    constexpr int BM = 16 * TM, BN = 16 * TN;
    constexpr int A_IT = BM / 8, B_IT = BN / 8, LPS = A_IT + B_IT;
    constexpr int STAGE = (BM + BN) * 128;
    constexpr int SROW = BN + 4;  // padded scratch row, floats
    // fp32 MFMAs take eight times the cycles of bf16 ones: their k-loop is worth a software pipeline
    // in every tile shape, the bf16 one only where a k-tile has 16 or more MFMAs
    constexpr bool PIPELINED = DT == SGPRS_F32 || TM * TN >= 8;
    constexpr int ITEMS = BM * BN / 4, PER = (ITEMS + NW * 64 - 1) / (NW * 64);
    static_assert((NS - 1) * LPS <= 63, "vmcnt range");
    static_assert(BM * SROW * 4 <= NS * STAGE, "a wavefront's partial tile fits its ring");

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = mt * BM, n0 = nt * BN;
    const int share = (int)((unsigned)a.ktiles / NW), extra = a.ktiles & (NW - 1);
    const int kt0 = wave * share + min(wave, extra), nkt = share + (wave < extra ? 1 : 0);
    unsigned char* ring = smem + wave * (NS * STAGE);

    // Row of instruction i: i*8 + lane/8; this lane's LDS slot (lane & 7) holds the global 16-byte
    // chunk (lane & 7) ^ (row & 7), which makes the fragment reads bank-conflict free.
    const int lrow = lane >> 3, chunk_off = ((lane & 7) ^ lrow) * 16;
    const unsigned b_off = (unsigned)((n0 + lrow) * a.w_row_bytes + chunk_off);
    // Requests of k-tile number j of this wavefront's share, one instruction (8 rows) each; past the
    // share the descriptor has size 0: nothing is fetched, the count of outstanding requests stays
    // the same for every wavefront.
    auto request_w = [&](int j, int slot, int i) {
#if __HIP_DEVICE_COMPILE__  // the buffer-resource builtins exist in the device pass only
        typedef __attribute__((address_space(3))) void* lds_ptr_t;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, j < nkt ? (int)a.w_bytes : 0, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(ring + slot * STAGE + (BM + i * 8) * 128), 16, b_off + i * 8 * a.w_row_bytes,
                                                 (kt0 + j) * 128, 0, 0);
#endif
    };
    // A share that fits the ring is requested at once, the weights before the pixel arithmetic.
    const bool at_once = share < NS;
    if (at_once) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int i = 0; i < B_IT; ++i) request_w(s, s, i);
    }
    // The epilogue's operands come next, so that they are there long before it runs.
    u32x4_t rres[PER];
    f32x4_t sc[PER], sh[PER];
#pragma unroll
    for (int v = 0; v < PER; ++v) {
        const int item = tid + v * NW * 64, px = item / (BN / 4), c = n0 + (item % (BN / 4)) * 4;
        rres[v] = u32x4_t{0u, 0u, 0u, 0u};
        sc[v] = sh[v] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (ITEMS % (NW * 64) == 0 || item < ITEMS) {
            sc[v] = load_global<f32x4_t>(a.scale + c);
            sh[v] = load_global<f32x4_t>(a.shift + c);
            if (a.res) {
                const unsigned char* rp = a.res + ((size_t)min(m0 + px, a.M - 1) * a.Cout + c) * ES;
                if constexpr (DT == SGPRS_BF16) {
                    const u32x2_t t = load_global<u32x2_t>(rp);
                    rres[v][0] = t[0]; rres[v][1] = t[1];
                } else {
                    rres[v] = load_global<u32x4_t>(rp);
                }
            }
        }
    }

    int a_base[A_IT];
    unsigned a_in[A_IT];  // filter rows (bits 0..) and columns (bits kTapMaskBits..) inside the image
#pragma unroll
    for (int i = 0; i < A_IT; ++i) {
        const int m = m0 + lrow + 8 * i;
        const int n = ks_div(m, a.pq_mul, a.pq_sh), rem = m - n * a.PQ;
        const int p = ks_div(rem, a.q_mul, a.q_sh), q = rem - p * a.Q;
        const int h0 = p * a.stride - a.pad, w0 = q * a.stride - a.pad;
        a_base[i] = (n * a.H + h0) * a.row_bytes + w0 * a.pixel_bytes + chunk_off;
        a_in[i] = (tap_mask(h0, a.H) | (tap_mask(w0, a.W) << kTapMaskBits)) & (unsigned)((m - a.M) >> 31);
    }
    const int tap0 = ks_div(kt0, a.ct_mul, a.ct_sh);
    int ic = kt0 - tap0 * a.cin_tiles, ir = a.taps == 3 ? tap0 / 3 : tap0, is = a.taps == 3 ? tap0 - ir * 3 : 0;
    unsigned a_voff[A_IT];
    auto enter_tap = [&]() {
        const int tap_off = ir * a.row_bytes + is * a.pixel_bytes;
        const unsigned need = (1u << ir) | (1u << kTapMaskBits << is);
#pragma unroll
        for (int i = 0; i < A_IT; ++i) a_voff[i] = (a_in[i] & need) == need ? (unsigned)(a_base[i] + tap_off) : 0x80000000u;
    };
    enter_tap();
    auto request_x = [&](int j, int slot, int i) {
#if __HIP_DEVICE_COMPILE__
        typedef __attribute__((address_space(3))) void* lds_ptr_t;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, j < nkt ? (int)a.x_bytes : 0, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(ring + slot * STAGE + i * 8 * 128), 16, a_voff[i], ic * 128, 0, 0);
#endif
    };
    auto next_channel_tile = [&]() {
        if (++ic == a.cin_tiles) {
            ic = 0;
            if (++is == a.taps) { is = 0; ++ir; }
            enter_tap();
        }
    };
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (!at_once) {
#pragma unroll
            for (int i = 0; i < B_IT; ++i) request_w(s, s, i);
        }
#pragma unroll
        for (int i = 0; i < A_IT; ++i) request_x(s, s, i);
        next_channel_tile();
    }

    f32x4_t acc[SETS][TM][TN];
#pragma unroll
    for (int s = 0; s < SETS; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[s][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int frow = lane & 15, fgrp = lane >> 4;
    const unsigned f_off = (unsigned)(frow * 128 + ((fgrp ^ (frow & 7)) << 4));  // second half of the k-tile: chunk + 4, i.e. bit 6 flipped
    struct Fragments { u32x4_t px[TM], w[TN]; };
    auto read_px = [&](Fragments& f, int slot, int ks, int i) {
        f.px[i] = *(const u32x4_t*)(ring + slot * STAGE + i * 16 * 128 + (f_off ^ (ks << 6)));
    };
    auto read_w = [&](Fragments& f, int slot, int ks, int j) {
        f.w[j] = *(const u32x4_t*)(ring + slot * STAGE + (BM + j * 16) * 128 + (f_off ^ (ks << 6)));
    };
    constexpr int HALF = TM * TN * (DT == SGPRS_BF16 ? 1 : 4);  // MFMAs of half a k-tile
    auto mfma = [&](const Fragments& f, int m, int set) {
        const int u = m / (TM * TN), i = m % (TM * TN) / TN, j = m % TN;
        f32x4_t& c = acc[set % SETS][i][j];
        if constexpr (DT == SGPRS_BF16)
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f.w[j]), __builtin_bit_cast(bf16x8_t, f.px[i]), c, 0, 0, 0);
        else
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(f.w[j][u]), __uint_as_float(f.px[i][u]), c, 0, 0, 0);
    };
    if (at_once) {
        // k-tile st has landed once only the pixel rows of the later ones are outstanding
        for_each_stage([&](auto st) {
            if (st < nkt) {
                wait_vmcnt<(NS - 1 - st) * A_IT>();
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    Fragments f;
#pragma unroll
                    for (int i = 0; i < TM; ++i) read_px(f, st, ks, i);
#pragma unroll
                    for (int j = 0; j < TN; ++j) read_w(f, st, ks, j);
#pragma unroll
                    for (int m = 0; m < HALF; ++m) mfma(f, m, 2 * (st & 1) + ks);
                }
            }
        }, std::make_integer_sequence<int, NS>());
    } else if constexpr (!PIPELINED) {
        int st = 0;
        for (int t = 0; t < nkt; ++t) {
            wait_vmcnt<(NS - 1) * LPS>();
            Fragments f[2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int i = 0; i < TM; ++i) read_px(f[ks], st, ks, i);
#pragma unroll
                for (int j = 0; j < TN; ++j) read_w(f[ks], st, ks, j);
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the stage may be overwritten
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < B_IT; ++i) request_w(t + NS, st, i);
#pragma unroll
            for (int i = 0; i < A_IT; ++i) request_x(t + NS, st, i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int m = 0; m < HALF; ++m) mfma(f[ks], m, 0);
            next_channel_tile();
            if (++st == NS) st = 0;
        }
    } else {
        // Software pipeline: while k-tile t is multiplied, its stage (whose fragments are in registers)
        // is requested anew, and the fragments of k-tile t + 1 are read.  One request or read goes
        // behind every few MFMAs: in a burst they would hold up the wavefront's MFMAs.
        Fragments f[2][2];
        int st = 0;
        wait_vmcnt<(NS - 1) * LPS>();
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int i = 0; i < TM; ++i) read_px(f[0][ks], 0, ks, i);
#pragma unroll
            for (int j = 0; j < TN; ++j) read_w(f[0][ks], 0, ks, j);
        }
        // Tied accumulators: written through the builtin, the compiler renames them within the loop and
        // copies them back (30-50 moves per k-tile, each waiting for its MFMA: 36 instead of 31 us for
        // fp32 14x14x256 at 16 images).  The hazard recogniser does not see into the assembly: the
        // operands come from LDS reads, the first accumulators and the epilogue are fenced by s_nop.
        auto mfma_tied = [&](const Fragments& f, int m, int set) {
#if __HIP_DEVICE_COMPILE__
            const int u = m / (TM * TN), i = m % (TM * TN) / TN, j = m % TN;
            f32x4_t& c = acc[set % SETS][i][j];
            if constexpr (DT == SGPRS_BF16)
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(f.w[j]), "v"(f.px[i]));
            else
                asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+a"(c) : "v"(f.w[j][u]), "v"(f.px[i][u]));
#endif
        };
        auto pin_accumulators = [&]() {  // writes above and reads below stay there
#if __HIP_DEVICE_COMPILE__
#pragma unroll
            for (int s = 0; s < SETS; ++s)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[s][i][j]));
#endif
        };
        auto step = [&](int t, auto odd, Fragments (&cur)[2], Fragments (&nxt)[2]) {
            constexpr int READS = 2 * (TM + TN);
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the stage may be overwritten
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < HALF; ++m) {
                mfma_tied(cur[0], m, 2 * odd);
#pragma unroll
                for (int k = m * LPS / HALF; k < (m + 1) * LPS / HALF; ++k) {
                    if (k < B_IT) request_w(t + NS, st, k);
                    else request_x(t + NS, st, k - B_IT);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            next_channel_tile();
            if (++st == NS) st = 0;
            wait_vmcnt<(NS - 1) * LPS>();
#pragma unroll
            for (int m = 0; m < HALF; ++m) {
                mfma_tied(cur[1], m, 2 * odd + 1);
#pragma unroll
                for (int k = m * READS / HALF; k < (m + 1) * READS / HALF; ++k) {
                    const int ks = k / (TM + TN), q = k % (TM + TN);
                    if (q < TM) read_px(nxt[ks], st, ks, q);
                    else read_w(nxt[ks], st, ks, q - TM);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        pin_accumulators();
#if __HIP_DEVICE_COMPILE__
        asm volatile("s_nop 7");
#endif
        for (int t = 0; t < nkt; t += 2) {
            step(t, std::integral_constant<int, 0>(), f[0], f[1]);
            if (t + 1 < nkt) step(t + 1, std::integral_constant<int, 1>(), f[1], f[0]);
        }
#if __HIP_DEVICE_COMPILE__
        asm volatile("s_nop 15\n\ts_nop 15");
#endif
        pin_accumulators();
    }
    __builtin_amdgcn_s_waitcnt(0);  // the (empty) requests still in flight write LDS too
    __builtin_amdgcn_sched_barrier(0);

    // D layout: channel 4*(lane/16) + e, pixel lane % 16.
    float* part = (float*)ring;
#pragma unroll
    for (int ti = 0; ti < TM; ++ti)
#pragma unroll
        for (int tj = 0; tj < TN; ++tj) {
            f32x4_t c = acc[0][ti][tj];
            if constexpr (SETS == 2) c += acc[1][ti][tj];
            if constexpr (SETS == 4) c = (c + acc[1][ti][tj]) + (acc[2][ti][tj] + acc[3][ti][tj]);
            *(f32x4_t*)(part + (ti * 16 + frow) * SROW + tj * 16 + fgrp * 4) = c;
        }
    __syncthreads();
    const unsigned relu_floor = a.relu ? kReluFloor : kNoReluFloor;
#pragma unroll
    for (int v = 0; v < PER; ++v) {
        const int item = tid + v * NW * 64, px = item / (BN / 4), c = (item % (BN / 4)) * 4;
        if (ITEMS % (NW * 64) != 0 && item >= ITEMS) break;
        const float* src = (const float*)smem + px * SROW + c;
        f32x4_t s = *(const f32x4_t*)src;
#pragma unroll
        for (int w = 1; w < NW; ++w) s += *(const f32x4_t*)(src + w * (NS * STAGE / 4));
        if (m0 + px >= a.M) continue;
        s = s * sc[v] + sh[v];
        const size_t o = ((size_t)(m0 + px) * a.Cout + n0 + c) * ES;
        if constexpr (DT == SGPRS_BF16) {
            s[0] += __uint_as_float(rres[v][0] << 16); s[1] += __uint_as_float(rres[v][0] & 0xffff0000u);
            s[2] += __uint_as_float(rres[v][1] << 16); s[3] += __uint_as_float(rres[v][1] & 0xffff0000u);
            store_global(a.y + o, u32x2_t{pack_bf16x2_relu(s[0], s[1], relu_floor), pack_bf16x2_relu(s[2], s[3], relu_floor)});
        } else {
            s += __builtin_bit_cast(f32x4_t, rres[v]);
            if (a.relu) {
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e] = fmaxf(s[e], 0.f);
            }
            store_global(a.y + o, s);
        }
    }
}

// Workgroup b runs on die b % 8.  With a multiple of eight channel tiles a die keeps its own eighth
// of them (die_cols; its L2 then holds an eighth of the weights, fetched once, for all pixel tiles);
// otherwise a die takes a contiguous range of die_tiles tiles, a pixel tile's channel tiles together.
__device__ __forceinline__ bool ks_place(const KsplitArgs& a, int b, int* mt, int* nt)
{
    const int die = b & 7, t = b >> 3;
    const int u = a.die_cols ? t : die * a.die_tiles + t;
    const int cols = a.die_cols ? a.die_cols : a.gn;
    *mt = ks_div(u, a.place_mul, a.place_sh);
    *nt = u - *mt * cols + die * a.die_cols;
    return *mt < a.gm;
}

// blockIdx.y selects the problem: a block's first 3x3 convolution and its 1x1 shortcut, which read
// the same input and have the same output shape, share a launch.  The arguments are read as one
// batch of scalar loads from the kernel-argument segment: left to itself the compiler loads them
// piecemeal where they are used, a chain of scalar-cache misses before the first request.
template <int DT, int TM, int TN, int NS, int SETS>
__global__ __launch_bounds__(kKsplitWaves * 64) void conv_ksplit_kernel(const KsplitLaunch launch)
{
    KsplitArgs a;
#if __HIP_DEVICE_COMPILE__
    typedef __attribute__((address_space(4))) const unsigned* arg_ptr_t;
    arg_ptr_t src = (arg_ptr_t)__builtin_amdgcn_kernarg_segment_ptr() + blockIdx.y * (sizeof(KsplitArgs) / 4);
    unsigned words[sizeof(KsplitArgs) / 4];
#pragma unroll
    for (unsigned i = 0; i < sizeof(KsplitArgs) / 4; ++i) words[i] = src[i];
    static_assert(sizeof(KsplitArgs) % 16 == 0, "pinned four words at a time");
#pragma unroll
    for (unsigned i = 0; i < sizeof(KsplitArgs) / 4; i += 4)
        asm volatile("" : "+s"(words[i]), "+s"(words[i + 1]), "+s"(words[i + 2]), "+s"(words[i + 3]));
    __builtin_memcpy(&a, words, sizeof(a));
#else
    a = launch.p[0];
#endif
    int mt, nt;
    if (ks_place(a, blockIdx.x, &mt, &nt)) ksplit_tile<DT, TM, TN, NS, SETS>(a, mt, nt);
}

// Name as a profiler prints it: v = tile variant + 16 * dtype, + 32 for four accumulator sets.
const char* ksplit_variant_name(int v)
{
    static char buf[8][96];
    static int next = 0;
    if (v < 0 || (v & 15) >= kKsplitVariants || v >= 64) return "?";
    const int* t = kKsplitShape[v & 15];
    char* out = buf[next++ & 7];
    const int dtype = v >> 4 & 1;
    snprintf(out, 96, "conv_ksplit_kernel<%d, %d, %d, %d, %d>", dtype, t[0], t[1], t[2], v >= 32 ? 4 : dtype == SGPRS_BF16 ? 1 : 2);
    return out;
}

template <int DT, int TM, int TN, int NS, int SETS>
static int launch_ks(const KsplitLaunch& l, int slots, int problems, hipStream_t stream)
{
    constexpr int lds = kKsplitWaves * NS * (TM + TN) * 16 * 128;
    static std::atomic<bool> raised{false};
    if (!raised) {
        SGPRS_HIP(hipFuncSetAttribute((const void*)conv_ksplit_kernel<DT, TM, TN, NS, SETS>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        raised = true;
    }
    SGPRS_LAUNCH((conv_ksplit_kernel<DT, TM, TN, NS, SETS>), dim3(slots, problems), dim3(kKsplitWaves * 64), lds, stream, l);
    SGPRS_HIP(hipGetLastError());
    return SGPRS_OK;
}

// fp32 up to 768 input channels: beyond, even four accumulator sets leave chains whose error is larger
// than split-K's over workgroups (relative to 64 bits, 7x7 3x3 convolution: 768 channels 3.5e-7 against
// 3.7e-7, 1024 channels 4.1e-7 against 3.2e-7).
bool ksplit_fits(const sgprs_conv_desc_t& d, int v)
{
    return is_igemm(d) && (d.dtype == SGPRS_BF16 || d.cin <= 768) && v >= 0 && v < kKsplitVariants && d.cout % (16 * kKsplitShape[v][1]) == 0;
}

// Estimated time (microseconds) of a tile shape: launch, then rounds of workgroups, each a fixed
// part (start, pixel arithmetic, reduction), the traffic of its k-tiles at the 110 GB/s one CU gets
// out of the L2 with 64-144 KB in flight, and, behind the first filling of the rings, the matrix
// work.  Fitted to 1368 measurements (nine layers, 1..16 images, 8..256 CUs, both types): 8 % off
// rms, and its choice is 1.5 % slower than the best tile on average.  With the block's shortcut d1 in
// the same launch, the shortcut's workgroups first fill what the last round leaves idle (324 paired
// launches: 10 % off rms without refitting).
double ksplit_cost(const sgprs_conv_desc_t& d, int v, int cus, const sgprs_conv_desc_t* d1)
{
    const int es = (int)dtype_size(d.dtype);
    const int *t = kKsplitShape[v], bm = 16 * t[0], bn = 16 * t[1], lds = kKsplitWaves * t[2] * (bm + bn) * 128;
    const long long M = (long long)d.n * out_dim(d.h, d.r, d.stride, d.pad) * out_dim(d.w, d.s, d.stride, d.pad);
    const long long wgs = (M + bm - 1) / bm * (d.cout / bn), occ = lds <= 80 * 1024 ? 2 : 1, room = cus * occ;
    // one CU's time per FLOP; a bf16 k-tile's MFMAs are mostly hidden behind its traffic
    const double us_per_flop = d.dtype == SGPRS_BF16 ? 0.26 / 9.8e6 : 1.0 / 0.614e6;
    auto rounds = [&](const sgprs_conv_desc_t& p, long long n) {
        const int ktiles = p.r * p.s * p.cin * es / 128, kt = (ktiles + kKsplitWaves - 1) / kKsplitWaves * kKsplitWaves;  // the longest share decides
        const double traffic = (bm + bn) * 128.0 * kt / 110e3, ring = std::min(traffic, lds / 110e3);
        const double mfma = 2.0 * bm * bn * (128 / es) * kt * us_per_flop;
        auto round = [&](long long per_cu) {
            return 0.64 + 0.2 * t[0] + 0.00031 * bm * bn + std::max(per_cu * traffic, ring + per_cu * mfma * (per_cu > 1 ? 1.06 : 1.0));
        };
        const long long full = n / room, rest = n - full * room;
        return full * round(occ) + 0.12 * (full + (rest > 0) - 1) + (rest ? round((rest + cus - 1) / cus) : 0.0);
    };
    double cost = 1.5 + rounds(d, wgs);
    if (d1) {
        const long long left = wgs - (room - wgs % room) % room;
        if (left > 0) cost += rounds(*d1, left);
    }
    return cost;
}

int ksplit_num_variants() { return kKsplitVariants; }

bool plan_ksplit(const sgprs_conv_desc_t& d, int cus, int* variant, double* cost_us)
{
    double best = 1e30;
    for (int v = 0; v < kKsplitVariants; ++v) {
        if (!ksplit_fits(d, v)) continue;
        const double cost = ksplit_cost(d, v, cus, nullptr);
        if (cost < best) { best = cost; *variant = v; *cost_us = cost; }
    }
    return best < 1e30;
}

static int fill(const sgprs_conv_desc_t& d, int variant, const void* x, const void* w, const float* scale, const float* shift,
                const void* res, void* y, KsplitArgs* out)
{
    const int es = (int)dtype_size(d.dtype), kt_el = 128 / es;
    const int* t = kKsplitShape[variant];
    KsplitArgs& a = *out;
    memset(&a, 0, sizeof(a));
    a.x = (const unsigned char*)x; a.w = (const unsigned char*)w; a.y = (unsigned char*)y;
    a.scale = scale; a.shift = shift; a.res = (const unsigned char*)res;
    const int P = out_dim(d.h, d.r, d.stride, d.pad);
    a.H = d.h; a.W = d.w; a.Cout = d.cout; a.Q = out_dim(d.w, d.s, d.stride, d.pad);
    a.taps = d.r; a.stride = d.stride; a.pad = d.pad; a.relu = d.relu;
    a.PQ = P * a.Q; a.M = d.n * a.PQ;
    a.cin_tiles = d.cin / kt_el; a.ktiles = d.r * d.s * a.cin_tiles;
    a.pixel_bytes = d.cin * es; a.row_bytes = d.w * d.cin * es; a.w_row_bytes = a.ktiles * 128;
    div_constants(a.PQ, &a.pq_mul, &a.pq_sh);
    div_constants(a.Q, &a.q_mul, &a.q_sh);
    div_constants(a.cin_tiles, &a.ct_mul, &a.ct_sh);
    const long long xb = (long long)d.n * d.h * d.w * d.cin * es, wb = (long long)d.cout * d.r * d.s * d.cin * es;
    if (d.r > 3 || d.s != d.r || d.cin % kt_el || d.cout % (16 * t[1]) || xb >= (1ll << 31) || wb >= (1ll << 31))
        return fail(SGPRS_ERR_INVALID_ARG, "internal: launch plan does not match the shape");
    a.x_bytes = (unsigned)xb; a.w_bytes = (unsigned)wb;
    a.gm = (a.M + 16 * t[0] - 1) / (16 * t[0]); a.gn = d.cout / (16 * t[1]);
    a.die_cols = a.gn % 8 == 0 ? a.gn / 8 : 0;
    a.die_tiles = (a.gm * a.gn + 7) / 8;
    div_constants(a.die_cols ? a.die_cols : a.gn, &a.place_mul, &a.place_sh);
    return SGPRS_OK;
}

// d1 == NULL: one convolution; otherwise the block's 1x1 shortcut goes along (no residuals then).
int launch_conv_ksplit(const sgprs_conv_desc_t& d, int variant, const void* x, const void* w, const float* scale, const float* shift,
                       const void* res, void* y, const sgprs_conv_desc_t* d1, const void* w1, const float* scale1,
                       const float* shift1, void* y1, hipStream_t stream, Profiler* prof)
{
    if (variant < 0 || variant >= kKsplitVariants) return fail(SGPRS_ERR_INVALID_ARG, "bad variant %d", variant);
    KsplitLaunch l;
    memset(&l, 0, sizeof(l));
    KsplitArgs &a0 = l.p[0], &a1 = l.p[1];
    int rc;
    if ((rc = fill(d, variant, x, w, scale, shift, res, y, &a0))) return rc;
    const double es = (double)dtype_size(d.dtype);
    double flops = 2.0 * a0.M * d.cout * (double)d.r * d.s * d.cin;
    double bytes = ((double)d.n * d.h * d.w * d.cin + (double)d.cout * d.r * d.s * d.cin + (double)a0.M * d.cout * (res ? 2 : 1)) * es;
    if (d1) {
        if ((rc = fill(*d1, variant, x, w1, scale1, shift1, nullptr, y1, &a1))) return rc;
        if (a1.gm != a0.gm || a1.gn != a0.gn) return fail(SGPRS_ERR_INVALID_ARG, "internal: paired convolutions of different output shapes");
        flops += 2.0 * a1.M * d1->cout * (double)d1->r * d1->s * d1->cin;
        bytes += ((double)d1->cout * d1->r * d1->s * d1->cin + (double)a1.M * d1->cout) * es;
    }
    // two sets hold a chain to 288 products up to K = 2304, four up to 4608; split-K gave deep 1x1
    // convolutions shorter chains still (768 channels: 1.85e-7, with two sets here 1.86e-7)
    const int key = d.dtype * 16 + variant + (d.dtype == SGPRS_F32 && (a0.ktiles > 72 || (d.r == 1 && d.cin > 512)) ? 32 : 0);
    if (prof && prof->on && (rc = prof->begin(stream, d1 ? kKindIgemmPair : kKindIgemm, kKsplitNames + key, flops, bytes))) return rc;
    const int slots = a0.die_tiles * 8;  // a multiple of 8 either way
    switch (key) {
#define X(v, tm, tn, ns)                                                                          \
        case v: rc = launch_ks<SGPRS_F32, tm, tn, ns, 2>(l, slots, d1 ? 2 : 1, stream); break;      \
        case 32 + v: rc = launch_ks<SGPRS_F32, tm, tn, ns, 4>(l, slots, d1 ? 2 : 1, stream); break; \
        case 16 + v: rc = launch_ks<SGPRS_BF16, tm, tn, ns, 1>(l, slots, d1 ? 2 : 1, stream); break;
        SGPRS_KSPLIT_VARIANTS(X)
#undef X
    }
    if (rc) return rc;
    if (prof && prof->on && (rc = prof->end(stream))) return rc;
    return SGPRS_OK;
}

}  // namespace sgprs
