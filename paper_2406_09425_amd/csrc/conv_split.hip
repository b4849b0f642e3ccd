// fp32 convolution on the bf16 matrix cores: implicit GEMM, K range split over the wavefronts of a workgroup.
//
// What bounds the fp32 layers of a batch is the fp32 matrix rate, a sixteenth of the bf16 one: 90 to 105 of
// 157 TFLOP/s were reached.  A float is the sum of three bf16 numbers (8 bits each; rounded, what that leaves
// rounded, and the rest, which is exact), and of the nine products of two such sums the three smallest stay
// below 2^-26 of the whole.  So six bf16 MFMAs, accumulated in fp32, take the place of eight fp32 MFMAs of twice
// the cycles each, and add up 32 products at a time where those add four: sums are rounded a fifth as often.
//   * Weights: a task keeps their planes in fragment order, one coalesced KiB from the L2 to registers each,
//     requested one k-tile (32 input channels of one tap) ahead; they never see the LDS.
//   * Pixels stay fp32 in memory.  A wavefront's ring of two k-tiles is filled by loads that write LDS directly;
//     a fragment is split (44 vector instructions) behind the 6 TN MFMAs of the one before.  A wavefront alone
//     on its SIMD issues an instruction only every 5 to 6 cycles, which would bound this loop; hence tiles of at most 256
//     registers, two wavefronts a SIMD, as two workgroups of four or, where tiles are few, one of eight.
//   * Partial tiles meet in LDS and are added in wavefront order.
// What leaves bf16's range of exponents (planes and products below 2^-126 may count as 0) costs a product at most 2^-122
// if weights are at most 2 and nothing of them is lost.  So a channel's weights are scaled by a power of two to a
// largest one of 1 to 2, exactly, and its scale the other way; layers where a channel's weights other than 0 lie more
// than 2^50 apart, or are not finite, keep the fp32 kernels.  K <= 4608 products then lose 2^-109 at most, 2^-29 of a
// sum of 2^-80.  A tile with a sum that is not finite, or nonzero and smaller, is multiplied again with the fp32
// MFMAs; so is one with a sum of 0 that reads a pixel value other than 0 below 2^-30 (above, no product is below 2^-80).
// That takes time (16 images on 256 CUs, us, layer 1 / the stride-2 block of layer 4): pixels around 1e-30 in every tile 32.6 -> 92.9 / 21.6 -> 54.2
// for the launch that reads them, pixels of 0 throughout 41.0 / 26.6, one infinity 34.4 / 44.4, filters decayed to 1e-25 none.
// Error relative to 64 bits, fp32 MFMAs in two to four chains / here: 56x56x64 1.6e-7 / 0.8e-7, 28x28x128 2.2e-7 /
// 1.0e-7, 14x14x256 3.0e-7 / 1.4e-7, 7x7x512 3.0e-7 / 1.9e-7; 40 random layers: half on average, 0.66 at most.
// 16 images on 256 CUs, us per launch inside the network, before / now: 56x56x64 40.6 / 31.0, 28x28x128 39.8 / 26.2,
// 14x14x256 36.3 / 25.2, 7x7x512 35.0 / 27.8, the three stride-2 blocks with their shortcuts 24.7 / 21.3, 28.3 / 18.3,
// 22.6 / 20.8.  With every SIMD busy the clock drops; 760 to 840 bf16 TFLOP/s is what the bf16 layers reach too.  The whole inference: 637.3 -> 488.3.  Tiles of 112 pixels (one wavefront a SIMD: 1.8 us per k-tile for 64 channels, 1.0 for the
// 64-pixel tile) and splitting the weights in the kernel (0.3 us more per k-tile) were slower.
#include <algorithm>
#include <utility>

#include "internal.h"
#include "tap_mask.h"

namespace sgprs {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kWeightRange = 50;

// Pixel and channel tiles (of 16), wavefronts that share the K range (tiles of 32 channels were never the best of a layer).
#define SGPRS_SPLIT_VARIANTS(X) X(0, 2, 4, 4) X(1, 4, 4, 4) X(2, 2, 4, 8) X(3, 4, 4, 8)
constexpr int kSplitShape[][3] = {
#define X(v, tm, tn, nw) {tm, tn, nw},
    SGPRS_SPLIT_VARIANTS(X)
#undef X
};
constexpr int kSplitVariants = sizeof(kSplitShape) / sizeof(kSplitShape[0]);

// One convolution.  Divisions m / d of 0 <= m < 2^31 are umulhi(2 m, mul) >> sh (see div_constants).
struct SplitArgs {
    const unsigned char* x;
    const unsigned char* w;
    unsigned char* y;
    const float* scale;
    const float* shift;
    const unsigned char* res;
    const unsigned char* planes;
    const float* plane_scale;          // scale for the sums of the planes' products
    unsigned x_bytes, w_bytes, planes_bytes;
    int H, W, Q, PQ, M, Cout;
    int taps, stride, pad;             // filter height and width
    int pixel_bytes, row_bytes, w_row_bytes;
    int ktiles, cin_tiles;
    unsigned pq_mul, q_mul, ct_mul, place_mul;
    int pq_sh, q_sh, ct_sh, place_sh;
    int gm, gn, die_cols, die_tiles;   // pixel tiles, channel tiles; see below
    int relu, unused[2];
};
struct SplitLaunch { SplitArgs p[2]; };

__device__ __forceinline__ int sp_div(int m, unsigned mul, int sh) { return (int)(__umulhi(2u * (unsigned)m, mul) >> sh); }
template <class T> __device__ __forceinline__ T sp_load(const void* p) { return *(const __attribute__((address_space(1))) T*)p; }
template <class T> __device__ __forceinline__ void sp_store(void* p, T v) { *(__attribute__((address_space(1))) T*)p = v; }
template <int N> __device__ __forceinline__ void sp_wait_vmcnt()
{
    static_assert(N <= 63, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
    __builtin_amdgcn_sched_barrier(0);
}

// A wavefront's LDS: its ring of two stages, which its partial tile (rows padded by four floats) replaces at the end.
constexpr int split_wave_bytes(int tm, int tn)
{
    const int ring = 2 * 16 * tm * 128, part = (16 * tm * (16 * tn + 4) * 4 + 1023) / 1024 * 1024;
    return ring > part ? ring : part;
}

// Operation o of 28 that split a row's eight floats: plane 0 is the value rounded to bf16, plane 1 what that
// leaves, rounded, plane 2 the rest, which has at most eight bits left.
constexpr int kSplitOps = 28;
__device__ __forceinline__ void split_op(u32x4_t (&d)[3], f32x4_t (&r)[2], int o)
{
#if __HIP_DEVICE_COMPILE__
    const int phase = o < 4 ? 0 : o < 12 ? 1 : o < 16 ? 2 : o < 24 ? 3 : 4;  // round, subtract, round, subtract, round
    if (phase % 2 == 0) {
        const int k = phase == 0 ? o : phase == 2 ? o - 12 : o - 24;
        const f32x2_t f = {r[k / 2][k % 2 * 2], r[k / 2][k % 2 * 2 + 1]};
        d[phase / 2][k] = __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2_t));
    } else {
        const int e = phase == 1 ? o - 4 : o - 16;
        const unsigned pair = d[phase / 2][e / 2];
        r[e / 4][e % 4] -= __uint_as_float(e % 2 ? pair & 0xffff0000u : pair << 16);
    }
#endif
}

// One tile of 16*TM pixels x 16*TN channels: pixel tile mt, channel tile nt.
template <int TM, int TN, int NW>
__device__ __forceinline__ void split_tile(const SplitArgs& a, int mt, int nt)
{
#if __HIP_DEVICE_COMPILE__
    constexpr int SETS = TM * TN > 8 ? 1 : 2;
    constexpr int BM = 16 * TM, BN = 16 * TN, A_IT = BM / 8;
    constexpr int STAGE = BM * 128, PART = split_wave_bytes(TM, TN);
    constexpr int SROW = BN + 4;  // padded scratch row, floats
    constexpr int ITEMS = BM * BN / 4, PER = (ITEMS + NW * 64 - 1) / (NW * 64);
    static_assert(NW * 64 % (BN / 4) == 0, "a thread's items share their channels");
    typedef __attribute__((address_space(3))) void* lds_ptr_t;

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = mt * BM, n0 = nt * BN;
    const int share = (int)((unsigned)a.ktiles / NW), extra = a.ktiles & (NW - 1);
    const int kt0 = wave * share + min(wave, extra), nkt = share + (wave < extra ? 1 : 0);
    unsigned char* ring = smem + wave * PART;
    int* found = (int*)(smem + NW * PART);  // see below

    // Weights of k-tile j of this wavefront's share: TN x 3 fragments, one coalesced KiB each, into set j % 2.
    u32x4_t pw[2][TN][3];
    auto load_w = [&](int j, int set) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.planes, 0, j < nkt ? (int)a.planes_bytes : 0, 0x00020000);
#pragma unroll
        for (int c = 0; c < TN; ++c)
#pragma unroll
            for (int p = 0; p < 3; ++p)
                pw[set][c][p] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16 + p * 1024, (((nt * TN + c) * a.ktiles) + kt0 + j) * 3072, 0);
    };
    load_w(0, 0);
    if (tid < 4) found[tid] = 0;

    // Pixels: row of instruction i is i*8 + lane/8; this lane's LDS slot (lane & 7) holds the global 16-byte
    // chunk (lane & 7) ^ (row & 7), which makes the fragment reads bank-conflict free.
    const int lrow = lane >> 3, chunk_off = ((lane & 7) ^ lrow) * 16;
    int a_base[A_IT];
    unsigned a_in[A_IT];  // filter rows (bits 0..) and columns (bits kTapMaskBits..) inside the image
#pragma unroll
    for (int i = 0; i < A_IT; ++i) {
        const int m = m0 + lrow + 8 * i;
        const int n = sp_div(m, a.pq_mul, a.pq_sh), rem = m - n * a.PQ;
        const int p = sp_div(rem, a.q_mul, a.q_sh), q = rem - p * a.Q;
        const int h0 = p * a.stride - a.pad, w0 = q * a.stride - a.pad;
        a_base[i] = (n * a.H + h0) * a.row_bytes + w0 * a.pixel_bytes + chunk_off;
        a_in[i] = (tap_mask(h0, a.H) | (tap_mask(w0, a.W) << kTapMaskBits)) & (unsigned)((m - a.M) >> 31);
    }
    int ic, ir, is;
    // Requests of k-tile number j of this wavefront's share, one instruction (8 rows) each; past the
    // share the descriptor has size 0: nothing is fetched, the count of outstanding requests stays.
    auto request = [&](int j, int slot) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, j < nkt ? (int)a.x_bytes : 0, 0x00020000);
        const int tap_off = ir * a.row_bytes + is * a.pixel_bytes;
        const unsigned need = (1u << ir) | (1u << kTapMaskBits << is);
#pragma unroll
        for (int i = 0; i < A_IT; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(ring + slot * STAGE + i * 8 * 128), 16,
                                                     (a_in[i] & need) == need ? (unsigned)(a_base[i] + tap_off) : 0x80000000u, ic * 128, 0, 0);
        if (++ic == a.cin_tiles) {
            ic = 0;
            if (++is == a.taps) { is = 0; ++ir; }
        }
    };
    const int tap0 = sp_div(kt0, a.ct_mul, a.ct_sh);
    auto first_tap = [&]() {
        ic = kt0 - tap0 * a.cin_tiles;
        ir = a.taps == 3 ? tap0 / 3 : tap0;
        is = a.taps == 3 ? tap0 - ir * 3 : 0;
    };
    first_tap();
    request(0, 0);
    request(1, 1);

    f32x4_t acc[SETS][TM][TN];
    auto clear = [&]() {
#pragma unroll
        for (int s = 0; s < SETS; ++s)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[s][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    clear();
    const int frow = lane & 15, fgrp = lane >> 4;
    const unsigned f_off = (unsigned)(frow * 128 + ((fgrp ^ (frow & 7)) << 4));  // floats 4g ..; floats 16 + 4g ..: chunk + 4, i.e. bit 6 flipped
    struct Raw { f32x4_t v[2]; };
    struct Planes { u32x4_t p[3]; };
    auto read_px = [&](int slot, int i) {
        const unsigned char* row = ring + slot * STAGE + i * 16 * 128;
        return Raw{{*(const f32x4_t*)(row + f_off), *(const f32x4_t*)(row + (f_off ^ 64u))}};
    };
    auto mfma = [&](f32x4_t& c, const u32x4_t& w, const u32x4_t& x) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, x), c, 0, 0, 0);
    };

    sp_wait_vmcnt<A_IT>();
    Raw rp[2];
    Planes pp[2];
    rp[0] = read_px(0, 0);
    rp[1] = read_px(0, 1);
#pragma unroll
    for (int o = 0; o < kSplitOps; ++o) split_op(pp[0].p, rp[0].v, o);
    // K-tile t, of parity B: pixel tile after pixel tile is multiplied while the next one is split and the one after
    // that read.  The weights of k-tile t + 1 are requested at its start, the pixels of t + 2 once those of t are read.
    auto tile = [&](int t, auto parity) {
        constexpr int B = decltype(parity)::value;
        load_w(t + 1, B ^ 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int g = B * TM + i;  // in pairs of k-tiles an even number
            if (i == TM - 2) {
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the stage may be overwritten
                sp_wait_vmcnt<TN * 3>();             // the pixels of t + 1: only its weights were requested later
                request(t + 2, B);
            }
            rp[g & 1] = i + 2 < TM ? read_px(B, i + 2) : read_px(B ^ 1, i + 2 - TM);
            __builtin_amdgcn_sched_barrier(0);
            // Products of planes p + q <= 2.  The largest ones have accumulators of their own or, where registers do not
            // allow that, a k-tile's products are summed from zero, the largest last: in one chain for all of them the
            // small ones would round the sum six times as often (error 1.4 times that of the fp32 MFMAs instead of half).
            constexpr int kP[6] = {0, 2, 1, 0, 1, 0}, kQ[6] = {2, 0, 1, 1, 0, 0}, N = 6 * TN;
            f32x4_t part[TN];
#pragma unroll
            for (int m = 0; m < N; ++m) {
                const int u = m / TN, j = m % TN;
                f32x4_t& c = SETS > 1 ? acc[u < 5 ? SETS - 1 : 0][i][j] : part[j];
                if (SETS == 1 && u == 0) c = f32x4_t{0.f, 0.f, 0.f, 0.f};
                mfma(c, pw[B][j][kP[u]], pp[g & 1].p[kQ[u]]);
#pragma unroll
                for (int o = m * kSplitOps / N; o < (m + 1) * kSplitOps / N; ++o) split_op(pp[(g + 1) & 1].p, rp[(g + 1) & 1].v, o);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (SETS == 1) {
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[0][i][j] += part[j];
            }
        }
    };
    for (int t = 0; t < nkt; t += 2) {
        tile(t, std::integral_constant<int, 0>());
        if (t + 1 < nkt) tile(t + 1, std::integral_constant<int, 1>());
    }

    const int c0 = n0 + (tid % (BN / 4)) * 4;
    for (bool exact = false;; exact = true) {
        __builtin_amdgcn_s_waitcnt(0);  // the (empty) requests still in flight write LDS too
        __builtin_amdgcn_sched_barrier(0);
        // the epilogue's operands arrive while the partial tiles are exchanged
        const f32x4_t sc = sp_load<f32x4_t>((exact ? a.scale : a.plane_scale) + c0), sh = sp_load<f32x4_t>(a.shift + c0);
        f32x4_t rres[PER];
#pragma unroll
        for (int v = 0; v < PER; ++v) {
            const int px = (tid + v * NW * 64) / (BN / 4);
            rres[v] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (a.res) rres[v] = sp_load<f32x4_t>(a.res + ((size_t)min(m0 + px, a.M - 1) * a.Cout + c0) * 4);
        }
        // D layout: channel 4*(lane/16) + e, pixel lane % 16.
        float* mine = (float*)ring;
#pragma unroll
        for (int ti = 0; ti < TM; ++ti)
#pragma unroll
            for (int tj = 0; tj < TN; ++tj) *(f32x4_t*)(mine + (ti * 16 + frow) * SROW + tj * 16 + fgrp * 4) = SETS > 1 ? acc[0][ti][tj] + acc[SETS - 1][ti][tj] : acc[0][ti][tj];
        __syncthreads();
        auto sum = [&](int px, int c) {
            const float* src = (const float*)smem + px * SROW + c;
            f32x4_t s = *(const f32x4_t*)src;
#pragma unroll
            for (int w = 1; w < NW; ++w) s += *(const f32x4_t*)(src + w * (PART / 4));
            return s;
        };
        unsigned least = ~0u, most = 0u;  // of the sums' magnitudes as whole numbers, twice, less one: 0 is the largest
#pragma unroll
        for (int v = 0; v < PER; ++v) {
            const int item = tid + v * NW * 64, px = item / (BN / 4), c = (item % (BN / 4)) * 4;
            if (ITEMS % (NW * 64) != 0 && item >= ITEMS) break;
            f32x4_t s = sum(px, c);
            if (m0 + px >= a.M) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned size = (__float_as_uint(s[e]) << 1) - 1;
                least = min(least, size);
                most = max(most, size);
            }
            s = s * sc + sh;
            s += rres[v];
            if (a.relu) {
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e] = fmaxf(s[e], 0.f);
            }
            sp_store(a.y + ((size_t)(m0 + px) * a.Cout + n0 + c) * 4, s);
        }
        if (exact) return;
        constexpr unsigned kInfinity = 0x7f800000u << 1, kSmallSum = 0x17800000u << 1, kSmallPixel = 0x30800000u << 1;
        if (most >= kInfinity - 1 || least < kSmallSum - 1) found[0] = 1;
        __syncthreads();
        if (!found[0]) return;
        // Rare: which of the two it is, a sum of 0 (of a channel that has weights) or one that the planes cannot hold.
#pragma nounroll
        for (int v = 0; v < PER; ++v) {
            const int item = tid + v * NW * 64, px = item / (BN / 4), c = (item % (BN / 4)) * 4;
            if ((ITEMS % (NW * 64) != 0 && item >= ITEMS) || m0 + px >= a.M) break;
            const f32x4_t s = sum(px, c);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned size = __float_as_uint(s[e]) << 1;
                if (size == 0 ? sc[e] != 0.f : size >= kInfinity || size < kSmallSum) found[size == 0 ? 2 : 1] = 1;
            }
        }
        __syncthreads();
        if (!found[1]) {
            if (!found[2]) return;
            // Sums of 0 are rare but where all pixels are 0, which this finds out in a part of the products' time.
            least = ~0u;
            first_tap();
            for (int t = 0; t < nkt; t += 2) {  // (past the share: zeros)
                request(t, 0);
                request(t + 1, 1);
                sp_wait_vmcnt<0>();
#pragma unroll
                for (int i = 0; i < 2 * TM; ++i) {
                    const Raw px = read_px(i / TM, i % TM);
#pragma unroll
                    for (int e = 0; e < 8; ++e) least = min(least, (__float_as_uint(px.v[e / 4][e % 4]) << 1) - 1);
                }
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the stages may be overwritten
                __builtin_amdgcn_sched_barrier(0);
            }
            if (least < kSmallPixel) found[3] = 1;
            __syncthreads();
            if (!found[3]) return;
        }
        clear();
        first_tap();
        const unsigned w_row = (unsigned)(n0 + frow) * a.w_row_bytes + fgrp * 16;
        const __amdgpu_buffer_rsrc_t w_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, (int)a.w_bytes, 0x00020000);
        for (int t = 0; t < nkt; ++t) {
            request(t, 0);
            f32x4_t w[TN][2];
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    w[j][h] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(w_rs, w_row + j * 16 * a.w_row_bytes + h * 64, (kt0 + t) * 128, 0));
            sp_wait_vmcnt<0>();
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const Raw px = read_px(0, i);
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[e / 4 % SETS][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[j][e / 4][e % 4], px.v[e / 4][e % 4], acc[e / 4 % SETS][i][j], 0, 0, 0);
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the stage may be overwritten
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#endif
}

// ---- weights in planes --------------------------------------------------------------
// Exponent of every output channel's largest weight, and the channel's scale with it (0 where all weights are 0);
// *unfit where the planes do not hold a channel's weights (see above) or that scale leaves the normal range.
__global__ __launch_bounds__(256) void weight_exponents_kernel(const f32x4_t* src, const float* scale, float* plane_scale, int* exponents, int* unfit, int quads)
{
    unsigned largest = 0u, least = ~0u;  // magnitudes as whole numbers; the least one but for 0, less one
    for (int i = threadIdx.x; i < quads; i += 256) {
        const f32x4_t v = src[(size_t)blockIdx.x * quads + i];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned bits = __float_as_uint(v[e]) & 0x7fffffffu;
            largest = max(largest, bits);
            least = min(least, bits - 1);
        }
    }
    __shared__ unsigned of_wave[4][2];
#pragma unroll
    for (int o = 32; o > 0; o /= 2) {
        largest = max(largest, (unsigned)__shfl_xor((int)largest, o));
        least = min(least, (unsigned)__shfl_xor((int)least, o));
    }
    if (threadIdx.x % 64 == 0) { of_wave[threadIdx.x / 64][0] = largest; of_wave[threadIdx.x / 64][1] = least; }
    __syncthreads();
    if (threadIdx.x) return;
    for (int w = 1; w < 4; ++w) { largest = max(largest, of_wave[w][0]); least = min(least, of_wave[w][1]); }
    int exponent = 0;
    float scaled = 0.f;
    if (largest >= 0x7f800000u) {
        *unfit = 1;
    } else if (largest) {
        exponent = ilogbf(__uint_as_float(largest));
        scaled = scale[blockIdx.x];
        const int scaled_exponent = scaled == 0.f ? 0 : ilogbf(scaled) + exponent;  // (an infinity's and a NaN's lie outside too)
        if (ilogbf(__uint_as_float(least + 1)) < exponent - kWeightRange || scaled_exponent < -126 || scaled_exponent > 126) *unfit = 1;
        scaled = ldexpf(scaled, exponent);
    }
    exponents[blockIdx.x] = exponent;
    plane_scale[blockIdx.x] = scaled;
}

// From [cout][tap][cin] fp32 to [cout / 16][tap][cin / 32][plane][lane][16 bytes]: lane l of a fragment holds, of
// channel l % 16, floats 4g .. 4g + 3 and 16 + 4g .. 16 + 4g + 3 of the 32, g = l / 16.
__global__ void split_weights_kernel(const f32x4_t* src, u32x4_t* dst, const int* exponents, int ktiles, int units)
{
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= units) return;
    const int lane = u & 63, rest = u >> 6, kt = rest % ktiles, row = rest / ktiles * 16 + (lane & 15);
    const f32x4_t* from = src + ((size_t)row * ktiles + kt) * 8 + (lane >> 4);
    f32x4_t r[2] = {from[0], from[4]};
    const int exponent = exponents[row];
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e / 4][e % 4] = ldexpf(r[e / 4][e % 4], -exponent);
    u32x4_t d[3];
#pragma unroll
    for (int o = 0; o < kSplitOps; ++o) split_op(d, r, o);
#pragma unroll
    for (int p = 0; p < 3; ++p) dst[((size_t)rest * 3 + p) * 64 + lane] = d[p];
}

static size_t plane_bytes(const sgprs_conv_desc_t& d)
{
    const long long bytes = 6ll * d.cout * d.r * d.s * d.cin;
    return is_igemm(d) && d.dtype == SGPRS_F32 && d.cout % 16 == 0 && bytes < (1ll << 31) ? (size_t)bytes : 0;
}

size_t split_weight_bytes(const sgprs_conv_desc_t& d) { return plane_bytes(d) ? plane_bytes(d) + d.cout * (sizeof(float) + sizeof(int)) : 0; }

int split_weights(const sgprs_conv_desc_t& d, const void* src, const float* scale, void* dst, int* unfit, hipStream_t stream)
{
    if (!split_weight_bytes(d)) return fail(SGPRS_ERR_INVALID_ARG, "internal: no planes for this shape");
    const int units = d.cout * d.r * d.s * (d.cin / 8);
    float* plane_scale = (float*)((unsigned char*)dst + plane_bytes(d));
    int* exponents = (int*)(plane_scale + d.cout);
    hipLaunchKernelGGL(weight_exponents_kernel, dim3(d.cout), dim3(256), 0, stream, (const f32x4_t*)src, scale, plane_scale, exponents, unfit, d.r * d.s * d.cin / 4);
    SGPRS_HIP(hipGetLastError());
    hipLaunchKernelGGL(split_weights_kernel, dim3((units + 255) / 256), dim3(256), 0, stream, (const f32x4_t*)src, (u32x4_t*)dst, exponents,
                       d.r * d.s * d.cin / 32, units);
    SGPRS_HIP(hipGetLastError());
    return SGPRS_OK;
}

// blockIdx.y selects the problem, as in conv_ksplit_kernel; so does the placement of tiles on dies.
template <int TM, int TN, int NW>
__global__ __launch_bounds__(NW * 64, 2) void conv_split_kernel(const SplitLaunch launch)
{
    SplitArgs a;
#if __HIP_DEVICE_COMPILE__
    typedef __attribute__((address_space(4))) const unsigned* arg_ptr_t;
    arg_ptr_t src = (arg_ptr_t)__builtin_amdgcn_kernarg_segment_ptr() + blockIdx.y * (sizeof(SplitArgs) / 4);
    unsigned words[sizeof(SplitArgs) / 4];
#pragma unroll
    for (unsigned i = 0; i < sizeof(SplitArgs) / 4; ++i) words[i] = src[i];
    static_assert(sizeof(SplitArgs) % 16 == 0, "pinned four words at a time");
#pragma unroll
    for (unsigned i = 0; i < sizeof(SplitArgs) / 4; i += 4)
        asm volatile("" : "+s"(words[i]), "+s"(words[i + 1]), "+s"(words[i + 2]), "+s"(words[i + 3]));
    __builtin_memcpy(&a, words, sizeof(a));
#else
    a = launch.p[0];
#endif
    const int die = blockIdx.x & 7, u = a.die_cols ? (int)(blockIdx.x >> 3) : die * a.die_tiles + (int)(blockIdx.x >> 3);
    const int cols = a.die_cols ? a.die_cols : a.gn;
    const int mt = sp_div(u, a.place_mul, a.place_sh), nt = u - mt * cols + die * a.die_cols;
    if (mt < a.gm) split_tile<TM, TN, NW>(a, mt, nt);
}

// Name as a profiler prints it.
const char* split_variant_name(int v)
{
    static char buf[kSplitVariants][64];
    if (v < 0 || v >= kSplitVariants) return "?";
    snprintf(buf[v], 64, "conv_split_kernel<%d, %d, %d>", kSplitShape[v][0], kSplitShape[v][1], kSplitShape[v][2]);
    return buf[v];
}

template <int TM, int TN, int NW> static int launch_sp(const SplitLaunch& l, int slots, int problems, hipStream_t stream)
{
    constexpr int lds = NW * split_wave_bytes(TM, TN) + 16;
    static std::atomic<bool> raised{false};
    if (!raised) {
        SGPRS_HIP(hipFuncSetAttribute((const void*)conv_split_kernel<TM, TN, NW>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        raised = true;
    }
    SGPRS_LAUNCH((conv_split_kernel<TM, TN, NW>), dim3(slots, problems), dim3(NW * 64), lds, stream, l);
    SGPRS_HIP(hipGetLastError());
    return SGPRS_OK;
}

// Up to 512 input channels: what the error was measured for.
bool split_fits(const sgprs_conv_desc_t& d, int v)
{
    return is_igemm(d) && d.dtype == SGPRS_F32 && d.cin <= 512 && v >= 0 && v < kSplitVariants && split_weight_bytes(d) && d.cout % (16 * kSplitShape[v][1]) == 0;
}

// Estimated time (us) of a launch.  A tile takes a fixed part (start, pixel arithmetic, exchange, epilogue) and a
// time per k-tile of a wavefront; four-wavefront workgroups run two to a CU, so that rounds overlap, and with most
// of the chip in them the clock drops: 1.4 times that per k-tile where every CU of 256 has several.  Fitted to
// the network's layers, 2 to 16 images, 64 to 256 CUs (within 10 % but for a few at 15 %).  Whole inferences with and
// without this kernel, 1 to 16 images on 8 to 256 CUs: 0.61 to 1.001 of the time (one image on 8 CUs 749 us against 1135).
double split_cost(const sgprs_conv_desc_t& d, int v, int cus, const sgprs_conv_desc_t* d1)
{
    static const double kFixed[kSplitVariants] = {4.3, 5.4, 4.3, 6.4}, kPerKtile[kSplitVariants] = {0.72, 0.985, 1.155, 1.64};
    const int tm = kSplitShape[v][0], tn = kSplitShape[v][1], nw = kSplitShape[v][2];
    const long long M = (long long)d.n * out_dim(d.h, d.r, d.stride, d.pad) * out_dim(d.w, d.s, d.stride, d.pad);
    const long long wgs = (M + 16 * tm - 1) / (16 * tm) * (d.cout / (16 * tn)), rounds = (wgs + cus - 1) / cus;
    const double per_cu = (double)wgs / cus, chip = std::min(cus, 256) / 256.0;
    auto share = [&](const sgprs_conv_desc_t& p) { return (p.r * p.s * p.cin / 32 + nw - 1) / nw * kPerKtile[v]; };  // the longest
    const double t0 = share(d), t1 = d1 ? share(*d1) : 0.0;
    if (nw == 8) {
        const double part = kFixed[v] - 1.7, slow = 1.0 + 0.15 * chip;
        return 1.0 + rounds * (part + t0 * slow) + (d1 ? rounds * (part + t1 * slow) : 0.0);
    }
    const double busy = (1.0 + 0.4 * chip), each = 1.5 * chip * tm * tn / 16;
    const double one = t0 * (1.0 + 0.25 * chip * std::min(1.0, per_cu) + 0.8 * (rounds - 1)), all = per_cu * (t0 * busy + each);
    return kFixed[v] + std::max(one, all) + (d1 ? std::max(1.0, per_cu) * (t1 * busy + each) : 0.0);
}

int split_num_variants() { return kSplitVariants; }

bool plan_split(const sgprs_conv_desc_t& d, int cus, int* variant, double* cost_us)
{
    double best = 1e30;
    for (int v = 0; v < kSplitVariants; ++v) {
        if (!split_fits(d, v)) continue;
        const double cost = split_cost(d, v, cus, nullptr);
        if (cost < best) { best = cost; *variant = v; *cost_us = cost; }
    }
    return best < 1e30;
}

static int fill(const sgprs_conv_desc_t& d, int variant, const void* x, const void* w, const void* planes, const float* scale, const float* shift,
                const void* res, void* y, SplitArgs* out)
{
    const int* t = kSplitShape[variant];
    SplitArgs& a = *out;
    memset(&a, 0, sizeof(a));
    a.x = (const unsigned char*)x; a.w = (const unsigned char*)w; a.y = (unsigned char*)y;
    a.scale = scale; a.shift = shift; a.res = (const unsigned char*)res; a.planes = (const unsigned char*)planes;
    a.plane_scale = (const float*)(a.planes + plane_bytes(d));
    const int P = out_dim(d.h, d.r, d.stride, d.pad);
    a.H = d.h; a.W = d.w; a.Cout = d.cout; a.Q = out_dim(d.w, d.s, d.stride, d.pad);
    a.taps = d.r; a.stride = d.stride; a.pad = d.pad; a.relu = d.relu;
    a.PQ = P * a.Q; a.M = d.n * a.PQ;
    a.cin_tiles = d.cin / 32; a.ktiles = d.r * d.s * a.cin_tiles;
    a.pixel_bytes = d.cin * 4; a.row_bytes = d.w * d.cin * 4; a.w_row_bytes = a.ktiles * 128;
    div_constants(a.PQ, &a.pq_mul, &a.pq_sh);
    div_constants(a.Q, &a.q_mul, &a.q_sh);
    div_constants(a.cin_tiles, &a.ct_mul, &a.ct_sh);
    const long long xb = (long long)d.n * d.h * d.w * d.cin * 4, wb = (long long)d.cout * d.r * d.s * d.cin * 4;
    if (!split_fits(d, variant) || d.r > 3 || d.s != d.r || d.cin % 32 || xb >= (1ll << 31) || wb >= (1ll << 31))
        return fail(SGPRS_ERR_INVALID_ARG, "internal: launch plan does not match the shape");
    a.x_bytes = (unsigned)xb; a.w_bytes = (unsigned)wb; a.planes_bytes = (unsigned)plane_bytes(d);
    a.gm = (a.M + 16 * t[0] - 1) / (16 * t[0]); a.gn = d.cout / (16 * t[1]);
    a.die_cols = a.gn % 8 == 0 ? a.gn / 8 : 0;
    a.die_tiles = (a.gm * a.gn + 7) / 8;
    div_constants(a.die_cols ? a.die_cols : a.gn, &a.place_mul, &a.place_sh);
    return SGPRS_OK;
}

// d1 == NULL: one convolution; otherwise the block's 1x1 shortcut goes along (no residuals then).
int launch_conv_split(const sgprs_conv_desc_t& d, int variant, const void* x, const void* w, const void* planes, const float* scale, const float* shift,
                      const void* res, void* y, const sgprs_conv_desc_t* d1, const void* w1, const void* planes1, const float* scale1,
                      const float* shift1, void* y1, hipStream_t stream, Profiler* prof)
{
    if (variant < 0 || variant >= kSplitVariants) return fail(SGPRS_ERR_INVALID_ARG, "bad variant %d", variant);
    SplitLaunch l;
    memset(&l, 0, sizeof(l));
    SplitArgs &a0 = l.p[0], &a1 = l.p[1];
    int rc;
    if ((rc = fill(d, variant, x, w, planes, scale, shift, res, y, &a0))) return rc;
    double flops = 2.0 * a0.M * d.cout * (double)d.r * d.s * d.cin;
    double bytes = ((double)d.n * d.h * d.w * d.cin + (double)d.cout * d.r * d.s * d.cin + (double)a0.M * d.cout * (res ? 2 : 1)) * 4.0;
    if (d1) {
        if ((rc = fill(*d1, variant, x, w1, planes1, scale1, shift1, nullptr, y1, &a1))) return rc;
        if (a1.gm != a0.gm || a1.gn != a0.gn) return fail(SGPRS_ERR_INVALID_ARG, "internal: paired convolutions of different output shapes");
        flops += 2.0 * a1.M * d1->cout * (double)d1->r * d1->s * d1->cin;
        bytes += ((double)d1->cout * d1->r * d1->s * d1->cin + (double)a1.M * d1->cout) * 4.0;
    }
    if (prof && prof->on && (rc = prof->begin(stream, d1 ? kKindIgemmPair : kKindIgemm, kSplitNames + variant, flops, bytes))) return rc;
    const int slots = a0.die_tiles * 8;  // a multiple of 8 either way
    switch (variant) {
#define X(v, tm, tn, nw) case v: rc = launch_sp<tm, tn, nw>(l, slots, d1 ? 2 : 1, stream); break;
        SGPRS_SPLIT_VARIANTS(X)
#undef X
    }
    if (rc) return rc;
    if (prof && prof->on && (rc = prof->end(stream))) return rc;
    return SGPRS_OK;
}

}  // namespace sgprs
