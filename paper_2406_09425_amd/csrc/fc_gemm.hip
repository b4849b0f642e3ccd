// The fully connected layer for batches of 32 images and more:
// logits[n][o] = sum_c w[o][c] v[n][c] + b[o], v the pooled vectors in fp32.
//
// Memory and matrix work are both small here (512 x 1000 weights); what bounds the layer is how its
// operands get to the matrix cores.  Fragment-shaped loads (a row per lane) reach a quarter of the
// load path's rate and left a 4096-image layer at 55 us (bf16); one wavefront per output with
// register weights re-reads the pooled vectors for every four outputs (fp32: 60 us at 433 images).
// Here (avg-pool + FC on 256 CUs: 433 images fp32 46.7 -> 16.7 us, 4096 images fp32 364 -> 128; 1820 images
// bf16 on 48 CUs 220 -> 145), as in the convolution that splits K over wavefronts, every wavefront moves its
// own share of the inputs into an LDS ring of its own with loads that write LDS directly, multiplies them
// without a barrier, and the partial tiles meet in LDS at the end, added in a fixed order.
// fp32 weights: MFMA 16x16x4, in chains of eight products that are added as trees: the error against 64
// bits is that of a register FC with shuffle sums (512 inputs 8.6e-8 relative, 2048 inputs 9.9e-8 against
// 1.23e-7), where one chain per wavefront had 2.1e-7 and 4.1e-7 and took 10 to 20 % less time.  bf16
// weights: the fp32 pooled values go in as a bf16 head plus a bf16 remainder (two MFMA 16x16x32; products
// of two bf16 are exact in fp32, so what is lost is below 2^-17 of a value), split when the fragment is read.
#include "internal.h"

namespace sgprs {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// 8 consecutive fp32 values as bf16 heads and remainders.
__device__ __forceinline__ void split_bf16(const u32x4_t a, const u32x4_t b, u32x4_t* hi, u32x4_t* lo)
{
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const f32x2_t f = {__uint_as_float(p < 2 ? a[2 * p] : b[2 * p - 4]), __uint_as_float(p < 2 ? a[2 * p + 1] : b[2 * p - 3])};
        const unsigned h = __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2_t));
        const f32x2_t r = {f[0] - __uint_as_float(h << 16), f[1] - __uint_as_float(h & 0xffff0000u)};
        (*hi)[p] = h;
        (*lo)[p] = __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf16x2_t));
    }
}

// 16*TM images x 16*TN outputs per workgroup; k-tiles of 32 inputs, ring of NS stages per wavefront.
// cin is a multiple of 512 and cout of 4 (checked by the launcher); images and outputs past the end
// read zeros (the buffers are the tile's own rows, so operands of any size are addressed with 32-bit
// offsets) and are not stored.  (fp32: at most 256 registers, so that the MFMAs write plain vector registers
// and their sums need no copies.)
template <int DT, int TM, int TN, int NS, int NW>
__global__ __launch_bounds__(NW * 64, DT == SGPRS_F32 ? 2 : 1) void fc_gemm_kernel(const float* __restrict__ v, const unsigned char* __restrict__ w,
                                                                                   const float* __restrict__ bias, float* __restrict__ y,
                                                                                   int nimg, int cin, int cout)
{
    constexpr int BM = 16 * TM, BN = 16 * TN, WROW = DT == SGPRS_BF16 ? 64 : 128;
    constexpr int A_IT = BM / 8, B_IT = BN * WROW / 1024, LPS = A_IT + B_IT;
    constexpr int STAGE = BM * 128 + BN * WROW, SROW = BN + 4, SETS = DT == SGPRS_BF16 ? 1 : 2;
    static_assert((NS - 1) * LPS <= 63, "vmcnt range");
    static_assert(BM * SROW * 4 <= NS * STAGE, "a wavefront's partial tile fits its ring");
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = blockIdx.y * BM, o0 = blockIdx.x * BN;
    const int nkt = cin / (32 * NW), kt0 = wave * nkt;  // an even number of k-tiles
    unsigned char* ring = smem + wave * (NS * STAGE);

    // LDS slots hold swizzled 16-byte chunks, so that a fragment read meets no bank twice: slot s of a
    // 128-byte row holds chunk s ^ (row & 7), of a 64-byte row chunk s ^ ((row >> 1) & 3).
    const unsigned v_off = (unsigned)((lane >> 3) * cin * 4 + (((lane & 7) ^ (lane >> 3)) << 4));
    const unsigned w_off = DT == SGPRS_BF16 ? (unsigned)((lane >> 2) * cin * 2 + (((lane & 3) ^ ((lane >> 3) & 3)) << 4))
                                            : (unsigned)((lane >> 3) * cin * 4 + (((lane & 7) ^ (lane >> 3)) << 4));
    const float* v_rows = v + (size_t)n0 * cin;
    const unsigned char* w_rows = w + (size_t)o0 * cin * (WROW / 32);
    const int v_bytes = min(BM, nimg - n0) * cin * 4, w_bytes = min(BN, cout - o0) * cin * (WROW / 32);
    auto request = [&](int t, int slot) {
#if __HIP_DEVICE_COMPILE__  // the buffer-resource builtins exist in the device pass only
        typedef __attribute__((address_space(3))) void* lds_ptr_t;
        const bool live = t < nkt;  // past the share: descriptors of size 0, the count of requests stays
        const __amdgpu_buffer_rsrc_t w_rs = __builtin_amdgcn_make_buffer_rsrc((void*)w_rows, 0, live ? w_bytes : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t v_rs = __builtin_amdgcn_make_buffer_rsrc((void*)v_rows, 0, live ? v_bytes : 0, 0x00020000);
        unsigned char* st = ring + slot * STAGE;
#pragma unroll
        for (int i = 0; i < B_IT; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rs, (lds_ptr_t)(st + BM * 128 + i * 1024), 16, w_off + i * (1024 / WROW) * cin * (WROW / 32),
                                                     (kt0 + t) * WROW, 0, 0);
#pragma unroll
        for (int i = 0; i < A_IT; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(v_rs, (lds_ptr_t)(st + i * 1024), 16, v_off + i * 8 * cin * 4, (kt0 + t) * 128, 0, 0);
#endif
    };
#pragma unroll
    for (int s = 0; s < NS; ++s) request(s, s);

    f32x4_t acc[SETS][TM][TN];
#pragma unroll
    for (int s = 0; s < SETS; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[s][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int frow = lane & 15, fgrp = lane >> 4;
    auto v_chunk = [&](const unsigned char* st, int i, int c) { return *(const u32x4_t*)(st + (i * 16 + frow) * 128 + ((c ^ (frow & 7)) << 4)); };
    // fp32: the 32 products of a k-tile are four
    // chains of two MFMAs from zero, added as a tree, even and odd k-tiles apart.  The tree of output tile
    // ij runs between the MFMAs of the next tile, the last tile's in the next k-tile (at first it adds zeros).
    static_assert(DT == SGPRS_BF16 || TM * TN % 2 == 0, "the two sets of chains alternate");
    f32x4_t chain[2][4];
#pragma unroll
    for (int c = 0; c < 4; ++c) chain[1][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto add_chains = [&](int ij, int set, int step) {
        f32x4_t(&c)[4] = chain[ij & 1];
        if (step == 0) c[0] += c[1];
        else if (step == 1) c[2] += c[3];
        else if (step == 2) c[0] += c[2];
        else acc[set % SETS][ij / TN][ij % TN] += c[0];
    };
    int slot = 0;
    auto k_tile = [&](int t, auto odd) {
        __builtin_amdgcn_s_waitcnt(((NS - 1) * LPS & 15) | (((NS - 1) * LPS >> 4) << 14) | 0x0F70);
        __builtin_amdgcn_sched_barrier(0);
        const unsigned char* st = ring + slot * STAGE;
        u32x4_t a[TM][2], b[TN][2];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) a[i][h] = v_chunk(st, i, DT == SGPRS_BF16 ? 2 * fgrp + h : fgrp + 4 * h);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const unsigned char* wr = st + BM * 128 + (j * 16 + frow) * WROW;
            if constexpr (DT == SGPRS_BF16) {
                b[j][0] = *(const u32x4_t*)(wr + ((fgrp ^ ((frow >> 1) & 3)) << 4));
            } else {
                b[j][0] = *(const u32x4_t*)(wr + ((fgrp ^ (frow & 7)) << 4));
                b[j][1] = *(const u32x4_t*)(wr + (((fgrp + 4) ^ (frow & 7)) << 4));
            }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the stage may be overwritten
        __builtin_amdgcn_sched_barrier(0);
        request(t + NS, slot);
        __builtin_amdgcn_sched_barrier(0);
        if (++slot == NS) slot = 0;
        if constexpr (DT == SGPRS_BF16) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                u32x4_t part[2];
                split_bf16(a[i][0], a[i][1], &part[0], &part[1]);
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[0][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, b[j][0]),
                                                                            __builtin_bit_cast(bf16x8_t, part[p]), acc[0][i][j], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int ij = 0; ij < TM * TN; ++ij)
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int i = ij / TN, j = ij % TN;
                    f32x4_t& c = chain[ij & 1][k / 2];
                    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
                    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(b[j][k >> 2][k & 3]), __uint_as_float(a[i][k >> 2][k & 3]),
                                                             k % 2 ? c : zero, 0, 0, 0);
                    if (k % 2) add_chains(ij ? ij - 1 : TM * TN - 1, ij ? odd : odd + 1, k / 2);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
    };
    for (int t = 0; t < nkt; t += 2) {
        k_tile(t, std::integral_constant<int, 0>());
        k_tile(t + 1, std::integral_constant<int, 1>());
    }
    if constexpr (DT == SGPRS_F32)
#pragma unroll
        for (int k = 0; k < 4; ++k) add_chains(TM * TN - 1, 1, k);
    __builtin_amdgcn_s_waitcnt(0);  // the (empty) requests still in flight write LDS too
    __builtin_amdgcn_sched_barrier(0);

    // D layout: output 4*(lane/16) + e, image lane % 16
    float* part = (float*)ring;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
            *(f32x4_t*)(part + (i * 16 + frow) * SROW + j * 16 + fgrp * 4) = SETS == 1 ? acc[0][i][j] : acc[0][i][j] + acc[SETS - 1][i][j];
    __syncthreads();
    for (int item = tid; item < BM * BN / 4; item += NW * 64) {
        const int img = item / (BN / 4), c = (item % (BN / 4)) * 4, o = o0 + c;
        const float* src = (const float*)smem + img * SROW + c;
        f32x4_t p[NW], s;
#pragma unroll
        for (int q = 0; q < NW; ++q) p[q] = *(const f32x4_t*)(src + q * (NS * STAGE / 4));
        if constexpr (DT == SGPRS_BF16) {
            s = ((p[0] + p[1]) + p[2]) + p[3];
        } else {
#pragma unroll
            for (int d = 1; d < NW; d *= 2)
#pragma unroll
                for (int q = 0; q < NW; q += 2 * d) p[q] += p[q + d];
            s = p[0];
        }
        if (n0 + img >= nimg || o >= cout) continue;
        if (bias) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += bias[o + e];
        }
        float* dst = y + (size_t)(n0 + img) * cout + o;  // (the caller's logits need not be 16-byte aligned)
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[e] = s[e];
    }
}

template <int DT, int TM, int TN, int NS, int NW = 4>
static int launch_tile(const float* v, const void* w, const float* bias, float* y, int n, int cin, int cout, hipStream_t stream)
{
    constexpr int lds = NW * NS * (16 * TM * 128 + 16 * TN * (DT == SGPRS_BF16 ? 64 : 128));
    static std::atomic<bool> raised{false};
    if (!raised) {
        SGPRS_HIP(hipFuncSetAttribute((const void*)fc_gemm_kernel<DT, TM, TN, NS, NW>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        raised = true;
    }
    const dim3 grid((cout + 16 * TN - 1) / (16 * TN), (n + 16 * TM - 1) / (16 * TM));
    SGPRS_LAUNCH((fc_gemm_kernel<DT, TM, TN, NS, NW>), grid, dim3(NW * 64), lds, stream, v, (const unsigned char*)w, bias, y, n, cin, cout);
    SGPRS_HIP(hipGetLastError());
    return SGPRS_OK;
}

bool fc_gemm_applicable(int n, int cin, int cout)
{
    // fewer images leave most of a tile's columns empty, and their logits match the one-launch kernel's bit for bit
    return n >= 32 && cin % 512 == 0 && cout % 4 == 0;
}

// 64x64 tiles halve the traffic of 32x32 ones; they need enough images to occupy the partition, and in
// fp32, where they cost matrix time, more than half a tile of them (32 images of 2048 inputs on 8 CUs:
// 48 us with 32x32 tiles, 93 with 64x64).  Small fp32 tiles: eight wavefronts halve the chain of k-tiles
// where a CU gets one tile, beyond that two workgroups of four (64 images of 512 inputs on 256 CUs 7.8 and
// 8.4 us, 433 images 17.7 with four and 19.1 with eight).
int launch_fc_gemm(int dtype, const float* v, const void* w, const float* bias, float* y, int n, int cin, int cout, hipStream_t stream, int cus)
{
    const bool big = (long long)((cout + 63) / 64) * ((n + 63) / 64) >= cus && (dtype == SGPRS_BF16 || n > 32);
    if (dtype == SGPRS_BF16)
        return big ? launch_tile<SGPRS_BF16, 4, 4, 2>(v, w, bias, y, n, cin, cout, stream) : launch_tile<SGPRS_BF16, 2, 2, 3>(v, w, bias, y, n, cin, cout, stream);
    if (big) return launch_tile<SGPRS_F32, 4, 4, 2>(v, w, bias, y, n, cin, cout, stream);
    return (long long)((cout + 31) / 32) * ((n + 31) / 32) > cus ? launch_tile<SGPRS_F32, 2, 2, 2>(v, w, bias, y, n, cin, cout, stream)
                                                                : launch_tile<SGPRS_F32, 2, 2, 2, 8>(v, w, bias, y, n, cin, cout, stream);
}

}  // namespace sgprs
