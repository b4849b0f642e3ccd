// The fully connected layer for batches of 32 images and more:
// logits[n][o] = sum_c w[o][c] v[n][c] + b[o], v the pooled vectors in fp32.
//
// Memory and matrix work are both small here (512 x 1000 weights); what bounds the layer is how its
// operands get to the matrix cores.  Fragment-shaped loads (a row per lane) reach a quarter of the
// load path's rate and left a 4096-image layer at 55 us (bf16); one wavefront per output with
// register weights re-reads the pooled vectors for every four outputs (fp32: 60 us at 433 images).
// Here (avg-pool + FC: 433 images fp32 on 128 CUs 72 -> 21 us, 4096 images fp32 359 -> 114, 1820 images
// bf16 on 48 CUs 220 -> 145), as in the convolution that splits K over wavefronts, every wavefront moves its own quarter of
// the inputs into an LDS ring of its own with loads that write LDS directly, multiplies them without a
// barrier, and the four partial tiles meet in LDS at the end, added in wavefront order.
// fp32 weights: MFMA 16x16x4.  bf16 weights: the fp32 pooled values go in as a bf16 head plus a bf16
// remainder (two MFMA 16x16x32; products of two bf16 are exact in fp32, so what is lost is below
// 2^-17 of a value), split when the fragment is read.
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
// offsets) and are not stored.
template <int DT, int TM, int TN, int NS>
__global__ __launch_bounds__(256) void fc_gemm_kernel(const float* __restrict__ v, const unsigned char* __restrict__ w,
                                                      const float* __restrict__ bias, float* __restrict__ y, int nimg, int cin, int cout)
{
    constexpr int BM = 16 * TM, BN = 16 * TN, WROW = DT == SGPRS_BF16 ? 64 : 128;
    constexpr int A_IT = BM / 8, B_IT = BN * WROW / 1024, LPS = A_IT + B_IT;
    constexpr int STAGE = BM * 128 + BN * WROW, SROW = BN + 4;
    static_assert((NS - 1) * LPS <= 63, "vmcnt range");
    static_assert(BM * SROW * 4 <= NS * STAGE, "a wavefront's partial tile fits its ring");
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = blockIdx.y * BM, o0 = blockIdx.x * BN;
    const int nkt = cin >> 7, kt0 = wave * nkt;
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

    f32x4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int frow = lane & 15, fgrp = lane >> 4;
    auto v_chunk = [&](const unsigned char* st, int i, int c) { return *(const u32x4_t*)(st + (i * 16 + frow) * 128 + ((c ^ (frow & 7)) << 4)); };
    int slot = 0;
    for (int t = 0; t < nkt; ++t) {
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
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, b[j][0]),
                                                                            __builtin_bit_cast(bf16x8_t, part[p]), acc[i][j], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(b[j][h][u]), __uint_as_float(a[i][h][u]),
                                                                             acc[i][j], 0, 0, 0);
        }
    }
    __builtin_amdgcn_s_waitcnt(0);  // the (empty) requests still in flight write LDS too
    __builtin_amdgcn_sched_barrier(0);

    // D layout: output 4*(lane/16) + e, image lane % 16
    float* part = (float*)ring;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) *(f32x4_t*)(part + (i * 16 + frow) * SROW + j * 16 + fgrp * 4) = acc[i][j];
    __syncthreads();
    for (int item = tid; item < BM * BN / 4; item += 256) {
        const int img = item / (BN / 4), c = (item % (BN / 4)) * 4, o = o0 + c;
        const float* src = (const float*)smem + img * SROW + c;
        f32x4_t s = *(const f32x4_t*)src;
#pragma unroll
        for (int q = 1; q < 4; ++q) s += *(const f32x4_t*)(src + q * (NS * STAGE / 4));
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

template <int DT, int TM, int TN, int NS>
static int launch_tile(const float* v, const void* w, const float* bias, float* y, int n, int cin, int cout, hipStream_t stream)
{
    constexpr int lds = 4 * NS * (16 * TM * 128 + 16 * TN * (DT == SGPRS_BF16 ? 64 : 128));
    static std::atomic<bool> raised{false};
    if (!raised) {
        SGPRS_HIP(hipFuncSetAttribute((const void*)fc_gemm_kernel<DT, TM, TN, NS>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        raised = true;
    }
    const dim3 grid((cout + 16 * TN - 1) / (16 * TN), (n + 16 * TM - 1) / (16 * TM));
    SGPRS_LAUNCH((fc_gemm_kernel<DT, TM, TN, NS>), grid, dim3(256), lds, stream, v, (const unsigned char*)w, bias, y, n, cin, cout);
    SGPRS_HIP(hipGetLastError());
    return SGPRS_OK;
}

bool fc_gemm_applicable(int n, int cin, int cout)
{
    // fewer images leave most of a tile's columns empty, and their logits match the one-launch kernel's bit for bit
    return n >= 32 && cin % 512 == 0 && cout % 4 == 0;
}

// 64x64 tiles halve the traffic of 32x32 ones; they need enough images to occupy the partition.
int launch_fc_gemm(int dtype, const float* v, const void* w, const float* bias, float* y, int n, int cin, int cout, hipStream_t stream, int cus)
{
    const bool big = (long long)((cout + 63) / 64) * ((n + 63) / 64) >= cus;
    if (dtype == SGPRS_BF16)
        return big ? launch_tile<SGPRS_BF16, 4, 4, 2>(v, w, bias, y, n, cin, cout, stream) : launch_tile<SGPRS_BF16, 2, 2, 3>(v, w, bias, y, n, cin, cout, stream);
    return big ? launch_tile<SGPRS_F32, 4, 4, 2>(v, w, bias, y, n, cin, cout, stream) : launch_tile<SGPRS_F32, 2, 2, 2>(v, w, bias, y, n, cin, cout, stream);
}

}  // namespace sgprs
