// 3x3 stride-1 convolution, bf16, for launches with at most one output tile per CU: the K range is split
// over the eight wavefronts of a workgroup, which share one copy of the input pixels that their tile needs.
//
// What bounds such a launch (timestamps of a one-image 14x14x256 layer, us): 1.3 between two launches, 0.35 until
// the kernel's arguments are there, then what a CU gets out of the L2, 64 bytes a clock (a request of 1 KiB
// takes 16 cycles to issue), and 0.7 for the reduction and the store.  The implicit-GEMM kernel that splits K
// the same way (conv_ksplit_kernel) fetches every pixel once per filter tap: 147 KiB for its 16x16 tile, half of
// it pixels.  Here the pixels (a rectangle of output pixels and its halo, all channels) are fetched once into
// LDS, so that larger tiles cost little more: 94 KiB for that tile, 196 instead of 295 for 64 pixels x 32
// channels.  The weights go through a ring of two halves in LDS per wavefront, requested without a barrier and
// awaited by counted vmcnt; partial tiles meet in LDS and are added in wavefront order.
// One image, us per launch in a chain, conv_ksplit_kernel / this one: 56x56x64 on 256 CUs 4.10 / 3.54, on 64 CUs
// 6.08 / 5.13; 28x28x128 on 64 CUs 5.77 / 4.79, on 32 CUs 7.21 / 6.26; 14x14x256 on 64 CUs 5.24 / 4.84, on 32 CUs
// 7.77 / 6.09; 7x7x512 on 256 CUs 5.25 / 4.83, on 32 CUs 7.20 / 6.38.  Two rounds of tiles a CU are slower than
// the LDS-patch kernel, fp32 (twice the bytes, sums in short chains) is no faster than conv_ksplit_kernel, and
// weights in fragment order straight to registers take as long as through the ring: none of these is built.
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace sgprs {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

// Pixel and channel tiles (of 16), k-tiles (128 bytes of one tap) in each half of a wavefront's ring.
#define SGPRS_KPATCH_VARIANTS(X) X(0, 1, 1, 3) X(1, 2, 1, 3) X(2, 2, 2, 1) X(3, 4, 2, 1) X(4, 4, 4, 1)
struct KpatchShape { int tm, tn, h; };
constexpr KpatchShape kKpatchShape[] = {
#define X(v, tm, tn, h) {tm, tn, h},
    SGPRS_KPATCH_VARIANTS(X)
#undef X
};
constexpr int kKpatchVariants = sizeof(kKpatchShape) / sizeof(kKpatchShape[0]);
constexpr int kKpatchWaves = 8, kLdsBytes = 160 * 1024;

// Divisions m / d of 0 <= m < 2^31 are umulhi(2 m, mul) >> sh (see div_constants), of the small numbers
// inside a patch (m * mul) >> 22 with 24-bit factors.
struct KpatchArgs {
    const unsigned char* x;
    const unsigned char* w;
    unsigned char* y;
    const float* scale;
    const float* shift;
    const unsigned char* res;
    unsigned x_bytes, w_bytes, y_bytes;
    int H, W, Q, NP, Cout;             // NP = images * output rows
    int pad, ktiles, cin_tiles;
    int pitch, row_bytes, image_bytes; // of x
    int units, patch_loads;            // 16-byte units of a pixel, KiB of the patch
    int TH, TW, PW, HE, multi;         // tile, patch width, patch rows of an image; multi: more than one image
    unsigned units_mul, pw_mul, tw_mul;
    unsigned he_mul, p_mul, ct_mul, cb_mul, place_mul;
    int he_sh, p_sh, ct_sh, cb_sh, place_sh;
    int swz_sh, swz_bits;
    int gm, gn, cb, die_cols, die_tiles;
    int relu, unused[1];
};
static_assert(sizeof(KpatchArgs) % 16 == 0, "pinned four words at a time");

__device__ __forceinline__ int kp_div(int m, unsigned mul, int sh) { return (int)(__umulhi(2u * (unsigned)m, mul) >> sh); }
__device__ __forceinline__ int kp_small_div(int m, unsigned mul) { return (int)((unsigned)__umul24((unsigned)m, mul) >> 22); }
template <class T> __device__ __forceinline__ T kp_load(const void* p) { return *(const __attribute__((address_space(1))) T*)p; }
template <class T> __device__ __forceinline__ void kp_store(void* p, T v) { *(__attribute__((address_space(1))) T*)p = v; }

// At most N vector memory operations outstanding.
template <int N> __device__ __forceinline__ void kp_wait_vmcnt()
{
    static_assert(N <= 63, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
    __builtin_amdgcn_sched_barrier(0);
}

// A wavefront's ring, which its partial tile (rows padded by four floats) replaces at the end.
constexpr int kp_ring_bytes(int tm, int tn, int h)
{
    const int ring = 2 * h * 16 * tn * 128, part = (16 * tm * (16 * tn + 4) * 4 + 1023) / 1024 * 1024;
    return ring > part ? ring : part;
}

// The arguments are read as one batch of scalar loads, as in conv_ksplit_kernel.
template <int TM, int TN, int H>
__global__ __launch_bounds__(kKpatchWaves * 64) void conv3x3_kpatch_kernel(const KpatchArgs launch)
{
    constexpr int NW = kKpatchWaves, BM = 16 * TM, BN = 16 * TN, B_IT = BN / 8;
    constexpr int STAGE = BN * 128, RING = kp_ring_bytes(TM, TN, H), PATCH = NW * RING;
    constexpr int SROW = BN + 4;  // padded scratch row, floats
    constexpr int ITEMS = BM * BN / 4, PER = (ITEMS + NW * 64 - 1) / (NW * 64);
    constexpr int OPERANDS = 2 + PER;  // epilogue loads
    static_assert(H <= 3 && H * B_IT + OPERANDS <= 63, "vmcnt range");
    static_assert(NW * 64 % (BN / 4) == 0, "a thread's items share their channels");

    KpatchArgs a;
#if __HIP_DEVICE_COMPILE__
    typedef __attribute__((address_space(4))) const unsigned* arg_ptr_t;
    arg_ptr_t src_args = (arg_ptr_t)__builtin_amdgcn_kernarg_segment_ptr();
    unsigned words[sizeof(KpatchArgs) / 4];
#pragma unroll
    for (unsigned i = 0; i < sizeof(KpatchArgs) / 4; ++i) words[i] = src_args[i];
#pragma unroll
    for (unsigned i = 0; i < sizeof(KpatchArgs) / 4; i += 4)
        asm volatile("" : "+s"(words[i]), "+s"(words[i + 1]), "+s"(words[i + 2]), "+s"(words[i + 3]));
    __builtin_memcpy(&a, words, sizeof(a));
#else
    a = launch;
#endif
    // Workgroup b runs on die b % 8; placement as in conv_ksplit_kernel.
    const int die = blockIdx.x & 7, u0 = a.die_cols ? (int)(blockIdx.x >> 3) : die * a.die_tiles + (int)(blockIdx.x >> 3);
    const int cols = a.die_cols ? a.die_cols : a.gn;
    const int mt = kp_div(u0, a.place_mul, a.place_sh), nt = u0 - mt * cols + die * a.die_cols;
    if (mt >= a.gm) return;

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = nt * BN;
    const int share = (int)((unsigned)a.ktiles / NW), extra = a.ktiles & (NW - 1);
    const int kt0 = wave * share + min(wave, extra), nkt = share + (wave < extra ? 1 : 0);
    unsigned char* ring = smem + wave * RING;

    // Weights: row of instruction i is i*8 + lane/8; this lane's LDS slot (lane & 7) holds the global 16-byte
    // chunk (lane & 7) ^ (row & 7).
    const int lrow = lane >> 3;
    const unsigned b_off = (unsigned)((n0 + lrow) * a.ktiles * 128 + ((lane & 7) ^ lrow) * 16);
    // Slot of a patch pixel's 16-byte unit: neighbouring pixels of one unit fall on different banks.
    auto swizzle = [&](int px) { return (int)__builtin_amdgcn_ubfe((unsigned)px, a.swz_sh, a.swz_bits); };
    auto request_w = [&](int j, int slot) {
#if __HIP_DEVICE_COMPILE__  // the buffer-resource builtins exist in the device pass only
        typedef __attribute__((address_space(3))) void* lds_ptr_t;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, (int)a.w_bytes, 0x00020000);
        if (j >= nkt) return;
#pragma unroll
        for (int i = 0; i < B_IT; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(ring + slot * STAGE + i * 1024), 16, b_off + i * 8 * a.ktiles * 128,
                                                     (kt0 + j) * 128, 0, 0);
#endif
    };
    // Everything but the last `later` k-tiles (at most H) and the `others` requested after them has landed.
    auto wait_for_half = [&](int later, auto others) {
        constexpr int O = decltype(others)::value;
        if (later >= H) kp_wait_vmcnt<H * B_IT + O>();
        else if (later <= 0) kp_wait_vmcnt<O>();
        else if (later == 1) kp_wait_vmcnt<(H > 1 ? B_IT : 0) + O>();
        else kp_wait_vmcnt<(H > 2 ? 2 * B_IT : 0) + O>();
    };
#pragma unroll
    for (int h = 0; h < H; ++h) request_w(h, h);

    // The patch: PW columns of rows E0 .. of the extended row space (every image with its halo rows).
    const int rb = a.cb > 1 ? kp_div(mt, a.cb_mul, a.cb_sh) : mt;
    const int g0 = rb * a.TH, q0 = (mt - rb * a.cb) * a.TW;
    auto extended = [&](int g) { return g + (a.multi ? kp_div(g, a.p_mul, a.p_sh) * 2 : 0); };
    const int E0 = extended(g0);
    for (int j = wave; j < a.patch_loads; j += NW) {
        const int u = j * 64 + lane, px = kp_small_div(u, a.units_mul), slot = u - (int)__umul24(px, a.units);
        const int pr = kp_small_div(px, a.pw_mul), pc = px - (int)__umul24(pr, a.PW);
        int row = E0 + pr, image = 0;
        if (a.multi) {
            const int n = kp_div(row, a.he_mul, a.he_sh);
            row -= n * a.HE;
            image = n * a.image_bytes;
        }
        const int hh = row - a.pad, ww = pc + q0 - a.pad;
        const bool ok = (unsigned)hh < (unsigned)a.H && (unsigned)ww < (unsigned)a.W;
        const unsigned off = (__umul24(hh, a.row_bytes) + image) + (__umul24(ww, a.pitch) + ((slot ^ swizzle(px)) << 4));
#if __HIP_DEVICE_COMPILE__
        typedef __attribute__((address_space(3))) void* lds_ptr_t;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, (int)a.x_bytes, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(smem + PATCH + j * 1024), 16, ok ? off : 0x80000000u, 0, 0, 0);
#endif
    }
#pragma unroll
    for (int h = 0; h < H; ++h) request_w(H + h, H + h);

    // While all that is on its way: the epilogue's operands (pixels past the image: out of bounds), which the
    // wait below counts ...
    const int c0 = n0 + (tid % (BN / 4)) * 4;
    const f32x4_t sc = kp_load<f32x4_t>(a.scale + c0), sh = kp_load<f32x4_t>(a.shift + c0);
    u32x2_t rres[PER];
    unsigned out_off[PER];
    bool live[PER];
#if __HIP_DEVICE_COMPILE__
    const __amdgpu_buffer_rsrc_t res_rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.res, 0, a.res ? (int)a.y_bytes : 0, 0x00020000);
#endif
#pragma unroll
    for (int v = 0; v < PER; ++v) {
        const int item = tid + v * NW * 64, px = item / (BN / 4);
        const int ty = kp_small_div(px, a.tw_mul), tx = px - ty * a.TW;
        live[v] = (ITEMS % (NW * 64) == 0 || item < ITEMS) & (ty < a.TH) & (g0 + ty < a.NP) & (q0 + tx < a.Q);
        const unsigned off = (unsigned)(((g0 + ty) * a.Q + q0 + tx) * a.Cout + c0) * 2u;
        out_off[v] = live[v] ? off : 0x80000000u;
#if __HIP_DEVICE_COMPILE__
        rres[v] = __builtin_amdgcn_raw_buffer_load_b64(res_rs, out_off[v], 0, 0);
#endif
    }
    // ... this lane's pixels (patch index of their first tap) and weight rows ...
    const int frow = lane & 15, fgrp = lane >> 4;
    int pp[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int px = i * 16 + frow, ty = kp_small_div(px, a.tw_mul), tx = px - ty * a.TW;
        pp[i] = ty < a.TH && g0 + ty < a.NP ? (extended(g0 + ty) - E0) * a.PW + tx : 0;
    }
    const unsigned w_off = (unsigned)(frow * 128 + ((fgrp ^ (frow & 7)) << 4));  // second half of the k-tile: chunk + 4, i.e. bit 6 flipped
    const int tap0 = kp_div(kt0, a.ct_mul, a.ct_sh), row0 = tap0 / 3;
    int ic = kt0 - tap0 * a.cin_tiles, is = tap0 - row0 * 3, tap_off = row0 * a.PW + is;
    const int last_off = 2 * (a.PW + 1);
    // ... and the fragment addresses of the next H k-tiles (past the last tap: of the last one).
    unsigned px_addr[H][TM];
    auto next_addresses = [&]() {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const int off = min(tap_off, last_off), chunk = (ic * 8 + fgrp) << 4;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int p = pp[i] + off;
                px_addr[h][i] = __umul24(p, a.pitch) + (chunk ^ (swizzle(p) << 4));
            }
            const bool tap_done = ++ic == a.cin_tiles;
            ic = tap_done ? 0 : ic;
            is += tap_done;
            const bool row_done = is == 3;
            is = row_done ? 0 : is;
            tap_off += row_done ? a.PW - 2 : (int)tap_done;
        }
    };
    next_addresses();

    f32x4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // this wavefront's part of the patch and the first half of its ring, then the others' parts
    wait_for_half(nkt - H, std::integral_constant<int, OPERANDS>());
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);

    struct Fragments { u32x4_t px[TM], w[TN]; };
    unsigned half = 0;
    for (int t0 = 0; t0 < nkt; t0 += H) {
        Fragments f[H][2];
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int i = 0; i < TM; ++i) f[h][ks].px[i] = *(const u32x4_t*)(smem + PATCH + (px_addr[h][i] ^ (ks << 6)));
#pragma unroll
                for (int j = 0; j < TN; ++j) f[h][ks].w[j] = *(const u32x4_t*)(ring + half + h * STAGE + j * 16 * 128 + (w_off ^ (ks << 6)));
            }
        const bool more = t0 + H < nkt;
        if (more) {
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the half may be overwritten
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < H; ++h) request_w(t0 + 2 * H + h, half / STAGE + h);
        }
#pragma unroll
        for (int h = 0; h < H; ++h)
            if (t0 + h < nkt) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f[h][ks].w[j]),
                                                                                __builtin_bit_cast(bf16x8_t, f[h][ks].px[i]), acc[i][j], 0, 0, 0);
            }
        if (more) {
            next_addresses();
            wait_for_half(nkt - t0 - 2 * H, std::integral_constant<int, 0>());
            half ^= H * STAGE;
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_sched_barrier(0);

    // D layout: channel 4*(lane/16) + e, pixel lane % 16.
    float* part = (float*)ring;
#pragma unroll
    for (int ti = 0; ti < TM; ++ti)
#pragma unroll
        for (int tj = 0; tj < TN; ++tj) *(f32x4_t*)(part + (ti * 16 + frow) * SROW + tj * 16 + fgrp * 4) = acc[ti][tj];
    __syncthreads();
    const unsigned relu_floor = a.relu ? kReluFloor : kNoReluFloor;
#pragma unroll
    for (int v = 0; v < PER; ++v) {
        const int item = tid + v * NW * 64, px = item / (BN / 4), c = (item % (BN / 4)) * 4;
        if (!live[v]) continue;
        const float* src = (const float*)smem + px * SROW + c;
        f32x4_t s = *(const f32x4_t*)src;
#pragma unroll
        for (int w = 1; w < NW; ++w) s += *(const f32x4_t*)(src + w * (RING / 4));
        s = s * sc + sh;
        s[0] += __uint_as_float(rres[v][0] << 16); s[1] += __uint_as_float(rres[v][0] & 0xffff0000u);
        s[2] += __uint_as_float(rres[v][1] << 16); s[3] += __uint_as_float(rres[v][1] & 0xffff0000u);
        kp_store(a.y + out_off[v], u32x2_t{pack_bf16x2_relu(s[0], s[1], relu_floor), pack_bf16x2_relu(s[2], s[3], relu_floor)});
    }
}

// Name as a profiler prints it.
const char* kpatch_variant_name(int v)
{
    static char buf[kKpatchVariants][96];
    if (v < 0 || v >= kKpatchVariants) return "?";
    snprintf(buf[v], 96, "conv3x3_kpatch_kernel<%d, %d, %d>", kKpatchShape[v].tm, kKpatchShape[v].tn, kKpatchShape[v].h);
    return buf[v];
}

template <int TM, int TN, int H> static int launch_kp(const KpatchArgs& a, int lds, hipStream_t stream)
{
    static std::atomic<bool> raised{false};
    if (!raised) {
        SGPRS_HIP(hipFuncSetAttribute((const void*)conv3x3_kpatch_kernel<TM, TN, H>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes));
        raised = true;
    }
    SGPRS_LAUNCH((conv3x3_kpatch_kernel<TM, TN, H>), dim3(a.die_tiles * 8), dim3(kKpatchWaves * 64), lds, stream, a);
    SGPRS_HIP(hipGetLastError());
    return SGPRS_OK;
}

static constexpr unsigned small_mul(int q) { return (unsigned)(((1 << 22) + q - 1) / q); }

struct KpatchTile { int th, tw, rows, pw, lds; long long tiles; };

// The tile of variant v with tw columns: as many rows (counted across the images) as its pixels allow; false
// if it does not fit the LDS.
static bool kpatch_tile_shape(const sgprs_conv_desc_t& d, int v, int tw, KpatchTile* t)
{
    const KpatchShape& s = kKpatchShape[v];
    const int P = out_dim(d.h, 3, 1, d.pad), Q = out_dim(d.w, 3, 1, d.pad);
    const long long NP = (long long)d.n * P;
    t->tw = tw;
    t->th = (int)std::min<long long>(16 * s.tm / tw, NP);
    if (t->th < 1) return false;
    const int crossings = d.n > 1 ? (t->th - 1 + P - 1) / P : 0;  // image borders inside a tile, at most
    t->rows = t->th + 2 + 2 * crossings;
    t->pw = tw + 2;
    const long long patch = (long long)t->rows * t->pw * d.cin * 2, units = d.cin / 8;
    const long long lds = (long long)kKpatchWaves * kp_ring_bytes(s.tm, s.tn, s.h) + (patch + 1023) / 1024 * 1024;
    if (lds > kLdsBytes) return false;
    // kp_small_div(m, small_mul(q)) is exact while m * q < 2^22 and m * small_mul(q) < 2^32
    auto small = [](long long m, long long q) { return m * q < 1ll << 22 && m * (long long)small_mul((int)q) < 1ll << 32; };
    if (!small(patch / 16 + 63, units) || !small(t->rows * t->pw + 63, t->pw) || !small(16 * s.tm, tw)) return false;
    t->lds = (int)lds;
    t->tiles = (NP + t->th - 1) / t->th * ((Q + tw - 1) / tw);
    return true;
}

// Estimated time (us) where every CU gets at most one tile: launch, a tile's chain, its k-tiles per wavefront,
// and its bytes at the 120 GB/s that a CU gets out of the L2.  Fitted to 27 launches of the network's layers (1 to
// 8 images, 32 to 256 CUs): 3 % off rms.  The 32x16 tile takes 0.55 us more where the longest share ends inside a
// half of the ring: 22 drawn layers of 384 channels, 7 k-tiles a share, were estimated 9 % faster than
// conv_ksplit_kernel and took 0.97 to 1.07 of its time (3 images of 24x15 on 248 CUs 5.57 us against 5.22).
static double kpatch_cost(const sgprs_conv_desc_t& d, int v, const KpatchTile& t)
{
    static const double kChain[kKpatchVariants] = {3.35, 3.6, 3.25, 3.6, 4.1}, kPerKtile[kKpatchVariants] = {0.0, 0.04, 0.08, 0.18, 0.3};
    const double kt = 9.0 * d.cin / 64, bytes = kt * 128 * 16 * kKpatchShape[v].tn + (double)t.rows * t.pw * d.cin * 2;
    const int share = (9 * d.cin / 64 + kKpatchWaves - 1) / kKpatchWaves;
    return kChain[v] + kPerKtile[v] * kt / kKpatchWaves + bytes / 120e3 + (v == 1 && share % kKpatchShape[v].h ? 0.55 : 0.0);
}

// Variant v's best tile: fewest tiles where a CU would get more than one (tests force such launches), least time otherwise.
static bool kpatch_best_tile(const sgprs_conv_desc_t& d, int v, int cus, KpatchTile* best, double* cost)
{
    const long long xb = (long long)d.n * d.h * d.w * d.cin * 2, wb = (long long)d.cout * 9 * d.cin * 2;
    if (v < 0 || v >= kKpatchVariants || d.dtype != SGPRS_BF16 || d.r != 3 || d.s != 3 || d.stride != 1 || d.cin % 64 || d.cout % (16 * kKpatchShape[v].tn) ||
        xb >= (1ll << 31) || wb >= (1ll << 31) || (long long)d.w * d.cin * 2 >= 1ll << 24 || d.h >= 1 << 22 || d.w >= 1 << 22 || d.pad >= 1 << 20)
        return false;
    const long long P = out_dim(d.h, 3, 1, d.pad), Q = out_dim(d.w, 3, 1, d.pad);
    if (d.n * (P + 2) >= 1ll << 30 || d.n * P * Q * d.cout * 2 >= 1ll << 31) return false;
    *cost = 1e30;
    for (int tw = 1; tw <= std::min<long long>(Q, 16 * kKpatchShape[v].tm); ++tw) {
        KpatchTile t;
        if (!kpatch_tile_shape(d, v, tw, &t)) continue;
        const long long wgs = t.tiles * (d.cout / (16 * kKpatchShape[v].tn));
        if (wgs >= 1ll << 28) continue;
        const double c = wgs <= cus ? kpatch_cost(d, v, t) : 1e6 + (double)wgs;
        if (c < *cost) { *cost = c; *best = t; }
    }
    return *cost < 1e30;
}

bool kpatch_fits(const sgprs_conv_desc_t& d, int v)
{
    KpatchTile t;
    double cost;
    return kpatch_best_tile(d, v, 256, &t, &cost);
}

bool plan_kpatch(const sgprs_conv_desc_t& d, int cus, int* variant, double* cost_us)
{
    *cost_us = 1e6;  // beyond: more than one tile per CU
    for (int v = 0; v < kKpatchVariants; ++v) {
        KpatchTile t;
        double cost;
        if (kpatch_best_tile(d, v, cus, &t, &cost) && cost < *cost_us) { *cost_us = cost; *variant = v; }
    }
    return *cost_us < 1e6;
}

int launch_conv3x3_kpatch(const sgprs_conv_desc_t& d, int variant, const void* x, const void* w, const float* scale, const float* shift,
                          const void* res, void* y, hipStream_t stream, int cus, Profiler* prof)
{
    struct Key { sgprs_conv_desc_t d; int variant, cus; };
    struct Plan { KpatchTile t; bool ok; };
    static thread_local PlanMemo<Key, Plan> local;
    static SharedPlanMemo<Key, Plan> memo;
    Key k;
    memset(&k, 0, sizeof(k));
    k.d = d; k.variant = variant; k.cus = cus;
    const Plan plan = memo.get(local, k, [&]() {
        Plan p;
        double cost;
        p.ok = kpatch_best_tile(d, variant, cus, &p.t, &cost);
        return p;
    });
    if (!plan.ok) return fail(SGPRS_ERR_INVALID_ARG, "internal: launch plan does not match the shape");
    const KpatchTile& t = plan.t;
    KpatchArgs a;
    memset(&a, 0, sizeof(a));
    a.x = (const unsigned char*)x; a.w = (const unsigned char*)w; a.y = (unsigned char*)y;
    a.scale = scale; a.shift = shift; a.res = (const unsigned char*)res;
    const int P = out_dim(d.h, 3, 1, d.pad);
    a.H = d.h; a.W = d.w; a.Q = out_dim(d.w, 3, 1, d.pad); a.NP = d.n * P; a.Cout = d.cout;
    a.pad = d.pad; a.relu = d.relu;
    a.cin_tiles = d.cin / 64; a.ktiles = 9 * a.cin_tiles;
    a.pitch = d.cin * 2; a.units = a.pitch / 16;
    a.row_bytes = d.w * a.pitch; a.image_bytes = d.h * a.row_bytes;
    a.x_bytes = (unsigned)((long long)d.n * a.image_bytes);
    a.w_bytes = (unsigned)((long long)d.cout * a.ktiles * 128);
    a.y_bytes = (unsigned)((long long)a.NP * a.Q * d.cout * 2);
    a.TH = t.th; a.TW = t.tw; a.PW = t.pw; a.HE = P + 2; a.multi = d.n > 1;
    a.patch_loads = (t.rows * t.pw * a.units + 63) / 64;
    a.units_mul = small_mul(a.units); a.pw_mul = small_mul(a.PW); a.tw_mul = small_mul(a.TW);
    div_constants(a.HE, &a.he_mul, &a.he_sh);
    div_constants(P, &a.p_mul, &a.p_sh);
    div_constants(a.cin_tiles, &a.ct_mul, &a.ct_sh);
    a.cb = (a.Q + t.tw - 1) / t.tw;
    div_constants(a.cb, &a.cb_mul, &a.cb_sh);
    // pixels of an odd number of 128 bytes alternate between the halves of the banks by themselves
    const bool even = a.cin_tiles % 2 == 0;
    a.swz_sh = even ? 0 : 1;
    a.swz_bits = even ? 4 : 3;
    a.gm = (int)t.tiles; a.gn = d.cout / (16 * kKpatchShape[variant].tn);
    a.die_cols = a.gn % 8 == 0 ? a.gn / 8 : 0;
    a.die_tiles = (a.gm * a.gn + 7) / 8;
    div_constants(a.die_cols ? a.die_cols : a.gn, &a.place_mul, &a.place_sh);
    int rc;
    const double M = (double)a.NP * a.Q;
    if (prof && prof->on && (rc = prof->begin(stream, kKindIgemm, kKpatchNames + variant, 2.0 * M * d.cout * 9 * d.cin, (double)a.x_bytes + a.w_bytes + (double)a.y_bytes * (res ? 2 : 1))))
        return rc;
    switch (variant) {
#define X(v, tm, tn, h) case v: rc = launch_kp<tm, tn, h>(a, t.lds, stream); break;
        SGPRS_KPATCH_VARIANTS(X)
#undef X
        default: rc = fail(SGPRS_ERR_INVALID_ARG, "bad variant %d", variant);
    }
    if (rc) return rc;
    if (prof && prof->on && (rc = prof->end(stream))) return rc;
    return SGPRS_OK;
}

}  // namespace sgprs
