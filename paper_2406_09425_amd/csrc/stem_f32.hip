// fp32 stem: conv 7x7/2 (3 -> 64) + folded BN + ReLU, alone or with the max-pool 3x3/2 behind it.
//
// What bounds it is the fp32 matrix rate (16x16x4: 32 cycles, 147-deep sums), and on one image the
// chain request -> MFMAs -> store of a single tile.  The kernels that widen a pixel to four channel
// slots spend 168 K positions on 147 products, read a 16-byte pixel and two weight fragments from
// LDS for every six MFMAs, and fetch their patch through registers.  Here:
//   * a wavefront owns 16 of the 64 output channels and keeps their whole filter in 37 registers;
//     it computes every pixel of the tile, so LDS serves pixels only, one 4-byte read per MFMA
//     (64 lanes x 4 bytes of the packed rows; 16 pixels lie 6 floats apart and the four K groups 5,
//     which is conflict-free);
//   * the input rows keep the image's 3-channel packing and are copied global -> LDS by loads that
//     write LDS directly, two buffers, the next tile's patch requested before this tile's MFMAs;
//     a piece outside the image is zero-filled by the buffer's bounds check;
//   * the sum's order is free, so K is dealt to the MFMA's four K groups such that every read is a
//     register plus an immediate: group g takes floats 5g..5g+4 of each of the 7 tap rows (35 steps),
//     and the 21st float of rows g and g + 4 (2 steps; row 7 does not exist and is read as zero):
//     148 positions for 147 products.
// Workgroups of four wavefronts, two per CU (78 KB of LDS).  The weights arrive through the LDS area
// that later stages the pooled kernel's conv pixels.
// Measured on 256 CUs, us (before: four channel slots per pixel): alone 1 image 8.0 (14.4); with the
// pool 16 images 52.2 (60.8), 62 TFLOP/s before and 72 now; the MFMAs of its busiest CU take 35 at 2.4 GHz
// (7 tiles of 10 x 37 MFMAs a SIMD, a fifth of them for pixels that neighbouring tiles share).
#include "internal.h"

namespace sgprs {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

struct StemF32Args {
    const unsigned char* x;
    const unsigned char* w;
    unsigned char* y;
    const float* scale;
    const float* shift;
    int H, W;          // input
    int P, Q;          // conv output
    int PP, PQ;        // pooled output
    int tiles_p, tiles_q, ntiles;
    unsigned x_bytes;
    int relu;
};

// A tile is CR x CC conv pixels.  Alone: CC = 16, the tile at multiples of CR and 16.  Pooled: the
// CR = 2 TP + 1, CC = 17 conv pixels behind TP x 8 pooled ones, starting one row and column early.
template <int CR, int CC, bool POOL>
__global__ __launch_bounds__(256, 2) void stem_f32_kernel(const StemF32Args a)
{
    constexpr int TP = POOL ? (CR - 1) / 2 : CR, TQ = POOL ? 8 : 16;   // tile step in output pixels
    constexpr int PX = CR * CC, NT = (PX + 15) / 16;                  // MFMA column tiles
    constexpr int ROWS = 2 * CR + 5;
    // The first input column of a tile is 2 * cc0 - 3, -60 bytes (pooled) or -36 (alone) from a multiple
    // of 48 bytes: the row starts LEAD floats earlier, on a 16-byte boundary.
    constexpr int LEAD = POOL ? 1 : 3;
    constexpr int PIECES = ((2 * CC + 5) * 3 + LEAD + 3) / 4;          // 16-byte pieces per staged row
    constexpr int PITCH = PIECES * 4;                                  // floats
    constexpr int UNITS = ROWS * PIECES, ROUNDS = (UNITS + 255) / 256;
    constexpr int PATCH = (UNITS + 63) / 64 * 1024;                    // whole 1 KiB instructions
    constexpr int W_BYTES = 64 * kStemK * 4;
    constexpr int SROW = 64 * 4 + 16;                                  // staged conv pixel
    static_assert(NT % 2 == 0, "pixel tiles go in pairs");
    static_assert(!POOL || NT * 16 * SROW <= W_BYTES, "the staged tile takes the weights' place");

    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* patch = smem + W_BYTES;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fcol = lane & 15, grp = lane >> 4;
    const int row_bytes = a.W * 12;

    struct TilePos { int n, p, q; };                                   // image, first output row and column
    auto position = [&](int tile) {
        const int per_image = a.tiles_p * a.tiles_q;
        TilePos t;
        t.n = tile / per_image;
        const int r = tile - t.n * per_image, tp = r / a.tiles_q;
        t.p = tp * TP;
        t.q = (r - tp * a.tiles_q) * TQ;
        return t;
    };
    auto request_patch = [&](const TilePos t, int buf) {
#if __HIP_DEVICE_COMPILE__
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, (int)a.x_bytes, 0x00020000);
        const int h_base = POOL ? 4 * t.p - 5 : 2 * t.p - 3, b_base = POOL ? 48 * t.q - 64 : 24 * t.q - 48;
#pragma unroll
        for (int it = 0; it < ROUNDS; ++it) {
            const int u = it * 256 + tid, row = u / PIECES, seg = u - row * PIECES;
            const int ih = h_base + row, b = b_base + 16 * seg;
            const bool ok = u < UNITS && (unsigned)ih < (unsigned)a.H && (unsigned)b < (unsigned)row_bytes;
            if ((it * 4 + wave) * 1024 < PATCH)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(patch + buf * PATCH + (it * 4 + wave) * 1024), 16,
                                                         ok ? (unsigned)((t.n * a.H + ih) * row_bytes + b) : 0x80000000u, 0, 0, 0);
        }
#endif
    };

    // Each die (workgroup b runs on die b % 8) walks its own contiguous share of the tiles: patches
    // overlap, and neighbours meet in one L2.
    int tile = blockIdx.x, tile_step = gridDim.x, tile_end = a.ntiles;
    if (gridDim.x % 8 == 0) {
        const int per_die = (a.ntiles + 7) / 8, die = blockIdx.x & 7;
        tile = die * per_die + ((int)blockIdx.x >> 3);
        tile_step = (int)gridDim.x >> 3;
        tile_end = min((die + 1) * per_die, a.ntiles);
    }
    if (tile >= tile_end) return;
    TilePos cur = position(tile);
    request_patch(cur, 0);
    // Weights: 64 rows of 7 x 8 taps (4 floats each); tap t of filter row r lands in the slot t ^ (channel & 7).
#if __HIP_DEVICE_COMPILE__
    {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, W_BYTES, 0x00020000);
#pragma unroll
        for (int it = 0; it < W_BYTES / 4096; ++it) {
            const int u = it * 256 + tid, row = u / 56, slot = u - row * 56;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(smem + (it * 4 + wave) * 1024), 16,
                                                     (unsigned)(row * 896 + (slot ^ (row & 7)) * 16), 0, 0, 0);
        }
    }
#endif
    const int ch = wave * 16 + grp * 4;                                // this lane's four output channels
    const f32x4_t sc = *(const f32x4_t*)(a.scale + ch), sh = *(const f32x4_t*)(a.shift + ch);

    // Float offset of this lane's K run for pixel 16 i + fcol of the tile (K group included)
    int poff[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        int t = 16 * i + fcol;
        if (t >= PX) t = 0;                                            // padding: computed, never used
        poff[i] = (2 * (t / CC)) * PITCH + 6 * (t % CC) + LEAD + 5 * grp;
    }
    const int last_off = grp * (PITCH - 5) + 20;                       // from there to float 20 of row grp

    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    float wk[37];
    {
        const unsigned char* base = smem + (wave * 16 + fcol) * 896;
        const int sw = fcol & 7;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int j = 5 * grp + i, tap = j / 3, c = j - 3 * tap;
            const unsigned char* src = base + ((tap ^ sw) << 4) + c * 4;
#pragma unroll
            for (int r = 0; r < 7; ++r) wk[r * 5 + i] = *(const float*)(src + r * 128);
        }
        const unsigned char* src = base + ((6 ^ sw) << 4) + 8;
        wk[35] = *(const float*)(src + grp * 128);
        const float w36 = *(const float*)(src + (grp < 3 ? grp + 4 : 0) * 128);
        wk[36] = grp < 3 ? w36 : 0.f;
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);                                // lgkmcnt(0)
    __syncthreads();                                                   // the weights' place may be overwritten

    for (int buf = 0;; buf ^= 1) {
        const int next = tile + tile_step;
        TilePos nxt = cur;
        if (next < tile_end) {
            nxt = position(next);
            request_patch(nxt, buf ^ 1);
        }
        const float* px = (const float*)(patch + buf * PATCH);
        const int cr0 = POOL ? 2 * cur.p - 1 : cur.p, cc0 = POOL ? 2 * cur.q - 1 : cur.q;
        // Steps come in eight groups per pair of pixel tiles: the 7 tap rows (5 steps), then the 21st floats
        // (2 steps).  A group is read while the one before it is multiplied; left to itself the compiler
        // reads each operand right before its MFMA and waits for it.
        float v[2][2][5];
        auto read_group = [&](int i0, int g, float (&d)[2][5]) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float* src = px + poff[i0 + u];
                if (g < 7) {
#pragma unroll
                    for (int i = 0; i < 5; ++i) d[u][i] = src[g * PITCH + i];
                } else {
                    d[u][0] = src[last_off];
                    d[u][1] = src[last_off + (grp < 3 ? 4 * PITCH : 0)];
                }
            }
        };
        read_group(0, 0, v[0]);
#pragma unroll
        for (int i0 = 0; i0 < NT; i0 += 2) {
            f32x4_t acc[2];
            acc[0] = acc[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                if (g < 7) read_group(i0, g + 1, v[(g + 1) & 1]);
                else if (i0 + 2 < NT) read_group(i0 + 2, 0, v[0]);
                __builtin_amdgcn_sched_barrier(0);
                float (&d)[2][5] = v[g & 1];
                if (g == 7) {
                    d[0][1] = grp < 3 ? d[0][1] : 0.f;
                    d[1][1] = grp < 3 ? d[1][1] : 0.f;
                }
#pragma unroll
                for (int i = 0; i < (g < 7 ? 5 : 2); ++i)
#pragma unroll
                    for (int u = 0; u < 2; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(wk[g * 5 + i], d[u][i], acc[u], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            // D layout: channel 4 * (lane / 16) + e, pixel lane % 16
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int t = 16 * (i0 + u) + fcol;
                const int cr = cr0 + t / CC, cc = cc0 + t % CC;
                const bool ok = t < PX && (unsigned)cr < (unsigned)a.P && (unsigned)cc < (unsigned)a.Q;
                f32x4_t r = acc[u] * sc + sh;
                if (POOL || a.relu) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) r[e] = fmaxf(r[e], 0.f);
                }
                if constexpr (POOL) {
                    // positions outside the conv output never win the maximum
#pragma unroll
                    for (int e = 0; e < 4; ++e) r[e] = ok ? r[e] : -INFINITY;
                    *(f32x4_t*)(smem + t * SROW + ch * 4) = r;
                } else if (ok) {
                    *(f32x4_t*)(a.y + (((size_t)cur.n * a.P + cr) * a.Q + cc) * 256 + ch * 4) = r;
                }
            }
        }
        if constexpr (POOL) {
            __syncthreads();
            // one item = (pooled pixel, four channels)
#pragma unroll
            for (int it = 0; it < TP * TQ * 16 / 256; ++it) {
                const int item = it * 256 + tid, c4 = item & 15, pix = item >> 4, lp = pix / TQ, lq = pix % TQ;
                const unsigned char* src = smem + (2 * lp * CC + 2 * lq) * SROW + c4 * 16;
                f32x4_t m = *(const f32x4_t*)src;
#pragma unroll
                for (int k = 1; k < 9; ++k) {
                    const f32x4_t t = *(const f32x4_t*)(src + (k / 3 * CC + k % 3) * SROW);
#pragma unroll
                    for (int e = 0; e < 4; ++e) m[e] = fmaxf(m[e], t[e]);
                }
                const int p = cur.p + lp, q = cur.q + lq;
                if (p < a.PP && q < a.PQ) *(f32x4_t*)(a.y + (((size_t)cur.n * a.PP + p) * a.PQ + q) * 256 + c4 * 16) = m;
            }
        }
        if (next >= tile_end) break;
        tile = next;
        cur = nxt;
        __builtin_amdgcn_s_waitcnt(0);                                 // the next patch has landed ...
        __syncthreads();                                               // ... for every wavefront; the staged pixels have been read
    }
}

template <int CR, int CC, bool POOL>
static int launch_tile(const StemF32Args& a, int cus, hipStream_t stream)
{
    constexpr int units = (2 * CR + 5) * (((2 * CC + 5) * 3 + (POOL ? 1 : 3) + 3) / 4);
    constexpr int lds = 64 * kStemK * 4 + 2 * ((units + 63) / 64 * 1024);
    static_assert(lds <= 80 * 1024, "two workgroups per CU");
    static std::atomic<bool> raised{false};
    if (!raised) {
        SGPRS_HIP(hipFuncSetAttribute((const void*)stem_f32_kernel<CR, CC, POOL>, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        raised = true;
    }
    SGPRS_LAUNCH((stem_f32_kernel<CR, CC, POOL>), dim3((unsigned)std::min<long long>(a.ntiles, 2ll * cus)), dim3(256), lds, stream, a);
    SGPRS_HIP(hipGetLastError());
    return SGPRS_OK;
}

// Rows in whole 16-byte pieces, offsets of 31 bits.
bool stem_f32_applicable(int n, int h, int w)
{
    return w % 4 == 0 && (long long)n * h * w * 12 < (1ll << 31);
}

// Tiles of `rows` x 8 pooled pixels.
static long long pooled_tiles(int n, int h, int w, int rows)
{
    const int pp = (out_dim(h, 7, 2, 3) - 1) / 2 + 1, pq = (out_dim(w, 7, 2, 3) - 1) / 2 + 1;
    return (long long)n * ((pp + rows - 1) / rows) * ((pq + 7) / 8);
}

bool stem_f32_one_round(int n, int h, int w, int cus) { return pooled_tiles(n, h, w, 4) <= cus; }

int launch_stem_f32(int n, int h, int w, const void* x, const void* wts, const float* scale, const float* shift, void* y,
                    int relu, bool pool, hipStream_t stream, int cus)
{
    StemF32Args a;
    a.x = (const unsigned char*)x; a.w = (const unsigned char*)wts; a.y = (unsigned char*)y;
    a.scale = scale; a.shift = shift; a.relu = relu;
    a.H = h; a.W = w;
    a.P = out_dim(h, 7, 2, 3); a.Q = out_dim(w, 7, 2, 3);
    a.PP = (a.P - 1) / 2 + 1; a.PQ = (a.Q - 1) / 2 + 1;
    a.x_bytes = (unsigned)((long long)n * h * w * 12);
    // alone, 8 rows of 16 pixels unless that leaves CUs idle
    const int tall = pool || (long long)n * ((a.P + 7) / 8) * ((a.Q + 15) / 16) >= 2ll * cus;
    // with the pool, 4 rows of pooled pixels unless tiles of 2 (more conv pixels computed twice) all run at once: the chain of
    // one tile is 6 x 37 MFMAs instead of 10 x 37
    const bool low = pool && pooled_tiles(n, h, w, 2) <= cus;
    const int tp = pool ? (low ? 2 : 4) : tall ? 8 : 4;
    a.tiles_p = ((pool ? a.PP : a.P) + tp - 1) / tp;
    a.tiles_q = pool ? (a.PQ + 7) / 8 : (a.Q + 15) / 16;
    const long long nt = (long long)n * a.tiles_p * a.tiles_q;
    if (nt >= (1ll << 31)) return fail(SGPRS_ERR_UNSUPPORTED, "too many stem tiles");
    a.ntiles = (int)nt;
    if (low) return launch_tile<5, 17, true>(a, cus, stream);
    if (pool) return launch_tile<9, 17, true>(a, cus, stream);
    return tall ? launch_tile<8, 16, false>(a, cus, stream) : launch_tile<4, 16, false>(a, cus, stream);
}

}  // namespace sgprs
