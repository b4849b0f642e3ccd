// Offline-phase host helpers: BN folding, weight packing, launch planning.
// (Paper, "Offline Phase": everything that can be prepared before a task is
// released is prepared once.)
#include <algorithm>
#include <cmath>
#include <cstring>

#include "internal.h"

namespace sgprs {

int check_conv_desc(const sgprs_conv_desc_t* d)
{
    if (!d) return fail(SGPRS_ERR_INVALID_ARG, "conv desc is NULL");
    if (!dtype_ok(d->dtype)) return fail(SGPRS_ERR_UNSUPPORTED, "dtype %d", d->dtype);
    if (d->n <= 0 || d->h <= 0 || d->w <= 0 || d->cin <= 0 || d->cout <= 0 || d->r <= 0 || d->s <= 0 ||
        d->stride <= 0 || d->pad < 0)
        return fail(SGPRS_ERR_INVALID_ARG, "non-positive conv dimension");
    if (d->h + 2 * d->pad < d->r || d->w + 2 * d->pad < d->s)
        return fail(SGPRS_ERR_INVALID_ARG, "kernel larger than padded input");
    if (!is_stem(*d) && !is_igemm(*d))
        return fail(SGPRS_ERR_UNSUPPORTED,
                    "conv %dx%d stride %d pad %d cin %d: supported are 1x1/3x3 stride 1/2 with "
                    "cin %% 32 == 0 and the 7x7 stride-2 pad-3 3-channel stem",
                    d->r, d->s, d->stride, d->pad, d->cin);
    if (d->cout % 64) return fail(SGPRS_ERR_UNSUPPORTED, "cout %d must be a multiple of 64", d->cout);
    if (is_igemm(*d) && d->dtype == SGPRS_BF16 && d->cin % 64)
        return fail(SGPRS_ERR_UNSUPPORTED, "bf16 conv needs cin %% 64 == 0 (got %d)", d->cin);
    const long long p = out_dim(d->h, d->r, d->stride, d->pad), q = out_dim(d->w, d->s, d->stride, d->pad);
    const long long in_el = (long long)d->n * d->h * d->w * d->cin, out_el = (long long)d->n * p * q * d->cout;
    if (in_el >= (1ll << 31) || out_el >= (1ll << 31))
        return fail(SGPRS_ERR_UNSUPPORTED, "tensor with 2^31 or more elements");
    return SGPRS_OK;
}

static size_t packed_elems(const sgprs_conv_desc_t& d)
{
    return is_stem(d) ? (size_t)d.cout * kStemK : (size_t)d.cout * d.r * d.s * d.cin;
}

// Position of w[k][c][r][s] in the packed array, or -1 for "not stored".
static inline size_t packed_index(const sgprs_conv_desc_t& d, int k, int c, int r, int s)
{
    if (is_stem(d)) return (size_t)k * kStemK + (size_t)r * kStemTapRow + s * 4 + c;
    return (((size_t)k * d.r + r) * d.s + s) * d.cin + c;
}

// Rough cost model (microseconds) used to pick a tile shape and split-K
// factor.  It only has to rank candidates; absolute accuracy is irrelevant.
struct Tile { int bm, bn; double eff; };
static const Tile kTiles[] = {{128, 128, 1.0}, {128, 64, 0.85}, {64, 64, 0.6}, {32, 128, 0.5}};

int igemm_num_variants() { return (int)(sizeof(kTiles) / sizeof(kTiles[0])); }

// Tuning overrides: written by sgprs_conv_tuning_override, read by whatever thread plans a launch
// (the lane launcher threads of a periodic run among them), hence atomics.
std::atomic<int> g_conv_force_kind{-1};
std::atomic<int> g_igemm_force_variant{-1};
std::atomic<int> g_igemm_force_splits{0};

std::atomic<int> g_plan_generation{0};

static ConvPlan plan_conv_uncached(const sgprs_conv_desc_t& d, int cus, bool has_residual, bool ksplit, bool fragments);

ConvPlan plan_conv(const sgprs_conv_desc_t& d, int cus, bool has_residual, bool ksplit, bool fragments)
{
    struct Key { sgprs_conv_desc_t d; int cus, res, ksplit, fragments, gen; };
    static thread_local PlanMemo<Key, ConvPlan> local;
    static SharedPlanMemo<Key, ConvPlan> memo;
    Key k;
    memset(&k, 0, sizeof(k));
    k.d = d; k.cus = cus; k.res = has_residual; k.ksplit = ksplit; k.fragments = fragments; k.gen = g_plan_generation.load();
    return memo.get(local, k, [&]() { return plan_conv_uncached(d, cus, has_residual, ksplit, fragments); });
}

static ConvPlan plan_conv_uncached(const sgprs_conv_desc_t& d, int cus, bool has_residual, bool ksplit, bool fragments)
{
    const int force_kind = g_conv_force_kind.load(), force_variant = g_igemm_force_variant.load(),
              force_splits = g_igemm_force_splits.load();
    if (force_variant >= 16 && kpatch_fits(d, force_variant - 16)) {
        ConvPlan p;
        p.kind = 6; p.variant = force_variant - 16; p.bm = 1;
        return p;
    }
    if (force_variant >= 8 && ksplit_fits(d, force_variant - 8)) {
        ConvPlan p;
        p.kind = 4; p.variant = force_variant - 8; p.bm = 1;
        return p;
    }
    if (force_kind == -1) {
        int rows = 0;
        if (plan_rows(d, cus, &rows)) {
            ConvPlan p;
            p.kind = 3; p.variant = rows; p.splits = 1;
            p.bm = 1;  // marks a valid plan
            return p;
        }
    }
    ConvPlan best;
    double best_cost = 1e30;
    if (force_kind != 0) {
        int v = 0, s = 1;
        double cost = 0.0;
        if (plan_patch(d, cus, &v, &s, &cost)) {
            best.kind = 1; best.variant = v; best.splits = s;
            best.bm = 1;  // marks a valid plan
            best_cost = cost;
            if (force_kind == 1) return best;
        }
        if (force_kind != 1 && !has_residual && plan_s2patch(d, cus, &v)) {
            best.kind = 2; best.variant = v; best.splits = 1;
            best.bm = 1;
            return best;
        }
        // a forced implicit-GEMM tile is for the layers that would take that family anyway
        if (best.bm && force_variant >= 0) return best;
        if (ksplit && force_variant < 0 && force_kind != 1 && plan_ksplit(d, cus, &v, &cost) && cost < best_cost) {
            best = ConvPlan();
            best.kind = 4; best.variant = v; best.bm = 1;
            best_cost = cost;
        }
        if (ksplit && force_variant < 0 && force_kind != 1 && plan_kpatch(d, cus, &v, &cost) && cost < best_cost) {
            best = ConvPlan();
            best.kind = 6; best.variant = v; best.bm = 1;
            best_cost = cost;
        }
        if (fragments && force_kind == -1 && force_variant < 0 && plan_split(d, cus, &v, &cost) && cost < best_cost) {
            best = ConvPlan();
            best.kind = 7; best.variant = v; best.bm = 1;
            best_cost = cost;
        }
        if (fragments && force_kind == -1 && force_variant < 0 && plan_wtile(d, cus, &v, &cost)) {
            // Its estimate holds for the clock that the launch leaves the chip; those of the other two were
            // fitted where few CUs ran, and fall short of what launches on most of the chip take (LDS
            // patches: 12.5 estimated, 12.4 us on 32 CUs, 14.0 on 256; K split: 14.9, 13.2 and 16.9).
            const double chip = std::min(cus, 256) / 256.0, scaled = cost * (1.0 - 0.18 * chip);
            // With one chunk of channels per wavefront it loses near a tie, and the next layer finds its input in other
            // dies' L2s (28x28x128, 20 images on 256 CUs: 10.4 -> 10.9 us, and 0.5 us more in each of the next two
            // launches; whole inference 200.0 -> 204.5, 12 images on 160 CUs 184.5 -> 188.0): 7 % against it.
            const double margin = d.cin / 64 == v ? 0.93 : 1.0;
            if ((best.kind >= 4 ? cost * (1.02 - 0.15 * chip) : scaled) < margin * best_cost) {
                best = ConvPlan();
                best.kind = 5; best.variant = v; best.bm = 1;
                best_cost = scaled;
            }
        }
    }
    const int P = out_dim(d.h, d.r, d.stride, d.pad), Q = out_dim(d.w, d.s, d.stride, d.pad);
    const long long M = (long long)d.n * P * Q;
    const int kt_el = d.dtype == SGPRS_BF16 ? 64 : 32;
    const int ktiles = d.r * d.s * d.cin / kt_el;
    // time of one 128x128 tile over one k-tile on one CU at a realistic rate
    const double us_per_ktile_128 = d.dtype == SGPRS_BF16 ? 0.45 : 1.8;
    // with two LDS stages a k-tile cannot take less than one trip to the L2 (bf16 14x14x256 -> 256/2
    // at one image, 18 k-tiles in a row: 10.1 us)
    const double us_per_ktile_min = 0.45, us_per_block = 2.9;
    for (int v = 0; v < igemm_num_variants(); ++v) {
        Tile t = kTiles[v];
        if (d.cout % t.bn) continue;
        // few output pixels (batch-1 layers of 28x28 and below): the 32-row tile wastes the fewest
        // rows and gives split-K the most workgroups; measured 3-7 % faster than 64x64 there
        if (t.bm == 32 && M <= 1024) t.eff = 0.8;
        if (force_variant >= 0 && force_variant < igemm_num_variants() && v != force_variant &&
            d.cout % kTiles[force_variant].bn == 0)
            continue;
        const long long gm = (M + t.bm - 1) / t.bm, gn = d.cout / t.bn;
        const long long blocks = gm * gn;
        const int occ = 2;  // workgroups resident per CU
        for (int s = 1; s <= 32; s *= 2) {
            if (s > 1 && ktiles / s < 2) break;
            // a forced split factor applies where the shape allows it (else the planner's own choice stands)
            if (force_variant >= 0 && force_splits > 1 && s != force_splits &&
                ktiles / force_splits >= 2)
                continue;
            if (force_variant >= 0 && force_splits == 1 && s != 1) continue;
            const int kt_per = (ktiles + s - 1) / s;
            if (s > 1 && (long long)(s - 1) * kt_per >= ktiles) continue;  // an empty split
            const double per_block =
                kt_per * std::max(us_per_ktile_min, us_per_ktile_128 * (t.bm * t.bn / 16384.0) / t.eff * occ) + us_per_block;
            const long long rounds = (blocks * s + (long long)cus * occ - 1) / ((long long)cus * occ);
            double cost = rounds * per_block;
            if (s > 1) {
                const double bytes = (double)M * d.cout * 4.0 * (s + 1);
                cost += 4.0 + bytes / (3.0e6 * cus / 256.0);
            }
            if (cost < best_cost) {
                best_cost = cost;
                best.kind = 0;
                best.variant = v; best.bm = t.bm; best.bn = t.bn; best.splits = s; best.ktiles = ktiles;
                best.grid_m = (int)gm; best.grid_n = (int)gn;
            }
        }
    }
    return best;
}

// What a paired launch whose estimate in a loop is `cost` takes inside a network whose inputs change, where its weights are cold and it
// has the clock that the launches around it leave (bf16).  Implicit GEMM by tile: fixed, k-tiles of a workgroup, workgroups per CU, k-tiles
// of the busiest CU, the same in steps of two thirds of a round (where the time of the 128x128 tiles jumps), k-tiles times the share of
// the chip in use, MB.
static double pair_in_network(const ConvPlan& p, const sgprs_conv_desc_t& d0, const sgprs_conv_desc_t& d1, int cus, double cost)
{
    if (p.kind != 0) return 1.05 * cost;
    const double blocks = (double)p.grid_m * p.grid_n, rounds = blocks / cus, active = std::min(rounds, 1.0) * cus / 256;
    if (p.variant > 2) return 0.9 * cost + 5.4 * active;
    static const double kNet[3][7] = {{4.5, 0.05, 1.8, 0.216, 0.142, 0.0, 0.094}, {2.3, 0.02, 1.2, 0.235, 0.0, 0.26, 0.04}, {-3.3, 0.40, 1.8, 0.03, 0.0, 0.29, 0.0}};
    const double* c = kNet[p.variant];
    const double mb = 2e-6 * ((double)d0.n * d0.h * d0.w * d0.cin + 10.0 * d0.cin * d0.cout + 2.0 * d0.n * out_dim(d0.h, 3, 2, 1) * out_dim(d0.w, 3, 2, 1) * d0.cout);
    return c[0] + c[2] * std::max(1.0, 2.0 * rounds) + c[6] * mb +
           p.ktiles * (c[1] + c[3] * std::ceil(rounds) + c[4] * std::ceil(1.5 * rounds) / 1.5 + c[5] * active);
}

// A down-sampling block's first 3x3 convolution and its 1x1 shortcut in one launch: the tile that is
// best for the two together.  The single-convolution estimates do not rank these launches: the
// implicit-GEMM workgroups of the shortcut run beside the main problem's (three to five fit a CU)
// where the K-split kernel, one or two to a CU, needs further rounds.  Implicit GEMM: launch and
// epilogue, the k-tiles of one workgroup or, if that is longer, of the busiest CU, and a part per
// workgroup and CU; fitted per tile to 324 launches in loops over one input (the network's three
// blocks, 1..128 images, 32..256 CUs, both types; 5-12 % off rms).  Whole inferences with inputs that
// change from pass to pass, plan of the single convolution against this one, us: bf16 one image on 32
// CUs 130.2 / 126.6, on 64 CUs stage by stage 104.5 / 103.5, on 256 CUs 78.2 / 78.3; fp32 on 256 CUs one
// image 117.6 / 116.2, 16 images 652.6 / 641.1; bf16 13 images on 96 CUs and 128 on 256 the same; 64
// images on 256 CUs 397.0 / 399.4, the one that loses: in a loop its 14x14x256 -> 512 pair takes 19.2 us
// with the 64x64 implicit-GEMM tiles chosen here and 23.4 with the K-split kernel, in the network it is
// the other way round by 2 us.  Near a tie the K-split kernel is the one that keeps its time inside the
// network (4 images on 96 CUs, whole inference: 156.0 us with it in the second block, 159.4 with implicit
// GEMM, whose launch alone is as fast): 5 % in its favour.
static ConvPlan plan_conv_pair_uncached(const sgprs_conv_desc_t& d0, const sgprs_conv_desc_t& d1, int cus, bool fragments)
{
    const ConvPlan single = plan_conv(d0, cus);
    const int P = out_dim(d0.h, d0.r, d0.stride, d0.pad), Q = out_dim(d0.w, d0.s, d0.stride, d0.pad);
    const int forced = g_igemm_force_variant.load() - kS2tileNames;
    if (fragments && s2tile_fits(d0, d1, forced)) {
        ConvPlan p;
        p.kind = 8; p.variant = forced; p.bm = 1;
        return p;
    }
    if (g_conv_force_kind.load() != -1 || g_igemm_force_variant.load() >= 0 || single.bm == 0 || (single.kind != 0 && single.kind != 4) ||
        !is_igemm(d1) || d1.cout != d0.cout || P != out_dim(d1.h, d1.r, d1.stride, d1.pad) || Q != out_dim(d1.w, d1.s, d1.stride, d1.pad))
        return single;
    static const double kCost[2][4][4] = {  // fp32, bf16: {fixed, per k-tile of a workgroup, per k-tile of the busiest CU, per workgroup and CU}
        {{0.0, 1.86, 1.86, 9.5}, {3.9, 0.98, 0.860, 3.4}, {6.1, 0.51, 0.478, 0.44}, {4.9, 0.54, 0.490, 0.50}},
        {{4.2, 0.50, 0.316, 2.6}, {4.1, 0.40, 0.235, 1.07}, {2.4, 0.38, 0.145, 0.75}, {2.0, 0.45, 0.189, 0.61}}};
    const int kt_el = d0.dtype == SGPRS_BF16 ? 64 : 32;
    const long long M = (long long)d0.n * P * Q;
    const int kt0 = d0.r * d0.s * d0.cin / kt_el, kt1 = d1.r * d1.s * d1.cin / kt_el;
    ConvPlan best;
    double best_cost = 1e30;
    for (int v = 0; v < igemm_num_variants(); ++v) {
        const Tile& t = kTiles[v];
        if (d0.cout % t.bn) continue;
        const long long gm = (M + t.bm - 1) / t.bm, gn = d0.cout / t.bn, blocks = gm * gn;
        const double* c = kCost[d0.dtype == SGPRS_BF16][v];
        const double busiest = std::max((double)((blocks + cus - 1) / cus * kt0), (double)blocks * (kt0 + kt1) / cus);
        const double cost = 1.05 * (c[0] + std::max(c[1] * kt0, c[2] * busiest) + c[3] * std::max(1.0, 2.0 * blocks / cus));
        if (cost < best_cost) {
            best_cost = cost;
            best.variant = v; best.bm = t.bm; best.bn = t.bn; best.splits = 1; best.ktiles = kt0;
            best.grid_m = (int)gm; best.grid_n = (int)gn;
        }
    }
    for (int v = 0; v < ksplit_num_variants(); ++v) {
        if (!ksplit_fits(d0, v) || !ksplit_fits(d1, v)) continue;
        const double cost = ksplit_cost(d0, v, cus, &d1);
        if (cost < best_cost) {
            best_cost = cost;
            best = ConvPlan();
            best.kind = 4; best.variant = v; best.bm = 1;
        }
    }
    for (int v = 0; v < split_num_variants() && fragments; ++v) {
        if (!split_fits(d0, v) || !split_fits(d1, v)) continue;
        const double cost = split_cost(d0, v, cus, &d1);
        if (cost < best_cost) {
            best_cost = cost;
            best = ConvPlan();
            best.kind = 7; best.variant = v; best.bm = 1;
        }
    }
    // Near a tie the launch chosen so far stays.  Of the three blocks' launches at 167 sizes (1 to 512 images, 8 to 256 CUs, inputs that change)
    // this choice is more than 2 % slower than the implicit GEMM and the K-split kernel at 4, by 2 to 9 % (27 images on 64 CUs, 28x28x128 -> 256:
    // 22.2 / 24.2 us), and leaves 1 % of all their time to the best launch of each size.
    int variant;
    double cost;
    if (fragments && plan_s2tile(d0, d1, cus, &variant, &cost) && cost < 0.98 * pair_in_network(best, d0, d1, cus, best_cost)) {
        best = ConvPlan();
        best.kind = 8; best.variant = variant; best.bm = 1;
    }
    return best.bm ? best : single;
}

ConvPlan plan_conv_pair(const sgprs_conv_desc_t& d0, const sgprs_conv_desc_t& d1, int cus, bool fragments)
{
    struct Key { sgprs_conv_desc_t d0, d1; int cus, fragments, gen; };
    static thread_local PlanMemo<Key, ConvPlan> local;
    static SharedPlanMemo<Key, ConvPlan> memo;
    Key k;
    memset(&k, 0, sizeof(k));
    k.d0 = d0; k.d1 = d1; k.cus = cus; k.fragments = fragments; k.gen = g_plan_generation.load();
    return memo.get(local, k, [&]() { return plan_conv_pair_uncached(d0, d1, cus, fragments); });
}

size_t conv_workspace_bytes(const sgprs_conv_desc_t& d, const ConvPlan& p)
{
    if (p.splits <= 1) return 0;
    const int P = out_dim(d.h, d.r, d.stride, d.pad), Q = out_dim(d.w, d.s, d.stride, d.pad);
    return (size_t)p.splits * d.n * P * Q * d.cout * sizeof(float);
}

}  // namespace sgprs

using namespace sgprs;

extern "C" {

int sgprs_fold_bn(const float* gamma, const float* beta, const float* mean, const float* var, float eps,
                  int c, float* scale, float* shift)
{
    if (!gamma || !beta || !mean || !var || !scale || !shift)
        return fail(SGPRS_ERR_INVALID_ARG, "NULL BN vector");
    if (c <= 0) return fail(SGPRS_ERR_INVALID_ARG, "c %d <= 0", c);
    for (int i = 0; i < c; ++i) {
        const double v = (double)var[i] + (double)eps;
        if (!(v > 0.0)) return fail(SGPRS_ERR_INVALID_ARG, "var[%d]+eps = %g is not positive", i, v);
        const double sc = (double)gamma[i] / std::sqrt(v);
        scale[i] = (float)sc;
        shift[i] = (float)((double)beta[i] - (double)mean[i] * sc);
    }
    return SGPRS_OK;
}

int sgprs_conv_packed_weight_bytes(const sgprs_conv_desc_t* d, size_t* bytes)
{
    int rc = check_conv_desc(d);
    if (rc) return rc;
    if (!bytes) return fail(SGPRS_ERR_INVALID_ARG, "bytes is NULL");
    *bytes = packed_elems(*d) * dtype_size(d->dtype);
    return SGPRS_OK;
}

int sgprs_pack_conv_weights(const sgprs_conv_desc_t* d, const float* w, void* packed, size_t bytes)
{
    int rc = check_conv_desc(d);
    if (rc) return rc;
    if (!w || !packed) return fail(SGPRS_ERR_INVALID_ARG, "NULL weight pointer");
    const size_t need = packed_elems(*d) * dtype_size(d->dtype);
    if (bytes < need) return fail(SGPRS_ERR_INVALID_ARG, "packed buffer %zu < %zu bytes", bytes, need);
    memset(packed, 0, need);
    for (int k = 0; k < d->cout; ++k)
        for (int c = 0; c < d->cin; ++c)
            for (int r = 0; r < d->r; ++r)
                for (int s = 0; s < d->s; ++s) {
                    const float v = w[(((size_t)k * d->cin + c) * d->r + r) * d->s + s];
                    const size_t o = packed_index(*d, k, c, r, s);
                    if (d->dtype == SGPRS_BF16) ((uint16_t*)packed)[o] = f32_to_bf16_bits(v);
                    else ((float*)packed)[o] = v;
                }
    return SGPRS_OK;
}

int sgprs_unpack_conv_weights(const sgprs_conv_desc_t* d, const void* packed, size_t bytes, float* w)
{
    int rc = check_conv_desc(d);
    if (rc) return rc;
    if (!w || !packed) return fail(SGPRS_ERR_INVALID_ARG, "NULL weight pointer");
    const size_t need = packed_elems(*d) * dtype_size(d->dtype);
    if (bytes < need) return fail(SGPRS_ERR_INVALID_ARG, "packed buffer %zu < %zu bytes", bytes, need);
    for (int k = 0; k < d->cout; ++k)
        for (int c = 0; c < d->cin; ++c)
            for (int r = 0; r < d->r; ++r)
                for (int s = 0; s < d->s; ++s) {
                    const size_t o = packed_index(*d, k, c, r, s);
                    w[(((size_t)k * d->cin + c) * d->r + r) * d->s + s] =
                        d->dtype == SGPRS_BF16 ? bf16_bits_to_f32(((const uint16_t*)packed)[o])
                                               : ((const float*)packed)[o];
                }
    return SGPRS_OK;
}

int sgprs_conv2d_workspace(const sgprs_conv_desc_t* d, int partition_cus, size_t* bytes)
{
    int rc = check_conv_desc(d);
    if (rc) return rc;
    if (!bytes) return fail(SGPRS_ERR_INVALID_ARG, "bytes is NULL");
    if (partition_cus <= 0) return fail(SGPRS_ERR_INVALID_ARG, "partition_cus %d <= 0", partition_cus);
    // The plan may depend on whether a residual is passed and on the kind of the partition's mask
    // (planning_cus), and a tuning override may switch to the kernels that split K over workgroups
    // after the caller has allocated: enough for all of them.
    *bytes = 0;
    if (!is_stem(*d))
        for (int cus : {partition_cus, planning_cus(partition_cus)})
            for (int res = 0; res < 2; ++res)
                *bytes = std::max({*bytes, conv_workspace_bytes(*d, plan_conv(*d, cus, res != 0)),
                                   conv_workspace_bytes(*d, plan_conv(*d, cus, res != 0, false))});
    return SGPRS_OK;
}

int sgprs_conv2d_plan(const sgprs_conv_desc_t* d, int partition_cus, int has_residual, int* family, int* detail)
{
    int rc = check_conv_desc(d);
    if (rc) return rc;
    if (!family || !detail) return fail(SGPRS_ERR_INVALID_ARG, "family or detail is NULL");
    if (partition_cus <= 0) return fail(SGPRS_ERR_INVALID_ARG, "partition_cus %d <= 0", partition_cus);
    if (is_stem(*d)) {
        *family = 4; *detail = 0;
        return SGPRS_OK;
    }
    const ConvPlan p = plan_conv(*d, planning_cus(partition_cus), has_residual != 0);
    if (p.bm == 0) return fail(SGPRS_ERR_UNSUPPORTED, "no tile shape fits cout %d", d->cout);
    *family = p.kind == 4 || p.kind == 6 ? 0 : p.kind;
    *detail = p.variant + (p.kind == 4 ? 8 : p.kind == 6 ? 16 : 0);
    return SGPRS_OK;
}

}  // extern "C"
