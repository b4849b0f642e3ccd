"""GPU parity of the per-operator entry points against the fp64 oracle.

Every case calls libsgprs through its C ABI (via the ctypes binding) on seeded
inputs and compares element by element with the oracle:
max|gpu - ref| <= 1e-4 * max|ref| for fp32 and <= 2e-2 * max|ref| for
bf16-storage / fp32-accumulate (the oracle is fed the bf16-rounded values).
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2406_09425_amd as S
from workloads import BN_EPS, make_bn, make_conv_weight, make_input, round_to_bf16

from gpu_util import (DevConv, assert_close, dev_empty, dev_f32, dev_nhwc, host_nchw, rel_err)

pytestmark = pytest.mark.gpu
DTYPES = [S.SGPRS_F32, S.SGPRS_BF16]
DT_ID = {S.SGPRS_F32: "f32", S.SGPRS_BF16: "bf16"}
PART_SIZES = (8, 64, "full")   # keys of the `pools` fixture


@pytest.fixture(scope="module")
def pools():
    info = S.Pool(1, 8)
    total = info.info()["total_cus"]
    info.destroy()
    ps = {c: S.Pool(1, c) for c in (8, 64, total)}
    ps["full"] = ps[total]
    yield ps
    for p in set(ps.values()):
        p.destroy()


def fc_gemm_applicable(n, cin, cout):
    """Whether the FC of n images takes the tiled kernel: the library's own rule."""
    return bool(getattr(S.lib(), "_ZN5sgprs18fc_gemm_applicableEiii")(n, cin, cout) & 1)


def conv_case(dtype, n, h, w, cin, cout, k, stride, pad, relu, with_res, seed, pool, cus, absx=False):
    bf = dtype == S.SGPRS_BF16
    x = make_input(90, seed, (n, cin, h, w), "absnormal" if absx else "normal", bf16=bf)
    wt = make_conv_weight(90, seed, 1, cout, cin, k, bf16=bf)
    g, b, m, v = make_bn(90, seed, 2, cout)
    ref = oracle.bn(oracle.conv2d(x, wt, stride, pad), g, b, m, v, BN_EPS)
    res = None
    if with_res:
        res = make_input(90, seed, ref.shape, bf16=bf, tensor_id=7)
        ref = oracle.add(ref, res)
    if relu:
        ref = oracle.relu(ref)
    d = S.ConvDesc(n, h, w, cin, cout, k, k, stride, pad, dtype, int(relu))
    dc = DevConv(d, wt, g, b, m, v, BN_EPS)
    xd = dev_nhwc(x, dtype)
    rd = dev_nhwc(res, dtype) if with_res else None
    yd = dev_empty((n, ref.shape[2], ref.shape[3], cout), dtype)
    keep = dc.run(xd, yd, rd, pool, 0, cus)
    pool.sync()
    del keep
    return host_nchw(yd), ref


IGEMM_SHAPES = [
    # n, h, w, cin, cout, k, stride, pad   (ResNet18 shapes at batch 1 + ragged ones)
    (1, 56, 56, 64, 64, 3, 1, 1),
    (1, 56, 56, 64, 128, 3, 2, 1),
    (1, 56, 56, 64, 128, 1, 2, 0),
    (1, 28, 28, 128, 128, 3, 1, 1),
    (1, 14, 14, 256, 256, 3, 1, 1),
    (1, 14, 14, 256, 512, 3, 2, 1),
    (1, 7, 7, 512, 512, 3, 1, 1),
    (1, 14, 14, 256, 512, 1, 2, 0),
    (3, 9, 13, 64, 64, 3, 1, 1),     # ragged M = 351
    (2, 11, 7, 128, 192, 3, 2, 1),   # odd sizes, cout 192 = 3 x 64
    (5, 5, 5, 64, 64, 1, 1, 0),      # 1x1 stride 1
]


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
@pytest.mark.parametrize("shape", IGEMM_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_conv_igemm_parity(pools, dtype, shape):
    for i, cus in enumerate((8, "full")):
        pool = pools[cus]
        ncus = pool.partition_cus(0)
        got, ref = conv_case(dtype, *shape, relu=True, with_res=True, seed=11 + i, pool=pool, cus=ncus)
        e = assert_close(got, ref, dtype, f"conv {shape} on {ncus} CUs")
        if dtype == S.SGPRS_F32:
            assert e < 2e-5, e  # fp32 accumulation error should sit far inside the tolerance


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
def test_conv_flags_no_relu_no_residual(pools, dtype):
    pool = pools["full"]
    got, ref = conv_case(dtype, 2, 14, 14, 128, 128, 3, 1, 1, relu=False, with_res=False, seed=21, pool=pool,
                         cus=pool.partition_cus(0))
    assert_close(got, ref, dtype, "conv without relu/residual")
    assert np.min(ref) < 0 and np.min(got) < 0


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
@pytest.mark.parametrize("shape", [(1, 224, 224), (2, 50, 70), (1, 30, 33)], ids=str)
def test_conv_stem_parity(pools, dtype, shape):
    n, h, w = shape
    for cus in (8, "full"):
        pool = pools[cus]
        got, ref = conv_case(dtype, n, h, w, 3, 64, 7, 2, 3, relu=True, with_res=False, seed=31, pool=pool,
                             cus=pool.partition_cus(0))
        assert_close(got, ref, dtype, f"stem {shape}")


@pytest.mark.parametrize("shape,relu", [((1, 1, 4), True), ((2, 31, 28), False), ((1, 33, 64), True), ((3, 130, 132), True),
                                        ((2, 224, 224), False)], ids=str)
def test_stem_f32_packed_rows(pools, shape, relu):
    """The fp32 stem on packed input rows (widths that are a multiple of four): one output pixel, tails
    in both directions, tiles of 4 and of 8 rows, one workgroup walking many tiles.  148 products and
    sums of |w x| per output: below 148 * 2^-24 = 9e-6 of the largest.  An infinite input pixel reaches
    the outputs whose window holds it and no other."""
    n, h, w = shape
    for cus in (8, "full"):
        pool = pools[cus]
        got, ref = conv_case(S.SGPRS_F32, n, h, w, 3, 64, 7, 2, 3, relu=relu, with_res=False, seed=33, pool=pool,
                             cus=pool.partition_cus(0))
        assert got.shape == ref.shape and rel_err(got, ref) <= 9e-6, shape
        x = make_input(90, 34, (n, 3, h, w))
        wt = make_conv_weight(90, 34, 1, 64, 3, 7)
        dc = DevConv(S.ConvDesc(n, h, w, 3, 64, 7, 7, 2, 3, S.SGPRS_F32, int(relu)), wt, *make_bn(90, 34, 2, 64), BN_EPS)
        ih, iw, outs = h // 2, w // 2, []
        for v in (0.0, np.inf):
            x[-1, 1, ih, iw] = v
            yd = dev_empty((n,) + ref.shape[2:] + (64,), S.SGPRS_F32)
            keep = dc.run(dev_nhwc(x, S.SGPRS_F32), yd, None, pool, 0, pool.partition_cus(0))
            pool.sync()
            outs.append(host_nchw(yd))
        p, q = np.meshgrid(np.arange(ref.shape[2]), np.arange(ref.shape[3]), indexing="ij")
        hit = (np.abs(2 * p - ih) <= 3) & (np.abs(2 * q - iw) <= 3)
        same = np.array_equal
        assert same(outs[0][:-1], outs[1][:-1]) and same(outs[0][-1][:, ~hit], outs[1][-1][:, ~hit])
        assert not np.isfinite(outs[1][-1][:, hit]).all()


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
def test_conv_is_deterministic_and_mask_independent(pools, dtype):
    shape = (1, 14, 14, 256, 256, 3, 1, 1)
    outs = {}
    for cus in (8, 64, "full"):
        pool = pools[cus]
        a, ref = conv_case(dtype, *shape, relu=True, with_res=True, seed=41, pool=pool, cus=pool.partition_cus(0))
        b, _ = conv_case(dtype, *shape, relu=True, with_res=True, seed=41, pool=pool, cus=pool.partition_cus(0))
        assert np.array_equal(a, b), "two runs of the same launch differ"
        assert_close(a, ref, dtype)
        outs[cus] = a
    # masks change the split-K factor at most: results agree to rounding
    assert rel_err(outs[8], outs["full"]) <= (1e-5 if dtype == S.SGPRS_F32 else 1e-2)


def test_pack_unpack_roundtrip_on_device_copy():
    d = S.ConvDesc(1, 8, 8, 64, 64, 3, 3, 1, 1, S.SGPRS_BF16, 0)
    w = make_conv_weight(90, 0, 3, 64, 64, 3, bf16=True)
    assert np.array_equal(S.sgprs_unpack_conv_weights(d, S.sgprs_pack_conv_weights(d, w)), w)


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
@pytest.mark.parametrize("shape", [(1, 64, 112, 112), (2, 16, 9, 11), (3, 64, 7, 8)], ids=str)
def test_maxpool_parity_exact(pools, dtype, shape):
    n, c, h, w = shape
    x = make_input(91, 0, shape, bf16=dtype == S.SGPRS_BF16)  # has negatives: padding must not win
    ref = oracle.maxpool2d(x)
    xd = dev_nhwc(x, dtype)
    for cus in PART_SIZES:   # the partition sizes the per-operator sweep times
        yd = dev_empty((n, ref.shape[2], ref.shape[3], c), dtype)
        S.sgprs_maxpool2d(dtype, n, h, w, c, xd.data_ptr(), yd.data_ptr(), pools[cus], 0)
        pools[cus].sync()
        assert np.array_equal(host_nchw(yd), ref), cus  # selection only: bit exact


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
def test_bn_relu_parity(pools, dtype):
    shape = (1, 128, 28, 28)
    x = make_input(92, 0, shape, bf16=dtype == S.SGPRS_BF16)
    g, b, m, v = make_bn(92, 0, 1, 128)
    ref = oracle.relu(oracle.bn(x, g, b, m, v, BN_EPS))
    sc, sh = S.sgprs_fold_bn(g, b, m, v, BN_EPS)
    xd, scd, shd = dev_nhwc(x, dtype), dev_f32(sc), dev_f32(sh)
    for cus in PART_SIZES:
        yd = dev_empty((1, 28, 28, 128), dtype)
        S.sgprs_bn_relu(dtype, 28 * 28, 128, xd.data_ptr(), scd.data_ptr(), shd.data_ptr(), yd.data_ptr(),
                        pools[cus], 0)
        pools[cus].sync()
        assert_close(host_nchw(yd), ref, dtype, f"bn_relu on {cus} CUs")


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
@pytest.mark.parametrize("relu", [False, True])
def test_add_parity(pools, dtype, relu):
    shape = (1, 512, 7, 7)
    bf = dtype == S.SGPRS_BF16
    a, b = make_input(93, 0, shape, bf16=bf), make_input(93, 1, shape, bf16=bf)
    ref = oracle.add(a, b)
    if relu:
        ref = oracle.relu(ref)
    ad, bd = dev_nhwc(a, dtype), dev_nhwc(b, dtype)
    for cus in PART_SIZES:
        yd = dev_empty((1, 7, 7, 512), dtype)
        S.sgprs_add_relu(dtype, a.size, ad.data_ptr(), bd.data_ptr(), yd.data_ptr(), relu, pools[cus], 0)
        pools[cus].sync()
        assert_close(host_nchw(yd), ref, dtype, f"add on {cus} CUs")
        if not relu:
            assert np.min(host_nchw(yd)) < 0


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
@pytest.mark.parametrize("n", [1, 5, 33, 515])
def test_avgpool_fc_parity(pools, dtype, n):
    """1 and 5 images: one launch; 33: two launches, in bf16 the FC on the matrix cores; 515 (ragged
    against the 4 images per workgroup of the streaming avg-pool and the 32 of the FC tiles): the
    many-image avg-pool kernel."""
    bf = dtype == S.SGPRS_BF16
    x = make_input(94, n, (n, 512, 7, 7), bf16=bf)
    w = make_conv_weight(94, n, 1, 1000, 512, 1, bf16=bf)[:, :, 0, 0]
    bias = (make_input(94, n, (1000,), tensor_id=2) * 0.1).astype(np.float32)
    ref = oracle.fc(oracle.global_avgpool(x), w, bias)
    xd = dev_nhwc(x, dtype)
    wd = torch.from_numpy(np.ascontiguousarray(w)).to(xd.dtype).cuda()
    bd = dev_f32(bias)
    ws = torch.empty(n * 512, dtype=torch.float32, device="cuda")
    for cus in PART_SIZES:
        yd = torch.full((n, 1000), float("nan"), dtype=torch.float32, device="cuda")
        S.sgprs_avgpool_fc(dtype, n, 49, 512, 1000, xd.data_ptr(), wd.data_ptr(), bd.data_ptr(), yd.data_ptr(),
                           ws.data_ptr(), pools[cus], 0)
        pools[cus].sync()
        got = yd.cpu().numpy().astype(np.float64)
        assert_close(got, ref, dtype, f"avgpool_fc on {cus} CUs")
    # the average pool alone: against the oracle, and the same bits as the two-kernel path's workspace
    pd = torch.full((n, 512), float("nan"), dtype=torch.float32, device="cuda")
    S.sgprs_global_avgpool(dtype, n, 49, 512, xd.data_ptr(), pd.data_ptr(), pools["full"], 0)
    pools["full"].sync()
    assert rel_err(pd.cpu().numpy().astype(np.float64), oracle.global_avgpool(x).reshape(n, 512)) < (1e-6 if not bf else 1e-6)
    if n > 8:
        assert torch.equal(pd.flatten(), ws)
    # without bias
    S.sgprs_avgpool_fc(dtype, n, 49, 512, 1000, xd.data_ptr(), wd.data_ptr(), None, yd.data_ptr(),
                       ws.data_ptr(), pools["full"], 0)
    pools["full"].sync()
    assert_close(yd.cpu().numpy().astype(np.float64), ref - bias, dtype, "avgpool_fc no bias")


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
@pytest.mark.parametrize("cin,hw", [(512, 49), (1024, 21), (512, 3)])
def test_avgpool_fc_one_launch_equals_two(pools, dtype, cin, hw):
    """Up to 8 images take the single fused launch, 9 on 8 CUs avg-pool then FC (test_avgpool_fc_launches_by_size has the
    names): the same bits."""
    bf = dtype == S.SGPRS_BF16
    x = make_input(96, cin + hw, (9, cin, hw, 1), bf16=bf)
    w = make_conv_weight(96, cin + hw, 1, 1000, cin, 1, bf16=bf)[:, :, 0, 0]
    bias = make_input(96, cin + hw, (1000,), tensor_id=2).astype(np.float32)
    xd = dev_nhwc(x, dtype).reshape(9, hw, cin)
    wd = torch.from_numpy(np.ascontiguousarray(w)).to(xd.dtype).cuda()
    bd = dev_f32(bias)
    ws = torch.empty(9 * cin, dtype=torch.float32, device="cuda")
    two = torch.full((9, 1000), float("nan"), dtype=torch.float32, device="cuda")
    one = torch.full((8, 1000), float("nan"), dtype=torch.float32, device="cuda")
    S.sgprs_avgpool_fc(dtype, 9, hw, cin, 1000, xd.data_ptr(), wd.data_ptr(), bd.data_ptr(), two.data_ptr(),
                       ws.data_ptr(), pools[8], 0)
    S.sgprs_avgpool_fc(dtype, 8, hw, cin, 1000, xd.data_ptr(), wd.data_ptr(), bd.data_ptr(), one.data_ptr(),
                       ws.data_ptr(), pools["full"], 0)
    pools[8].sync()
    pools["full"].sync()
    assert torch.isfinite(one).all()
    assert torch.equal(one, two[:8])
    ref = oracle.fc(oracle.global_avgpool(x), w, bias)
    assert_close(two.cpu().numpy().astype(np.float64), ref, dtype, "two launches")
    assert_close(one.cpu().numpy().astype(np.float64), ref[:8], dtype, "one launch")


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
@pytest.mark.parametrize("cin,cout,hw", [(512, 1000, 21), (512, 1, 21), (512, 31, 21), (512, 33, 21), (1024, 1000, 21), (1024, 33, 21),
                                         (512, 1000, 49), (512, 33, 1), (512, 31, 3), (512, 33, 64), (512, 33, 65), (512, 31, 130),
                                         (1024, 33, 49), (1024, 33, 65)])
def test_avgpool_fc_rows_per_wavefront_same_bits(dtype, cin, cout, hw):
    """The images of one tensor in calls of 1 to 31 on 8, 32 and 256 CUs (4 or 8 output rows per wavefront, one launch or two,
    ragged output blocks; maps smaller than the four wavefronts, 7x7, and around the 64 positions that are requested at
    once): logits and, beyond 8 images, pooled vectors are the same bits."""
    td = torch.bfloat16 if dtype == S.SGPRS_BF16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(cout)
    x = torch.randn((31, hw, cin), generator=g, device="cuda").to(td)
    w = torch.randn((cout, cin), generator=g, device="cuda").to(td)
    b = torch.randn((cout,), generator=g, device="cuda")
    pooled = x.double().mean(1)
    ref = pooled @ w.double().t() + b.double()
    torch.cuda.synchronize()
    first = None
    for cus in (8, 32, 256):
        pool = S.Pool(1, cus)
        for n in (31, 17, 16, 9, 8, 4, 1):
            y = torch.full((n + 1, cout), float("nan"), device="cuda")
            ws = torch.full((n * cin,), float("nan"), device="cuda")
            torch.cuda.synchronize()
            S.sgprs_avgpool_fc(dtype, n, hw, cin, cout, x.data_ptr(), w.data_ptr(), b.data_ptr(), y.data_ptr(), ws.data_ptr(), pool, 0)
            pool.sync()
            first = y[:n].clone() if first is None else first
            assert torch.equal(y[:n], first[:n]), (cus, n)
            assert torch.isnan(y[n]).all()
            # cin fp32 products and their sums: 2^-24 each, of terms whose size is that of the products; and the sums of a quarter of the
            # positions, of the four quarters and the division, of terms whose size is that of the inputs
            bound = 2.0 ** -24 * ((cin + 18) * (pooled[:n].abs() @ w.double().abs().t() + b.double().abs()) +
                                  (hw / 4 + 5) * (x[:n].double().abs().mean(1) @ w.double().abs().t()))
            assert ((y[:n].double() - ref[:n]).abs() <= bound).all(), (cus, n)
            if n > 8:
                assert (ws.double() - pooled[:n].flatten()).abs().max() < 1e-6
            else:
                assert torch.isnan(ws).all()
        pool.destroy()


def test_error_paths_enqueue_nothing(pools):
    pool = pools["full"]
    x = torch.zeros(64, device="cuda")
    with pytest.raises(S.SgprsError) as e:
        S.sgprs_maxpool2d(S.SGPRS_F32, 1, 4, 4, 4, x.data_ptr(), x.data_ptr(), pool, 0)  # aliasing
    assert e.value.status == -1
    with pytest.raises(S.SgprsError):
        S.sgprs_maxpool2d(S.SGPRS_F32, 1, 4, 4, 4, x.data_ptr(), x.data_ptr() + 256, pool, 3)  # bad partition
    with pytest.raises(S.SgprsError) as e:
        S.sgprs_conv2d_workspace(S.ConvDesc(1, 8, 8, 48, 64, 3, 3, 1, 1, 0, 0), 256)  # cin % 32
    assert e.value.status == -5
    with pytest.raises(S.SgprsError):
        S.sgprs_add_relu(S.SGPRS_F32, 12, x.data_ptr(), x.data_ptr(), x.data_ptr(), False, pool, 0)


# ---- the LDS-patch 3x3 kernel, every tile variant forced in turn ----------------
PATCH_SHAPES = [
    # n, h, w, cin, cout: tiles straddle image boundaries, ragged last tile, several channel blocks/chunks
    (5, 14, 14, 64, 64),
    (3, 28, 28, 64, 128),
    (9, 7, 7, 128, 64),
    (2, 56, 56, 64, 64),
    (7, 9, 11, 128, 128),
]


@pytest.mark.parametrize("variant", range(5))
@pytest.mark.parametrize("shape", PATCH_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_conv3x3_patch_variants_parity(pools, variant, shape):
    n, h, w, cin, cout = shape
    pool = pools["full"]
    dtype = S.SGPRS_BF16
    try:
        for splits in (1, 2):
            S.sgprs_conv_tuning_override(1, variant, splits)
            for with_res in (True, False):
                got, ref = conv_case(dtype, n, h, w, cin, cout, 3, 1, 1, relu=with_res, with_res=with_res,
                                     seed=50 + variant, pool=pool, cus=pool.partition_cus(0))
                assert_close(got, ref, dtype, f"patch variant {variant} splits {splits} {shape}")
    finally:
        S.sgprs_conv_tuning_override(-1, 0, 1)


S2_SHAPES = [
    # n, h, w, cin, cout: several row tiles and image borders inside a tile, ragged last tile, 2-8 channel blocks
    (9, 14, 14, 64, 128),
    (3, 28, 28, 64, 128),
    (2, 56, 56, 64, 128),
    (20, 14, 14, 256, 512),
    (5, 10, 6, 128, 192),
    (7, 8, 12, 192, 64),
]


@pytest.mark.parametrize("variant", range(2))
@pytest.mark.parametrize("shape", S2_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_conv3x3s2_patch_variants_parity(pools, variant, shape):
    """The stride-2 patch kernel alone (no shortcut), both tile shapes, forced; shapes it
    declines fall back to the implicit GEMM and must match just the same."""
    n, h, w, cin, cout = shape
    pool = pools["full"]
    try:
        S.sgprs_conv_tuning_override(3, variant, 1)
        for relu in (True, False):
            got, ref = conv_case(S.SGPRS_BF16, n, h, w, cin, cout, 3, 2, 1, relu=relu, with_res=False, seed=80 + variant,
                                 pool=pool, cus=pool.partition_cus(0))
            assert_close(got, ref, S.SGPRS_BF16, f"stride-2 patch variant {variant} relu {relu} {shape}")
        # with a residual the planner must leave this kernel out (it has no residual input)
        got, ref = conv_case(S.SGPRS_BF16, n, h, w, cin, cout, 3, 2, 1, relu=True, with_res=True, seed=83, pool=pool,
                             cus=pool.partition_cus(0))
        assert_close(got, ref, S.SGPRS_BF16, f"stride-2 with residual {shape}")
    finally:
        S.sgprs_conv_tuning_override(-1, 0, 1)


# ---- the row-streaming 3x3 kernel of the 64 -> 64 layers -----------------------------
ROWS_CASES = [
    # batch, image height, partition, rows per stream and job the planner picks: one job per CU, jobs that cross
    # the middle of an image (7, 14) or cover whole images (28), several jobs per workgroup (batch 16 on 8 CUs),
    # and a 28-row image (two jobs of 2 x 7 rows)
    (2, 56, 8, 7), (4, 56, 8, 14), (8, 56, 8, 28), (16, 56, 64, 7), (16, 56, 8, 28), (4, 28, 8, 7),
]


@pytest.mark.parametrize("case", ROWS_CASES, ids=lambda c: "n%d-h%d-%dcu-S%d" % c)
def test_conv3x3_rows_parity(pools, case):
    """56-pixel rows, 64 -> 64 channels in bf16 on partitions where every CU gets whole jobs: the planner
    picks the row-streaming kernel; element by element against the oracle with and without residual
    and ReLU, and against the LDS-patch kernel (tuning override 5) on the same inputs."""
    n, h, cus, rows = case
    pool = pools[cus]
    dtype = S.SGPRS_BF16
    d = S.ConvDesc(n, h, 56, 64, 64, 3, 3, 1, 1, dtype, 1)
    assert S.sgprs_conv2d_plan(d, cus, True) == (3, rows)
    assert S.sgprs_conv2d_plan(d, cus, False) == (3, rows)
    for with_res, relu in ((True, True), (False, True), (False, False), (True, False)):
        got, ref = conv_case(dtype, n, h, 56, 64, 64, 3, 1, 1, relu=relu, with_res=with_res, seed=70 + n, pool=pool, cus=cus)
        assert_close(got, ref, dtype, f"rows kernel {case} res {with_res} relu {relu}")
        try:
            S.sgprs_conv_tuning_override(5, 0, 1)
            assert S.sgprs_conv2d_plan(d, cus, with_res)[0] == 1
            other, _ = conv_case(dtype, n, h, 56, 64, 64, 3, 1, 1, relu=relu, with_res=with_res, seed=70 + n, pool=pool, cus=cus)
        finally:
            S.sgprs_conv_tuning_override(-1, 0, 1)
        # the same bf16 inputs, fp32 sums in another order: at most a bf16 step apart
        assert np.all(np.abs(got - other) <= np.maximum(np.abs(other), 1e-2) * 2.0 ** -7)


def test_masks_that_leave_a_die_empty_are_rejected_and_odd_masks_work():
    """Mask bit i selects a CU of die i % 8.  A mask without a CU on some die is refused with a
    clear error; a mask of 9 CUs (two on die 0) is fine, and the forced patch kernels on it (a grid
    of 8 workgroups walking the padded, die-keyed work-item space) match the oracle."""
    n_xcd = S.Pool(1, 8).info()["n_xcd"]
    for bits in ((1 << 1) - 1, (1 << 4) - 1, (1 << 7) - 1):
        mask = np.zeros((1, 8), dtype=np.uint32)
        mask[0, 0] = bits
        if n_xcd > 1:
            with pytest.raises(S.SgprsError) as e:
                S.Pool(1, 0, masks=mask)
            assert e.value.status == -1 and "die" in str(e.value)
    mask = np.zeros((1, 8), dtype=np.uint32)
    mask[0, 0] = (1 << 9) - 1
    pool = S.Pool(1, 0, masks=mask)
    assert pool.partition_cus(0) == 9
    dtype = S.SGPRS_BF16
    try:
        for variant, shape in ((0, (1, 28, 28, 128, 128)), (1, (3, 14, 14, 64, 256)), (3, (2, 14, 14, 64, 512)),
                               (4, (2, 28, 28, 64, 128))):
            S.sgprs_conv_tuning_override(1, variant, 1)
            n, h, w, cin, cout = shape
            got, ref = conv_case(dtype, n, h, w, cin, cout, 3, 1, 1, relu=True, with_res=True, seed=120,
                                 pool=pool, cus=9)
            assert_close(got, ref, dtype, f"patch variant {variant} {shape} on 9 CUs")
        for variant, shape in ((0, (3, 28, 28, 64, 128)), (1, (9, 14, 14, 64, 512))):
            S.sgprs_conv_tuning_override(3, variant, 1)
            n, h, w, cin, cout = shape
            got, ref = conv_case(dtype, n, h, w, cin, cout, 3, 2, 1, relu=True, with_res=False, seed=130,
                                 pool=pool, cus=9)
            assert_close(got, ref, dtype, f"stride-2 patch variant {variant} {shape} on 9 CUs")
    finally:
        S.sgprs_conv_tuning_override(-1, 0, 1)
        pool.destroy()


def test_conv_planner_choices_agree(pools):
    """Automatic choice, implicit GEMM only and a forced patch variant give the
    same result to bf16 rounding on a batch large enough for the patch kernel."""
    pool = pools["full"]
    shape = (64, 14, 14, 64, 64, 3, 1, 1)
    outs = []
    try:
        for kind in (-1, 0, 1):
            S.sgprs_conv_tuning_override(kind, 3, 1)
            got, ref = conv_case(S.SGPRS_BF16, *shape, relu=True, with_res=True, seed=61, pool=pool,
                                 cus=pool.partition_cus(0))
            assert_close(got, ref, S.SGPRS_BF16, f"kind {kind}")
            outs.append(got)
    finally:
        S.sgprs_conv_tuning_override(-1, 0, 1)
    assert rel_err(outs[0], outs[1]) < 1e-2 and rel_err(outs[2], outs[1]) < 1e-2


@pytest.mark.parametrize("dtype", [S.SGPRS_F32, S.SGPRS_BF16], ids=["f32", "bf16"])
def test_igemm_forced_tiles_and_splits_parity(pools, dtype):
    """Every implicit-GEMM tile shape, with the planner's split factor and with
    forced ones, on a stride-2 3x3 and a 1x1 layer (ragged last row tile)."""
    pool = pools["full"]
    shapes = [(3, 14, 14, 64, 128, 3, 2, 1), (3, 14, 14, 64, 128, 1, 2, 0)]
    try:
        for variant in range(4):
            for splits in (0, 1, 2):
                for shape in shapes:
                    S.sgprs_conv_tuning_override(2, variant, splits)
                    got, ref = conv_case(dtype, *shape, relu=True, with_res=True, seed=70 + variant, pool=pool,
                                         cus=pool.partition_cus(0))
                    assert_close(got, ref, dtype, f"igemm variant {variant} splits {splits} {shape}")
    finally:
        S.sgprs_conv_tuning_override(-1, 0, 1)


# ---- implicit GEMM with K split over the wavefronts of a workgroup -----------------------
KSPLIT_SHAPES = [
    # n, h, w, cin, cout, k, stride, pad: ragged pixel tiles; fewer k-tiles than wavefronts (1x1); shares of 2..9
    # k-tiles, i.e. inside and beyond the ring; channel tiles per die (512) and pixel ranges per die (64, 192)
    (1, 5, 5, 64, 64, 1, 1, 0),
    (3, 9, 13, 64, 192, 3, 1, 1),
    (2, 11, 7, 128, 64, 3, 2, 1),
    (1, 7, 7, 512, 512, 3, 1, 1),
    (1, 14, 14, 256, 512, 1, 2, 0),
    # padding wider than the filter: whole windows before and past the image, in rows and columns, beyond
    # what a 32-bit shift holds (pad 33), strided, two images so that the neighbour's pixels are there to be read
    (2, 5, 7, 64, 64, 3, 1, 4),
    (2, 4, 3, 64, 64, 1, 1, 2),
    (1, 3, 2, 64, 64, 3, 2, 33),
    (2, 6, 5, 128, 64, 1, 2, 3),
]


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
@pytest.mark.parametrize("variant", range(8))
def test_conv_ksplit_tiles_parity(pools, dtype, variant):
    pool = pools["full"]
    try:
        S.sgprs_conv_tuning_override(2, 8 + variant, 0)
        for shape in KSPLIT_SHAPES:
            n, h, w, cin, cout, k, stride, pad = shape
            d = S.ConvDesc(n, h, w, cin, cout, k, k, stride, pad, dtype, 1)
            assert S.sgprs_conv2d_plan(d, pool.partition_cus(0)) == (0, 8 + variant)
            for with_res in (True, False):
                got, ref = conv_case(dtype, *shape, relu=with_res, with_res=with_res, seed=140 + variant, pool=pool,
                                     cus=pool.partition_cus(0))
                e = assert_close(got, ref, dtype, f"ksplit tile {variant} {shape}")
                if dtype == S.SGPRS_F32:
                    assert e < 2e-5, e  # fp32 accumulation over K <= 4608: about sqrt(K) * 2^-24
    finally:
        S.sgprs_conv_tuning_override(-1, 0, 1)


@pytest.mark.parametrize("variant", range(8))
@pytest.mark.parametrize("shape", [(1, 7, 7, 512, 512, 3, 1, 1), (1, 14, 14, 256, 256, 3, 1, 1), (1, 14, 14, 768, 64, 1, 1, 0)], ids=str)
def test_conv_ksplit_f32_keeps_its_chains_short(pools, variant, shape):
    """fp32 sums are kept in chains of at most 288 products (64 for the 1x1): each step adds a rounding error
    of about 2^-24 / sqrt(6) of the running sum, sqrt(288 / 2) of them in the root mean square, plus the partial
    sums' and the epilogue's roundings.  A single chain per wavefront (1152, 576 or 192 products) is past the line."""
    n, h, w, cin, cout, k, stride, pad = shape
    pool, chain = pools["full"], 64 if k == 1 else 288
    try:
        S.sgprs_conv_tuning_override(2, 8 + variant, 0)
        got, ref = conv_case(S.SGPRS_F32, *shape, relu=False, with_res=False, seed=160, pool=pool, cus=pool.partition_cus(0))
    finally:
        S.sgprs_conv_tuning_override(-1, 0, 1)
    e = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert e <= 2.0 ** -24 / 6.0 ** 0.5 * (chain / 2 + 20) ** 0.5, e


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
@pytest.mark.parametrize("n,cin,cout,cus", [(32, 512, 36, 8), (70, 1024, 100, 8), (129, 2048, 36, "full"), (65, 512, 1000, 64)], ids=str)
def test_fc_gemm_tiles_parity(pools, dtype, n, cin, cout, cus):
    """The FC of 32 images and more: small tiles (the large ones: the tests below), ragged in images and
    outputs, ring shares of 2 to 16 k-tiles, without a bias and with one.  fp32: sums of up to 2048 products,
    about sqrt(2048) * 2^-24; bf16: exact weights, pooled values to 2^-17."""
    bf = dtype == S.SGPRS_BF16
    x = make_input(97, n, (n, cin, 2, 1), bf16=bf)
    w = make_conv_weight(97, n, 1, cout, cin, 1, bf16=bf)[:, :, 0, 0]
    bias = make_input(97, n, (cout,), tensor_id=2).astype(np.float32) if n % 2 else np.zeros(cout, np.float32)
    ref = oracle.fc(oracle.global_avgpool(x), w, bias)
    xd = dev_nhwc(x, dtype)
    wd = torch.from_numpy(np.ascontiguousarray(w)).to(xd.dtype).cuda()
    bd = dev_f32(bias) if n % 2 else None
    ws = torch.empty(n * cin, dtype=torch.float32, device="cuda")
    lg = torch.full((n + 1, cout), float("nan"), dtype=torch.float32, device="cuda")
    pool = pools[cus]
    S.sgprs_avgpool_fc(dtype, n, 2, cin, cout, xd.data_ptr(), wd.data_ptr(), bd.data_ptr() if n % 2 else None, lg.data_ptr(),
                       ws.data_ptr(), pool, 0)
    pool.sync()
    got = lg.cpu().numpy().astype(np.float64)
    assert np.all(np.isnan(got[n]))    # nothing is written past the last image
    assert rel_err(got[:n], ref) <= (2e-5 if bf else 4e-6)


@pytest.mark.parametrize("n,cin,cus", [(64, 512, "full"), (39, 512, "full"), (40, 1024, "full"), (65, 512, 64), (200, 512, 8), (130, 2048, 8), (64, 2048, "full")], ids=str)
def test_fc_f32_keeps_its_chains_short(pools, n, cin, cus):
    """fp32 FC of 32 images and more, in each of its tile shapes and with the register kernel that fewer than
    40 images on most of the chip keep: products are summed in chains of eight, the
    rest is trees (16 roundings cover their levels).  Each rounding is about 2^-24 / sqrt(6) of its sum; a
    chain of eight adds 8 / 2 of them in the mean square, the quarter of the inputs that one wavefront
    multiplies (128 products and more) would be past the line.  One position per image: pooling is exact."""
    assert fc_gemm_applicable(n, cin, 1000)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn((n, 1, cin), generator=g, device="cuda")
    w = torch.randn((1000, cin), generator=g, device="cuda")
    ws, lg = torch.empty(n * cin, device="cuda"), torch.empty((n, 1000), device="cuda")
    torch.cuda.synchronize()
    S.sgprs_avgpool_fc(S.SGPRS_F32, n, 1, cin, 1000, x.data_ptr(), w.data_ptr(), None, lg.data_ptr(), ws.data_ptr(), pools[cus], 0)
    pools[cus].sync()
    ref = x[:, 0].double().cpu().numpy() @ w.double().cpu().numpy().T
    e = np.linalg.norm(lg.double().cpu().numpy() - ref) / np.linalg.norm(ref)
    assert e <= 2.0 ** -24 / 6.0 ** 0.5 * (8 / 2 + 16) ** 0.5, e


@pytest.mark.parametrize("dtype", DTYPES, ids=DT_ID.get)
def test_fc_gemm_weights_beyond_two_gib(pools, dtype):
    """More than 2^31 bytes of weights: the first and last outputs and those around byte 2^31, against fp64
    (bf16: pooled values to 2^-17; fp32: sums of 2048 products)."""
    n, cin = 33, 2048
    es = 2 if dtype == S.SGPRS_BF16 else 4
    mid = (1 << 31) // (cin * es)
    cout = mid + 132
    assert fc_gemm_applicable(n, cin, cout)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    x = torch.randn((n, 1, cin), generator=g, device="cuda").to(torch.bfloat16 if es == 2 else torch.float32)
    w = torch.empty((cout, cin), device="cuda", dtype=x.dtype).normal_(generator=g)
    ws = torch.empty(n * cin, device="cuda")
    lg = torch.full((n, cout), float("nan"), device="cuda")
    pool = pools["full"]
    torch.cuda.synchronize()
    S.sgprs_avgpool_fc(dtype, n, 1, cin, cout, x.data_ptr(), w.data_ptr(), None, lg.data_ptr(), ws.data_ptr(), pool, 0)
    pool.sync()
    assert bool(torch.isfinite(lg).all())
    rows = [0, 1, 65, mid - 1, mid, mid + 1, cout - 2, cout - 1]
    ref = x[:, 0].double().cpu().numpy() @ w[rows].double().cpu().numpy().T
    assert rel_err(lg[:, rows].double().cpu().numpy(), ref) <= (2e-5 if es == 2 else 4e-6)


WTILE_SHAPES = [
    # n, h, w, cin, cout, cus: the network's layers, several rounds of tiles on few CUs ...
    (2, 56, 56, 64, 64, 8), (3, 28, 28, 128, 128, 8), (5, 14, 14, 256, 256, "full"), (9, 7, 7, 512, 512, 64),
    # ... tiles of one or several images, cut in rows and in columns, with remainders, and single rows and columns
    (1, 60, 41, 192, 64, 64), (9, 5, 5, 128, 64, 8), (3, 9, 13, 256, 128, "full"), (1, 2, 130, 64, 192, 8), (3, 1, 6, 128, 64, 8),
    (2, 17, 1, 64, 64, 64), (1, 1, 1, 256, 64, "full")]


@pytest.mark.parametrize("ks,shape", [(ks, s) for ks in (1, 2, 4) for s in WTILE_SHAPES if s[3] // 64 % ks == 0], ids=str)
def test_conv3x3_wtile_parity(pools, ks, shape):
    """The kernel whose weights come in fragment order (tasks keep such a copy), by its launcher: `ks` wavefronts
    share a tile.  Weights in fragment order are those of the packed layout, 16 bytes at a time."""
    n, h, w, cin, cout, cus = shape
    pool, lib = pools[cus], S.lib()
    for relu, with_res in ((1, True), (0, False)):
        x = make_input(98, ks, (n, cin, h, w), bf16=True)
        wt = make_conv_weight(98, ks, 1, cout, cin, 3, bf16=True)
        g, b, m, v = make_bn(98, ks, 2, cout)
        ref = oracle.bn(oracle.conv2d(x, wt, 1, 1), g, b, m, v, BN_EPS)
        res = make_input(98, ks, ref.shape, bf16=True, tensor_id=7) if with_res else None
        if with_res:
            ref = oracle.add(ref, res)
        if relu:
            ref = oracle.relu(ref)
        d = S.ConvDesc(n, h, w, cin, cout, 3, 3, 1, 1, S.SGPRS_BF16, relu)
        dc = DevConv(d, wt, g, b, m, v, BN_EPS)
        wf = torch.zeros_like(dc.w)
        xd = dev_nhwc(x, S.SGPRS_BF16)
        rd = dev_nhwc(res, S.SGPRS_BF16) if with_res else None
        yd = dev_empty((n + 1, h, w, cout), S.SGPRS_BF16)
        torch.cuda.synchronize()
        ptr = lambda t: ctypes.c_void_p(t.data_ptr() if t is not None else None)
        stream = ctypes.c_void_p(pool.stream(0))
        assert getattr(lib, "_ZN5sgprs16repack_fragmentsERK17sgprs_conv_desc_tPKvPvP12ihipStream_t")(ctypes.byref(d), ptr(dc.w), ptr(wf), stream) == 0
        assert getattr(lib, "_ZN5sgprs20launch_conv3x3_wtileERK17sgprs_conv_desc_tiPKvS4_PKfS6_S4_PvP12ihipStream_tiPNS_8ProfilerE")(
            ctypes.byref(d), ks, ptr(xd), ptr(wf), ptr(dc.scale), ptr(dc.shift), ptr(rd), ptr(yd), stream, pool.partition_cus(0), None) == 0
        pool.sync()
        packed = dc.w.cpu().numpy().reshape(cout // 64, 4, 16, 9, cin // 64, 2, 4, 16)  # block, tile, channel, tap, chunk, half, group
        assert np.array_equal(wf.cpu().numpy().reshape(-1), packed.transpose(0, 4, 3, 5, 1, 6, 2, 7).reshape(-1))
        assert bool(torch.isnan(yd[n].float()).all())  # nothing is written past the last image
        assert_close(host_nchw(yd[:n]), ref, S.SGPRS_BF16, f"wtile {ks} {shape}")


KPATCH_SHAPES = [
    # the network's layers, several images to a tile, odd maps and channel counts (pixels of an odd number of 128 bytes) ...
    (1, 56, 56, 64, 64, 3, 1, 1), (1, 14, 14, 256, 256, 3, 1, 1), (3, 7, 7, 512, 512, 3, 1, 1), (5, 3, 2, 64, 64, 3, 1, 1), (2, 9, 13, 192, 128, 3, 1, 1),
    (1, 1, 1, 320, 64, 3, 1, 1), (1, 2, 90, 64, 192, 3, 1, 1),
    # ... and windows partly or wholly outside the image
    (2, 6, 5, 128, 64, 3, 1, 0), (2, 5, 7, 64, 64, 3, 1, 4), (1, 2, 3, 64, 64, 3, 1, 21)]


@pytest.mark.parametrize("variant", range(5))
def test_conv3x3_kpatch_tiles_parity(pools, variant):
    """Every tile of the kernel that keeps a tile's input pixels in LDS, also where a CU gets more than one of them."""
    kpatch_fits = getattr(S.lib(), "_ZN5sgprs11kpatch_fitsERK17sgprs_conv_desc_ti")
    try:
        S.sgprs_conv_tuning_override(2, 16 + variant, 0)
        for shape in KPATCH_SHAPES:
            n, h, w, cin, cout, k, stride, pad = shape
            pool = pools[8 if cin == 64 else "full"]
            d = S.ConvDesc(n, h, w, cin, cout, k, k, stride, pad, S.SGPRS_BF16, 1)
            takes = kpatch_fits(ctypes.byref(d), variant) & 1  # cout, and what the LDS holds beside the weights
            assert (S.sgprs_conv2d_plan(d, pool.partition_cus(0)) == (0, 16 + variant)) == takes, shape
            if not takes:
                continue
            for with_res in (True, False):
                got, ref = conv_case(S.SGPRS_BF16, *shape, relu=with_res, with_res=with_res, seed=170 + variant, pool=pool, cus=pool.partition_cus(0))
                assert_close(got, ref, S.SGPRS_BF16, f"tile {variant} {shape}")
    finally:
        S.sgprs_conv_tuning_override(-1, 0, 1)


SPLIT_SHAPES = [
    # n, h, w, cin, cout, k, stride, pad: the network's layers, ragged pixel tiles and channel counts ...
    (1, 56, 56, 64, 64, 3, 1, 1), (2, 14, 14, 256, 256, 3, 1, 1), (3, 7, 7, 512, 512, 3, 1, 1), (3, 9, 13, 96, 192, 3, 2, 1),
    # ... fewer k-tiles than wavefronts, shares of one and of odd numbers of them, windows outside the image
    (1, 5, 3, 32, 64, 1, 2, 0), (1, 11, 7, 160, 64, 1, 1, 0), (1, 1, 1, 32, 128, 3, 1, 1), (2, 5, 7, 64, 64, 3, 1, 4), (1, 3, 2, 64, 64, 3, 2, 33)]


def split_planes(lib, pool, d, dc):
    """The weights' planes with their scales and exponents, and whether the planes do not hold the weights."""
    planes = torch.zeros(6 * d.cout * d.cin * d.r * d.s + 8 * d.cout, dtype=torch.uint8, device="cuda")
    unfit = torch.zeros(1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert getattr(lib, "_ZN5sgprs13split_weightsERK17sgprs_conv_desc_tPKvPKfPvPiP12ihipStream_t")(
        ctypes.byref(d), ctypes.c_void_p(dc.w.data_ptr()), ctypes.c_void_p(dc.scale.data_ptr()), ctypes.c_void_p(planes.data_ptr()), ctypes.c_void_p(unfit.data_ptr()), ctypes.c_void_p(pool.stream(0))) == 0
    pool.sync()
    return planes, bool(unfit.item())


def split_case(lib, pool, variant, d, dc, x, res, guard=1, second=None):
    """`second`: descriptor and operands of the shortcut that goes along; its output is returned too."""
    ptr = lambda t: ctypes.c_void_p(t.data_ptr() if t is not None else None)
    p, q = (d.h + 2 * d.pad - d.r) // d.stride + 1, (d.w + 2 * d.pad - d.s) // d.stride + 1
    planes, unfit = split_planes(lib, pool, d, dc)
    assert not unfit
    y = torch.full((d.n + guard, p, q, d.cout), float("nan"), device="cuda")
    along = [None] * 6
    if second:
        d1, dc1 = second
        planes1, unfit = split_planes(lib, pool, d1, dc1)
        assert not unfit
        y1 = torch.full_like(y, float("nan"))
        along = [ctypes.byref(d1), ptr(dc1.w), ptr(planes1), ptr(dc1.scale), ptr(dc1.shift), ptr(y1)]
    torch.cuda.synchronize()
    stream = ctypes.c_void_p(pool.stream(0))
    assert getattr(lib, "_ZN5sgprs17launch_conv_splitERK17sgprs_conv_desc_tiPKvS4_S4_PKfS6_S4_PvPS1_S4_S4_S6_S6_S7_P12ihipStream_tPNS_8ProfilerE")(
        ctypes.byref(d), variant, ptr(x), ptr(dc.w), ptr(planes), ptr(dc.scale), ptr(dc.shift), ptr(res), ptr(y), *along, stream, None) == 0
    pool.sync()
    assert bool(torch.isnan(y[d.n:]).all())  # nothing is written past the last image
    if second:
        assert bool(torch.isnan(y1[d.n:]).all())
        return y[:d.n], y1[:d.n]
    return y[:d.n]


@pytest.mark.parametrize("variant", range(4))
def test_conv_split_tiles_parity(pools, variant):
    """fp32 by three bf16 planes of every operand (tasks keep the weights' planes), by its launcher.  The planes are
    exact, what is left out stays below 2^-26: the error is held to the line of the fp32 kernel's chains of
    288 products (see above), over K <= 4608."""
    lib, pool = S.lib(), pools["full"]
    fits = getattr(lib, "_ZN5sgprs10split_fitsERK17sgprs_conv_desc_ti")
    for shape in SPLIT_SHAPES:
        n, h, w, cin, cout, k, stride, pad = shape
        for relu, with_res in ((1, True), (0, False)):
            x, wt = make_input(99, variant, (n, cin, h, w)), make_conv_weight(99, variant, 1, cout, cin, k)
            g, b, m, v = make_bn(99, variant, 2, cout)
            ref = oracle.bn(oracle.conv2d(x, wt, stride, pad), g, b, m, v, BN_EPS)
            res = make_input(99, variant, ref.shape, tensor_id=7) if with_res else None
            ref = oracle.relu(oracle.add(ref, res)) if with_res else ref
            d = S.ConvDesc(n, h, w, cin, cout, k, k, stride, pad, S.SGPRS_F32, relu)
            assert fits(ctypes.byref(d), variant) & 1
            dc = DevConv(d, wt, g, b, m, v, BN_EPS)
            y = split_case(lib, pool, variant, d, dc, dev_nhwc(x, S.SGPRS_F32), dev_nhwc(res, S.SGPRS_F32) if with_res else None)
            got = host_nchw(y)
            assert_close(got, ref, S.SGPRS_F32, f"split tile {variant} {shape}")
            e = np.linalg.norm(got - ref) / np.linalg.norm(ref)
            assert e <= 2.0 ** -24 / 6.0 ** 0.5 * (288 / 2 + 20) ** 0.5, (shape, e)


@pytest.mark.parametrize("variant", range(4))
@pytest.mark.parametrize("lost", [False, True])
def test_conv_split_with_its_shortcut(pools, variant, lost):
    """A down-sampling block's first convolution and its 1x1 shortcut in one launch, every tile; `lost`: the shortcut's
    sums are too small for the planes where an image is, and only there, so that one of the two is multiplied again."""
    for n, h, w, cin, cout in ((2, 56, 56, 64, 128), (3, 14, 14, 256, 512), (1, 9, 13, 96, 192), (1, 2, 1, 32, 64)):
        x = make_input(97, variant, (n, cin, h, w))
        if lost:
            x[:, :, ::2, ::2] *= np.float32(2.0 ** -110)  # what the shortcut reads
        convs, refs = [], []
        for k, relu in ((3, 1), (1, 0)):
            wt = make_conv_weight(97, variant, k, cout, cin, k)
            g, b, m, v = make_bn(97, variant, k, cout)
            if lost and k == 1:
                g, m, b = g * np.float32(2.0 ** 110), m * np.float32(2.0 ** -110), b
            ref = oracle.bn(oracle.conv2d(x, wt, 2, k // 2), g, b, m, v, BN_EPS)
            d = S.ConvDesc(n, h, w, cin, cout, k, k, 2, k // 2, S.SGPRS_F32, relu)
            convs.append((d, DevConv(d, wt, g, b, m, v, BN_EPS)))
            refs.append(oracle.relu(ref) if relu else ref)
        got = split_case(S.lib(), pools["full"], variant, *convs[0], dev_nhwc(x, S.SGPRS_F32), None, second=convs[1])
        for y, ref in zip(got, refs):
            assert np.linalg.norm(host_nchw(y) - ref) <= 2.0 ** -24 / 6.0 ** 0.5 * (288 / 2 + 20) ** 0.5 * np.linalg.norm(ref)


PLANES_END = {  # factors of pixels and weights
    "infinities": (1.0, 1.0), "rounds to infinity": (1.0, 1.0), "tiny": (1e-36, 1.0), "huge": (1e30, 1.0), "zeros": (0.0, 1.0),
    # pixels whose lower planes, or all of them, are lost below 2^-126, with weights that make ordinary sums of them ...
    "tiny, huge weights": (2.0 ** -116, 2.0 ** 60), "subnormal, huge weights": (2.0 ** -128, 2.0 ** 80), "lost, huge weights": (2.0 ** -141, 2.0 ** 60),
    "few and lost": (2.0 ** -141, 2.0 ** 60), "subnormal": (1e-39, 2.0 ** 20),
    # ... and the reverse
    "huge, tiny weights": (1e30, 1e-36), "huge, subnormal weights": (1e30, 1e-39), "large, tiny weights": (1e20, 1e-35), "dead filters": (1.0, 1.0)}


@pytest.mark.parametrize("variant", range(4))
@pytest.mark.parametrize("what", PLANES_END)
def test_conv_split_where_the_planes_end(pools, variant, what):
    """Values that three bf16 planes do not hold: a channel's weights are scaled, or the tile is multiplied again with
    the fp32 MFMAs, and each output is infinite, NaN or accurate as in plain fp32."""
    gen = torch.Generator().manual_seed(5)
    x, wt = torch.randn((1, 9, 9, 64), generator=gen) * PLANES_END[what][0], (torch.randn((64, 64, 3, 3), generator=gen) / 24 * PLANES_END[what][1]).numpy()
    if what == "infinities":
        x[0, 3, 3, 5], x[0, 7, 7, 9], x[0, 1, 8, 0] = float("inf"), -float("inf"), float("nan")
    elif what == "rounds to infinity":
        x[0, 3, 3, 5] = 3.4e38
    elif what == "few and lost":
        x[0, :, :, 1:], x[0, 4:] = 0.0, 0.0
    elif what == "dead filters":
        wt[[7, 40]] *= np.float32(1e-30)
        wt[[9, 63]] = 0.0
    d = S.ConvDesc(1, 9, 9, 64, 64, 3, 3, 1, 1, S.SGPRS_F32, 0)
    one, zero = np.ones(64, np.float32), np.zeros(64, np.float32)
    scale = np.float32(2.0 ** 60) * one if what == "huge, subnormal weights" else one
    y = split_case(S.lib(), pools["full"], variant, d, DevConv(d, wt, scale, zero, zero, one, 0.0), x.cuda(), None).double().cpu() / float(scale[0])
    ref = torch.nn.functional.conv2d(x.double().permute(0, 3, 1, 2), torch.from_numpy(wt).double(), padding=1).permute(0, 2, 3, 1)
    finite = torch.isfinite(ref)
    assert torch.equal(torch.isnan(y), torch.isnan(ref)) and torch.equal(y[torch.isinf(ref)], ref[torch.isinf(ref)])
    for c in ([7, 40], [9, 63], slice(None)):
        assert float((y - ref)[..., c][finite[..., c]].norm()) <= 3.1e-7 * float(ref[..., c][finite[..., c]].norm())


def test_weights_that_the_planes_do_not_hold(pools):
    """Told when the planes are made: a channel's weights more than 2^50 apart, or not finite, or a scale that
    the weights' exponent takes out of the normal range."""
    d = S.ConvDesc(1, 9, 9, 64, 64, 3, 3, 1, 1, S.SGPRS_F32, 0)
    one, zero = np.ones(64, np.float32), np.zeros(64, np.float32)
    base = np.random.default_rng(3).uniform(0.5, 1.0, (64, 64, 3, 3)).astype(np.float32)
    for value, want in ((0.0, False), (2.0 ** -50, False), (-2.0 ** -50, False), (2.0 ** -52, True), (2.0 ** 51, True), (2.0 ** 127, True),
                        (1e-45, True), (np.inf, True), (np.nan, True)):
        for where in ((0, 0, 0, 0), (63, 63, 2, 2), (31, 17, 1, 0)):
            wt = base.copy()
            wt[where] = value
            assert split_planes(S.lib(), pools["full"], d, DevConv(d, wt, one, zero, zero, one, 0.0))[1] == want, (value, where)
    for scale, factor, want in ((1.0, 1e-30, False), (1.0, 1e-42, True), (1e38, 1e-42, False), (1.0, 0.0, False), (1e-45, 0.0, False),
                                (0.0, 1e30, False), (2.0 ** 90, 2.0 ** 9, False), (2.0 ** 90, 2.0 ** 38, True), (-1e-38, 1.0, True)):
        assert split_planes(S.lib(), pools["full"], d, DevConv(d, base * np.float32(factor), one * np.float32(scale), zero, zero, one, 0.0))[1] == want, (scale, factor)
