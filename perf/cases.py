"""What this framework is used for, as timed cases.

A user of the library holds a pool of CU-masked partitions and ResNet18 tasks (weights packed and
uploaded once) and then, over and over, runs whole inferences (`Task.run`), single stages handed
out by the scheduler (`Task.stage_run`), the static multi-tenant executor (`Pool.run_static`), or
one operator on a partition (`sgprs_conv2d`, `sgprs_maxpool2d`, ...).  Each case here is one such
pass with its sizes; `draw` gives further cases of the same ranges:

  net      whole inferences, batch 1..128 (bf16) or 1..16 (fp32), on 8..256 CUs
  stages   the six stages of a small batch through the per-stage entry point
  tenants  1..8 independent instances, each pinned to one of the pool's partitions
  conv     one convolution with folded BN (ReLU, residual): the network's layers and ragged maps
  maxpool, bn_relu, add_relu, avgpool, avgpool_fc   the remaining operators, from one image (a
           call that is all latency) to tensors far beyond the caches
"""
import math
import weakref

import torch

import paper_2406_09425_amd as S
from workloads import BN_EPS, CONV_SPECS, FC_IN, NUM_CLASSES

_DT = {"bf16": S.SGPRS_BF16, "f32": S.SGPRS_F32}
_TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
_ES = {"bf16": 2, "f32": 4}

# FLOP of one image's convolutions and FC, and the network's weights
_NET_FLOPS = 2.0 * FC_IN * NUM_CLASSES + sum(2.0 * cout * cin * k * k * ((h + 2 * pad - k) // stride + 1) ** 2
                                             for _, cin, cout, k, stride, pad, h in CONV_SPECS)
_NET_WEIGHTS = sum(cin * cout * k * k for _, cin, cout, k, _, _, _ in CONV_SPECS) + FC_IN * NUM_CLASSES
# values per image at the stage boundaries (input of stage 0, then the outputs of stages 0..5)
_BOUNDARY = [3 * 224 * 224, 64 * 56 * 56, 64 * 56 * 56, 128 * 28 * 28, 256 * 14 * 14, 512 * 7 * 7, NUM_CLASSES]


def listed():
    return [
        # the throughput workload: one bf16 batch that has the whole chip
        dict(name="net_bf16_b64_256cu", kind="net", dtype="bf16", batch=64, cus=256),
        # one frame as it arrives, whole chip: pure latency
        dict(name="net_bf16_b1_256cu", kind="net", dtype="bf16", batch=1, cus=256),
        dict(name="net_f32_b1_256cu", kind="net", dtype="f32", batch=1, cus=256),
        # one frame on one of eight equal partitions
        dict(name="net_bf16_b1_32cu", kind="net", dtype="bf16", batch=1, cus=32),
        # a ragged batch on a partition of a mixed pool
        dict(name="net_bf16_b13_96cu", kind="net", dtype="bf16", batch=13, cus=96),
        # a single-precision batch
        dict(name="net_f32_b16_256cu", kind="net", dtype="f32", batch=16, cus=256),
        # an offline batch: the largest
        dict(name="net_bf16_b128_256cu", kind="net", dtype="bf16", batch=128, cus=256),
        # the multi-tenant pool: eight instances on eight partitions of 32 CUs
        dict(name="tenants_bf16_8x32cu", kind="tenants", dtype="bf16", n=8, cus=32, batch=1, rounds=4),
        # what the scheduler issues for one job: six stages, one by one
        dict(name="stages_bf16_b1_64cu", kind="stages", dtype="bf16", batch=1, cus=64),
        # operators of the CU-scaling experiment: the dominant convolution, the smallest call of
        # all (residual add of one 512x7x7 map), and the max-pool of a 64-image batch
        dict(name="conv_bf16_b1_256x14x14", kind="conv", dtype="bf16", n=1, h=14, w=14, cin=256, cout=256, k=3, stride=1,
             relu=True, res=False, cus=256),
        dict(name="add_bf16_512x7x7", kind="add_relu", dtype="bf16", n=1, hw=49, c=512, cus=256),
        dict(name="maxpool_bf16_b64_64x112x112", kind="maxpool", dtype="bf16", n=64, h=112, w=112, c=64, cus=256),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    known = [{k: v for k, v in c.items() if k != "name"} for c in listed()]
    while True:
        case = _draw(rng)
        if case not in known:
            return case


def _draw(rng):
    kind = rng.choices(["net", "stages", "tenants", "conv", "maxpool", "bn_relu", "add_relu", "avgpool", "avgpool_fc"],
                       [10, 1, 1, 4, 1, 1, 1, 1, 1])[0]
    dtype = rng.choice(["bf16", "bf16", "f32"])
    cus = rng.choice([8 * rng.randint(1, 32), 8 * rng.randint(1, 32), 8 * rng.randint(1, 32), 256])
    slow = 1 if dtype == "bf16" else 8
    if kind == "net":  # a partition gets as many images as it can turn around in about a millisecond
        return dict(kind=kind, dtype=dtype, batch=_log_int(rng, 1, max(1, cus // (2 * slow))), cus=cus)
    if kind == "stages":
        return dict(kind=kind, dtype=dtype, batch=_log_int(rng, 1, max(1, cus // 16)), cus=cus)
    if kind == "tenants":
        n = rng.randint(1, 8)
        return dict(kind=kind, dtype="bf16", n=n, cus=8 * rng.randint(1, 32 // n), batch=rng.randint(1, 2), rounds=rng.randint(1, 4))
    if kind == "conv":
        k, stride, relu, res = 3, rng.choice([1, 1, 2]), True, rng.random() < 0.5
        if rng.random() < 0.5:
            _, cin, cout, k, stride, _, h = rng.choice(CONV_SPECS)
            w, relu, res = h, k != 1, res and stride == 1
        else:
            cin, cout = (64 * rng.choice([1, 2, 3, 4, 6, 8]) for _ in range(2))
            h, w = rng.randint(5, 60), rng.randint(5, 60)
        case = dict(kind=kind, dtype=dtype, n=1, h=h, w=w, cin=cin, cout=cout, k=k, stride=stride, relu=relu, res=res, cus=cus)
        most = 1e11 * cus / 256 / slow / work(case)["flops"]
        return dict(case, n=_log_int(rng, 1, max(1, min(128, int(most)))))
    n = _log_int(rng, 1, 64)
    if kind == "maxpool":
        return dict(kind=kind, dtype=dtype, n=n, h=rng.randint(14, 112), w=rng.randint(14, 112), c=rng.choice([32, 64, 96, 128]), cus=cus)
    if kind in ("bn_relu", "add_relu"):
        return dict(kind=kind, dtype=dtype, n=n, hw=rng.randint(7, 56) * rng.randint(7, 56), c=rng.choice([64, 128, 256, 512]), cus=cus)
    return dict(kind=kind, dtype=dtype, n=_log_int(rng, 1, 4096), hw=rng.randint(5, 8) * rng.randint(5, 8), c=512, cus=cus)


# ---- inputs --------------------------------------------------------------------------------------
# A program opens one pool and keeps it; states of the same shape share it and the last one closes it.
_pools = weakref.WeakValueDictionary()


def _pool(n_p, cus):
    p = _pools.get((n_p, cus))
    if p is None:
        p = _pools[(n_p, cus)] = S.Pool(n_p, cus)
    return p


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, std=1.0):
    return torch.randn(shape, generator=g, device="cuda") * std


def _bn(g, c):
    gamma = torch.rand(c, generator=g, device="cuda") + 0.5
    var = torch.rand(c, generator=g, device="cuda") + 0.5
    return gamma, _normal(g, (c,), 0.1), _normal(g, (c,), 0.1), var


def _task(g, dtype, batch):
    """A ResNet18 instance with He-normal weights and plausible BN statistics."""
    p = dict(conv_w=[], gamma=[], beta=[], mean=[], var=[])
    for _, cin, cout, k, _, _, _ in CONV_SPECS:
        p["conv_w"].append(_normal(g, (cout, cin, k, k), math.sqrt(2.0 / (cin * k * k))).cpu().numpy())
        for key, v in zip(("gamma", "beta", "mean", "var"), _bn(g, cout)):
            p[key].append(v.cpu().numpy())
    p["fc_w"] = _normal(g, (NUM_CLASSES, FC_IN), math.sqrt(2.0 / FC_IN)).cpu().numpy()
    p["fc_b"] = _normal(g, (NUM_CLASSES,), 0.1).cpu().numpy()
    return S.Task(p, _DT[dtype], batch, BN_EPS)


def _net_state(g, dtype, batch):
    return dict(task=_task(g, dtype, batch), x=_normal(g, (batch, 224, 224, 3)).to(_TORCH[dtype]),
                out=torch.zeros((batch, NUM_CLASSES), device="cuda"))


def _conv_out(case):
    pad = case["k"] // 2
    return tuple((case[d] + 2 * pad - case["k"]) // case["stride"] + 1 for d in ("h", "w"))


def prepare(case, seed):
    g, kind, dtype = _gen(seed), case["kind"], case["dtype"]
    tdt = _TORCH[dtype]
    st = dict(case=case, dt=_DT[dtype])
    if kind == "net":
        st.update(_net_state(g, dtype, case["batch"]))
    elif kind == "stages":
        st.update(task=_task(g, dtype, case["batch"]), x=_normal(g, (case["batch"], 224, 224, 3)).to(tdt))
        st["out"] = [torch.zeros((case["batch"], v), device="cuda", dtype=tdt if j < 5 else torch.float32)
                     for j, v in enumerate(_BOUNDARY[1:])]
        st["ptr"] = [st["x"].data_ptr()] + [o.data_ptr() for o in st["out"]]
    elif kind == "tenants":
        st["nets"] = [_net_state(g, dtype, case["batch"]) for _ in range(case["n"])]
        st["tasks"] = [s["task"] for s in st["nets"]]
        st["in_ptr"] = [s["x"].data_ptr() for s in st["nets"]]
        st["out_ptr"] = [s["out"].data_ptr() for s in st["nets"]]
        st["out"] = [s["out"] for s in st["nets"]]
    elif kind == "conv":
        n, h, w, cin, cout, k = (case[f] for f in ("n", "h", "w", "cin", "cout", "k"))
        p, q = _conv_out(case)
        d = S.ConvDesc(n, h, w, cin, cout, k, k, case["stride"], k // 2, st["dt"], int(case["relu"]))
        wt = _normal(g, (cout, cin, k, k), math.sqrt(2.0 / (cin * k * k))).cpu().numpy()
        scale, shift = S.sgprs_fold_bn(*(v.cpu().numpy() for v in _bn(g, cout)), BN_EPS)
        st.update(desc=d, w=torch.from_numpy(S.sgprs_pack_conv_weights(d, wt)).cuda(), scale=torch.from_numpy(scale).cuda(),
                  shift=torch.from_numpy(shift).cuda(), x=_normal(g, (n, h, w, cin)).to(tdt),
                  res=_normal(g, (n, p, q, cout)).to(tdt) if case["res"] else None,
                  out=torch.zeros((n, p, q, cout), device="cuda", dtype=tdt))
        st["ws_bytes"] = S.sgprs_conv2d_workspace(d, case["cus"])
        st["ws"] = torch.empty(max(st["ws_bytes"], 16), device="cuda", dtype=torch.uint8)
    elif kind == "maxpool":
        n, h, w, c = (case[f] for f in ("n", "h", "w", "c"))
        st["x"] = _normal(g, (n, h, w, c)).to(tdt)
        st["out"] = torch.zeros((n, (h - 1) // 2 + 1, (w - 1) // 2 + 1, c), device="cuda", dtype=tdt)
    else:
        n, hw, c = case["n"], case["hw"], case["c"]
        st["x"] = _normal(g, (n, hw, c)).to(tdt)
        if kind == "bn_relu":
            scale, shift = S.sgprs_fold_bn(*(v.cpu().numpy() for v in _bn(g, c)), BN_EPS)
            st.update(scale=torch.from_numpy(scale).cuda(), shift=torch.from_numpy(shift).cuda(), out=torch.zeros_like(st["x"]))
        elif kind == "add_relu":
            st.update(b=_normal(g, (n, hw, c)).to(tdt), out=torch.zeros_like(st["x"]))
        elif kind == "avgpool":
            st["out"] = torch.zeros((n, c), device="cuda")
        else:
            st.update(w=_normal(g, (NUM_CLASSES, c), math.sqrt(2.0 / c)).to(tdt), bias=_normal(g, (NUM_CLASSES,), 0.1),
                      ws=torch.zeros((n, c), device="cuda"), out=torch.zeros((n, NUM_CLASSES), device="cuda"))
    st["pool"] = _pool(case["n"] if kind == "tenants" else 1, case["cus"])
    torch.cuda.synchronize()  # the partitions' streams are not ordered after torch's
    return st


# ---- one pass ------------------------------------------------------------------------------------
def _run_net(st, case):
    st["task"].run(case["batch"], st["x"].data_ptr(), st["out"].data_ptr(), st["pool"], 0)


def _run_stages(st, case):
    for j in range(6):
        st["task"].stage_run(j, case["batch"], st["ptr"][j], st["ptr"][j + 1], st["pool"], 0)


def _run_tenants(st, case):
    st["pool"].run_static(st["tasks"], st["in_ptr"], st["out_ptr"], case["batch"], range(case["n"]), case["rounds"])


def _run_conv(st, case):
    S.sgprs_conv2d(st["desc"], st["x"].data_ptr(), st["w"].data_ptr(), st["scale"].data_ptr(), st["shift"].data_ptr(),
                   st["res"].data_ptr() if case["res"] else None, st["out"].data_ptr(), st["ws"].data_ptr(), st["ws_bytes"],
                   st["pool"], 0)


def _run_maxpool(st, case):
    S.sgprs_maxpool2d(st["dt"], case["n"], case["h"], case["w"], case["c"], st["x"].data_ptr(), st["out"].data_ptr(), st["pool"], 0)


def _run_bn_relu(st, case):
    S.sgprs_bn_relu(st["dt"], case["n"] * case["hw"], case["c"], st["x"].data_ptr(), st["scale"].data_ptr(), st["shift"].data_ptr(),
                    st["out"].data_ptr(), st["pool"], 0)


def _run_add_relu(st, case):
    S.sgprs_add_relu(st["dt"], st["x"].numel(), st["x"].data_ptr(), st["b"].data_ptr(), st["out"].data_ptr(), True, st["pool"], 0)


def _run_avgpool(st, case):
    S.sgprs_global_avgpool(st["dt"], case["n"], case["hw"], case["c"], st["x"].data_ptr(), st["out"].data_ptr(), st["pool"], 0)


def _run_avgpool_fc(st, case):
    S.sgprs_avgpool_fc(st["dt"], case["n"], case["hw"], case["c"], NUM_CLASSES, st["x"].data_ptr(), st["w"].data_ptr(),
                       st["bias"].data_ptr(), st["out"].data_ptr(), st["ws"].data_ptr(), st["pool"], 0)


_RUN = dict(net=_run_net, stages=_run_stages, tenants=_run_tenants, conv=_run_conv, maxpool=_run_maxpool, bn_relu=_run_bn_relu,
            add_relu=_run_add_relu, avgpool=_run_avgpool, avgpool_fc=_run_avgpool_fc)


def run(state):
    case = state["case"]
    _RUN[case["kind"]](state, case)
    return state["out"]


# ---- what a pass cannot do without ---------------------------------------------------------------
def work(case):
    kind, es = case["kind"], _ES[case["dtype"]]
    if kind in ("net", "stages", "tenants"):
        b = case["batch"]
        one = _BOUNDARY[0] * b * es + _NET_WEIGHTS * es + NUM_CLASSES * b * 4
        if kind == "stages":  # every stage's output is asked for, and is the next one's input
            one += 2 * sum(_BOUNDARY[1:6]) * b * es
        times = case["n"] * case["rounds"] if kind == "tenants" else 1
        return dict(bytes=one * times, flops=_NET_FLOPS * b * times)
    if kind == "conv":
        p, q = _conv_out(case)
        n, cin, cout, kk = case["n"], case["cin"], case["cout"], case["k"] ** 2
        y = n * p * q * cout
        return dict(bytes=(n * case["h"] * case["w"] * cin + cin * cout * kk + y * (2 if case["res"] else 1)) * es + 8 * cout,
                    flops=2.0 * y * cin * kk)
    if kind == "maxpool":
        h, w = case["h"], case["w"]
        per = h * w + ((h - 1) // 2 + 1) * ((w - 1) // 2 + 1)
        return dict(bytes=case["n"] * case["c"] * per * es, flops=0)
    n, hw, c = case["n"], case["hw"], case["c"]
    if kind == "bn_relu":
        return dict(bytes=2 * n * hw * c * es + 8 * c, flops=2 * n * hw * c)
    if kind == "add_relu":
        return dict(bytes=3 * n * hw * c * es, flops=n * hw * c)
    if kind == "avgpool":
        return dict(bytes=n * hw * c * es + 4 * n * c, flops=n * hw * c)
    return dict(bytes=n * hw * c * es + NUM_CLASSES * (c * es + 4 + 4 * n), flops=n * hw * c + 2.0 * n * c * NUM_CLASSES)


def tolerance(case):
    kind, bf16 = case["kind"], case["dtype"] == "bf16"
    if kind in ("maxpool", "add_relu"):  # selections, and one correctly rounded sum per value
        return "exact"
    if kind in ("avgpool", "avgpool_fc"):  # fp32 sums and fp32 results whatever the storage type
        return dict(rel=1e-5)
    return dict(rel=1e-2 if bf16 else 1e-5)
