"""What a program built on this library spends its time on, as timed cases.

Three kinds of work, each through the public Python entry points:

  net    a network-shaped pass (``api.KernelList.run``): every fused kernel of a network, each launch on tensors
         of its own, under the transferred records that the stored sweep outcome chose.  At another batch size,
         image size or sequence length than the stored one the same records are re-applied to the new shapes,
         which is what they are for; a record that does not apply leaves its kernel on the default schedule.
  op     one operator call (``api.tt_conv2d_bias_relu``, ``tt_dense_bias_relu``, ``tt_batch_matmul``,
         ``tt_dwconv``).  ``records`` says under which schedule: "transfer" is the fastest donor record of the
         stored pools for that shape, found by ``api.tt_transfer_sweep`` when the program starts and kept;
         "default" is a call without a schedule, as a program without a pool makes it.
  sweep  the search itself: ``api.tt_transfer_sweep`` of a network's kernels over a stored pool with the default
         protocol, the donor schedules' times on the new shapes being what the user waits for.

Tensors are channels-last (NHWC activations, KRSC filters), as the library stores them.
"""
import dataclasses
import json
import math
import os

import torch

from paper_2201_05587_amd import api, tune
from paper_2201_05587_amd import workloads as wl

TUNED = os.path.join(os.path.dirname(os.path.abspath(api.__file__)), "tuned")
# network -> (stored sweep outcome, the kernels it was made for)
NETWORKS = {
    "resnet50": ("cfg5", lambda b, seq: wl.resnet50_kernels(b, wl.BF16, with_dense=False)),
    "resnet18": ("cfg2", lambda b, seq: wl.resnet18_kernels(b, wl.F32)),
    "bert": ("cfg3", lambda b, seq: wl.bert_kernels(seq=seq, batch=b)),
    "mobilenetv2": ("cfg4", lambda b, seq: wl.mobilenetv2_kernels(b, wl.F32)),
}
POOLS = ("cfg1", "cfg2", "cfg3", "cfg4", "cfg5")


def _net(network, batch, seq=0, image=224):
    """`seq`: tokens of a transformer's sequence; `image`: edge of a convolutional network's input."""
    return {"kind": "net", "network": network, "batch": batch, "seq": seq, "image": 0 if seq else image}


def _conv(cls, dtype, records, n, c, h, w, k, f, stride):
    return {"kind": "op", "op": "conv", "cls": cls, "dtype": dtype, "records": records, "n": n, "c": c, "h": h,
            "w": w, "k": k, "f": f, "stride": stride}


def _gemm(cls, dtype, records, batch, m, n, k, trans_b=1):
    return {"kind": "op", "op": "bmm" if cls == wl.CLS_BATCH_MATMUL else "dense", "cls": cls, "dtype": dtype,
            "records": records, "batch": batch, "m": m, "n": n, "k": k, "trans_b": trans_b}


def _dw(records, n, c, h, w, stride):
    return {"kind": "op", "op": "dw", "cls": wl.CLS_DWCONV_BIAS_RELU6, "dtype": wl.F32, "records": records, "n": n,
            "c": c, "h": h, "w": w, "stride": stride}


def _sweep(network, batch, seq):
    return {"kind": "sweep", "network": network, "batch": batch, "seq": seq, "image": 0}


def listed():
    return [
        # image classification at a throughput batch: the library's benchmark, 53 convolutions
        dict(_net("resnet50", 32), name="resnet50_b32_bf16"),
        # the same work at batch 1 in single precision: 22 kernels of a few microseconds, latency counts
        dict(_net("resnet18", 1), name="resnet18_b1_f32"),
        # a transformer encoder layer's products, 1024 tokens
        dict(_net("bert", 8, 128), name="bert_s128_b8_bf16"),
        # depthwise and pointwise layers, bound by memory
        dict(_net("mobilenetv2", 16), name="mobilenetv2_b16_f32"),
        # one ordinary 3x3 layer, called by itself
        dict(_conv(wl.CLS_CONV2D_BIAS_RELU, wl.F32, "transfer", 1, 64, 56, 56, 64, 3, 1), name="conv3x3_64_56_f32"),
        # an odd residual layer: cropped input of unequal sides, channel counts that fill no tile
        dict(_conv(wl.CLS_CONV2D_BIAS_ADD_RELU, wl.BF16, "transfer", 5, 88, 31, 45, 104, 3, 1),
             name="conv3x3_ragged_res_bf16"),
        # a layer of a program that has no pool yet
        dict(_conv(wl.CLS_CONV2D_BIAS_RELU, wl.BF16, "default", 8, 128, 28, 28, 128, 3, 1), name="conv3x3_default_bf16"),
        # the large matrix product
        dict(_gemm(wl.CLS_DENSE_ADD, wl.BF16, "transfer", 1, 4096, 4096, 4096), name="dense_4096_bf16"),
        # the smallest call: the classifier of one image
        dict(_gemm(wl.CLS_DENSE_ADD, wl.F32, "default", 1, 1, 1000, 512), name="dense_1x512_1000_f32"),
        # attention over an odd number of tokens: probabilities times values
        dict(_gemm(wl.CLS_BATCH_MATMUL, wl.BF16, "transfer", 192, 197, 64, 197, 0), name="bmm_pv_197_bf16"),
        # a depthwise layer with an odd map
        dict(_dw("transfer", 4, 120, 57, 57, 1), name="dw_120_57_f32"),
        # the search for a layer's schedules: six kernels, every same-class record of the stored pool
        dict(_sweep("bert", 8, 128), name="sweep_bert_s128_b8"),
    ]


# ---- drawn cases ---------------------------------------------------------------------------------------------------
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """Channel counts: mostly multiples of 16 or 8, some of anything."""
    v, u = _log(rng, lo, hi), rng.random()
    unit = 16 if u < 0.55 else 8 if u < 0.8 else 1
    return max(unit, v // unit * unit)


def draw(rng):
    known = [{k: v for k, v in c.items() if k != "name"} for c in listed()]
    while True:
        case = _draw(rng)
        if case not in known:
            return case


def _draw(rng):
    u = rng.random()
    if u < 0.3:
        network = rng.choice(["resnet50", "resnet18", "bert", "mobilenetv2"])
        if network == "bert":
            seq = _log(rng, 16, 384)
            return _net(network, _log(rng, 1, max(1, min(32, 4096 // seq))), seq)
        # every map's edge is a whole multiple of image / 32
        image = 32 * rng.randint(4, 8)
        batch = {"resnet50": 32, "resnet18": 8, "mobilenetv2": 16}[network] * 224 ** 2 // image ** 2
        return _net(network, _log(rng, 1, batch), image=image)
    if u < 0.38:
        seq = _log(rng, 16, 128)
        return _sweep("bert", _log(rng, 1, max(1, 1024 // seq)), seq)
    records = "default" if rng.random() < 0.3 else "transfer"
    op = rng.choice(["conv", "conv", "conv", "dense", "bmm", "dw"])
    if op == "conv":
        dtype = rng.choice([wl.F32, wl.BF16, wl.BF16])
        f, stride = rng.choice([1, 1, 3, 3, 3, 5]), rng.choice([1, 1, 1, 2])
        h = _log(rng, 7, 112)
        w = h if rng.random() < 0.6 else max(7, h + rng.randint(-h // 3, h // 3))
        if rng.random() < 0.1:  # a stem
            case = _conv(wl.CLS_CONV2D_BIAS_RELU, dtype, records, _log(rng, 1, 32), 3, 2 * h, 2 * w,
                         _channels(rng, 16, 96), 7, 2)
        else:
            cls = rng.choice([0, 1, 1, 2] if dtype == wl.BF16 else [0, 1, 1, 2, 3])
            case = _conv(cls, dtype, records, _log(rng, 1, 32), _channels(rng, 16, 1024), h, w, _channels(rng, 16, 1024),
                         f, stride)
    elif op == "dense":
        dtype = rng.choice([wl.F32, wl.BF16, wl.BF16])
        case = _gemm(rng.choice([4, 5, 6] if dtype == wl.BF16 else [4]), dtype, records, 1, _log(rng, 1, 4096),
                     _channels(rng, 16, 4096), _channels(rng, 64, 4096))
    elif op == "bmm":
        seq, hd = _log(rng, 16, 512), rng.choice([32, 64, 64, 96, 128])
        qk = rng.random() < 0.5
        case = _gemm(wl.CLS_BATCH_MATMUL, wl.BF16, records, _log(rng, 1, 192), seq, seq if qk else hd, hd if qk else seq,
                     1 if qk else 0)
    else:
        h = _log(rng, 7, 112)
        case = _dw(records, _log(rng, 1, 16), _channels(rng, 16, 960), h, h if rng.random() < 0.6 else h + rng.randint(1, 9),
                   rng.choice([1, 1, 2]))
    # keep a call within the work of the largest product above (single precision: a sixteenth of it) and 200 MB
    most = 4096.0 ** 3 * 2 / (1 if case["dtype"] == wl.BF16 else 16)
    size = "n" if op in ("conv", "dw") else "batch" if op == "bmm" else "m"
    while case[size] > 1 and (work(case)["flops"] > most or work(case)["bytes"] > 200e6):
        case[size] = (case[size] + 1) // 2
    while op == "conv" and work(case)["flops"] > most:
        case["c"] = max(16, case["c"] // 2)
    return case


# ---- shapes, records, tensors ----------------------------------------------------------------------------------------
def _kernel(case):
    dt = case["dtype"]
    if case["op"] == "conv":
        p = case["f"] // 2
        shape = wl.ConvShape(case["n"], case["c"], case["h"], case["w"], case["k"], case["f"], case["f"], case["stride"],
                             case["stride"], p, p, dt)
    elif case["op"] == "dw":
        shape = wl.ConvShape(case["n"], case["c"], case["h"], case["w"], case["c"], 3, 3, case["stride"], case["stride"],
                             1, 1, dt)
    else:
        shape = wl.GemmShape(case["batch"], case["m"], case["n"], case["k"], case["trans_b"], dt)
    return wl.Kernel(case["cls"], shape)


def _kernels(case):
    """The launches of a case, one entry each (a sweep times every distinct kernel)."""
    if case["kind"] == "op":
        return [_kernel(case)]
    ks = NETWORKS[case["network"]][1](case["batch"], case["seq"])
    if case["image"] not in (0, 224):
        ks = [dataclasses.replace(k, shape=dataclasses.replace(k.shape, h=k.shape.h * case["image"] // 224,
                                                               w=k.shape.w * case["image"] // 224))
              if k.is_conv() else k for k in ks]
    return [k for k in ks for _ in range(k.use_count if case["kind"] == "net" else 1)]


def _tensors(kernel, gen):
    """A kernel's tensors on the GPU: activations U(-1, 1) (N(0, 1) for the matrix products), weights
    N(0, 1 / fan_in), small biases, residuals U(-1, 1)."""
    s, dt = kernel.shape, api.torch_dtype(kernel.shape.dtype)

    def uniform(shape, a=1.0):
        return ((torch.rand(shape, generator=gen, device="cuda") * 2 - 1) * a).to(dt)

    def normal(shape, sd=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * sd).to(dt)

    if kernel.is_conv():
        dw = kernel.cls == wl.CLS_DWCONV_BIAS_RELU6
        t = {"x": uniform((s.n, s.h, s.w, s.c)),
             "w": normal((3, 3, s.c), 1 / 3.0) if dw else normal((s.k, s.r, s.s, s.c), (s.c * s.r * s.s) ** -0.5),
             "bias": uniform((s.k,), 0.1)}
        if kernel.cls == wl.CLS_CONV2D_BIAS_ADD_RELU:
            t["res"] = uniform((s.n, s.ho, s.wo, s.k))
        return t
    if kernel.cls == wl.CLS_BATCH_MATMUL:
        return {"a": normal((s.batch, s.m, s.k)),
                "b": normal((s.batch, s.n, s.k) if s.trans_b else (s.batch, s.k, s.n), s.k ** -0.5)}
    return {"x": normal((s.m, s.k)), "w": normal((s.n, s.k), s.k ** -0.5), "bias": uniform((s.n,), 0.1)}


def _device_kernel(kernel, gen, ws_bytes):
    s, t = kernel.shape, _tensors(kernel, gen)
    dt = api.torch_dtype(s.dtype)
    if kernel.is_conv():
        t["y"] = torch.empty((s.n, s.ho, s.wo, s.k), dtype=dt, device="cuda")
    elif kernel.cls == wl.CLS_BATCH_MATMUL:
        t["c"] = torch.empty((s.batch, s.m, s.n), dtype=dt, device="cuda")
    else:
        t["y"] = torch.empty((s.m, s.n), dtype=dt, device="cuda")
    return api.DeviceKernel(kernel.cls, s, t, 1, kernel.name, ws_bytes)


def _dtype_of(record):
    """The data type of the kernel a pool record was tuned on (the last entry of its shape)."""
    conv = record.cls in wl.CONV_CLASSES or record.cls == wl.CLS_DWCONV_BIAS_RELU6
    return record.donor_shape[11 if conv else 5]


def _workspace(kernel, records):
    plans = [api.tt_schedule_apply(r, kernel.cls, kernel.shape) for r in records]
    return max([int(p.workspace_bytes) for p in plans if p.status == api.TT_OK], default=0)


def _stored_records(network):
    with open(os.path.join(TUNED, NETWORKS[network][0] + ".json")) as f:
        return {e["name"]: e["transfer"] for e in json.load(f)["kernels"]}


def _net_records(network, kernels):
    """The stored choice for every kernel, re-applied to this shape; None (the default) where it does not apply.
    The kernels of a network come in the same order at every size, though not always under the same name."""
    made_for = {"resnet50": (32, 0), "resnet18": (1, 0), "bert": (8, 128), "mobilenetv2": (16, 0)}[network]
    stored = _stored_records(network)
    ref = [k for k in NETWORKS[network][1](*made_for) for _ in range(k.use_count)]
    out = []
    for k, r in zip(kernels, ref):
        rec = stored[r.name] and api.make_schedule(**stored[r.name])
        if rec is not None and not api.tt_schedule_apply(rec, k.cls, k.shape).runnable():
            rec = None
        out.append(rec)
    return out


_transferred = {}  # the records a program found when it started


def _transferred_record(case, kernel, gen):
    key = tuple(sorted((k, v) for k, v in case.items() if k != "name"))
    if key not in _transferred:
        pool = [r for p in POOLS for r in tune.load_pool(os.path.join(TUNED, p + ".pool"))
                if r.cls == kernel.cls and _dtype_of(r) == kernel.shape.dtype]
        dk = _device_kernel(kernel, gen, _workspace(kernel, pool))
        rows, _, _, _ = api.tt_transfer_sweep([dk], pool)
        chosen = rows[0]["chosen"]
        _transferred[key] = pool[chosen].copy() if chosen >= 0 else None
    return _transferred[key]


# ---- the measured interface --------------------------------------------------------------------------------------------
def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    kernels = _kernels(case)
    if case["kind"] == "net":
        records = _net_records(case["network"], kernels)
        dks = [_device_kernel(k, gen, api.workspace_bytes(r, k.cls, k.shape)) for k, r in zip(kernels, records)]
        return {"kind": "net", "dks": dks, "list": api.KernelList(dks, records)}
    if case["kind"] == "sweep":
        pool = tune.load_pool(os.path.join(TUNED, NETWORKS[case["network"]][0] + ".pool"))
        dks = [_device_kernel(k, gen, _workspace(k, [r for r in pool if r.cls == k.cls])) for k in kernels]
        return {"kind": "sweep", "dks": dks, "pool": pool}
    k = kernels[0]
    state = {"kind": case["op"], "cls": k.cls, "shape": api.to_c_shape(k.shape), "sched": None}
    if case["records"] == "transfer":
        state["sched"] = _transferred_record(case, k, gen)
        gen.manual_seed(int(seed))
    state.update(_tensors(k, gen))
    return state


def run(state):
    kind = state["kind"]
    if kind == "net":
        state["list"].run()
        return [dk.output() for dk in state["dks"]]
    if kind == "sweep":
        api.tt_transfer_sweep(state["dks"], state["pool"])
        return [dk.output() for dk in state["dks"]]
    if kind == "conv":
        return api.tt_conv2d_bias_relu(state["x"], state["w"], state["bias"], state.get("res"), state["shape"], state["cls"],
                                       state["sched"])
    if kind == "dense":
        return api.tt_dense_bias_relu(state["x"], state["w"], state["bias"], state["shape"], state["cls"], state["sched"])
    if kind == "bmm":
        return api.tt_batch_matmul(state["a"], state["b"], state["shape"], state["sched"])
    return api.tt_dwconv(state["x"], state["w"], state["bias"], state["shape"], state["sched"])


def work(case):
    """Every tensor of every launch once; a sweep launches each (kernel, record) pair at least three times to
    warm up, once to size its samples and once for each of ten samples."""
    ks, times = _kernels(case), 1
    total = {"bytes": 0.0, "flops": 0.0}
    if case["kind"] == "sweep":
        pool = tune.load_pool(os.path.join(TUNED, NETWORKS[case["network"]][0] + ".pool"))
    for k in ks:
        if case["kind"] == "sweep":
            times = 14 * (1 + sum(r.cls == k.cls for r in pool))
        total["bytes"] += times * k.algorithmic_bytes()
        total["flops"] += times * k.flops()
    return total


def tolerance(case):
    """Sums in single precision in another order; bf16 outputs are rounded once to 8 bits."""
    dtypes = {k.shape.dtype for k in _kernels(case)}
    return {"rel": 1e-2} if wl.BF16 in dtypes else {"rel": 1e-5}
