"""What is measured: the work a user of this library has it do, over the range of sizes it is used at.

Whole integer networks run through `netrun.GpuNet` (classification at serving batch sizes from a single picture to a
full batch, restoration of luma planes from small pictures to a 2560x1600 frame), and single calls through `binding`
(one convolution layer, one stand-alone rescaled addition).  A network's weights and calibration integers are the
stored ones of its configuration (a user's model does not change between calls); its pictures come from the seed.
All results are integers and have to be the same bit for bit.
"""
import functools
import json
import math
import os

import numpy as np
import torch

from paper_2006_11735_amd import binding as B
from paper_2006_11735_amd import convert
from paper_2006_11735_amd.netrun import GpuNet
from workloads import nets as W

CALIB = os.path.join(os.path.dirname(os.path.abspath(W.__file__)), "calib")
# residual networks: constructor, stored calibration, largest batch
RESNETS = {"resnet18": (W.resnet18, "cfg5_seed0", 64), "resnet50": (W.resnet50, "cfg3_seed0", 64),
           "resnet50_pc": (W.resnet50, "cfg3_seed0_pc", 64), "resnet152": (W.resnet152, "cfg4_seed0", 128)}


def listed():
    return [
        # one integer layer called on its own: the smallest call there is
        {"name": "layer_56x56x64", "kind": "layer", "n": 1, "h": 56, "w": 56, "cin": 64, "cout": 64, "k": 3, "stride": 1, "skip": False},
        # one picture classified as it arrives: the latency end of serving
        {"name": "resnet50_b1", "kind": "resnet", "net": "resnet50", "batch": 1},
        # the handful of requests a server collects within its deadline
        {"name": "resnet50_b9", "kind": "resnet", "net": "resnet50", "batch": 9},
        # the benchmark's own configuration: throughput
        {"name": "resnet50_b64", "kind": "resnet", "net": "resnet50", "batch": 64},
        # the same network with one multiplier and shift per output channel
        {"name": "resnet50_pc_b64", "kind": "resnet", "net": "resnet50_pc", "batch": 64},
        # basic blocks: the small classifier
        {"name": "resnet18_b64", "kind": "resnet", "net": "resnet18", "batch": 64},
        # the largest throughput workload
        {"name": "resnet152_b128", "kind": "resnet", "net": "resnet152", "batch": 128},
        # super-resolution of one luma plane
        {"name": "vdsr_256x256", "kind": "vdsr", "h": 256, "w": 256, "full8": False},
        # the same with 8-bit activations on a picture that is no multiple of anything
        {"name": "vdsr8_181x243", "kind": "vdsr", "h": 181, "w": 243, "full8": True},
        # artefact removal on a 720p frame, and on the largest frame
        {"name": "vrcnn_720x1280", "kind": "vrcnn", "h": 720, "w": 1280},
        {"name": "vrcnn_1600x2560", "kind": "vrcnn", "h": 1600, "w": 2560},
        # a residual merge as a pass of its own (the 56x56x256 maps of a batch of 64)
        {"name": "add_u8_200704x256", "kind": "add", "pixels": 200704, "c": 256, "b_s32": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "resnet", "resnet", "resnet", "vdsr", "vrcnn", "add"])
    if kind == "layer":
        # layers as the networks have them: maps from 7x7 to 112x112, 16 to 512 channels
        stride = rng.choice([1, 1, 2])
        return {"kind": kind, "n": _log(rng, 1, 16), "h": _log(rng, 7, 112), "w": _log(rng, 7, 112), "cin": 16 * _log(rng, 1, 32),
                "cout": 16 * _log(rng, 1, 32), "k": rng.choice([1, 3]), "stride": stride, "skip": rng.random() < 0.3}
    if kind == "resnet":
        net = rng.choice(sorted(RESNETS))
        return {"kind": kind, "net": net, "batch": _log(rng, 1, RESNETS[net][2])}
    if kind == "vdsr":
        return {"kind": kind, "h": _log(rng, 96, 384), "w": _log(rng, 96, 384), "full8": rng.random() < 0.3}
    if kind == "vrcnn":
        h = _log(rng, 240, 1600)
        return {"kind": kind, "h": h, "w": int(round(h * rng.uniform(1.25, 1.6)))}
    return {"kind": kind, "pixels": _log(rng, 3136, 200704), "c": 16 * _log(rng, 4, 16), "b_s32": rng.random() < 0.5}


def _net_of(case):
    """(network, stored calibration's name)"""
    if case["kind"] == "resnet":
        make, calib, _ = RESNETS[case["net"]]
        return make(case["batch"]), calib
    if case["kind"] == "vdsr":
        return W.vdsr(case["h"], case["w"]), "cfg1_seed0_a255" if case["full8"] else "cfg1_seed0"
    return W.vrcnn(case["h"], case["w"]), "cfg2_seed0"


@functools.lru_cache(maxsize=None)
def _model(make_key, calib):
    """The stored model of a family: its weights (which depend on no picture size and no batch) and its integers."""
    if make_key in RESNETS:
        net = RESNETS[make_key][0](1)
    else:
        net = W.vdsr(96, 96) if make_key == "vdsr" else W.vrcnn(96, 96)
    with open(os.path.join(CALIB, calib + ".json")) as f:
        integers = json.load(f)
    return {op["name"]: (W.weight_tensor(op, 0), W.bias_tensor(op, 0)) for op in W.conv_ops(net)}, integers


def _bytes(shape, lo, hi, gen, dtype):
    return torch.randint(lo, hi + 1, shape, device="cuda", dtype=torch.int32, generator=gen).to(dtype)


def _prepare_layer(case, gen):
    n, h, w, cin, cout, k = (case[q] for q in ("n", "h", "w", "cin", "cout", "k"))
    # accumulators of uniform bytes times uniform weights: the bound sits at the 99.9th percentile (3.09 sigma)
    sigma = (127 * 127 / 3) * math.sqrt(k * k * cin)
    mul, shift = convert.bound_params(int(3.09 * sigma), 127)
    d = B.conv_desc(n=n, h=h, w=w, cin=cin, in_c_stride=cin, cout=cout, kh=k, kw=k, stride_h=case["stride"], stride_w=case["stride"],
                    pad_h=k // 2, pad_w=k // 2, out_c_stride=cout, mul=mul, shift=shift)
    ho, wo = B.iconv2d_out_hw(d)
    res = None
    if case["skip"]:
        d.res_mode, d.res_dtype, d.res_c_stride = B.ICNN_RES_PRE, B.ICNN_U8, cout
        d.res_mul, d.res_shift = convert.mul_shift(127, int(3.09 * sigma))
        res = _bytes((n, ho, wo, cout), 0, 127, gen, torch.uint8)
    x = _bytes((n, h, w, cin), 0, 127, gen, torch.uint8)
    wt = _bytes((cout, k, k, cin), -127, 127, gen, torch.int8)
    bias = _bytes((cout,), -4096, 4096, gen, torch.int32)
    packed = torch.empty(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda")
    B.iconv2d_prepack_weights(d, wt, packed)
    ws_bytes = B.iconv2d_workspace_bytes(d)
    ws = torch.zeros(ws_bytes, dtype=torch.uint8, device="cuda") if ws_bytes else None
    y = torch.empty((n, ho, wo, cout), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()                                      # the plain weights go away with this function
    return {"kind": "layer", "args": (d, x, packed, bias, res, y, ws), "y": y}


def _prepare_add(case, gen):
    px, c, s32 = case["pixels"], case["c"], case["b_s32"]
    # main path and skip operand in the sizes a merge sees: a stored map, and a stored map or a projection's int32 sums
    d = B.add_desc(count_pixels=px, c=c, a_c_stride=c, b_c_stride=c, out_c_stride=c, out_mode=B.ICNN_OUT_CLAMP_U8, lo=0, hi=127,
                   mul=23000, shift=15, a_dtype=B.ICNN_U8, b_dtype=B.ICNN_S32 if s32 else B.ICNN_U8, b_mul=17000, b_shift=27 if s32 else 15)
    a = _bytes((px, c), 0, 127, gen, torch.uint8)
    b = _bytes((px, c), -200000, 200000, gen, torch.int32) if s32 else _bytes((px, c), 0, 127, gen, torch.uint8)
    return {"kind": "add", "d": d, "a": a, "b": b, "y": torch.empty((px, c), dtype=torch.uint8, device="cuda")}


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    if case["kind"] == "layer":
        return _prepare_layer(case, gen)
    if case["kind"] == "add":
        return _prepare_add(case, gen)
    net, calib = _net_of(case)
    weights, integers = _model(case.get("net", case["kind"]), calib)
    g = GpuNet(net, 0, integers, weights=weights)
    shape = net["buffers"]["raw"]["shape"]
    g.set_input(np.random.default_rng(int(seed)).integers(0, 256, shape, dtype=np.uint8))
    return {"kind": "net", "net": g}


def run(state):
    if state["kind"] == "layer":
        B.iconv2d_brelu(*state["args"])
        return state["y"]
    if state["kind"] == "add":
        B.iadd_rescale(state["d"], state["a"], state["b"], state["y"])
        return state["y"]
    g = state["net"]
    g.run()
    return {name: g.buf[name] for name in g.net["outputs"]}


def work(case):
    if case["kind"] == "layer":
        n, h, w, cin, cout, k, s = (case[q] for q in ("n", "h", "w", "cin", "cout", "k", "stride"))
        px = n * ((h + 2 * (k // 2) - k) // s + 1) * ((w + 2 * (k // 2) - k) // s + 1)
        return {"bytes": n * h * w * cin + cout * k * k * cin + 4 * cout + px * cout * (2 if case["skip"] else 1),
                "flops": 2 * px * cout * k * k * cin}
    if case["kind"] == "add":
        return {"bytes": case["pixels"] * case["c"] * (6 if case["b_s32"] else 3), "flops": 0}
    net, _ = _net_of(case)
    total = int(np.prod(net["buffers"]["raw"]["shape"]))
    total += sum(op["cout"] * (op["kh"] * op["kw"] * op["cin"] + 4) for op in W.conv_ops(net))
    for name in net["outputs"]:
        b = net["buffers"][name]
        total += int(np.prod(b["shape"])) * (4 if b["dtype"] == "s32" else 1)
    return {"bytes": total, "flops": 2 * W.conv_macs(net)}


def tolerance(case):
    return "exact"
