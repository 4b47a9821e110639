"""What `netrun` plans for networks other than the stored configurations: channel slices, buffers that are used again, pitches the fused
launches do not take.  Every plan is run on the CPU (tests/cpu_library.py) and has to give the oracle's bytes."""
import pytest
import torch

import bench
import cpu_library
from oracle import calibrate as K
from oracle import net as ONet
from workloads import nets as W

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="plans are run without a GPU")


@pytest.fixture(autouse=True)
def library(monkeypatch):
    return cpu_library.install(monkeypatch)


def builder(n, h, w, c, top=W.ACT_MAX):
    b = W._Builder("net", n, h, w, c, n)
    b.net["input_range"] = [0, top]
    return b


def integers(net):
    """Requantisation that keeps outputs spread over their range, without a calibration run: uniform bytes times uniform weights"""
    conv = {}
    for op in W.conv_ops(net):
        sigma = 127 * 127 / 3 * (op["kh"] * op["kw"] * op["cin"]) ** 0.5
        mul, shift = K.bound_params(int(2 * sigma), K.MAX_INT)
        conv[op["name"]] = dict(mul=mul, shift=shift, bound_q=K.MAX_INT, lo=0, hi=255, res_mul=20000, res_shift=15 if op["res_dtype"] == "s32" else 5)
    pool = {op["dst"]: dict(mul=K.mul_shift(64, 1)[0], shift=K.mul_shift(64, 1)[1], bound_q=K.MAX_INT) for op in net["ops"] if op["op"] == "avgpool"}
    return {"conv": conv, "avgpool": pool, "max_int": K.MAX_INT}


def straight(layers, last_total=None):
    b = builder(1, 64, 64, 64)
    cur = "raw"
    for i in range(layers):
        last = i + 1 == layers
        cur = b.conv("c%d" % i, cur, "out" if last else "t%d" % i, 64, 3, dst_c_total=last_total if last else None)
    b.net["outputs"] = ["out"]
    return b.net


def test_a_run_of_layers_is_one_chain():
    net = straight(3)
    g = cpu_library.check(net, integers(net))
    assert [st[0] for st in g.steps] == ["chain"]


def test_a_chain_the_library_refuses_runs_layer_by_layer():
    net = straight(3, last_total=72)                   # the last layer writes 64 of 72 channels: no 16-byte pitch
    g = cpu_library.check(net, integers(net))
    assert [st[0] for st in g.steps] == ["conv"] * 3 and not g.fused and not g.fused_chain


def test_buffers_used_in_turn():
    # a -> b, b -> a, a -> out: a chain from a to a would write what its other workgroups read
    b = builder(1, 64, 64, 64)
    b.conv("c0", "raw", "a", 64, 3)
    b.conv("c1", "a", "b", 64, 3)
    b.conv("c2", "b", "a", 64, 3)
    b.conv("c3", "a", "out", 64, 3)
    b.net["outputs"] = ["out"]
    cpu_library.check(b.net, integers(b.net))


def test_a_layer_that_reads_another_slice_than_the_last_one_written():
    # p fills cat[0:64], q cat[64:128], r reads cat[0:64]: r follows q in the list and takes nothing from it
    b = builder(1, 64, 64, 64)
    b.conv("p", "raw", "cat", 64, 3, dst_c_total=128)
    b.conv("q", "raw", "cat", 64, 3, dst_c_total=128, dst_c_offset=64)
    b.conv("r", "cat", "out", 64, 3, src_c=64)
    b.net["outputs"] = ["out"]
    g = cpu_library.check(b.net, integers(b.net))
    assert not g.fused_chain


def test_a_layer_that_reads_more_than_the_last_one_wrote():
    b = builder(1, 64, 64, 64)
    b.conv("p", "raw", "cat", 64, 3, dst_c_total=128, dst_c_offset=64)
    b.conv("q", "raw", "cat", 64, 3, dst_c_total=128)
    b.conv("r", "cat", "out", 64, 3)                   # all 128 channels
    b.net["outputs"] = ["out"]
    cpu_library.check(b.net, integers(b.net))


def test_a_pool_over_more_channels_than_the_layer_before_it_wrote():
    b = builder(1, 32, 32, 3, 255)
    b.conv("side", "raw", "cat", 32, 7, stride=2, pad=3, in_sub128=True, dst_c_total=64, dst_c_offset=32)
    b.conv("stem", "raw", "cat", 32, 7, stride=2, pad=3, in_sub128=True, dst_c_total=64)
    b.maxpool("cat", "pool")
    b.net["outputs"] = ["pool"]
    g = cpu_library.check(b.net, integers(b.net))
    assert not g.fused_pool
    b = builder(1, 32, 32, 3, 255)
    b.conv("stem", "raw", "t", 32, 7, stride=2, pad=3, in_sub128=True)
    b.maxpool("t", "pool")
    b.net["outputs"] = ["pool"]
    assert cpu_library.check(b.net, integers(b.net)).fused_pool


def block(middle=None, pad=0, inplace=False, projection=None, res_mode="pre"):
    """An identity (or, with a projection, opening) bottleneck block of 64 channels.  middle: the second layer reads that many channels;
    pad: of the first layer, taken back by the second"""
    b = builder(1, 16, 16, 64)
    b.conv("c0", "raw", "x", 64, 1)
    if middle:
        b.conv("side", "raw", "t", middle - 64, 1, dst_c_total=middle, dst_c_offset=64)
    b.conv("c1", "x", "t", 64, 1, pad=pad, dst_c_total=middle)
    b.conv("c2", "t", "u", 64, 3, pad=1 - pad)
    skip = "x"
    if projection:
        skip = b.conv("proj", "x", "sk", projection, 1, out_mode="raw_s32", role="projection")
    b.conv("c3", "u", "x" if inplace else "y", projection or 64, 1, res=skip, res_mode=res_mode)
    b.net["outputs"] = ["x" if inplace else "y"]
    return b.net


@pytest.mark.parametrize("kw, kinds", [
    (dict(), ["conv", "block"]), (dict(middle=128), ["conv"] * 5), (dict(pad=1), ["conv"] * 4), (dict(projection=256), ["conv", "projblock"]),
    (dict(projection=256, res_mode="post"), ["conv"] * 5), (dict(inplace=True), ["conv"] * 4), (dict(projection=256, pad=1), ["conv"] * 3 + ["dual"]),
], ids=str)
def test_bottleneck_blocks_of_other_forms(kw, kinds):
    net = block(**kw)
    assert [st[0] for st in cpu_library.check(net, integers(net)).steps] == kinds


def test_a_merge_that_overwrites_what_its_projection_reads():
    b = builder(1, 16, 16, 64)
    b.conv("c0", "raw", "x", 64, 1)
    b.conv("c1", "x", "t", 64, 1)
    b.conv("proj", "x", "sk", 64, 1, out_mode="raw_s32", role="projection")
    b.conv("c2", "t", "x", 64, 1, res="sk", res_mode="pre")
    b.net["outputs"] = ["x"]
    cpu_library.check(b.net, integers(b.net))


def test_two_branches_on_one_channel_range():
    # the second branch overwrites the first one's channels
    b = builder(1, 64, 64, 64)
    b.conv("a", "raw", "t", 32, 5, dst_c_total=48)
    b.conv("b", "raw", "t", 16, 3, dst_c_total=48, dst_c_offset=16)
    b.conv("c", "t", "out", 16, 1, src_c=32)
    b.net["outputs"] = ["out"]
    g, want = cpu_library.planned(b.net, integers(b.net))
    assert (g.result("out") == want["out"]).all() and [st[0] for st in g.steps] == ["conv"] * 3


def test_a_pair_that_returns_to_its_first_buffer():
    # t -> y -> t: every workgroup has read its own pixels of t before it writes them
    b = builder(1, 48, 48, 64)
    b.conv("c0", "raw", "t", 64, 1)
    b.conv("c1", "t", "y", 256, 1)
    b.conv("c2", "y", "t", 64, 1)
    b.net["outputs"] = ["y", "t"]
    g = cpu_library.check(b.net, integers(b.net))
    assert [st[0] for st in g.steps] == ["conv", "pair"]


@pytest.mark.parametrize("next_dst, height, kinds", [("v", 16, ["conv", "conv", "triple"]), (None, 16, ["conv", "conv", "triple"]),
                                                     ("t", 16, ["conv", "conv", "triple", "conv"]), ("u", 16, ["conv", "conv", "triple", "conv"]),
                                                     ("v", 15, ["conv", "conv", "conv", "conv", "conv"])], ids=str)
def test_a_block_boundary_of_256_channels(next_dst, height, kinds):
    # the 3x3 layer's input has neighbours' readers, and its output is written too: the next block's first layer stays outside if it goes there
    b = builder(1, height, 16, 64)
    b.conv("c0", "raw", "x", 1024, 1)
    b.conv("c1", "x", "t", 256, 1)
    b.conv("c2", "t", "u", 256, 3)
    b.conv("c3", "u", "y", 1024, 1, res="x", res_mode="pre")
    if next_dst:
        b.conv("d1", "y", next_dst, 256, 1)
    b.net["outputs"] = ["y"] + ([next_dst] if next_dst else [])
    g, want = cpu_library.planned(b.net, integers(b.net))
    assert [st[0] for st in g.steps] == kinds
    for name in ["y"] + ([next_dst] if next_dst else ["u"]):
        assert (g.result(name) == want[name]).all(), name


def merges(second_reader=False, output=False, overwrite=False, unread=False):
    """x -> projection -> sk and x -> t -> merge with sk.  second_reader: another merge reads sk; output: sk is a result; overwrite: x is
    written again before the merge; unread: no merge at all"""
    b = builder(1, 16, 16, 64)
    b.conv("c0", "raw", "x", 64, 1)
    b.conv("c1", "x", "t", 64, 1)
    b.conv("proj", "x", "sk", 64, 1, out_mode="raw_s32", role="projection")
    if overwrite:
        b.conv("again", "t", "x", 64, 1)
    if not unread:
        b.conv("c2", "t", "y", 64, 1, res="sk", res_mode="pre")
    if second_reader:
        b.conv("c3", "y", "z", 64, 1, res="sk", res_mode="pre")
    b.net["outputs"] = ["z" if second_reader else "t" if unread else "y"] + (["sk"] if output else [])
    return b.net


@pytest.mark.parametrize("kw", [{}, dict(second_reader=True), dict(output=True), dict(overwrite=True), dict(unread=True, output=True), dict(unread=True)], ids=str)
def test_projections_and_who_reads_them(kw):
    net = merges(**kw)
    g = cpu_library.check(net, integers(net))
    assert bool(g.fused_proj) == (not kw)


@pytest.mark.parametrize("make, per_channel, kinds", [
    (lambda: W.vdsr(64, 72, depth=9), False, {"conv", "chain"}),
    (lambda: W.vrcnn(64, 72), False, {"conv", "twin", "twin_last"}),
    (lambda: W.resnet(2, [2, 1, 1, 1], "tiny", image=64, calib_images=2, classes=10), False, {"convpool", "projblock", "block", "dual", "conv", "avgpool"}),
    (lambda: W.resnet(2, [2, 1, 1, 1], "tiny", image=64, calib_images=2, classes=10), True,
     {"convpool_pc", "projblock_pc", "block_pc", "dual_pc", "conv", "conv_pc", "avgpool"}),
    (lambda: W.resnet_basic(2, [1, 1, 1, 1], "tiny18", image=64, calib_images=2, classes=10), False, {"convpool", "conv", "avgpool"}),
], ids=["vdsr", "vrcnn", "bottleneck", "bottleneck_pc", "basic"])
def test_small_networks_of_every_kind(make, per_channel, kinds, monkeypatch):
    net = make()
    calib, _ = ONet.calibrate(net, 0, per_channel=per_channel)
    g = cpu_library.check(net, calib)
    assert {st[0] for st in g.steps} == kinds
    # the benchmark counts every convolution once: in any launch it is part of, also when the batch runs as two halves
    monkeypatch.setattr(type(g), "HALVES_MIN_PIXELS", 0)
    halves = cpu_library.planned(net, calib)[0]
    assert halves.parts == min(2, net["buffers"]["raw"]["shape"][0])
    for q in (g, halves):
        work = [bench.step_work(q, i) for i in range(len(q.steps))]
        assert sum(w[0] for w in work if w is not None) == 2 * W.conv_macs(net)
        assert {st[0] for st, w in zip(q.steps, work) if w is None} <= {"maxpool", "avgpool"}
        assert all(bench.step_name(q, i).startswith(q.steps[i][1]["name"][:4]) for i, w in enumerate(work) if w is not None)
