"""A batch run as two halves side by side (GpuNet's parts, icnn_run_lanes): the same bytes as the batch in one piece."""
import json

import numpy as np
import pytest
import torch

from oracle import net as ONet
from workloads import nets as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("images", [2, 3, 5])
@pytest.mark.parametrize("per_channel", [False, True])
def test_halves_of_a_small_batch(images, per_channel, monkeypatch):
    from paper_2006_11735_amd import binding as B
    from paper_2006_11735_amd.netrun import GpuNet
    net = W.resnet(images, [2, 1, 1, 1], "tiny", image=64, calib_images=2, classes=10)
    calib, _ = ONet.calibrate(net, 0, per_channel=per_channel)
    monkeypatch.setattr(GpuNet, "HALVES_MIN_PIXELS", 0)
    g = GpuNet(net, 0, calib)
    assert isinstance(g._calls, B.Lanes) and len(g.fused) == len(set(g.fused))
    want = ONet.run(net, 0, calib)
    g.set_input()

    def check():
        for name in net["buffers"]:
            if name not in g.fused:
                assert (g.result(name) == want[name]).all(), name
    g.run()
    check()
    for i in range(len(g.steps)):                  # step by step on one stream
        g.run_step(i)
    check()
    # captured: the side stream joins the capture and leaves it again
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        g.run()
        s.synchronize()
        with torch.cuda.graph(graph, stream=s):
            g.run()
    for _ in range(3):
        for name in net["buffers"]:
            if name != net["input"]:
                g.buf[name].zero_()
        graph.replay()
        torch.cuda.synchronize()
        check()
        g.run()
        check()


@pytest.mark.parametrize("images", [83, 85])
def test_a_batch_on_either_side_of_the_rule(images, monkeypatch):
    from paper_2006_11735_amd import binding as B
    from paper_2006_11735_amd.netrun import GpuNet
    net = W.resnet18(images)
    calib = json.load(open(ONet.stored_calib_path("cfg5", 0)))
    x = np.random.default_rng(1).integers(0, 256, net["buffers"]["raw"]["shape"], dtype=np.uint8)
    g = GpuNet(net, 0, calib)
    assert isinstance(g._calls, B.Lanes) == (images == 85)
    monkeypatch.setattr(GpuNet, "HALVES_MIN_PIXELS", 1 << 40)
    one = GpuNet(net, 0, calib)
    for q in (g, one):
        q.set_input(x)
        q.run()
    for name in net["buffers"]:
        if name not in g.fused and name not in one.fused:
            assert torch.equal(g.buf[name], one.buf[name]), name


def test_lanes_refuse_what_they_cannot_hold():
    from paper_2006_11735_amd import binding as B
    calls = [B.Calls([]) for _ in range(17)]
    with pytest.raises(B.IcnnError):
        B.Lanes(calls)
    lanes = B.Lanes(calls[:2])
    lanes.run()
    lanes._lists = calls[:3]
    with pytest.raises(B.IcnnError):
        lanes.run()
