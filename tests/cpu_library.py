"""The library without a GPU, for tests of what `netrun` plans: every call goes through the library's own host checks (which refuse it as
on a GPU) and, once they accept it, is computed by the oracle layer by layer, the middle tensors of a fused launch in temporaries.

A fused launch computes its workgroups in no order, so a call whose output overlaps what others of its workgroups read has no
defined result: the stand-in fails the test instead of picking one.
"""
import contextlib

import numpy as np
import torch

from oracle import net as ONet
from oracle import oracle as O

_OUT = {0: "brelu", 1: "clamp_u8", 2: "linear_s8", 3: "raw_s32"}
_RES = {0: "none", 1: "pre", 2: "post"}
_BYTES = {0: 1, 1: 1, 2: 4}


def _bytes_of(t, pitch, offset, channels, item):
    """(first byte, end, pitch, width) in bytes of a channel slice"""
    at = t.data_ptr() + offset * item
    return at, t.data_ptr() + t.numel() * t.element_size(), pitch * item, channels * item


def _overlap(a, b):
    if a[0] >= b[1] or b[0] >= a[1]:
        return False
    if a[2] == b[2]:                                   # slices of one buffer
        d = (b[0] - a[0]) % a[2]
        return not (d >= a[3] and d + b[3] <= a[2])
    return True


class CpuLibrary:
    def __init__(self, B):
        self.B = B
        self.weights, self.params = {}, {}
        self.real = {name: getattr(B, name) for name in self.NAMES}

    NAMES = ("iconv2d_brelu", "iconv2d_brelu_pc", "iconv2d_dual_brelu", "iconv2d_dual_brelu_pc", "iconv2d_bottleneck_brelu",
             "iconv2d_bottleneck_brelu_pc", "iconv2d_bottleneck_dual_brelu", "iconv2d_bottleneck_dual_brelu_pc", "iconv2d_pair_brelu",
             "iconv2d_pair_brelu_pc", "iconv2d_triple_brelu", "iconv2d_triple_brelu_pc", "iconv2d_twin_brelu", "iconv2d_twin_last_brelu", "iconv2d_maxpool_brelu", "iconv2d_maxpool_brelu_pc",
             "iconv2d_chain_brelu", "imaxpool2d_u8", "iavgpool_global_u8")

    # ---- what a GpuNet prepares
    def prepack_weights(self, desc, w, packed, stream=None):
        self.weights[packed.data_ptr()] = w.numpy().copy(), packed

    def prepack_params(self, desc, arrs, packed, stream=None):
        self.params[packed.data_ptr()] = [a.numpy().copy() for a in arrs], packed

    # ---- one layer
    def layer(self, d, x, wp, bias, res=None, out=None, pc=None):
        """x, res, out: numpy [n, h, w, pitch]; the written (or a new) output array"""
        assert d.stride_h == d.stride_w and d.pad_h == d.pad_w and x.shape == (d.n, d.h, d.w, x.shape[3])
        kw = {}
        if pc is not None:
            kw = dict(zip(("mul_c", "shift_c", "res_mul_c", "res_shift_c"), self.params[pc.data_ptr()][0]))
        if d.out_mode == 3:
            kw.pop("mul_c", None), kw.pop("shift_c", None)
        mode = _RES[d.res_mode] if res is not None else "none"
        return O.conv2d(x.copy(), self.weights[wp.data_ptr()][0], bias.numpy(), stride=d.stride_h, pad=d.pad_h, mul=d.mul, shift=d.shift,
                        bound_q=d.bound_q, lo=d.lo, hi=d.hi, out_mode=_OUT[d.out_mode], res=None if res is None else res.copy(), res_mode=mode,
                        res_mul=d.res_mul, res_shift=d.res_shift, in_sub128=bool(d.in_sub128), cin=d.cin, out=out,
                        out_c_offset=d.out_c_offset if out is not None else 0, **kw)

    @staticmethod
    def reads(d, x):
        return _bytes_of(x, d.in_c_stride, 0, d.cin, 1)

    @staticmethod
    def writes(d, y):
        return _bytes_of(y, d.out_c_stride, d.out_c_offset, d.cout, 4 if d.out_mode == 3 else 1)

    def no_race(self, outs, ins, in_place=False):
        """in_place: the kernel's workgroups have read all of their own pixels before they write them"""
        for o in outs:
            for i in ins:
                assert not _overlap(o, i) or (in_place and o[1:3] == i[1:3]), "a fused launch writes what its other workgroups read"

    # ---- the calls, computed
    def iconv2d_brelu(self, d, x, wp, b, res, y, ws=None):
        self.layer(d, x.numpy(), wp, b, None if res is None else res.numpy(), y.numpy())

    def iconv2d_brelu_pc(self, d, x, wp, b, pc, res, y, ws=None):
        self.layer(d, x.numpy(), wp, b, None if res is None else res.numpy(), y.numpy(), pc)

    def iconv2d_dual_brelu(self, dm, xm, wm, bm, dp, xp, wp, bp, y, pc=None):
        self.no_race([self.writes(dm, y)], [self.reads(dm, xm), self.reads(dp, xp)])
        self.layer(dm, xm.numpy(), wm, bm, self.layer(dp, xp.numpy(), wp, bp), y.numpy(), pc)

    def iconv2d_dual_brelu_pc(self, dm, xm, wm, bm, pc, dp, xp, wp, bp, y):
        self.iconv2d_dual_brelu(dm, xm, wm, bm, dp, xp, wp, bp, y, pc)

    def iconv2d_bottleneck_brelu(self, d1, x, w1, b1, d2, w2, b2, d3, w3, b3, res, y, pcs=(None, None, None)):
        self.no_race([self.writes(d3, y)], [self.reads(d1, x)])
        t = self.layer(d2, self.layer(d1, x.numpy(), w1, b1, pc=pcs[0]), w2, b2, pc=pcs[1])
        self.layer(d3, t, w3, b3, None if res is None else res.numpy(), y.numpy(), pcs[2])

    def iconv2d_bottleneck_brelu_pc(self, d1, x, w1, b1, p1, d2, w2, b2, p2, d3, w3, b3, p3, res, y):
        self.iconv2d_bottleneck_brelu(d1, x, w1, b1, d2, w2, b2, d3, w3, b3, res, y, (p1, p2, p3))

    def iconv2d_bottleneck_dual_brelu(self, d1, x, w1, b1, d2, w2, b2, d3, w3, b3, dp, wp, bp, y, pcs=(None, None, None)):
        self.no_race([self.writes(d3, y)], [self.reads(d1, x)])
        t = self.layer(d2, self.layer(d1, x.numpy(), w1, b1, pc=pcs[0]), w2, b2, pc=pcs[1])
        self.layer(d3, t, w3, b3, self.layer(dp, x.numpy(), wp, bp), y.numpy(), pcs[2])

    def iconv2d_bottleneck_dual_brelu_pc(self, d1, x, w1, b1, p1, d2, w2, b2, p2, d3, w3, b3, p3, dp, wp, bp, y):
        self.iconv2d_bottleneck_dual_brelu(d1, x, w1, b1, d2, w2, b2, d3, w3, b3, dp, wp, bp, y, (p1, p2, p3))

    def iconv2d_pair_brelu(self, d3, t, w3, b3, res, y, d1, w1, b1, z, pcs=(None, None)):
        ins = [self.reads(d3, t)] + ([] if res is None else [_bytes_of(res, d3.res_c_stride, 0, d3.cout, 1)])
        self.no_race([self.writes(d3, y), self.writes(d1, z)], ins, in_place=True)
        self.no_race([self.writes(d1, z)], [self.writes(d3, y)])
        wide = self.layer(d3, t.numpy(), w3, b3, None if res is None else res.numpy(), y.numpy(), pcs[0])
        self.layer(d1, wide[..., d3.out_c_offset:d3.out_c_offset + d3.cout], w1, b1, out=z.numpy(), pc=pcs[1])

    def iconv2d_pair_brelu_pc(self, d3, t, w3, b3, p3, res, y, d1, w1, b1, p1, z):
        self.iconv2d_pair_brelu(d3, t, w3, b3, res, y, d1, w1, b1, z, (p3, p1))

    def iconv2d_triple_brelu(self, d2, t, w2, b2, t2, d3, w3, b3, res, y, d1, w1, b1, z, lanes=1, pcs=(None, None, None)):
        outs = ([] if t2 is None else [self.writes(d2, t2)]) + [self.writes(d3, y)] + ([] if d1 is None else [self.writes(d1, z)])
        self.no_race(outs, [self.reads(d2, t)])
        if res is not None:
            self.no_race(outs, [_bytes_of(res, d3.res_c_stride, 0, d3.cout, 1)], in_place=True)
        for k, o in enumerate(outs):
            self.no_race([o], outs[:k])
        mid = self.layer(d2, t.numpy(), w2, b2, out=None if t2 is None else t2.numpy(), pc=pcs[0])
        wide = self.layer(d3, mid[..., d2.out_c_offset if t2 is not None else 0:][..., :d2.cout], w3, b3, None if res is None else res.numpy(), y.numpy(), pcs[1])
        if d1 is not None:
            self.layer(d1, wide[..., d3.out_c_offset:d3.out_c_offset + d3.cout], w1, b1, out=z.numpy(), pc=pcs[2])

    def iconv2d_triple_brelu_pc(self, d2, t, w2, b2, p2, t2, d3, w3, b3, p3, res, y, d1, w1, b1, p1, z, lanes=1):
        self.iconv2d_triple_brelu(d2, t, w2, b2, t2, d3, w3, b3, res, y, d1, w1, b1, z, lanes, (p2, p3, p1))

    def iconv2d_twin_brelu(self, da, x, wa, ba, ya, db, wb, bb, yb):
        self.no_race([self.writes(da, ya), self.writes(db, yb)], [self.reads(da, x)])
        self.no_race([self.writes(da, ya)], [self.writes(db, yb)])
        self.layer(da, x.numpy(), wa, ba, out=ya.numpy())
        self.layer(db, x.numpy(), wb, bb, out=yb.numpy())

    def iconv2d_twin_last_brelu(self, da, x, wa, ba, db, wb, bb, dc, wc, bc, res, y):
        self.no_race([self.writes(dc, y)], [self.reads(da, x)])
        t = np.zeros((da.n, da.h, da.w, dc.cin), dtype=np.uint8)
        self.layer(da, x.numpy(), wa, ba, out=t)
        self.layer(db, x.numpy(), wb, bb, out=t)
        self.layer(dc, t, wc, bc, None if res is None else res.numpy(), y.numpy())

    def iconv2d_maxpool_brelu(self, d, k, stride, pad, x, wp, b, y, pc=None):
        pooled = O.maxpool2d(self.layer(d, x.numpy(), wp, b, pc=pc), k, stride, pad)
        y.numpy()[..., d.out_c_offset:d.out_c_offset + d.cout] = pooled

    def iconv2d_maxpool_brelu_pc(self, d, k, stride, pad, x, wp, b, pc, y):
        self.iconv2d_maxpool_brelu(d, k, stride, pad, x, wp, b, y, pc)

    def iconv2d_chain_brelu(self, descs, x, packs, biases, y):
        self.no_race([self.writes(descs[-1], y)], [self.reads(descs[0], x)])
        cur = x.numpy()
        for i, (d, w, b) in enumerate(zip(descs, packs, biases)):
            cur = self.layer(d, cur, w, b, out=y.numpy() if i + 1 == len(descs) else None)

    def imaxpool2d_u8(self, n, h, w, c, k, stride, pad, x, y):
        y.numpy()[...] = O.maxpool2d(x.numpy(), k, stride, pad)

    def iavgpool_global_u8(self, n, h, w, c, mul, shift, bound_q, x, y):
        y.numpy()[...] = O.avgpool_global(x.numpy(), mul, shift, bound_q)

    # ---- a call: refused by the library, or computed here
    def call(self, name):
        def f(*args, stream=None):
            try:
                self.real[name](*args, stream=0)
            except self.B.IcnnError as e:
                if e.code != self.B.ICNN_E_LAUNCH:             # accepted, and no GPU to launch on
                    raise
            else:
                raise AssertionError("there is a GPU")
            getattr(self, name)(*args)
        return f


def install(monkeypatch):
    """Puts the stand-in under `netrun` (its B, its table of functions, its device)."""
    from paper_2006_11735_amd import binding as B
    from paper_2006_11735_amd import netrun
    assert not torch.cuda.is_available()
    lib = CpuLibrary(B)
    calls = {name: lib.call(name) for name in lib.NAMES}
    table = {kind: calls[f.__name__] for kind, f in netrun.GpuNet._FUNCTIONS.items()}
    for name, f in calls.items():
        monkeypatch.setattr(B, name, f)
    monkeypatch.setattr(netrun.GpuNet, "_FUNCTIONS", table)
    monkeypatch.setattr(B, "iconv2d_prepack_weights", lib.prepack_weights)
    monkeypatch.setattr(B, "iconv2d_prepack_channel_params", lib.prepack_params)
    monkeypatch.setattr(B, "channel_params", lambda *arrs: arrs)
    monkeypatch.setattr(B, "Lanes", list)
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    monkeypatch.setattr(torch.cuda, "device", lambda *a: contextlib.nullcontext())
    return lib


def planned(net, calib, seed=0, **kw):
    """The network as it is planned, run once: (GpuNet, the oracle's buffers)"""
    from paper_2006_11735_amd.netrun import GpuNet
    g = GpuNet(net, seed, calib, device="cpu", **kw)
    for name, t in g.buf.items():                      # what the calls made while planning left behind must not help
        t.fill_(0 if name == net["input"] else 77)
    g.set_input()
    for i in range(len(g.steps)):
        g.run_step(i)
    return g, ONet.run(net, seed, calib)


def check(net, calib, **kw):
    """Plans and runs `net`; every stored buffer equals the oracle's."""
    g, want = planned(net, calib, **kw)
    for name in net["buffers"]:
        if name not in g.fused:
            got = g.buf[name].numpy()
            writers = [op for op in net["ops"] if op["dst"] == name]
            seen = np.zeros(got.shape[3], dtype=bool)
            for op in writers:
                seen[op.get("dst_c_offset", 0):op.get("dst_c_offset", 0) + op.get("cout", got.shape[3])] = True
            assert (got[..., seen] == want[name][..., seen]).all(), name
    assert not set(net["outputs"]) & set(g.fused)
    return g
