"""Runs a synthetic integer network (workloads.nets) on the GPU through the C
boundary.  This is harness code: it owns the device buffers (torch tensors),
prepacks the weights once, and then issues one library call per layer.  All
arithmetic happens inside the library.
"""
import numpy as np
import torch

from workloads import nets as W
from . import binding as B

_OUT = {"brelu": B.ICNN_OUT_BRELU_U8, "clamp_u8": B.ICNN_OUT_CLAMP_U8,
        "linear_s8": B.ICNN_OUT_LINEAR_S8, "raw_s32": B.ICNN_OUT_RAW_S32}
_RES = {"none": B.ICNN_RES_NONE, "pre": B.ICNN_RES_PRE, "post": B.ICNN_RES_POST}
_DT = {"u8": B.ICNN_U8, "s8": B.ICNN_S8, "s32": B.ICNN_S32}


class GpuNet:
    def __init__(self, net, seed, calib, images=None, device="cuda:0", fuse=True, weights=None, fuse_blocks=None):
        """fuse: run a projection conv and the block's last conv that consumes it as one
        iconv2d_dual_brelu launch where the library accepts that (the int32 skip buffer then
        stays untouched).  fuse_blocks (default: as fuse): run an identity bottleneck block (1x1, 3x3, 1x1 with
        the block input as skip operand) as one iconv2d_bottleneck_brelu launch where the library accepts
        that (its two middle buffers then stay untouched).  weights: optional {layer: (int8 [cout,kh,kw,cin], int32 [cout])}, e.g.
        from paper_2006_11735_amd.convert, instead of the seeded synthetic tensors."""
        self.weights = weights
        if not torch.cuda.is_available():
            raise RuntimeError("GpuNet needs a GPU: there is no CPU fallback")
        self.net, self.seed, self.calib = net, seed, calib
        self.device = torch.device(device)
        n_full = net["buffers"]["raw"]["shape"][0]
        self.images = n_full if images is None else min(images, n_full)
        self.buf = {}
        for name, b in net["buffers"].items():
            shape = [self.images] + b["shape"][1:]
            dt = torch.int32 if b["dtype"] == "s32" else torch.uint8
            self.buf[name] = torch.zeros(shape, dtype=dt, device=self.device)
        self.steps = []
        self.fused = []                     # names of int32 skip buffers that are never written
        self.fused_proj = {}                # main conv name -> the projection op fused into it
        self.fused_block = {}               # last conv name -> (first, middle) conv ops fused into its launch
        self.fused_block_pc = {}            # the same with requantisation per output channel
        self.fused_pool = {}                # first conv name -> the max-pool op fused into its launch
        self.fused_pair = {}                # block-closing conv name -> the next block's opening conv op in its launch
        self.fused_triple = {}              # block-closing conv name -> (3x3 conv op before it, next block's opening conv op or None) in its launch
        self.fused_twin = {}                # branch name -> the other branch's op in its launch
        self.fused_twin_last = {}           # last conv name -> the ops of the two branches before it in its launch
        self.fused_chain = {}               # last conv name -> the conv ops before it in its launch
        self.fused_projblock = {}           # last conv name -> (first, middle, projection) conv ops fused into its launch
        self._packed = {}                   # conv name -> its packed weights, bias and per-channel parameters, shared by the parts
        blocks = fuse if fuse_blocks is None else fuse_blocks
        full, parts, at = self.buf, self._parts(), 0
        self.parts = len(parts)
        lists = []
        for images in parts:
            self.buf = {name: t[at:at + images] for name, t in full.items()}
            at += images
            self._build(fuse, blocks)
            lists.append(self.steps)
        self.buf = full
        self.steps = [st for part in lists for st in part]
        self.step_images = [images for images, part in zip(parts, lists) for _ in part]       # images that step i works on
        self.fused = list(dict.fromkeys(self.fused))
        calls = [B.Calls([(kind, args) for kind, _, args in part]) for part in lists]
        with torch.cuda.device(self.device):
            self._calls = calls[0] if len(calls) == 1 else B.Lanes(calls)
        torch.cuda.synchronize(self.device)

    # A layer of 16384 pixels gives each of the 256 compute units one tile of 64; a layer with a few more runs two rounds, the second nearly
    # empty, and the next layer waits for it.  Beyond that size a batch therefore runs as two halves side by side on two streams,
    # one half's last rounds filled with the other's next layer (halves / whole, us): 50-layer network 751 / 805 at batch 84, 977 / 1072 at 128;
    # the 152-layer one 1818 / 1832 at 84, 2223 / 2506 at 128; per channel 1042 / 1071 at 84; the 18-layer one 317 / 357 at 84.  Below it the
    # networks differ: the 152-layer one loses 3 % at 68 and is level at 76, the 50-layer one gains 2 % at 64, the 18-layer one 6 % from 44 on.
    # Pictures of restoration networks are hundreds of rounds each.
    HALVES_MIN_PIXELS = 256 * 64
    HALVES_MAX_MAP = 32 * 32

    def _parts(self):
        """Images per part: the whole batch, or two halves.  Decided by the median convolution layer's output map."""
        maps = sorted(int(np.prod(self.net["buffers"][op["dst"]]["shape"][1:3])) for op in self.net["ops"] if op["op"] == "conv")
        mid = maps[len(maps) // 2]
        if self.images < 2 or mid > self.HALVES_MAX_MAP or mid * self.images <= self.HALVES_MIN_PIXELS:
            return [self.images]
        return [self.images - self.images // 2, self.images // 2]

    def _build(self, fuse, blocks):
        """The calls (self.steps) for the images in self.buf."""
        net, calib = self.net, self.calib
        self.steps = []
        pending = {}                        # skip buffer name -> prepared projection step
        readers = self._readers()
        for at, op in enumerate(net["ops"]):
            if op["op"] == "conv":
                step = self._prep_conv(op)
                if fuse and op["role"] == "projection" and op["out_mode"] == "raw_s32" and self._can_wait(at, readers):
                    pending[op["dst"]] = step
                    continue
                if op["res"] in pending:
                    proj = pending.pop(op["res"])
                    dual = self._try_fuse(step, proj)
                    if dual is not None:
                        self.fused.append(op["res"])
                        self.fused_proj[op["name"]] = proj[1]
                        self.steps.append(dual)
                        continue
                    self.steps.append(proj)
                self.steps.append(step)
            elif op["op"] == "maxpool":
                n, h, w, c = self.buf[op["src"]].shape
                args = (n, h, w, c, op["k"], op["stride"], op["pad"], self.buf[op["src"]], self.buf[op["dst"]])
                self.steps.append(("maxpool", op, args))
            elif op["op"] == "avgpool":
                n, h, w, c = self.buf[op["src"]].shape
                cal = calib["avgpool"][op["dst"]]
                args = (n, h, w, c, cal["mul"], cal["shift"], cal["bound_q"], self.buf[op["src"]],
                        self.buf[op["dst"]])
                self.steps.append(("avgpool", op, args))
            else:
                raise ValueError(op["op"])
        if blocks:
            self._fuse_blocks()
            self._fuse_projection_blocks()
            self._fuse_first_layer()
            self._fuse_triples()
            self._fuse_pairs()
            self._fuse_twin_last()
            self._fuse_twins()
            self._fuse_chains()

    def _can_wait(self, at, readers):
        """Whether op `at` may be issued with the one op that reads its result, a later merge: nothing between them writes what it reads
        or writes, and nobody else sees the result."""
        ops = self.net["ops"]
        op, use = ops[at], readers.get(ops[at]["dst"], [])
        if len(use) != 1 or use[0].get("res") != op["dst"] or op["dst"] in self.net["outputs"] or op["dst_c_offset"] != 0:
            return False
        merge = [i for i, o in enumerate(ops) if o is use[0]][0]
        return merge > at and not any(o["dst"] in (op["src"], op["dst"]) for o in ops[at + 1:merge])

    def _fuse_first_layer(self):
        """A picture convolution followed by the max-pool of its output, nothing else reading that output: one
        iconv2d_maxpool_brelu launch where the library accepts it (the convolution's buffer then stays untouched)."""
        readers = self._readers()
        steps, i = [], 0
        while i < len(self.steps):
            pair = self.steps[i:i + 2]
            if len(pair) == 2 and pair[0][0] in ("conv", "conv_pc") and pair[1][0] == "maxpool":
                oc, op_ = pair[0][1], pair[1][1]
                if self._only_feeds(oc, op_, readers):
                    pc = pair[0][0] == "conv_pc"
                    d, x, wp, bias = pair[0][2][:4]
                    dd = B.conv_desc(**{k: getattr(d, k) for k, _ in d._fields_})
                    pooled = self.buf[op_["dst"]]
                    dd.out_c_stride, dd.out_c_offset = pooled.shape[3], 0
                    args = (dd, op_["k"], op_["stride"], op_["pad"], x, wp, bias) + ((pair[0][2][4],) if pc else ()) + (pooled,)
                    if self._accepts(B.iconv2d_maxpool_brelu_pc if pc else B.iconv2d_maxpool_brelu, args):
                        self.fused.append(oc["dst"])
                        self.fused_pool[oc["name"]] = op_
                        steps.append(("convpool_pc" if pc else "convpool", oc, args))
                        i += 2
                        continue
            steps.append(self.steps[i])
            i += 1
        self.steps = steps

    # By whether requantisation is per channel: below these the three layers by themselves, which spread their weights over the whole chip,
    # are level or faster (50-layer network, fused / apart, us: per layer the library itself takes them apart below 1176 pixels, six images 226 / 227, 16 267 / 283,
    # 64 526 / 559; per channel four images 249 / 237, nine 272 / 266, 16 314 / 309, 24 360 / 355, 32 = 6272 pixels 423 / 425, 48 560 / 600, 64 630 / 674; with two
    # launches side by side the layers are level or faster: 88 images 819 / 794, 96 863 / 847, 128 1074 / 1076).
    TRIPLE_MIN_PIXELS = {False: 256, True: 6272}

    def _fuse_triples(self):
        """A block's 3x3 convolution, the 1x1 convolution that closes the block and, where it follows, the 1x1 convolution that opens the
        next one: one iconv2d_triple_brelu call where the library accepts it (one launch, or one per layer where it takes a small call
        apart).  All three outputs are written, the 3x3 layer's too."""
        steps, i = [], 0
        while i < len(self.steps):
            run = self.steps[i:i + 3]
            kinds = [st[0] for st in run]
            if len(run) >= 2 and kinds[0] == kinds[1] and kinds[0] in ("conv", "conv_pc") and run[0][1]["kh"] == 3:
                pc = kinds[0] == "conv_pc"
                o2, o3 = run[0][1], run[1][1]
                if np.prod(self.buf[o2["dst"]].shape[:3]) >= self.TRIPLE_MIN_PIXELS[pc] and not (pc and self.parts > 1) and o3["src"] == o2["dst"] and o3["kh"] == 1 and o2["dst_c_offset"] == 0 and o2["cout"] == o3["cin"]:
                    d2, t, w2, b2, r2, t2 = self._conv_args(run[0])
                    d3, _t2, w3, b3, res, y = self._conv_args(run[1])
                    head = (d2, t, w2, b2) + ((run[0][2][4],) if pc else ()) + (t2, d3, w3, b3) + ((run[1][2][4],) if pc else ()) + (res, y)
                    fn = B.iconv2d_triple_brelu_pc if pc else B.iconv2d_triple_brelu
                    tails = [(None, (None,) * (5 if pc else 4) + (self.parts,))]
                    if len(run) == 3 and kinds[2] == kinds[0]:
                        o1 = run[2][1]
                        if o1["src"] == o3["dst"] and o1["kh"] == 1 and o3["dst_c_offset"] == 0 and o1["cin"] == o3["cout"] and o1["cout"] == o3["cin"]:
                            d1, _y, w1, b1, _r1, z = self._conv_args(run[2])
                            tails.insert(0, (o1, (d1, w1, b1) + ((run[2][2][4],) if pc else ()) + (z, self.parts)))
                    took = None
                    for o1, tail in tails:
                        if r2 is None and self._accepts(fn, head + tail):
                            took = o1, head + tail
                            break
                    if took is not None:
                        o1, args = took
                        self.fused_triple[o3["name"]] = (o2, o1)
                        if o1 is not None:
                            self.fused_pair[o3["name"]] = o1
                        steps.append(("triple_pc" if pc else "triple", o3, args))
                        i += 2 if o1 is None else 3
                        continue
            steps.append(self.steps[i])
            i += 1
        self.steps = steps

    # What the three-layer launches and the blocks leave: per channel the 256 -> 1024 -> 256 boundaries of a batch in two halves, per layer those whose
    # 3x3 layer _fuse_triples does not take (no stored network has one).  The figures are those of the 50-layer network without these launches, from when the
    # layers by themselves were the tile kernels; in two halves per channel, the one case left in a stored network, the pairs are now behind (fused / apart: 88
    # images 835 / 794 us, 96 884 / 847, 128 1134 / 1076).
    # The fused pair streams both layers' weights through every workgroup's 64-pixel tile: it wins where the tiles
    # fit the chip in about one round and the wide tensor is at most 1024 channels (measured at batch 64: 17.6 us
    # against 23.8 us for 12544 pixels of 256 -> 1024 -> 256; level at 50176 pixels of 128 -> 512 -> 128; a loss,
    # 22.9 us against 19.0 us, at 3136 pixels of 512 -> 2048 -> 512).
    # Below the other bound (by narrow width and whether requantisation is per channel) the two layers by themselves are the faster
    # choice: the fused time hardly depends on the tiles as long as each has a compute unit of its own, the layers' does.
    #   256 -> 1024 -> 256: 13.2 us fused; apart 12.0 at 784 pixels, 13.1 at 1960, 14.0 at 2156, 14.6 at 3920: up to 2048 pixels the second
    #   layer's work units are all on the chip at once (conv_lat.hip).  50-layer network, its five pairs fused / apart: 8 images 332 / 327 us,
    #   10: 351 / 348, 11: 387 / 387, 16: 399 / 402, 64: 748 / 774.
    #   Per channel: 18.7 us fused at few pixels; the same network: 16 images 500 / 490 us, 40: 726 / 711, 48: 826 / 842, 64: 904 / 919.  Up to
    #   8192 pixels the first layer by itself is one round of two 128 x 128 tiles per compute unit.
    #   128 -> 512 -> 128: 7.4 us fused and 9.7 apart at 784 pixels already; per channel never (the 50-layer network fused / apart: one image 263 / 265,
    #   nine 292 / 285, 16 337 / 332, 32 489 / 477).
    PAIR_MAX_PIXELS = 64 * 512
    PAIR_MIN_PIXELS = {(256, False): 2049, (256, True): 8193, (128, True): PAIR_MAX_PIXELS + 1}
    PAIR_MAX_WIDE = 1024

    def _fuse_pairs(self):
        """The 1x1 convolution that closes a block followed by the 1x1 convolution that opens the next one: one
        iconv2d_pair_brelu launch where the library accepts it and the shape is one the fused kernel wins on.  Both
        outputs are still written (the first is the next block's skip operand)."""
        steps, i = [], 0
        while i < len(self.steps):
            two = self.steps[i:i + 2]
            if len(two) == 2 and two[0][0] == two[1][0] and two[0][0] in ("conv", "conv_pc"):
                pc = two[0][0] == "conv_pc"
                o3, o1 = two[0][1], two[1][1]
                d3, t, w3, b3, res, y = self._conv_args(two[0])
                d1, _y, w1, b1, _r1, z = self._conv_args(two[1])
                if (o1["src"] == o3["dst"] and o3["kh"] == 1 and o1["kh"] == 1 and o3["dst_c_offset"] == 0 and
                        o1["cout"] == o3["cin"] and o1["cin"] == o3["cout"] and
                        self.PAIR_MIN_PIXELS.get((o3["cin"], pc), 0) <= d3.n * d3.h * d3.w <= self.PAIR_MAX_PIXELS and o3["cout"] <= self.PAIR_MAX_WIDE):
                    if pc:
                        fn, args = B.iconv2d_pair_brelu_pc, (d3, t, w3, b3, two[0][2][4], res, y, d1, w1, b1, two[1][2][4], z)
                    else:
                        fn, args = B.iconv2d_pair_brelu, (d3, t, w3, b3, res, y, d1, w1, b1, z)
                    if self._accepts(fn, args):
                        self.fused_pair[o3["name"]] = o1
                        steps.append(("pair_pc" if pc else "pair", o3, args))
                        i += 2
                        continue
            steps.append(self.steps[i])
            i += 1
        self.steps = steps

    # (240 x 320 in 26.8 us against 31.2 with the layers apart, 600 x 850 in 67 against 78; below a few of the fused kernel's tiles the layers
    # are left apart.)
    TWIN_LAST_MIN_PIXELS = 64 * 64

    def _fuse_twin_last(self):
        """Two branches of one input and the single-channel convolution of their concatenation, nothing else reading that: one
        iconv2d_twin_last_brelu launch where the library accepts it (the concatenation's buffer then stays untouched)."""
        readers = self._readers()
        steps, i = [], 0
        while i < len(self.steps):
            trio = self.steps[i:i + 3]
            if [st[0] for st in trio] == ["conv"] * 3:
                a, b, (dc, _t, wc, bc, rc, y, _ws) = (st[2] for st in trio)
                oa, ob, oc = (st[1] for st in trio)
                if oa["kh"] < ob["kh"]:
                    a, b, oa, ob = b, a, ob, oa
                (da, x, wa, ba, ra), (db, _x, wb, bb, rb) = a[:5], b[:5]
                if (oa["src"] == ob["src"] and oa["dst"] == ob["dst"] == oc["src"] and readers.get(oa["dst"]) == [oc] and ra is None and rb is None and
                        oa["dst"] not in self.net["outputs"] and oc["dst"] != oa["src"] and
                        da.n * da.h * da.w >= self.TWIN_LAST_MIN_PIXELS):
                    args = (da, x, wa, ba, db, wb, bb, dc, wc, bc, rc, y)
                    if self._accepts(B.iconv2d_twin_last_brelu, args):
                        self.fused.append(oa["dst"])
                        self.fused_twin_last[oc["name"]] = (oa, ob)
                        steps.append(("twin_last", oc, args))
                        i += 3
                        continue
            steps.append(self.steps[i])
            i += 1
        self.steps = steps

    # The twin launch reads the input once and writes whole pixels of the shared buffer.  It wins at every picture size (with the launch
    # behind it: 240 x 320 in 26.8 us against 37.3 with two launches, 600 x 850 in 67 against 98); a picture of fewer pixels than a few of
    # its tiles is left to the layers.
    TWIN_MIN_PIXELS = 64 * 64

    def _fuse_twins(self):
        """Two consecutive convolutions of the same input whose kernels differ by two pixels (the branches of a
        concatenation): one iconv2d_twin_brelu launch where the library accepts it."""
        steps, i = [], 0
        while i < len(self.steps):
            two = self.steps[i:i + 2]
            if len(two) == 2 and two[0][0] == "conv" and two[1][0] == "conv":
                (da, xa, wa, ba, ra, ya, _wsa), (db, xb, wb, bb, rb, yb, _wsb) = two[0][2], two[1][2]
                oa, ob = two[0][1], two[1][1]
                if oa["kh"] < ob["kh"]:
                    (da, wa, ba, ya, oa), (db, wb, bb, yb, ob) = (db, wb, bb, yb, ob), (da, wa, ba, ya, oa)
                if (oa["src"] == ob["src"] and oa["kh"] == ob["kh"] + 2 and ra is None and rb is None and
                        oa["dst"] != oa["src"] and ob["dst"] != ob["src"] and da.n * da.h * da.w >= self.TWIN_MIN_PIXELS):
                    args = (da, xa, wa, ba, ya, db, wb, bb, yb)
                    if self._accepts(B.iconv2d_twin_brelu, args):
                        self.fused_twin[oa["name"]] = ob
                        steps.append(("twin", oa, args))
                        i += 2
                        continue
            steps.append(self.steps[i])
            i += 1
        self.steps = steps

    # A chain's launches recompute borders to save launches; on pictures smaller than a few tiles there is nothing to gain
    # over the layers, which cost a launch each either way.
    CHAIN_MIN_PIXELS = 64 * 64

    def _fuse_chains(self):
        """Runs of convolutions that feed each other and nothing else: as few iconv2d_chain_brelu launches as the library
        advises, where it accepts them (the tensors between the layers of a launch then stay untouched)."""
        readers = self._readers()
        steps, i = [], 0
        while i < len(self.steps):
            run = [self.steps[i]]
            while i + len(run) < len(self.steps):
                a, b = run[-1], self.steps[i + len(run)]
                if a[0] != "conv" or b[0] != "conv" or not self._only_feeds(a[1], b[1], readers):
                    break
                run.append(b)
            run, lengths = self._chain_part(run)
            if len(run) < 2:
                steps.append(self.steps[i])
                i += 1
                continue
            at = 0
            for n in lengths:
                part, at = run[at:at + n], at + n
                if n == 1:
                    steps.append(part[0])
                    continue
                args = ([st[2][0] for st in part], part[0][2][1], [st[2][2] for st in part], [st[2][3] for st in part], part[-1][2][5])
                if not self._accepts(B.iconv2d_chain_brelu, args):
                    steps += part
                    continue
                self.fused += [st[1]["dst"] for st in part[:-1]]
                self.fused_chain[part[-1][1]["name"]] = [st[1] for st in part[:-1]]
                steps.append(("chain", part[-1][1], args))
            i += len(run)
        self.steps = steps

    def _chain_part(self, run):
        """The leading layers of a run that chains can hold (none: an empty list), and how many of them each launch takes."""
        d = run[0][2][0] if run[0][0] == "conv" else None
        if d is None or d.n * d.h * d.w < self.CHAIN_MIN_PIXELS:
            return [], []

        def split(part):
            try:
                return B.iconv2d_chain_split([st[2][0] for st in part])
            except B.IcnnError as e:
                if e.code not in (B.ICNN_E_UNSUPPORTED, B.ICNN_E_SHAPE):
                    raise
                return None
        if split(run[:1]) is None:
            return [], []
        while True:                                    # (what does not fit is the last layer of a run, if any)
            lengths = split(run)
            if lengths is not None:
                return run, lengths
            run = run[:-1]

    @staticmethod
    def _accepts(fn, args):
        """Issues a fused call, which is also its warm-up launch; False if the library does not take it: layers that are valid by
        themselves (their workspace has been asked for) and do not fit together are refused as a shape or a parameter, too."""
        try:
            fn(*args)
        except B.IcnnError as e:
            if e.code not in (B.ICNN_E_UNSUPPORTED, B.ICNN_E_SHAPE, B.ICNN_E_PARAM):
                raise
            return False
        return True

    @staticmethod
    def _conv_args(step):
        """descriptor, input, weights, bias, skip operand, output of a "conv" or "conv_pc" step"""
        args = step[2]
        return args[:4] + args[4 + (step[0] == "conv_pc"):][:2]

    def _readers(self):
        """buffer name -> the ops that read it"""
        readers = {}
        for op in self.net["ops"]:
            readers.setdefault(op["src"], []).append(op)
            if op.get("res") is not None:
                readers.setdefault(op["res"], []).append(op)
        return readers

    def _only_feeds(self, a, b, readers):
        """Whether op b reads what op a writes, all of it and nothing beside it, and nothing else ever does: the tensor between
        them may stay on chip."""
        width = self.net["buffers"][a["dst"]]["shape"][3]
        return (b["src"] == a["dst"] and readers.get(a["dst"]) == [b] and a["dst"] not in self.net["outputs"] and
                a["dst_c_offset"] == 0 and a["cout"] == b.get("cin", width))

    def _fuse_projection_blocks(self):
        """A stage's opening bottleneck block whose last layer already runs with its projection as one dual step: the
        two layers before it join that launch (iconv2d_bottleneck_dual_brelu) where the library accepts it; the block's
        two middle buffers then stay untouched as well."""
        readers = self._readers()
        steps, i = [], 0
        while i < len(self.steps):
            trio = self.steps[i:i + 3]
            if [st[0] for st in trio] in (["conv", "conv", "dual"], ["conv_pc", "conv_pc", "dual_pc"]):
                pc = trio[2][0] == "dual_pc"
                o1, o2, o3 = (st[1] for st in trio)
                proj = self.fused_proj[o3["name"]]
                chain = proj["src"] == o1["src"] and self._only_feeds(o1, o2, readers) and self._only_feeds(o2, o3, readers)
                if chain:
                    d1, x, w1, b1 = trio[0][2][:4]
                    d2, _x2, w2, b2 = trio[1][2][:4]
                    if pc:
                        dm, _xm, wm, bm, pcm, dp, _xp, wp, bp, y = trio[2][2]
                        fn = B.iconv2d_bottleneck_dual_brelu_pc
                        args = (d1, x, w1, b1, trio[0][2][4], d2, w2, b2, trio[1][2][4], dm, wm, bm, pcm, dp, wp, bp, y)
                    else:
                        dm, _xm, wm, bm, dp, _xp, wp, bp, y = trio[2][2]
                        fn, args = B.iconv2d_bottleneck_dual_brelu, (d1, x, w1, b1, d2, w2, b2, dm, wm, bm, dp, wp, bp, y)
                    if self._accepts(fn, args):
                        self.fused += [o1["dst"], o2["dst"]]
                        self.fused_projblock[o3["name"]] = (o1, o2, proj)
                        steps.append(("projblock_pc" if pc else "projblock", o3, args))
                        i += 3
                        continue
            steps.append(self.steps[i])
            i += 1
        self.steps = steps

    # With 128 middle channels a block is one workgroup after another's worth of weights per 64 pixels; its three layers spread them over the
    # chip, but are three launches.  The 50-layer network with its three such blocks fused / layer by layer: 165 / 173 us at one image of 28 x 28 (13
    # workgroups), 177 / 184 at two, 205 / 214 at four, 232 / 241 at nine, 341 / 367 at 32, 527 / 545 at 64.  Fewer pixels than that were not looked at and stay apart.
    BLOCK128_MIN_PIXELS = 784

    def _fuse_blocks(self):
        """Replaces every run of three per-layer conv steps that forms an identity bottleneck block by one fused step."""
        readers = self._readers()
        steps, i = [], 0
        while i < len(self.steps):
            trio = self.steps[i:i + 3]
            if [st[0] for st in trio] in (["conv"] * 3, ["conv_pc"] * 3):
                pc = trio[0][0] == "conv_pc"
                o1, o2, o3 = (st[1] for st in trio)
                chain = o3["res"] == o1["src"] and self._only_feeds(o1, o2, readers) and self._only_feeds(o2, o3, readers)
                d1 = trio[0][2][0]
                if chain and (o1["cout"] != 128 or d1.n * d1.h * d1.w >= self.BLOCK128_MIN_PIXELS):
                    (d1, x, w1, b1, _r1, _y1), (d2, _x2, w2, b2, _r2, _y2), (d3, _x3, w3, b3, res, y) = (self._conv_args(st) for st in trio)
                    if pc:
                        pc1, pc2, pc3 = (st[2][4] for st in trio)
                        fn, args = B.iconv2d_bottleneck_brelu_pc, (d1, x, w1, b1, pc1, d2, w2, b2, pc2, d3, w3, b3, pc3, res, y)
                    else:
                        fn, args = B.iconv2d_bottleneck_brelu, (d1, x, w1, b1, d2, w2, b2, d3, w3, b3, res, y)
                    if self._accepts(fn, args):
                        self.fused += [o1["dst"], o2["dst"]]
                        (self.fused_block_pc if pc else self.fused_block)[o3["name"]] = (o1, o2)
                        steps.append(("block_pc" if pc else "block", o3, args))
                        i += 3
                        continue
            steps.append(self.steps[i])
            i += 1
        self.steps = steps

    def _prep_conv(self, op):
        cal = self.calib["conv"][op["name"]]
        src, dst = self.buf[op["src"]], self.buf[op["dst"]]
        n, h, w, cbuf = src.shape
        # bytes above 127 can occur in activations bounded above 127, or in a full-range input that is
        # not re-normalised
        top = self.calib.get("max_int", 127) if op["src"] != self.net["input"] else self.net["input_range"][1]
        in_kind = B.ICNN_IN_U8_FULL if (top > 127 and not op["in_sub128"]) else B.ICNN_IN_U8_LE127
        d = B.conv_desc(
            n=n, h=h, w=w, cin=op["cin"], in_c_stride=cbuf, in_signed=in_kind, in_sub128=int(op["in_sub128"]),
            cout=op["cout"], kh=op["kh"], kw=op["kw"], stride_h=op["stride"], stride_w=op["stride"],
            pad_h=op["pad"], pad_w=op["pad"], out_c_stride=dst.shape[3], out_c_offset=op["dst_c_offset"],
            mul=cal.get("mul", 1), shift=cal.get("shift", 0), bound_q=cal.get("bound_q", 127),
            lo=cal.get("lo", 0), hi=cal.get("hi", 255), out_mode=_OUT[op["out_mode"]],
            res_mode=_RES[op["res_mode"]])
        res = None
        if op["res"] is not None:
            res = self.buf[op["res"]]
            d.res_dtype = _DT[op["res_dtype"]]
            d.res_c_stride = res.shape[3]
            d.res_mul, d.res_shift = cal.get("res_mul", 1), cal.get("res_shift", 0)
        wp, bias, pcp = self._packed.get(op["name"]) or self._pack(op, d, cal)
        if pcp is not None and res is not None:
            # the descriptor's own pair bounds the per-channel skip ratios (what the fused block's
            # overflow proof needs; the plain per-channel call does not read it)
            d.res_mul, d.res_shift = max(zip(cal["res_mul_c"], cal["res_shift_c"]), key=lambda t: t[0] / 2.0 ** t[1])
        ws_bytes = B.iconv2d_workspace_bytes(d)
        ws = torch.zeros(ws_bytes, dtype=torch.uint8, device=self.device) if ws_bytes else None       # zero-filled once: its counter block
        if pcp is not None:
            return ("conv_pc", op, (d, src, wp, bias, pcp, res, dst, ws))
        return ("conv", op, (d, src, wp, bias, res, dst, ws))

    def _pack(self, op, d, cal):
        """The layer's packed weights, its bias and, with requantisation per output channel, those parameters packed (else None)."""
        w_np = self.weights[op["name"]][0] if self.weights is not None else W.weight_tensor(op, self.seed)
        w_dev = torch.from_numpy(np.ascontiguousarray(w_np, dtype=np.int8)).to(self.device)
        wp = torch.empty(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device=self.device)
        B.iconv2d_prepack_weights(d, w_dev, wp)
        b_np = self.weights[op["name"]][1] if self.weights is not None else W.bias_tensor(op, self.seed)
        bias = torch.from_numpy(np.ascontiguousarray(b_np, dtype=np.int32)).to(self.device)
        pcp = None
        if "mul_c" in cal or "res_mul_c" in cal:
            # per-output-channel requantisation: the integers go to the device as they are
            def col(key, fallback):
                v = cal.get(key)
                if v is None:
                    v = [cal.get(fallback[0], fallback[1])] * op["cout"]
                return torch.tensor(v, dtype=torch.int32, device=self.device)
            arrs = [col("mul_c", ("mul", 1)), col("shift_c", ("shift", 0))]
            if op["res"] is not None:
                arrs += [col("res_mul_c", ("res_mul", 1)), col("res_shift_c", ("res_shift", 0))]
            pcp = torch.empty(B.iconv2d_packed_channel_params_bytes(d), dtype=torch.uint8, device=self.device)
            B.iconv2d_prepack_channel_params(d, B.channel_params(*arrs), pcp)
        torch.cuda.synchronize(self.device)       # the unpacked tensors may be released after the packing ran
        self._packed[op["name"]] = wp, bias, pcp
        return self._packed[op["name"]]

    def _try_fuse(self, main, proj):
        if proj[0] != "conv":
            return None
        dp, xp, wp, bp, _r, _sk, _w = proj[2]
        if main[0] == "conv_pc":
            dm, xm, wm, bm, pcp, _res, y, _ws = main[2]
            kind, fn, args = "dual_pc", B.iconv2d_dual_brelu_pc, (dm, xm, wm, bm, pcp, dp, xp, wp, bp, y)
        else:
            dm, xm, wm, bm, _res, y, _ws = main[2]
            kind, fn, args = "dual", B.iconv2d_dual_brelu, (dm, xm, wm, bm, dp, xp, wp, bp, y)
        return (kind, main[1], args) if self._accepts(fn, args) else None

    def set_input(self, x_raw=None):
        if x_raw is None:
            x_raw = W.input_tensor(self.net, self.seed, self.images)
        self.buf["raw"].copy_(torch.from_numpy(np.ascontiguousarray(x_raw)).to(self.device))

    def run(self, stream=None):
        self._calls.run(stream)

    def run_step(self, i, stream=None):
        kind, _, args = self.steps[i]
        self._FUNCTIONS[kind](*args, stream=stream)

    _FUNCTIONS = {"conv": B.iconv2d_brelu, "conv_pc": B.iconv2d_brelu_pc, "dual": B.iconv2d_dual_brelu, "dual_pc": B.iconv2d_dual_brelu_pc,
                  "pair": B.iconv2d_pair_brelu, "pair_pc": B.iconv2d_pair_brelu_pc, "triple": B.iconv2d_triple_brelu,
                  "triple_pc": B.iconv2d_triple_brelu_pc, "twin": B.iconv2d_twin_brelu, "twin_last": B.iconv2d_twin_last_brelu, "chain": B.iconv2d_chain_brelu,
                  "projblock": B.iconv2d_bottleneck_dual_brelu, "projblock_pc": B.iconv2d_bottleneck_dual_brelu_pc,
                  "block": B.iconv2d_bottleneck_brelu, "block_pc": B.iconv2d_bottleneck_brelu_pc, "convpool": B.iconv2d_maxpool_brelu,
                  "convpool_pc": B.iconv2d_maxpool_brelu_pc, "maxpool": B.imaxpool2d_u8, "avgpool": B.iavgpool_global_u8}

    def result(self, name):
        return self.buf[name].cpu().numpy()
