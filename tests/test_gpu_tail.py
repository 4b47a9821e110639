"""GPU parity of two branches and the single-channel layer behind them in one launch (iconv2d_twin_last_brelu) against the oracle's
three layers, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import calibrate as K
from oracle import oracle as O

pytestmark = pytest.mark.gpu


def run_tail(seed, n, h, w, *, off_a=0, xbuf=48, res="post", out_mode="clamp_u8", any_form=False):
    """(GPU output, oracle output) of 3x3 48 -> 16 beside 1x1 48 -> 32, concatenated, then 3x3 48 -> 1."""
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    g = np.random.default_rng(seed)
    off_b = 16 if off_a == 0 else 0
    x = g.integers(0, 128, size=(n, h, w, xbuf), dtype=np.uint8)
    wts = [g.integers(-127, 128, size=s, dtype=np.int8) for s in ((16, 3, 3, 48), (32, 1, 1, 48), (1, 3, 3, 48))]
    bias = [g.integers(-4096, 4097, size=c).astype(np.int32) for c in (16, 32, 1)]
    mid = np.zeros((n, h, w, 48), dtype=np.uint8)
    ms = []
    for wt, b, k, off in ((wts[0], bias[0], 3, off_a), (wts[1], bias[1], 1, off_b)):
        m, s = K.bound_params(K.percentile_999(O.conv2d(x, wt, b, cin=48, pad=k // 2, out_mode="raw_s32")))
        if any_form:                             # a pair the 32-bit requantisation does not take
            m, s = (m << 12) | 1, s + 12
        ms.append((m, s))
        mid = O.conv2d(x, wt, b, cin=48, pad=k // 2, mul=m, shift=s, out=mid, out_c_offset=off)
    raw = O.conv2d(mid, wts[2], bias[2], cin=48, pad=1, out_mode="raw_s32")
    mc, sc = K.bound_params(max(1, int(np.abs(raw).max())))
    skip = g.integers(0, 256, size=(n, h, w, 1), dtype=np.uint8)
    kw = dict(mul=mc, shift=sc, out_mode=out_mode)
    if out_mode == "clamp_u8":
        kw.update(lo=0, hi=255)
    rm, rs = (1, 0) if res == "post" else (20001, 6)
    if res:
        kw.update(res=skip, res_mode=res, res_mul=rm, res_shift=rs)
    want = O.conv2d(mid, wts[2], bias[2], cin=48, pad=1, **kw)

    descs, packs = [], []
    for wt, k, off, (m, s) in ((wts[0], 3, off_a, ms[0]), (wts[1], 1, off_b, ms[1]), (wts[2], 3, 0, (mc, sc))):
        d = B.conv_desc(n=n, h=h, w=w, cin=48, in_c_stride=xbuf if len(descs) < 2 else 48, cout=wt.shape[0], kh=k, kw=k, pad_h=k // 2, pad_w=k // 2,
                        out_c_stride=48 if len(descs) < 2 else 1, out_c_offset=off, mul=m, shift=s, bound_q=127)
        descs.append(d)
        packs.append(torch.zeros(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda:0"))
        B.iconv2d_prepack_weights(d, dev(wt), packs[-1])
    d = descs[2]
    d.out_mode = B.ICNN_OUT_RAW_S32 if out_mode == "raw_s32" else B.ICNN_OUT_CLAMP_U8
    d.lo, d.hi = 0, 255
    if res:
        d.res_mode, d.res_dtype, d.res_c_stride = (B.ICNN_RES_POST if res == "post" else B.ICNN_RES_PRE), B.ICNN_U8, 1
        d.res_mul, d.res_shift = rm, rs
    y = torch.zeros((n, h, w, 1), dtype=torch.int32 if out_mode == "raw_s32" else torch.uint8, device="cuda:0")
    B.iconv2d_twin_last_brelu(descs[0], dev(x), packs[0], dev(bias[0]), descs[1], packs[1], dev(bias[1]), d, packs[2], dev(bias[2]),
                              dev(skip) if res else None, y)
    torch.cuda.synchronize()
    return y.cpu().numpy(), want


TAILS = [
    # n, h, w and what differs from the restoration network's layers
    (1, 16, 30, {}),                        # one strip of one tile; the picture's last row is the tile's last
    (1, 1, 1, {}),
    (1, 17, 31, {}),                        # one row, one column beyond a tile
    (1, 15, 61, {"off_a": 32}),
    (2, 40, 90, {"xbuf": 64}),
    (1, 200, 300, {}),                      # a tile or less per workgroup: every unit but a strip's first starts with a warm-up
    (3, 97, 203, {"res": "pre"}),
    (1, 530, 700, {}),                      # several tiles per workgroup, units that cross strips
    (2, 333, 517, {"any_form": True}),
    (1, 64, 64, {"res": None, "out_mode": "raw_s32"}),
]


@pytest.mark.parametrize("case", TAILS, ids=lambda c: "x".join(map(str, c[:3])))
def test_branches_and_last_layer(case):
    n, h, w, kw = case
    got, want = run_tail(h * 1000 + w, n, h, w, **kw)
    assert np.array_equal(got, want)
