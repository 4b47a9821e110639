"""The requantisation forms of the convolution epilogues at the places where they can go wrong: accumulators on both sides of each rounding
step and of both clamps, against exact integers.  The input is zero, so channel c's accumulator is its bias.  A single layer uses the 32-bit,
the 64-bit multiply-add and the general form; the 24-bit factors' high half is the two-branch kernel's (the second test)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def exact(t, mul, shift, hi):
    q = (int(t) * mul + ((1 << shift) >> 1)) >> shift
    return min(max(q, 0), hi)


def rounding_accumulators(mul, shift, hi):
    steps = []
    for k in list(range(0, 5)) + list(range(max(0, hi - 3), hi + 3)):
        t = ((2 * k + 1) << shift) // (2 * mul)            # where [t mul / 2^shift] goes from k to k + 1
        steps += [t - 1, t, t + 1, t + 2]
    rng = np.random.default_rng(shift)
    top = ((2 * hi + 1) << shift) // (2 * mul) + 2
    steps += [-1, -5, -(1 << 30), 1 << 30] + [int(v) for v in rng.integers(-top, top + 1, size=64)]
    return [t for t in steps if abs(t) <= 1 << 30]


@pytest.mark.parametrize("tile", [-1, 1, 4])
@pytest.mark.parametrize("mul, shift, hi", [
    (16385, 24, 127),            # product fits 32 bits
    (16385, 25, 255), (16385, 26, 127), (32767, 26, 127), (32767, 27, 255), (16385, 30, 127), (16385, 31, 255), (16385, 33, 3),   # products beyond 32 bits
    (32767, 23, 127),            # one bit more than the high half takes
    (16385, 34, 1), (1 << 23, 40, 7), ((1 << 30) + 1, 40, 127), (3, 1, 255), (1, 0, 255),
])
def test_rounding_steps_and_clamps(tile, mul, shift, hi):
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    steps = rounding_accumulators(mul, shift, hi)
    rng = np.random.default_rng(shift)
    cout = (len(steps) + 63) // 64 * 64
    bias = np.array(steps + [0] * (cout - len(steps)), dtype=np.int32)
    n = 200                                                # pixels: several tiles of every kernel
    d = B.conv_desc(n=1, h=n, w=1, cin=64, in_c_stride=64, cout=cout, kh=1, kw=1, out_c_stride=cout, mul=mul, shift=shift, bound_q=hi)
    wp = torch.zeros(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda:0")
    B.iconv2d_prepack_weights(d, dev(rng.integers(-127, 128, size=(cout, 1, 1, 64), dtype=np.int8)), wp)
    y = torch.zeros((n, cout), dtype=torch.uint8, device="cuda:0")
    B.icnn_set_tuning("tile", tile)
    try:
        B.iconv2d_brelu(d, torch.zeros((n, 64), dtype=torch.uint8, device="cuda:0"), wp, dev(bias), None, y)
        torch.cuda.synchronize()
    finally:
        B.icnn_set_tuning("reset")
    want = np.array([exact(t, mul, shift, hi) for t in bias], dtype=np.uint8)
    assert (y.cpu().numpy() == want[None, :]).all()


# (mul, shift, bound): the 24-bit factors' high half where mul * 2^(33 - shift) < 2^24, the 32-bit form where only the product fits
HIGH_HALF = [(16385, 24, 127), (16385, 26, 127), (32767, 26, 127), (32767, 27, 127), (16385, 30, 15), (16385, 31, 3), (16385, 33, 1), (16383, 23, 255), (3, 13, 127)]
PRODUCT = [(32767, 23, 127), (16385, 23, 255), (16385, 20, 127), (3, 1, 255), (32767, 15, 127)]


@pytest.mark.parametrize("a, b", [(p, q) for form in (HIGH_HALF, PRODUCT) for p, q in zip(form, form[1:] + form[:1])], ids=str)
@pytest.mark.parametrize("cout_b", [16, 32])
def test_two_branch_forms(a, b, cout_b):
    # a 5x5 layer of 32 channels beside a 3x3 layer of 16 (two output rows to an accumulator) or 32, each branch with parameters of its own:
    # conv_rows_twin_kernel in these two forms where a branch's shift is 33 or its ratio one half and more, with one wide product elsewhere
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    high = [mul << (33 - shift) < 1 << 24 for mul, shift, _ in (a, b)]
    assert high[0] == high[1] and high[0] == (a in HIGH_HALF)
    if not high[0]:
        assert all(((hi + 1) << shift) < 1 << 32 for _, shift, hi in (a, b))
    h, w = 37, 70                                          # several tiles, hanging over both edges
    steps = [rounding_accumulators(*p) for p in (a, b)]
    x = torch.zeros((1, h, w, 64), dtype=torch.uint8, device="cuda:0")
    rng = np.random.default_rng(1)
    couts, ks, offs = (32, cout_b), (5, 3), (0, 32)
    descs = [B.conv_desc(n=1, h=h, w=w, cin=64, in_c_stride=64, cout=c, kh=k, kw=k, pad_h=k // 2, pad_w=k // 2, out_c_stride=32 + cout_b, out_c_offset=o,
                         mul=p[0], shift=p[1], bound_q=p[2]) for p, c, k, o in zip((a, b), couts, ks, offs)]
    packs = []
    for d in descs:
        packs.append(torch.zeros(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda:0"))
        B.iconv2d_prepack_weights(d, dev(rng.integers(-127, 128, size=(d.cout, d.kh, d.kw, 64), dtype=np.int8)), packs[-1])
    for at in range(0, max(-(-len(s) // c) for s, c in zip(steps, couts))):
        bias = [np.array([s[(at * c + i) % len(s)] for i in range(c)], dtype=np.int32) for s, c in zip(steps, couts)]
        y = torch.full((1, h, w, 32 + cout_b), 99, dtype=torch.uint8, device="cuda:0")
        B.iconv2d_twin_brelu(descs[0], x, packs[0], dev(bias[0]), y, descs[1], packs[1], dev(bias[1]), y)
        torch.cuda.synchronize()
        want = np.array([exact(t, *p) for p, v in zip((a, b), bias) for t in v], dtype=np.uint8)
        assert (y.cpu().numpy() == want).all()


# bytes by a product 2^8 times as large: multipliers on both sides of 2^23 (mul * 2^(32 - shift)), sums at int32's ends, with a skip operand that saturates them
@pytest.mark.parametrize("mul, shift", [(32767, 24), (32767, 23), (16385, 24), (1, 10), (1, 9), (3, 32), (8388607, 32), (5000001, 32)])
@pytest.mark.parametrize("kernel, cin, cout, k", [("flat", 128, 128, 1), ("keep", 64, 64, 3), ("lat", 64, 64, 1), ("tile", 64, 64, 3)])
@pytest.mark.parametrize("skip", [None, (20000, 5), (255, 0), (8388608, 1)], ids=str)
def test_byte_form(mul, shift, kernel, cin, cout, k, skip):
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    rng = np.random.default_rng([mul, shift])
    steps = rounding_accumulators(mul, shift, 127) + [2 ** 31 - 1, -2 ** 31, 2 ** 31 - 2, -2 ** 31 + 1, 0]
    rm, rs = skip or (0, 0)
    n, px = (len(steps) + cout - 1) // cout, 70
    res = rng.integers(0, 256, size=(px, cout), dtype=np.uint8)
    res[:4] = np.array([[0], [1], [127], [255]], np.uint8)
    d = B.conv_desc(n=1, h=px, w=1, cin=cin, in_c_stride=cin, cout=cout, kh=k, kw=k, pad_h=k // 2, pad_w=k // 2, out_c_stride=cout, mul=mul, shift=shift, bound_q=127)
    if skip:
        d.res_mode, d.res_dtype, d.res_c_stride, d.res_mul, d.res_shift = B.ICNN_RES_PRE, B.ICNN_U8, cout, rm, rs
    wp = torch.zeros(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda:0")
    B.iconv2d_prepack_weights(d, dev(rng.integers(-127, 128, size=(cout, k, k, cin), dtype=np.int8)), wp)
    x = torch.zeros((px, cin), dtype=torch.uint8, device="cuda:0")
    for at in range(n):
        bias = np.array([steps[(at * cout + i) % len(steps)] for i in range(cout)], dtype=np.int64)
        if skip:                                           # (half of them so that the sum, not the bias, is at the step)
            bias[::2] = np.clip(bias[::2] - ((int(res[2, 0]) * rm + ((1 << rs) >> 1)) >> rs), -2 ** 31, 2 ** 31 - 1)
        y = torch.zeros((px, cout), dtype=torch.uint8, device="cuda:0")
        B.icnn_set_tuning(kernel, 1)
        try:
            B.iconv2d_brelu(d, x, wp, dev(bias.astype(np.int32)), dev(res) if skip else None, y)
            torch.cuda.synchronize()
        finally:
            B.icnn_set_tuning("reset")
        t = np.broadcast_to(bias, (px, cout)).astype(object)
        if skip:
            t = np.clip(t + ((res.astype(object) * rm + ((1 << rs) >> 1)) >> rs), -2 ** 31, 2 ** 31 - 1)
        want = np.clip((t * mul + (1 << (shift - 1))) >> shift, 0, 127).astype(np.uint8)
        assert (y.cpu().numpy() == want).all()
