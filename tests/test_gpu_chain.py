"""GPU parity of a run of 3x3 layers in one launch (iconv2d_chain_brelu) against the oracle's separate layers, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import calibrate as K
from oracle import oracle as O

pytestmark = pytest.mark.gpu


def run_chain(seed, n, h, w, layers, *, top=127, xbuf=64, ybuf=64, yoff=0, last_mode="brelu", wide_shift=False):
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    g = np.random.default_rng(seed)
    x = g.integers(0, top + 1, size=(n, h, w, xbuf), dtype=np.uint8)
    cur, descs, packs, biases = x, [], [], []
    canvas = g.integers(0, 256, size=(n, h, w, ybuf), dtype=np.uint8)
    want = canvas.copy()
    for i in range(layers):
        wt = g.integers(-127, 128, size=(64, 3, 3, 64), dtype=np.int8)
        b = g.integers(-4096, 4097, size=64).astype(np.int32)
        raw = O.conv2d(cur, wt, b, cin=64, pad=1, out_mode="raw_s32")
        mul, shift = K.bound_params(K.percentile_999(raw), top)
        if wide_shift:
            mul, shift = mul << 9, shift + 9          # the same ratio with an odd multiplier above 2^24: the 64-bit forms
            mul += 1
        last = i + 1 == layers
        mode = dict(out_mode=last_mode) if last else {}
        if last and last_mode == "clamp_u8":
            mode.update(lo=3, hi=200)
        if last:
            O.conv2d(cur, wt, b, cin=64, pad=1, mul=mul, shift=shift, bound_q=top, out=want, out_c_offset=yoff, **mode)
        else:
            cur_next = O.conv2d(cur, wt, b, cin=64, pad=1, mul=mul, shift=shift, bound_q=top)
        d = B.conv_desc(n=n, h=h, w=w, cin=64, in_c_stride=xbuf if i == 0 else 64, cout=64, kh=3, kw=3, pad_h=1, pad_w=1,
                        in_signed=B.ICNN_IN_U8_FULL if top > 127 else B.ICNN_IN_U8_LE127, mul=mul, shift=shift, bound_q=top,
                        out_c_stride=ybuf if last else 64, out_c_offset=yoff if last else 0)
        if last and last_mode == "clamp_u8":
            d.out_mode, d.lo, d.hi = B.ICNN_OUT_CLAMP_U8, 3, 200
        pk = torch.zeros(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda:0")
        B.iconv2d_prepack_weights(d, dev(wt), pk)
        descs.append(d), packs.append(pk), biases.append(dev(b))
        if not last:
            cur = cur_next
    xd, yd = dev(x), dev(canvas)
    B.iconv2d_chain_brelu(descs, xd, packs, biases, yd)
    torch.cuda.synchronize()
    assert want[..., yoff:yoff + 64].max() > 0
    assert (yd.cpu().numpy() == want).all()


@pytest.mark.parametrize("case", [
    # n, h, w, layers
    (1, 64, 64, 3), (1, 1, 1, 2), (2, 5, 3, 4), (1, 37, 70, 2), (1, 18, 18, 3), (1, 19, 18, 3), (3, 23, 41, 6), (1, 40, 52, 1), (1, 96, 81, 5),
], ids=lambda c: "x".join(map(str, c)))
def test_chain_matches_layers(case):
    run_chain(sum(case), *case)


def test_chain_of_8_bit_activations():
    run_chain(1, 1, 45, 51, 4, top=255)
    run_chain(2, 2, 17, 16, 3, top=255, last_mode="clamp_u8")


def test_chain_pitches_offsets_and_requantisation_forms():
    run_chain(3, 1, 33, 29, 2, xbuf=80, ybuf=112, yoff=32)
    run_chain(4, 1, 33, 29, 3, last_mode="clamp_u8")
    run_chain(5, 1, 20, 20, 3, wide_shift=True)


def test_split_covers_the_run_and_refuses_other_shapes():
    from paper_2006_11735_amd import binding as B
    d = B.conv_desc(n=1, h=256, w=256, cin=64, in_c_stride=64, cout=64, kh=3, kw=3, pad_h=1, pad_w=1, out_c_stride=64, mul=20000, shift=24)
    for n in (1, 2, 7, 18):
        lens = B.iconv2d_chain_split([d] * n)
        assert sum(lens) == n and all(1 <= v <= 6 for v in lens)
    e = B.conv_desc(n=1, h=256, w=256, cin=64, in_c_stride=64, cout=32, kh=3, kw=3, pad_h=1, pad_w=1, out_c_stride=32, mul=20000, shift=24)
    with pytest.raises(B.IcnnError) as err:
        B.iconv2d_chain_split([d, e])
    assert err.value.code == B.ICNN_E_UNSUPPORTED
    with pytest.raises(B.IcnnError) as err:
        B.iconv2d_chain_brelu([d] * 7, 4096, [8192] * 7, [12288] * 7, 16384, stream=0)
    assert err.value.code == B.ICNN_E_UNSUPPORTED
