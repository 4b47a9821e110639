"""Host-side checks of the C boundary that need no GPU: the library loads, exports every
symbol the header declares, and rejects bad arguments before launching anything."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def binding():
    from paper_2006_11735_amd import binding as B
    return B


def header_functions():
    text = open(os.path.join(ROOT, "include", "icnn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return set(re.findall(r"\b(i[a-z0-9_]+)\s*\(", text)) - {"int32_t", "int64_t", "int8_t"}


def test_library_exports_every_declared_symbol():
    B = binding()
    names = header_functions()
    assert {"iconv2d_brelu", "iadd_rescale", "iconcat", "icnn_last_error"} <= names
    lib = ctypes.CDLL(B.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), n
    assert names == set(B.EXPORTS)
    assert B.icnn_version() >= 100


def good(B, **kw):
    base = dict(n=1, h=56, w=56, cin=64, in_c_stride=64, cout=64, kh=3, kw=3, pad_h=1, pad_w=1,
                out_c_stride=64, mul=23124, shift=26, bound_q=127)
    base.update(kw)
    return B.conv_desc(**base)


def test_conv_descriptor_validation():
    B = binding()
    assert B.iconv2d_validate(good(B)) == 0
    assert B.iconv2d_out_hw(good(B, stride_h=2, stride_w=2)) == (28, 28)
    bad = [
        (dict(n=0), B.ICNN_E_SHAPE), (dict(cin=0), B.ICNN_E_SHAPE), (dict(kh=0), B.ICNN_E_SHAPE),
        (dict(stride_h=0), B.ICNN_E_SHAPE), (dict(pad_h=-1), B.ICNN_E_SHAPE),
        (dict(h=1, w=1, pad_h=0, pad_w=0), B.ICNN_E_SHAPE),
        (dict(in_c_stride=63), B.ICNN_E_SHAPE), (dict(out_c_stride=63), B.ICNN_E_SHAPE),
        (dict(out_c_offset=1), B.ICNN_E_SHAPE), (dict(out_c_offset=-1, out_c_stride=128), B.ICNN_E_SHAPE),
        (dict(cin=8192, in_c_stride=8192), B.ICNN_E_SHAPE),          # K = 73728 > 65535
        (dict(mul=0), B.ICNN_E_PARAM), (dict(mul=-5), B.ICNN_E_PARAM),
        (dict(shift=-1), B.ICNN_E_PARAM), (dict(shift=63), B.ICNN_E_PARAM),
        (dict(bound_q=0), B.ICNN_E_PARAM), (dict(bound_q=256), B.ICNN_E_PARAM),
        (dict(out_mode=7), B.ICNN_E_PARAM), (dict(res_mode=3), B.ICNN_E_PARAM),
        (dict(in_signed=1, in_sub128=1), B.ICNN_E_PARAM), (dict(in_signed=3), B.ICNN_E_PARAM),
        (dict(in_signed=2, in_sub128=1), B.ICNN_E_PARAM),
        (dict(in_signed=2, cin=4096, in_c_stride=4096), B.ICNN_E_SHAPE),    # K = 36864 > 32767 with inputs up to 255
        (dict(out_mode=B.ICNN_OUT_CLAMP_U8, lo=5, hi=4), B.ICNN_E_PARAM),
        (dict(out_mode=B.ICNN_OUT_CLAMP_U8, lo=0, hi=256), B.ICNN_E_PARAM),
        (dict(res_mode=B.ICNN_RES_PRE, res_dtype=5, res_c_stride=64), B.ICNN_E_PARAM),
        (dict(res_mode=B.ICNN_RES_PRE, res_c_stride=32), B.ICNN_E_SHAPE),
        (dict(res_mode=B.ICNN_RES_PRE, res_c_stride=64, res_mul=0), B.ICNN_E_PARAM),
        (dict(res_mode=B.ICNN_RES_PRE, res_c_stride=64, res_shift=63), B.ICNN_E_PARAM),
        (dict(res_mode=B.ICNN_RES_POST, res_c_stride=64, out_mode=B.ICNN_OUT_RAW_S32), B.ICNN_E_PARAM),
    ]
    for kw, code in bad:
        assert B.iconv2d_validate(good(B, **kw)) == code, kw
        assert B.icnn_last_error() != ""
    # raw int32 output ignores mul / shift / bound
    assert B.iconv2d_validate(good(B, out_mode=B.ICNN_OUT_RAW_S32, mul=0, shift=99, bound_q=0)) == 0
    assert B.iconv2d_packed_weight_bytes(good(B)) == 4 * 9 * 2048 + 128 * 4      # fragments + one weight sum per padded channel
    assert B.iconv2d_workspace_bytes(good(B)) == 0


def test_entry_points_reject_bad_arguments_before_any_launch():
    B = binding()
    d = good(B)
    with pytest.raises(B.IcnnError) as e:
        B.iconv2d_brelu(d, None, None, None, None, None, None, stream=0)
    assert e.value.code == B.ICNN_E_NULL
    with pytest.raises(B.IcnnError) as e:
        B.iconv2d_brelu(d, 4096, 4096 + 8, 8192, None, 12288, None, stream=0)     # packed weights misaligned
    assert e.value.code == B.ICNN_E_ALIGN
    with pytest.raises(B.IcnnError) as e:
        B.iconv2d_brelu(good(B, res_mode=B.ICNN_RES_PRE, res_c_stride=64), 4096, 8192, 12288, None, 16384,
                        None, stream=0)
    assert e.value.code == B.ICNN_E_NULL
    with pytest.raises(B.IcnnError) as e:
        B.iconv2d_prepack_weights(d, None, 4096, stream=0)
    assert e.value.code == B.ICNN_E_NULL
    a = B.add_desc(count_pixels=10, c=16, a_c_stride=16, b_c_stride=16, out_c_stride=16, hi=127)
    for kw, code in ((dict(b_mul=0), B.ICNN_E_PARAM), (dict(shift=63), B.ICNN_E_PARAM),
                     (dict(a_c_stride=8), B.ICNN_E_SHAPE), (dict(count_pixels=-1), B.ICNN_E_SHAPE),
                     (dict(out_mode=B.ICNN_OUT_BRELU_U8), B.ICNN_E_PARAM), (dict(a_dtype=9), B.ICNN_E_PARAM),
                     (dict(lo=9, hi=3), B.ICNN_E_PARAM)):
        bad = B.add_desc(count_pixels=10, c=16, a_c_stride=16, b_c_stride=16, out_c_stride=16, hi=127)
        for k, v in kw.items():
            setattr(bad, k, v)
        with pytest.raises(B.IcnnError) as e:
            B.iadd_rescale(bad, 4096, 8192, 12288, stream=0)
        assert e.value.code == code, kw
    with pytest.raises(B.IcnnError) as e:
        B.iadd_rescale(a, None, 8192, 12288, stream=0)
    assert e.value.code == B.ICNN_E_NULL
    with pytest.raises(B.IcnnError) as e:
        B.iconcat([4096] * 17, [1] * 17, [1] * 17, [1] * 17, [0] * 17, 127, 4, 8192, 17, stream=0)
    assert e.value.code == B.ICNN_E_SHAPE
    with pytest.raises(B.IcnnError) as e:
        B.iconcat([4096, 8192], [8, 8], [8, 8], [1, 1], [0, 0], 127, 4, 12288, 15, stream=0)
    assert e.value.code == B.ICNN_E_SHAPE
    with pytest.raises(B.IcnnError) as e:
        B.iconcat([4096, 8192], [8, 8], [8, 8], [1, 0], [0, 0], 127, 4, 12288, 16, stream=0)
    assert e.value.code == B.ICNN_E_PARAM
    with pytest.raises(B.IcnnError) as e:
        B.imaxpool2d_u8(1, 8, 8, 16, 3, 2, 3, 4096, 8192, stream=0)
    assert e.value.code == B.ICNN_E_SHAPE
    with pytest.raises(B.IcnnError) as e:
        B.iavgpool_global_u8(1, 7, 7, 16, 0, 20, 127, 4096, 8192, stream=0)
    assert e.value.code == B.ICNN_E_PARAM
    with pytest.raises(B.IcnnError) as e:
        B.irenormalize_u8(16, None, 4096, stream=0)
    assert e.value.code == B.ICNN_E_NULL


def test_twin_layers_are_refused_on_the_host_where_the_fused_kernel_does_not_take_them():
    """iconv2d_twin_brelu checks both descriptors, the pointers and the pair's shape before anything is launched."""
    B = binding()

    def branch(k, cout, off, **kw):
        args = dict(h=32, w=64, cout=cout, kh=k, kw=k, pad_h=k // 2, pad_w=k // 2, out_c_stride=48, out_c_offset=off)
        args.update(kw)
        return good(B, **args)
    x, wa, wb, ba, bb, y = 4096, 8192, 12288, 16384, 20480, 24576
    cases = [
        ((branch(5, 32, 0), branch(5, 16, 32)), B.ICNN_E_UNSUPPORTED),                      # kernels of one size
        ((branch(7, 32, 0), branch(5, 16, 32)), B.ICNN_E_UNSUPPORTED),                      # no 7x7 form
        ((branch(5, 32, 0), branch(3, 16, 32, h=16)), B.ICNN_E_SHAPE),                      # different pictures
        ((branch(5, 32, 0), branch(3, 16, 32, cin=48, in_c_stride=48)), B.ICNN_E_SHAPE),    # different inputs
        ((branch(5, 32, 0, res_mode=B.ICNN_RES_PRE, res_c_stride=32), branch(3, 16, 32)), B.ICNN_E_UNSUPPORTED),
        ((branch(5, 32, 0, in_signed=B.ICNN_IN_U8_FULL), branch(3, 16, 32, in_signed=B.ICNN_IN_U8_FULL)), B.ICNN_E_UNSUPPORTED),
        ((branch(5, 32, 0, cin=32, in_c_stride=32), branch(3, 16, 32, cin=32, in_c_stride=32)), B.ICNN_E_UNSUPPORTED),
    ]
    for (da, db), code in cases:
        with pytest.raises(B.IcnnError) as e:
            B.iconv2d_twin_brelu(da, x, wa, ba, y, db, wb, bb, y, stream=0)
        assert e.value.code == code, (da.kh, db.kh, e.value.code)
    with pytest.raises(B.IcnnError) as e:
        B.iconv2d_twin_brelu(branch(5, 32, 0), x, wa, ba, y, branch(3, 16, 32), wb, bb, None, stream=0)
    assert e.value.code == B.ICNN_E_NULL
    with pytest.raises(B.IcnnError) as e:
        B.iconv2d_twin_brelu(branch(5, 32, 0), x + 8, wa, ba, y, branch(3, 16, 32), wb, bb, y, stream=0)
    assert e.value.code == B.ICNN_E_UNSUPPORTED                                              # misaligned input


def test_a_chain_refuses_an_output_over_its_input():
    B = binding()
    x, w, bias = 1 << 20, 1 << 30, 1 << 31
    size = 16 * 16 * 64

    def code(y, in_pitch=64, out_pitch=64, offset=0):
        first, last = good(B, h=16, w=16, in_c_stride=in_pitch), good(B, h=16, w=16, out_c_stride=out_pitch, out_c_offset=offset)
        with pytest.raises(B.IcnnError) as e:
            B.iconv2d_chain_brelu([first, last], x, [w] * 2, [bias] * 2, y, stream=0)
        return e.value.code
    overlapping = [(x,), (x + size - 64,), (x - size + 64,), (x, 128, 128, 0), (x, 128, 128, 32), (x + 32, 128, 128, 0), (x - 16, 128, 128, 0),
                   (x, 128, 192, 64)]
    for case in overlapping:
        assert code(*case) == B.ICNN_E_UNSUPPORTED, case
    import torch
    if not torch.cuda.is_available():                    # accepted: the launch itself fails where there is no GPU
        for case in [(x + size,), (x - size,), (x, 128, 128, 64), (x + 64, 128, 128, 0), (x - 64, 128, 128, 0), (x, 192, 192, 112)]:
            assert code(*case) == B.ICNN_E_LAUNCH, case


def test_chain_split_by_plane_size():
    # what the launches have been timed at (18 layers of 3x3 x 64): few pixels in long chains, large planes layer by layer where the kernel
    # with two-dimensional tiles takes them, in chains where inputs go up to 255
    B = binding()

    def split(h, w, full=False, n=18):
        kind = B.ICNN_IN_U8_FULL if full else B.ICNN_IN_U8_LE127
        return B.iconv2d_chain_split([good(B, h=h, w=w, in_signed=kind, bound_q=255 if full else 127)] * n)
    assert split(64, 64) == [6, 6, 6] and split(320, 320) == [2] * 9 and split(256, 256) == [2, 4, 4, 4, 4]
    for h, w in ((384, 512), (480, 640), (720, 1280), (1600, 2560)):
        assert split(h, w) == [1] * 18, (h, w)
        assert min(split(h, w, full=True)) >= 2, (h, w)
    assert max(split(256, 384)) > 1 and min(split(256, 384, full=True)) > 1
    # inputs that go up to 255 from the second layer on: only those layers change their own cost
    d = [good(B, h=720, w=1280)] * 4 + [good(B, h=720, w=1280, in_signed=B.ICNN_IN_U8_FULL)] * 4
    assert B.iconv2d_chain_split(d) == [1, 1, 1, 1, 2, 2]
    for n in (1, 2, 7, 255):
        assert sum(split(100, 130, n=n)) == n


def test_fused_launches_refuse_outputs_over_what_other_workgroups_read():
    B = binding()
    import torch
    accepted = None if torch.cuda.is_available() else B.ICNN_E_LAUNCH      # the launch itself fails where there is no GPU
    x, t, y, z, w, bias = (k << 24 for k in range(1, 7))

    def code(fn, *args):
        with pytest.raises(B.IcnnError) as e:
            fn(*args, stream=0)
        return e.value.code

    def one(cin, cout, **kw):
        return good(B, **{**dict(h=16, w=16, cin=cin, in_c_stride=cin, cout=cout, kh=1, kw=1, pad_h=0, pad_w=0, out_c_stride=cout), **kw})
    mid = good(B, h=16, w=16)
    skip = dict(res_mode=B.ICNN_RES_PRE, res_c_stride=64, res_mul=3, res_shift=5)
    proj = dict(res_mode=B.ICNN_RES_PRE, res_dtype=B.ICNN_S32, res_c_stride=256, res_mul=3, res_shift=12)
    raw = one(64, 256, out_mode=B.ICNN_OUT_RAW_S32)
    last = one(64, 256, **proj)
    wide = one(256, 1024, res_mode=B.ICNN_RES_PRE, res_c_stride=1024, res_mul=3, res_shift=5)
    pix = 16 * 16
    cases = [
        # (overlapping?, call)
        (True, (B.iconv2d_bottleneck_brelu, one(64, 64), x, w, bias, mid, w, bias, one(64, 64, **skip), w, bias, x, x)),
        (False, (B.iconv2d_bottleneck_brelu, one(64, 64), x, w, bias, mid, w, bias, one(64, 64, **skip), w, bias, x, y)),
        (True, (B.iconv2d_bottleneck_dual_brelu, one(64, 64), x, w, bias, mid, w, bias, last, w, bias, raw, w, bias, x - pix * 255)),
        (False, (B.iconv2d_bottleneck_dual_brelu, one(64, 64), x, w, bias, mid, w, bias, last, w, bias, raw, w, bias, x - pix * 256)),
        (True, (B.iconv2d_dual_brelu, last, t, w, bias, raw, x, w, bias, x)),
        (True, (B.iconv2d_dual_brelu, last, t, w, bias, raw, x, w, bias, t)),
        (False, (B.iconv2d_dual_brelu, last, t, w, bias, raw, x, w, bias, y)),
        # a pair may write over its own pixels' inputs, not over its other output or another pixel's input
        (False, (B.iconv2d_pair_brelu, wide, t, w, bias, x, y, one(1024, 256), w, bias, t)),
        (False, (B.iconv2d_pair_brelu, wide, t, w, bias, x, x, one(1024, 256), w, bias, z)),
        (True, (B.iconv2d_pair_brelu, wide, t, w, bias, x, y, one(1024, 256), w, bias, t + 256)),
        (True, (B.iconv2d_pair_brelu, wide, t, w, bias, x, y, one(1024, 256), w, bias, y)),
        (True, (B.iconv2d_pair_brelu, wide, t, w, bias, x, y, one(1024, 256), w, bias, x + 1024 * 16)),
        (True, (B.iconv2d_maxpool_brelu, good(B, h=32, w=32, cin=3, in_c_stride=3, kh=7, kw=7, stride_h=2, stride_w=2, pad_h=3, pad_w=3, in_sub128=1), 3, 2, 1,
                x, w, bias, x + 16)),
        (False, (B.iconv2d_maxpool_brelu, good(B, h=32, w=32, cin=3, in_c_stride=3, kh=7, kw=7, stride_h=2, stride_w=2, pad_h=3, pad_w=3, in_sub128=1), 3, 2, 1,
                 x, w, bias, y)),
    ]

    def branch(k, cout, offset, **kw):
        return good(B, **{**dict(h=32, w=64, cout=cout, kh=k, kw=k, pad_h=k // 2, pad_w=k // 2, out_c_stride=48, out_c_offset=offset), **kw})
    cases += [
        (False, (B.iconv2d_twin_brelu, branch(5, 32, 0), x, w, bias, y, branch(3, 16, 32), w, bias, y)),
        (True, (B.iconv2d_twin_brelu, branch(5, 32, 0), x, w, bias, y, branch(3, 16, 16), w, bias, y)),
        (True, (B.iconv2d_twin_brelu, branch(5, 32, 0), x, w, bias, x, branch(3, 16, 32), w, bias, y)),
        (True, (B.iconv2d_twin_brelu, branch(5, 32, 0), x, w, bias, y, branch(3, 16, 32), w, bias, x + 64 * 64)),
    ]
    narrow = dict(cin=48, in_c_stride=48)
    tail = good(B, h=32, w=64, cout=1, out_c_stride=1, **narrow)
    for at, over in ((y, False), (x, True), (x + 32 * 64 * 48 - 1, True), (x + 32 * 64 * 48, False)):
        cases.append((over, (B.iconv2d_twin_last_brelu, branch(3, 16, 0, **narrow), x, w, bias, branch(1, 32, 16, **narrow), w, bias, tail, w, bias, None, at)))
    for over, call in cases:
        if over:
            assert code(*call) == B.ICNN_E_UNSUPPORTED, call
        elif accepted is not None:
            assert code(*call) == accepted, call


def test_every_tuning_name_of_the_header_is_known():
    B = binding()
    text = open(os.path.join(ROOT, "include", "icnn.h")).read()
    part = text[text.index("Kernel-selection override"):text.index("int icnn_set_tuning")]
    names = set(re.findall(r'"([a-z0-9_]+)"', part)) - {"reset"}
    assert {"tile", "no_fc", "no_lat", "lat", "ksplit", "no_pic"} <= names
    try:
        for name in sorted(names):
            B.icnn_set_tuning(name, 0)
            with pytest.raises(B.IcnnError) as e:
                B.icnn_set_tuning(name, 99)
            assert e.value.code == B.ICNN_E_PARAM and "outside" in str(e.value), name
        with pytest.raises(B.IcnnError) as e:
            B.icnn_set_tuning("colour", 1)
        assert "unknown" in str(e.value)
    finally:
        B.icnn_set_tuning("reset")


def test_tuning_overrides_are_validated():
    B = binding()
    try:
        B.icnn_set_tuning("tile", 3)
        B.icnn_set_tuning("halo_always", 1)
        for name, value in (("tile", 5), ("tile", -2), ("stages", 1), ("stages", 7), ("no_fc", 2), ("colour", 1)):
            with pytest.raises(B.IcnnError) as e:
                B.icnn_set_tuning(name, value)
            assert e.value.code == B.ICNN_E_PARAM, (name, value)
    finally:
        B.icnn_set_tuning("reset")
