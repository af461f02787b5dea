"""Transposed convolution by residue classes of the output (matrix-unit kernel): strides
larger than the filter (classes without a tap), strides that share a factor with the
dilation, strides beyond the output, images whose size does not divide by the stride,
k-tiles that span taps, and rows stored one element at a time."""
import numpy as np
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T

pytestmark = pytest.mark.gpu

BF16, F16, F32 = wl.DTYPE_BF16, wl.DTYPE_F16, wl.DTYPE_F32

CASES = [  # n, H, W, Cin, Cout, KH, KW, stride, pad, out_pad, dil
    (2, 9, 7, 64, 72, 2, 3, (3, 4), (0, 1), (2, 1), (1, 1)),       # filter smaller than the stride: empty classes
    (1, 8, 9, 32, 40, 3, 3, (4, 6), (2, 1), (1, 3), (2, 4)),       # gcd(stride, dil) = 2
    (1, 7, 6, 32, 32, 5, 4, (2, 2), (3, 2), (1, 1), (2, 2)),       # dil a multiple of the stride: odd rows have no tap
    (3, 1, 2, 64, 64, 3, 3, (7, 5), (1, 2), (0, 0), (1, 1)),       # stride beyond the output
    (5, 13, 11, 40, 136, 4, 4, (2, 2), (1, 1), (1, 0), (1, 1)),    # a k-tile spans taps
    (2, 24, 23, 128, 256, 4, 4, (2, 2), (1, 1), (0, 0), (1, 1)),
]


@pytest.mark.parametrize("dtype,out_dtype,cfg", [(BF16, BF16, 0), (BF16, BF16, 1), (BF16, BF16, 6), (F16, F32, None)])
@pytest.mark.parametrize("case", CASES)
def test_residue_classes(case, dtype, out_dtype, cfg):
    import paper_2603_06731_amd as pbk
    n, H, W, Cin, Cout, KH, KW, stride, pad, out_pad, dil = case
    w = wl.Workload("convT_classes", "conv", dtype, out_dtype, C.EPI_BIAS_RELU, n=n, H=H, W=W, Cin=Cin, Cout=Cout,
                    KH=KH, KW=KW, stride=stride, pad=pad, out_pad=out_pad, dil=dil, transposed=1,
                    dist_b=("normal", float(np.sqrt(2.0 / (KH * KW * Cin)))))
    host = wl.make_inputs(w)
    with T.forced_kernel(None if cfg is None else f"mfma:{cfg}"):
        st, out = T.run_workload(w, T.upload(host))
    assert st == 0, pbk.pbk_status_string(st)
    assert "mfma" in pbk.pbk_last_kernel()
    ref, pre = T.oracle_full(w, host)
    err = T.rel_err(T.to_host_f64(out, w.out_dtype).reshape(ref.shape), ref, pre)
    assert err <= T.TIGHT[out_dtype], err        # the bound of the output rounding, as for every convolution


@pytest.mark.parametrize("cfg", [0, 1, 2, 6])
@pytest.mark.parametrize("case", [
    (2, 9, 7, 32, 40, 2, 2, (2, 2), (0, 0), (0, 0), (1, 1)),        # one tap per class, half a k-tile of channels
    (3, 11, 5, 72, 136, 2, 2, (2, 2), (0, 0), (1, 0), (1, 1)),      # ... a k-tile and a ragged one; classes of unequal size
    (2, 13, 12, 8, 264, 1, 1, (1, 1), (0, 0), (0, 0), (1, 1)),      # a single class: rows of C in order
    (1, 6, 9, 200, 72, 3, 3, (3, 4), (1, 1), (0, 0), (2, 3)),       # three k-tiles of 64 and a remainder; classes without a tap
    (2, 10, 9, 40, 48, 3, 5, (2, 2), (1, 2), (1, 1), (1, 1)),       # classes of one tap beside classes of two, three and six
    (1, 1, 300, 24, 32, 2, 3, (4, 2), (0, 1), (0, 0), (1, 1)),      # one image row, stride beyond the output along h
])
def test_single_tap_classes(case, cfg):
    """A class that one tap meets walks its channels as they are, whatever their number."""
    test_residue_classes(case, BF16, BF16, cfg)


def transpose(x, w, bias, geom, force=None):
    """geom: n, H, W, Cin, Cout, KH, KW, stride, pad, dil; bf16 operands, bias epilogue.  Returns (y, kernel name)."""
    import torch
    import paper_2603_06731_amd as pbk
    n, H, W, Cin, Cout, KH, KW, s, p, d = geom
    OH, OW = ((size - 1) * s[i] - 2 * p[i] + d[i] * (k - 1) + 1 for i, (size, k) in enumerate(((H, KH), (W, KW))))
    y = torch.full((n, OH, OW, Cout), float("nan"), dtype=torch.bfloat16, device="cuda")
    with T.forced_kernel(force):
        st = pbk.pbk_conv2d_transpose_nhwc(x, w, y, bias, n, H, W, Cin, Cout, KH, KW, *s, *p, 0, 0, *d, BF16, BF16, 1.0, C.EPI_BIAS)
    assert st == 0, pbk.pbk_status_string(st)
    return y, pbk.pbk_last_kernel()


def operands(geom, seed):
    import torch
    n, H, W, Cin, Cout, KH, KW = geom[:7]
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(n, H, W, Cin, generator=g, device="cuda", dtype=torch.bfloat16)
    w = torch.randn(KH, KW, Cin, Cout, generator=g, device="cuda", dtype=torch.bfloat16) * Cin ** -0.5
    return x, w, torch.randn(Cout, generator=g, device="cuda")


def close(got, ref):
    """One rounding to bf16 (2^-9 of the value; twice that) and fp32 sums of order one."""
    return bool(((got.float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all())


@pytest.mark.parametrize("cfg", [1, 2])
def test_rows_far_beyond_the_image(cfg):
    """A dilation that puts the last tap's rows 2^31 bytes behind the image: the class's pixel offsets wrap and the tap's offset brings
    them back."""
    dil, taps = 4096, 5
    geom = (1, 4, 1, 65536, 8, taps, 1, (1, 1), (0, 0), (dil, 1))
    assert (taps - 1) * dil * 65536 * 2 >= 2 ** 31
    x, w, bias = operands(geom, 1)
    y, kern = transpose(x, w, bias, geom, f"mfma:{cfg}")
    assert ("classes" in kern) == (cfg == 2), kern
    ref = bias.double().expand(y.shape[1], 8).clone()
    for kh in range(taps):
        ref[kh * dil:kh * dil + 4] += x[0, :, 0].double() @ w[kh, 0].double()
    assert close(y[0, :, 0], ref)


@pytest.mark.parametrize("force", [None, "mfma:2"])
def test_more_classes_than_a_launch_holds(force):
    """A stride of 4096 over a 2 x 2 image: 2^24 classes, one tile of 256 threads each.  All taps then, on the same matrix units."""
    s, Cin = 4096, 128
    geom = (1, 2, 2, Cin, 8, 2, 2, (s, s), (0, 0), (1, 1))
    x, w, bias = operands(geom, 2)
    y, kern = transpose(x, w, bias, geom, force)
    assert "mfma" in kern and "classes" not in kern, kern
    for ih in range(2):
        for iw in range(2):
            for kh in range(2):
                for kw in range(2):
                    at = y[0, ih * s + kh, iw * s + kw]
                    assert close(at, bias + x[0, ih, iw].float() @ w[kh, kw].float()), (ih, iw, kh, kw)
                    at.copy_(bias)
    assert bool((y == bias.bfloat16()).all())


@pytest.mark.parametrize("force", [None, "mfma:2", "mfma:14"])
def test_more_tiles_than_a_launch_holds(force):
    """Strides of 4096 and 3000: 12 million classes, fewer than a launch holds with 256 threads each, more than with the 512 of these tiles."""
    s, Cin = (4096, 3000), 128
    assert 2 ** 23 <= s[0] * s[1] < 2 ** 24
    geom = (1, 2, 2, Cin, 8, 2, 2, s, (0, 0), (1, 1))
    x, w, bias = operands(geom, 6)
    y, kern = transpose(x, w, bias, geom, force)
    assert "mfma" in kern and "classes" not in kern, kern
    for ih in range(2):
        for iw in range(2):
            for kh in range(2):
                for kw in range(2):
                    at = y[0, ih * s[0] + kh, iw * s[1] + kw]
                    assert close(at, bias + x[0, ih, iw].float() @ w[kh, kw].float()), (ih, iw, kh, kw)
                    at.copy_(bias)
    assert bool((y == bias.bfloat16()).all())


@pytest.mark.parametrize("case", CASES)
def test_residue_classes_ring(case):
    """The classes themselves, also where the automatic choice keeps all taps in the loop."""
    import paper_2603_06731_amd as pbk
    test_residue_classes(case, F16, F16, 2)
    assert "classes" in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()


@pytest.mark.parametrize("n,hw,Cin,Cout,k,stride,dil,kernel", [
    (2, 14, 40, 64, 2, 2, 1, "s2"), (2, 14, 48, 64, 2, 2, 1, "classes"),         # saved 120, 144
    (2, 14, 512, 64, 1, 2, 1, "s2"), (2, 14, 64, 64, 3, 1, 1, "s2"), (2, 14, 64, 64, 3, 2, 2, "s2"),      # nothing saved
    (2, 14, 64, 64, 3, 4, 2, "classes"),                                         # a stride that shares a factor with the dilation
    (8, 64, 64, 256, 2, 2, 1, "128x256x32"), (8, 64, 128, 256, 2, 2, 1, "classes"),                         # wide tiles: saved 192, 384
    (8, 64, 208, 256, 2, 2, 1, "128x256x32"), (8, 64, 216, 256, 2, 2, 1, "classes"),                        # ... channels across k-tiles: 624, 648
    (8, 64, 56, 248, 2, 2, 1, "classes"), (1, 32, 56, 256, 2, 2, 1, "classes"),  # not wide: columns, tiles
])
def test_dispatch(n, hw, Cin, Cout, k, stride, dil, kernel):
    """Classes or all taps, with the automatic choice, on either side of each line."""
    import torch
    geom = (n, hw, hw, Cin, Cout, k, k, (stride, stride), (0, 0), (dil, dil))
    x, w, bias = operands(geom, 5)
    y, kern = transpose(x, w, bias, geom)
    assert kern.endswith(kernel) or (kernel[0] == "1" and kernel in kern), kern
    # image 0: every input pixel painted through every tap
    E = (hw - 1) * stride + 1
    ref = bias.expand(y.shape[1], y.shape[2], Cout).clone()
    for kh in range(k):
        for kw in range(k):
            part = x[0].reshape(hw * hw, Cin).float() @ w[kh, kw].float()
            ref[kh * dil:kh * dil + E:stride, kw * dil:kw * dil + E:stride] += part.reshape(hw, hw, Cout)
    assert close(y[0], ref)


def test_weights_of_2_gib():
    """k-tiles that lie inside one tap start at a 64-bit address: the weights may be of any size."""
    geom = (1, 4, 4, 8192, 8192, 4, 4, (2, 2), (1, 1), (1, 1))
    x, w, bias = operands(geom, 3)
    y, kern = transpose(x, w, bias, geom)
    assert "mfma" in kern, kern
    ref = bias.expand(10, 10, 8192).clone()
    for kh in range(4):
        for kw in range(4):
            # input pixel (ih, iw) paints output pixel (2 ih - 1 + kh, 2 iw - 1 + kw): one row and column of margin
            ref[kh:kh + 7:2, kw:kw + 7:2] += (x.reshape(16, 8192).float() @ w[kh, kw].float()).reshape(4, 4, 8192)
    assert close(y[0], ref[1:9, 1:9])


@pytest.mark.parametrize("dtype,out_dtype", [(BF16, BF16), (F16, F32)])
@pytest.mark.parametrize("case,tiles64", [
    ((2, 9, 7, 128, 72, 2, 3, (3, 4), (0, 1), (2, 1), (1, 1)), True),      # classes without a tap, columns beyond the tile
    ((1, 8, 9, 40, 40, 5, 5, (4, 6), (2, 1), (1, 3), (2, 4)), True),       # gcd(stride, dil) = 2; a wave's weight rows span taps
    ((3, 11, 5, 72, 136, 4, 4, (2, 2), (1, 1), (1, 0), (1, 1)), True),     # rounds that span taps, classes of unequal size
    ((1, 13, 11, 32, 32, 5, 7, (2, 2), (3, 2), (1, 1), (1, 1)), True),     # four taps a round
    ((2, 6, 9, 192, 64, 4, 3, (2, 1), (1, 1), (0, 0), (1, 1)), True),      # taps that begin inside a round, a stride of one
    ((1, 5, 6, 1032, 24, 3, 3, (2, 2), (1, 1), (0, 0), (1, 3)), True),     # more channels than a round, dilation
    ((8, 32, 32, 64, 64, 4, 4, (2, 2), (1, 1), (0, 0), (1, 1)), False),    # 1024 tiles
    ((2, 16, 16, 32, 64, 3, 3, (2, 2), (1, 1), (1, 1), (1, 1)), True),     # two taps by two: 128
    ((2, 16, 16, 24, 64, 3, 3, (2, 2), (1, 1), (1, 1), (1, 1)), False)])   # ... 96
def test_tiles_of_64_columns(case, tiles64, dtype, out_dtype):
    """The automatic choice of the 64-wide tiles, whose k advances by rounds of 128 over taps and channels."""
    import paper_2603_06731_amd as pbk
    test_residue_classes(case, dtype, out_dtype, None)
    assert pbk.pbk_last_kernel().endswith("tile64_32x64_s3_classes") == tiles64, pbk.pbk_last_kernel()


@pytest.mark.parametrize("Cin,Cout,hw,tiles64", [(128, 64, 32, True), (128, 64, 33, False), (136, 64, 33, True), (128, 72, 24, True)])
def test_tiles_of_64_columns_single_round(Cin, Cout, hw, tiles64):
    """One tap a class: 128 values of k, a single round, up to 256 tiles; two rounds, and more than 64 columns, beyond."""
    import paper_2603_06731_amd as pbk
    test_residue_classes((2, hw, hw, Cin, Cout, 2, 2, (2, 2), (0, 0), (0, 0), (1, 1)), BF16, BF16, None)
    assert ("tile64" in pbk.pbk_last_kernel()) == tiles64, pbk.pbk_last_kernel()
