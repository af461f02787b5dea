"""The gathering kernel's rows of taps (a row of the filter as one tap of KW Cin channels): images whose rows a piece leaves on either side, rows of
taps of every length modulo a piece, NaN and infinity around what may be read; against the oracle."""
import numpy as np
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T

pytestmark = pytest.mark.gpu

BF16, F16 = wl.DTYPE_BF16, wl.DTYPE_F16
CASES = [  # n, H, W, Cin, Cout, KH, KW, stride, pad, dil_h
    (2, 9, 11, 3, 64, 7, 7, (2, 2), (3, 3), 1),         # windows that are wider than what is left of a row
    (1, 5, 3, 3, 24, 3, 3, (1, 1), (1, 1), 1),          # rows of nine values
    (2, 4, 8, 1, 40, 3, 8, (1, 1), (0, 0), 1),          # one channel: rows of exactly a piece
    (1, 6, 9, 1, 16, 2, 9, (1, 1), (1, 4), 1),
    (3, 8, 7, 2, 33, 3, 5, (1, 2), (2, 4), 2),          # padding beyond a whole piece, dilated rows, odd Cout
    (2, 12, 10, 11, 65, 3, 3, (1, 1), (1, 1), 1),
    (1, 10, 9, 35, 128, 5, 3, (2, 1), (2, 1), 1),
    (1, 7, 6, 100, 72, 3, 7, (1, 1), (1, 3), 1),        # more than one k-tile a row of taps
    (1, 3, 2, 5, 512, 3, 3, (1, 1), (2, 2), 1),         # an image smaller than the filter
    (5, 33, 31, 3, 32, 5, 5, (1, 1), (0, 0), 1),
    (1, 40, 40, 9, 130, 7, 7, (1, 1), (3, 3), 1),
]


@pytest.mark.parametrize("force", ["gather:0", "gather:1", "gather:4"])
@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("case", CASES)
def test_conv(case, dtype, force):
    import torch
    import paper_2603_06731_amd as pbk
    n, H, W, Cin, Cout, KH, KW, stride, pad, dh = case
    w = wl.Workload("taps", "conv", dtype, dtype, C.EPI_BIAS_RELU, n=n, H=H, W=W, Cin=Cin, Cout=Cout, KH=KH, KW=KW, stride=stride, pad=pad, dil=(dh, 1),
                    dist_b=("normal", float(np.sqrt(2.0 / (KH * KW * Cin)))))
    host = wl.make_inputs(w)
    dev = T.upload(host)
    with T.forced_kernel(force):
        st, out = T.run_workload(w, dev)
    assert st == 0 and "gather" in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()
    ref, pre = T.oracle_full(w, host)
    err = T.rel_err(T.to_host_f64(out, w.out_dtype).reshape(ref.shape), ref, pre)
    assert err <= T.TIGHT[dtype], err


@pytest.mark.parametrize("case", [CASES[0], CASES[4], CASES[5], CASES[7]])
def test_nan_reaches_only_its_windows(case):
    """A NaN and an infinity in one pixel each: every output whose window holds neither is finite and right."""
    import torch
    import paper_2603_06731_amd as pbk
    n, H, W, Cin, Cout, KH, KW, (sh, sw), (ph, pw), dh = case
    g = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn((n, H, W, Cin), generator=g, device="cuda").bfloat16()
    w = (torch.randn((KH, KW, Cin, Cout), generator=g, device="cuda") * (KH * KW * Cin) ** -0.5).bfloat16()
    OH, OW = (H + 2 * ph - dh * (KH - 1) - 1) // sh + 1, (W + 2 * pw - KW) // sw + 1
    y = torch.empty((n, OH, OW, Cout), device="cuda", dtype=torch.bfloat16)
    bad = x.clone()
    marked = torch.zeros((n, 1, H, W), dtype=torch.float32)
    for k, (i, j) in enumerate([(H // 2, 0), (0, W - 1)]):
        bad[n - 1, i, j, Cin // 2] = float("nan") if k else float("inf")
        marked[n - 1, 0, i, j] = 1.0
    hit = torch.nn.functional.conv2d(marked, torch.ones(1, 1, KH, KW), stride=(sh, sw), padding=(ph, pw), dilation=(dh, 1))[:, 0] > 0
    for inputs, clean in ((bad, ~hit), (x, torch.ones_like(hit))):
        y.fill_(float("nan"))
        assert pbk.pbk_conv2d_nhwc(inputs, w, y, None, n, H, W, Cin, Cout, KH, KW, sh, sw, ph, pw, dh, 1, BF16, BF16, 1.0, C.EPI_NONE,
                                   torch.cuda.current_stream()) == 0 and "gather" in pbk.pbk_last_kernel()
        ref = torch.nn.functional.conv2d(x.double().cpu().permute(0, 3, 1, 2), w.double().cpu().permute(3, 2, 0, 1), stride=(sh, sw), padding=(ph, pw),
                                         dilation=(dh, 1)).permute(0, 2, 3, 1)
        got = y.double().cpu()
        assert torch.all((got - ref).abs()[clean] <= 2.0 ** -8 * ref.abs()[clean] + 1e-4)
    assert hit.any() and not hit.all()


@pytest.mark.parametrize("n,hw,Cin,k,split", [
    (2, 16, 1, 8, False), (2, 30, 1, 9, False),         # one k-tile, three
    (1, 16, 35, 3, True), (1, 16, 11, 5, False),        # four tiles of 64 rows: six k-tiles, five
    (9, 16, 3, 11, False), (9, 16, 11, 7, True),        # 36 tiles: seven, nine
    (11, 16, 11, 7, True), (11, 16, 13, 7, True),       # 44: nine (two parts), eleven (three)
    (17, 16, 3, 11, False), (17, 16, 11, 7, True),      # 68: two parts from eight on
])
def test_parts(n, hw, Cin, k, split):
    """Workgroups share a tile by the k-tiles that are walked, not by those of a tap each: none is without one."""
    import paper_2603_06731_amd as pbk
    w = wl.Workload("taps_parts", "conv", BF16, BF16, C.EPI_BIAS_RELU, n=n, H=hw, W=hw, Cin=Cin, Cout=24, KH=k, KW=k, pad=(k // 2, (k - 1) // 2) if k % 2 else (0, 0),
                    dist_b=("normal", float(np.sqrt(2.0 / (k * k * Cin)))))
    host = wl.make_inputs(w)
    with T.forced_kernel(None):
        st, out = T.run_workload(w, T.upload(host))
    assert st == 0 and "gather_64x128x64" in pbk.pbk_last_kernel() and ("split" in pbk.pbk_last_kernel()) == split, pbk.pbk_last_kernel()
    ref, pre = T.oracle_full(w, host)
    err = T.rel_err(T.to_host_f64(out, w.out_dtype).reshape(ref.shape), ref, pre)
    assert err <= T.TIGHT[BF16], err


@pytest.mark.parametrize("force,Cin,KW,W,dil_w,rows", [
    (None, 3, 7, 20, 1, True), (None, 3, 7, 20, 2, False), (None, 9, 1, 20, 1, False), (None, 7, 1, 20, 1, False),      # taps apart, a single one
    (None, 1, 8, 20, 1, True), (None, 1, 7, 20, 1, False), (None, 1, 8, 7, 1, False),                                    # a row of taps, and an image's, of eight values
    ("gather:0", 3, 3, 20, 1, True), ("gather:0", 127, 3, 20, 1, False), ("gather:1", 127, 3, 20, 1, True), ("gather:4", 127, 3, 20, 1, True),   # as long as a tap each
    ("gather:4", 64, 3, 20, 1, True), ("gather:3", 3, 7, 20, 1, False),                                                  # 64-bit addresses
])
def test_choice(force, Cin, KW, W, dil_w, rows):
    """Which convolutions walk a row of taps as one: either side of each line, by the kernel's name."""
    import paper_2603_06731_amd as pbk
    w = wl.Workload("taps_choice", "conv", F16, F16, C.EPI_BIAS, n=1, H=24, W=W, Cin=Cin, Cout=33, KH=9, KW=KW, pad=(4, KW // 2 * dil_w), dil=(1, dil_w),
                    dist_b=("normal", float(np.sqrt(1.0 / (9 * KW * Cin)))))
    host = wl.make_inputs(w)
    with T.forced_kernel(force or "gather"):
        st, out = T.run_workload(w, T.upload(host))
    assert st == 0 and "gather" in pbk.pbk_last_kernel() and ("rows_gather" in pbk.pbk_last_kernel()) == rows, pbk.pbk_last_kernel()
    ref, pre = T.oracle_full(w, host)
    err = T.rel_err(T.to_host_f64(out, w.out_dtype).reshape(ref.shape), ref, pre)
    assert err <= T.TIGHT[F16], err
