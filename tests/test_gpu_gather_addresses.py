"""The gathering kernel's convolution with 64-bit addresses, which image tensors and weights from 2 GiB on take: chosen by hand for small
problems on each of its tiles, split and not, against the oracle; and by itself for two image tensors of that size."""
import numpy as np
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T
import test_gpu_gather as G
import test_gpu_gather_split as S
from test_gpu_few_tiles import TOL

pytestmark = pytest.mark.gpu

BF16, F16, F32 = wl.DTYPE_BF16, wl.DTYPE_F16, wl.DTYPE_F32

CASES = [c[:10] for c in S.CONVS] + [
    (1, 20, 19, 64, 136, 3, 3, (1, 1), (1, 1), (1, 1)),       # whole pieces only
    (2, 15, 17, 9, 40, 5, 3, (1, 2), (2, 1), (2, 1)),
    (1, 9, 9, 12, 40, 1, 2, (1, 1), (0, 0), (1, 1)),          # one k-tile
    (4, 70, 70, 20, 40, 3, 3, (1, 1), (1, 1), (1, 1)),        # more 64-row tiles than compute units: not the deep form
]


@pytest.mark.parametrize("force", ["gather:2", "gather:3"])
@pytest.mark.parametrize("dtype,out_dtype", [(BF16, BF16), (F16, F32)])
@pytest.mark.parametrize("case", CASES)
def test_conv(case, dtype, out_dtype, force):
    import paper_2603_06731_amd as pbk
    n, H, W, Cin, Cout, KH, KW, stride, pad, dil = case
    w = wl.Workload("gather_addresses", "conv", dtype, out_dtype, C.EPI_BIAS_RELU, n=n, H=H, W=W, Cin=Cin, Cout=Cout, KH=KH, KW=KW,
                    stride=stride, pad=pad, dil=dil, dist_b=("normal", float(np.sqrt(2.0 / (KH * KW * Cin)))))
    host = wl.make_inputs(w)
    with T.forced_kernel(force):
        st, out = T.run_workload(w, T.upload(host))
    name = pbk.pbk_last_kernel()
    assert st == 0 and "_a64" in name and ("gather_64x128" if force == "gather:3" else "gather_128x128x32") in name, name
    if force == "gather:3" and case in [c[:10] for c in S.CONVS]:
        assert ("split" in name) == [c[10] for c in S.CONVS if c[:10] == case][0], name
    if case == CASES[-1] and force == "gather:3":
        assert "64x128x32" in name, name
    ref, pre = T.oracle_full(w, host)
    err = T.rel_err(T.to_host_f64(out, w.out_dtype).reshape(ref.shape), ref, pre)
    assert err <= TOL[out_dtype], err


@pytest.mark.parametrize("n,H,W,Cin,Cout,stride,pad,kernel", [
    (32, 1024, 1024, 32, 16, 1, 1, "128x128x32_w2x2_a64"),            # 2 GiB: aligned, but beyond the kernel for aligned operands
    (2, 2048, 2048, 136, 32, 64, 0, "64x128x64_w4x2_a64_split"),      # 2.1 GiB in two images, few outputs
])
def test_image_tensors_from_2_gib(n, H, W, Cin, Cout, stride, pad, kernel):
    """Sampled outputs, those of the first and the last image's corners among them, against 64-bit sums."""
    import torch
    import paper_2603_06731_amd as pbk
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((n, H, W, Cin), generator=g, device="cuda", dtype=torch.bfloat16)
    assert x.numel() * 2 >= 1 << 31
    w = (torch.randn((3, 3, Cin, Cout), generator=g, device="cuda") * (9 * Cin) ** -0.5).bfloat16()
    OH, OW = (H + 2 * pad - 3) // stride + 1, (W + 2 * pad - 3) // stride + 1
    y = torch.full((n, OH, OW, Cout), float("nan"), device="cuda", dtype=torch.bfloat16)
    st = pbk.pbk_conv2d_nhwc(x, w, y, None, n, H, W, Cin, Cout, 3, 3, stride, stride, pad, pad, 1, 1, BF16, BF16, 1.0, C.EPI_NONE,
                             torch.cuda.current_stream())
    assert st == 0 and pbk.pbk_last_kernel().endswith(kernel), pbk.pbk_last_kernel()
    s = 4000
    sn, sh, sw = (torch.randint(m, (s,), generator=g, device="cuda") for m in (n, OH, OW))
    for i, c in enumerate([(a, b, d) for a in (0, n - 1) for b in (0, OH - 1) for d in (0, OW - 1)]):
        sn[i], sh[i], sw[i] = c
    ref = torch.zeros((s, Cout), device="cuda", dtype=torch.float64)
    for kh in range(3):
        for kw in range(3):
            ih, iw = sh * stride - pad + kh, sw * stride - pad + kw
            ok = (ih >= 0) & (ih < H) & (iw >= 0) & (iw < W)
            ref += (x[sn, ih.clamp(0, H - 1), iw.clamp(0, W - 1)].double() * ok[:, None]) @ w[kh, kw].double()
    # one rounding to bf16 (2^-9 of the value), fp32 sums of 9 Cin terms of order (9 Cin)^-1/2
    assert torch.all((y[sn, sh, sw].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4)
