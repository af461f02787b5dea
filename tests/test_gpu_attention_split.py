"""Attention whose key tiles are dealt to two groups of waves, against the definition evaluated in float64."""
import pytest

import workloads as wl
import pbk_testlib as T

pytestmark = pytest.mark.gpu

BF16, F16 = wl.DTYPE_BF16, wl.DTYPE_F16

CASES = [  # batch, Nq, Nk, row padding
    (1, 1, 1, 0),            # the second group has no key
    (2, 5, 65, 8),           # its only tile holds one key
    (2, 130, 130, 8),        # three tiles: halves of two and one
    (1, 300, 200, 0),        # causal: queries that see no key (NaN), tiles with no visible key
    (3, 129, 256, 0),        # whole tiles
    (1, 64, 707, 8),         # tiles without a bounds test in both halves
    (1, 450, 450, 0),
]


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_split(D, dtype, causal):
    import torch
    import paper_2603_06731_amd as pbk
    tdt = torch.bfloat16 if dtype == BF16 else torch.float16
    for b, Nq, Nk, pad in CASES:
        g = torch.Generator().manual_seed(b * 1000 + Nk)
        ld = D + pad
        # (rows padded with NaN: nothing outside the views may be read into the result)
        q, k, v = (torch.full((b, n, ld), float("nan")) for n in (Nq, Nk, Nk))
        for x in (q, k, v):
            x[..., :D] = torch.randn(x[..., :D].shape, generator=g)
        k[:, Nk // 2, :D] *= 6.0                     # scores that move the reference point
        q, k, v = q.to(tdt), k.to(tdt), v.to(tdt)
        out = torch.zeros(b, Nq, ld, dtype=tdt, device="cuda")
        alpha = D ** -0.5
        dims = (b, Nq, Nk, D, ld, ld, ld, ld, Nq * ld, Nk * ld, Nk * ld, Nq * ld)
        with T.forced_kernel("mfma:2"):
            if causal:
                st = pbk.pbk_attention_causal(q.cuda(), k.cuda(), v.cuda(), out, *dims, dtype, alpha)
            else:
                st = pbk.pbk_attention(q.cuda(), k.cuda(), v.cuda(), None, out, *dims, 0, 0, dtype, alpha)
        assert st == 0 and "kv64x2" in pbk.pbk_last_kernel()
        qd, kd, vd = (x[..., :D].double() for x in (q, k, v))
        s = qd @ kd.transpose(1, 2).contiguous() * alpha
        if causal:
            s = s.masked_fill(torch.arange(Nk)[None, :] > torch.arange(Nq)[:, None] + Nk - Nq, float("-inf"))
        w = torch.softmax(s, -1)
        ref = w @ vd
        got = out.cpu().double()
        assert torch.all(got[..., D:] == 0)
        got = got[..., :D]
        assert torch.equal(torch.isnan(got), torch.isnan(ref))
        # weights rounded to 16 bits (u of their value), then the output: u (sum w |v| + |o|), with fp32 sums below that
        u = 2.0 ** -8 if dtype == BF16 else 2.0 ** -11
        bound = u * ((w @ vd.abs()) + ref.abs()) + 1e-5
        ok = (got - ref).abs() <= bound
        assert torch.all(ok | torch.isnan(ref)), (b, Nq, Nk, float(((got - ref).abs() / bound).nan_to_num().max()))


@pytest.mark.parametrize("batch,Nq,Nk,D,causal,split", [
    (2, 1024, 1024, 64, 1, True), (2, 65, 96, 64, 1, True), (2, 65, 95, 64, 1, False), (1, 64, 1024, 64, 0, True), (1, 64, 1023, 64, 0, False),
    (1, 64, 1024, 128, 0, False), (1, 100, 1024, 128, 0, True), (1, 100, 2048, 128, 1, True),
    (48, 1024, 1024, 32, 0, True), (48, 1023, 1023, 32, 0, False), (49, 1024, 1024, 32, 0, False), (16, 4096, 4096, 32, 1, True),
    (17, 4096, 4096, 32, 1, False), (16, 4096, 4096, 64, 0, False), (22, 1500, 1500, 64, 1, False), (16, 4096, 4096, 64, 1, True),
])
def test_dispatch(batch, Nq, Nk, D, causal, split):
    """Either side of each line of the rule, with the automatic choice."""
    import torch
    import paper_2603_06731_amd as pbk
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn(batch, n, D, generator=g, device="cuda").bfloat16() for n in (Nq, Nk, Nk))
    out = torch.empty_like(q)
    dims = (batch, Nq, Nk, D, D, D, D, D, Nq * D, Nk * D, Nk * D, Nq * D)
    with T.forced_kernel(None):
        if causal:
            st = pbk.pbk_attention_causal(q, k, v, out, *dims, BF16, D ** -0.5)
        else:
            st = pbk.pbk_attention(q, k, v, None, out, *dims, 0, 0, BF16, D ** -0.5)
    assert st == 0 and ("kv64x" in pbk.pbk_last_kernel()) == split, pbk.pbk_last_kernel()
    qd, kd, vd = q[-1].double(), k[-1].double(), v[-1].double()      # the last batch entry
    s = qd @ kd.T * D ** -0.5
    if causal:
        s = s.masked_fill(torch.arange(Nk, device="cuda")[None, :] > torch.arange(Nq, device="cuda")[:, None] + Nk - Nq, float("-inf"))
    w = torch.softmax(s, -1)
    ref = w @ vd
    assert torch.all((out[-1].double() - ref).abs() <= 2.0 ** -8 * (w @ vd.abs() + ref.abs()) + 1e-5)


@pytest.mark.parametrize("batch,Nk,D,causal,split", [
    (240, 2048, 128, 0, True), (241, 2048, 128, 0, False), (256, 2048, 128, 1, False), (256, 3071, 128, 1, False), (256, 3072, 128, 0, True),
    (256, 2048, 64, 0, True),
])
def test_dispatch_a_round_of_entries(batch, Nk, D, causal, split):
    """As many entries as compute units, one query tile each."""
    test_dispatch(batch, 64, Nk, D, causal, split)
