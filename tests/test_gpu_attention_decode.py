"""Attention of a few queries against a long context (the kernel that splits the keys over the waves) against the CPU oracle's
definition evaluated in float64."""
import pytest

import workloads as wl
import pbk_testlib as T

pytestmark = pytest.mark.gpu

BF16, F16 = wl.DTYPE_BF16, wl.DTYPE_F16

CASES = [  # batch, Nq, Nk, row padding
    (1, 1, 1, 0),            # one key: one wave has work
    (3, 16, 31, 8),          # a ragged single step
    (2, 3, 33, 0),           # two steps, the second with one key
    (2, 5, 3, 0),            # causal: more queries than keys (rows that see none are NaN)
    (5, 8, 520, 8),          # a step more than the waves
    (70, 2, 1300, 0),
]


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("D,split", [(32, 1), (64, 1), (64, 2), (128, 1), (128, 2), (128, 4)])
def test_decode(D, split, dtype, causal):
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
        with T.forced_kernel(f"decode:{split}"):
            if causal:
                st = pbk.pbk_attention_causal(q.cuda(), k.cuda(), v.cuda(), out, *dims, dtype, alpha)
            else:
                st = pbk.pbk_attention(q.cuda(), k.cuda(), v.cuda(), None, out, *dims, 0, 0, dtype, alpha)
        assert st == 0 and "decode" in pbk.pbk_last_kernel()
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


@pytest.mark.parametrize("batch,Nq,Nk,D,kernel", [
    # queries and keys
    (16, 16, 512, 64, "decode"), (16, 17, 512, 64, "q128"), (16, 1, 128, 128, "decode"), (16, 1, 127, 128, "q128"),
    # workgroups per entry
    (64, 1, 256, 128, "kv32_c4"), (65, 1, 256, 128, "kv32_c2"), (128, 2, 256, 128, "kv32_c2"), (129, 2, 256, 128, "kv32_c1"),
    (128, 1, 128, 64, "kv32_c2"), (64, 1, 256, 32, "kv32_c1"),
    # up to 256 entries, one or two queries at D = 64
    (160, 2, 255, 64, "q128"), (160, 2, 256, 64, "decode"), (160, 3, 128, 64, "decode"), (200, 1, 383, 64, "q128"), (200, 1, 384, 64, "decode"),
    (256, 1, 128, 128, "decode"),
    # more than 256 entries
    (257, 1, 1024, 128, "q128"), (512, 1, 512, 64, "q128"), (639, 1, 1536, 64, "q128"), (640, 1, 1535, 64, "q128"), (640, 1, 1536, 64, "decode"),
    (640, 8, 1023, 128, "q128"), (640, 8, 1024, 128, "decode"), (512, 1, 128, 32, "decode"), (513, 1, 255, 32, "q128"), (513, 1, 256, 32, "decode"),
])
def test_dispatch(batch, Nq, Nk, D, kernel):
    """Either side of each line of the rule, with the automatic choice."""
    import torch
    import paper_2603_06731_amd as pbk
    g = torch.Generator(device="cuda").manual_seed(batch + Nk)
    q, k, v = (torch.randn(batch, n, D, generator=g, device="cuda").bfloat16() for n in (Nq, Nk, Nk))
    out = torch.empty_like(q)
    with T.forced_kernel(None):
        st = pbk.pbk_attention_causal(q, k, v, out, batch, Nq, Nk, D, D, D, D, D, Nq * D, Nk * D, Nk * D, Nq * D, BF16, D ** -0.5)
    assert st == 0 and kernel in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()
    s = torch.stack([q[b].double() @ k[b].double().T * D ** -0.5 for b in range(batch)])
    s = s.masked_fill(torch.arange(Nk, device="cuda")[None, :] > torch.arange(Nq, device="cuda")[:, None] + Nk - Nq, float("-inf"))
    w = torch.softmax(s, -1)
    for b in range(0, batch, max(1, batch // 16)):
        vb = v[b].double()
        ref = w[b] @ vb
        # (the bound of test_decode)
        assert torch.all((out[b].double() - ref).abs() <= 2.0 ** -8 * (w[b] @ vb.abs() + ref.abs()) + 1e-5), b


@pytest.mark.parametrize("batch,kernel", [((1 << 22) - 1, "decode"), (1 << 22, "q128")])
def test_launch_limit(batch, kernel):
    """1024 threads per entry: one entry fewer than a launch can hold, and as many as it cannot (they run on the kernel of
    whole sequences).  K and V are shared (stride 0)."""
    import torch
    import paper_2603_06731_amd as pbk
    D, Nk = 32, 256
    g = torch.Generator(device="cuda").manual_seed(batch)
    q = torch.randn(batch, D, generator=g, device="cuda").bfloat16()
    k, v = (torch.randn(Nk, D, generator=g, device="cuda").bfloat16() for _ in range(2))
    out = torch.full_like(q, float("nan"))
    with T.forced_kernel(None):
        st = pbk.pbk_attention(q, k, v, None, out, batch, 1, Nk, D, D, D, D, D, D, 0, 0, D, 0, 0, BF16, D ** -0.5)
    assert st == 0 and kernel in pbk.pbk_last_kernel(), (st, pbk.pbk_last_kernel())
    w = torch.softmax(q.float() @ k.float().T.contiguous() * D ** -0.5, -1)
    ref, mag = w @ v.float(), w @ v.float().abs()
    # one rounding of the weights and one of the output, 2^-8 each
    assert bool(((out.float() - ref).abs() <= 2 ** -8 * (mag + ref.abs()) + 1e-5).all())
