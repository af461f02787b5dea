"""Attention with 64 queries per workgroup and two or four groups of waves, against the definition evaluated in float64."""
import pytest

import workloads as wl
import pbk_testlib as T

pytestmark = pytest.mark.gpu

BF16, F16 = wl.DTYPE_BF16, wl.DTYPE_F16

CASES = [  # batch, Nq, Nk, row padding
    (1, 1, 1, 0),            # one group has a key
    (2, 33, 65, 8),          # the second of two groups has one key
    (2, 64, 200, 0),         # four tiles, the last ragged: one for each of four groups
    (3, 65, 257, 8),         # five: groups of two, two and one, the last without
    (1, 300, 200, 0),        # causal: queries that see no key (NaN), tiles with no visible key
    (5, 129, 1024, 0),       # whole tiles, without a bounds test in every group; causal: entries in either direction
    (2, 450, 450, 8),
]


def attend(pbk, q, k, v, out, D, dtype, causal):
    b, Nq, ld = q.shape
    Nk = k.shape[1]
    dims = (b, Nq, Nk, D, ld, ld, ld, ld, Nq * ld, Nk * ld, Nk * ld, Nq * ld)
    if causal:
        return pbk.pbk_attention_causal(q, k, v, out, *dims, dtype, D ** -0.5)
    return pbk.pbk_attention(q, k, v, None, out, *dims, 0, 0, dtype, D ** -0.5)


def check(q, k, v, got, D, dtype, causal):
    import torch
    Nq, Nk = q.shape[1], k.shape[1]
    qd, kd, vd = (x[..., :D].double() for x in (q, k, v))
    s = qd @ kd.transpose(1, 2).contiguous() * D ** -0.5
    if causal:
        hidden = torch.arange(Nk, device=s.device)[None, :] > torch.arange(Nq, device=s.device)[:, None] + Nk - Nq
        s = s.masked_fill(hidden, float("-inf"))
    w = torch.softmax(s, -1)
    ref, got = w @ vd, got[..., :D].double()
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    # weights rounded to 16 bits (u of their value), then the output: u (sum w |v| + |o|), with fp32 sums below that
    u = 2.0 ** -8 if dtype == BF16 else 2.0 ** -11
    bound = u * ((w @ vd.abs()) + ref.abs()) + 1e-5
    assert torch.all(((got - ref).abs() <= bound) | torch.isnan(ref)), (Nq, Nk, float(((got - ref).abs() / bound).nan_to_num().max()))


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("D,force,name", [(32, "mfma:3", "q64_kv64x2"), (64, "mfma:3", "q64_kv64x2"), (128, "mfma:3", "q64_kv64x2"),
                                          (32, "mfma:4", "q64_kv64x4"), (64, "mfma:4", "q64_kv64x4")])
def test_sizes(D, force, name, dtype, causal):
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
        with T.forced_kernel(force):
            st = attend(pbk, q.cuda(), k.cuda(), v.cuda(), out, D, dtype, causal)
        assert st == 0 and name in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()
        assert torch.all(out[..., D:] == 0)
        check(q, k, v, out.cpu(), D, dtype, causal)


@pytest.mark.parametrize("batch,Nq,Nk,D,causal,name", [
    (4, 65, 96, 64, 0, "q64_kv64x2"), (4, 65, 95, 64, 0, "q128_kv64_"), (4, 64, 96, 128, 0, "q128_kv64_"), (128, 128, 128, 128, 1, "q64_kv64x2"),
    (129, 128, 128, 128, 1, "q128_kv64_"), (2, 64, 2048, 64, 0, "q64_kv64x4"), (2, 200, 2047, 64, 1, "q64_kv64x2"), (2, 200, 2048, 128, 1, "q64_kv64x2"),
    (16, 2048, 2048, 64, 1, "q64_kv64x2"), (16, 2048, 2048, 64, 0, "q128_kv64x2"), (25, 1280, 1280, 64, 1, "q64_kv64x2"), (25, 1279, 1279, 64, 1, "q128_kv64x2"),
    (4, 150, 128, 32, 1, "q64_kv64x2"), (4, 150, 129, 32, 1, "q128_kv64_"), (4, 192, 192, 32, 1, "q128_kv64_"), (4, 193, 193, 32, 1, "q64_kv64x2"),
    (4, 150, 150, 32, 0, "q64_kv64x2"), (4, 176, 176, 64, 1, "q64_kv64x2"), (4, 177, 177, 128, 1, "q128_kv64_"),
    (24, 2048, 2048, 64, 1, "q64_"), (25, 2048, 2048, 64, 1, "q128_kv64_"), (48, 1024, 1024, 32, 0, "q64_"), (49, 1024, 1024, 32, 0, "q128_kv64_"),
])
def test_dispatch(batch, Nq, Nk, D, causal, name):
    """Either side of each line of the rule, with the automatic choice; the last entry in full."""
    import torch
    import paper_2603_06731_amd as pbk
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn(batch, n, D, generator=g, device="cuda").bfloat16() for n in (Nq, Nk, Nk))
    out = torch.empty_like(q)
    with T.forced_kernel(None):
        st = attend(pbk, q, k, v, out, D, BF16, causal)
    assert st == 0 and name in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()
    check(q[-1:], k[-1:], v[-1:], out[-1:], D, BF16, causal)
