"""The matrix-core attention against a float64 one, at the edges of its tiles of 32 tokens (and of the halves of them)."""
import ctypes

import pytest
import torch

from paper_2411_12780_amd import binding as P

pytestmark = pytest.mark.gpu
GUARD = 4096


def attention(B, T, H, qkv, dout):
    f = P.lib().ppll_internal_attention
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int] * 3 + [ctypes.c_void_p] * 6
    D = 64 * H
    out = torch.full((B * T * D + GUARD,), 7.0, dtype=torch.bfloat16, device="cuda")
    dqkv = torch.full((B * T * 3 * D + GUARD,), 7.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B * H * T + GUARD,), 7.0, device="cuda")
    status = f(B, T, H, qkv.data_ptr(), out.data_ptr(), lse.data_ptr(), dout.data_ptr(), dqkv.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return status, out, lse, dqkv


@pytest.mark.parametrize("B,H", [(3, 2), (1, 5)])
@pytest.mark.parametrize("T", [1, 5, 16, 17, 32, 33, 48, 49, 65, 96, 97, 113, 128, 129, 145, 160, 161, 192, 197, 208, 225, 256])
def test_attention_at_the_edges_of_its_tiles(T, B, H):
    g = torch.Generator(device="cuda").manual_seed(100 * T + B)
    D = 64 * H
    qkv = torch.randn(B, T, 3 * D, generator=g, device="cuda").to(torch.bfloat16)
    dout = torch.randn(B, T, D, generator=g, device="cuda").to(torch.bfloat16)
    status, out, lse, dqkv = attention(B, T, H, qkv, dout)
    assert status == 0
    for t, n in ((out, B * T * D), (dqkv, B * T * 3 * D), (lse, B * H * T)):
        assert bool((t[n:] == 7.0).all())     # nothing beyond the end

    heads = lambda t: t.reshape(B, T, H, 64).transpose(1, 2).double().contiguous()
    rows = lambda t: t.transpose(1, 2).reshape(B, T, D)
    tr = lambda t: t.transpose(-1, -2).contiguous()
    q, k, v = (heads(t) for t in qkv.split(D, dim=2))
    do = heads(dout)
    s = q @ tr(k) / 8
    p = torch.softmax(s, -1)
    o = p @ v
    dp = do @ tr(v)
    d = (do * o).sum(-1, keepdim=True)
    ds = p * (dp - d)
    # What is rounded to bf16 (2^-9 of a value at most): probabilities or dS before the second product, the result, and behind the
    # backward's <dO, O> the forward's output; exponents and sums are fp32, far below.  On the scale of the sums of magnitudes, which
    # the difference dP - <dO, O> falls short of.
    big = p * (dp.abs() + d.abs() + (do * o).abs().sum(-1, keepdim=True) + (do.abs() * (p @ v.abs())).sum(-1, keepdim=True))
    want = {"out": (o, p @ v.abs()), "dq": (ds @ k / 8, big @ k.abs() / 8), "dk": (tr(ds) @ q / 8, tr(big) @ q.abs() / 8),
            "dv": (tr(p) @ do, tr(p) @ do.abs())}
    got = dict(zip(("dq", "dk", "dv"), dqkv[:B * T * 3 * D].view(B, T, 3 * D).split(D, dim=2)), out=out[:B * T * D].view(B, T, D))
    for name, (ref, size) in want.items():
        assert bool(((got[name].double() - rows(ref)).abs() <= 2.0 ** -8 * (rows(ref).abs() + rows(size)) + 1e-6).all()), name
    assert float((lse[:B * H * T].view(B, H, T).double() - torch.logsumexp(s, -1)).abs().max()) <= 1e-5
    again = attention(B, T, H, qkv, dout)
    assert all(torch.equal(x, y) for x, y in zip((out, lse, dqkv), again[1:]))


@pytest.mark.parametrize("T", [17, 129])
def test_scores_far_from_zero(T):
    # keys of which the softmax takes one each, and rows beyond the last token whose exponent would overflow
    g = torch.Generator(device="cuda").manual_seed(T)
    qkv = torch.randn(2, T, 192, generator=g, device="cuda").to(torch.bfloat16)
    qkv[..., :64] = 30.0
    qkv[..., 64:128] = -30.0 + qkv[..., 64:128]
    dout = torch.randn(2, T, 64, generator=g, device="cuda").to(torch.bfloat16)
    status, out, lse, dqkv = attention(2, T, 1, qkv, dout)
    assert status == 0 and bool(torch.isfinite(out.float()).all()) and bool(torch.isfinite(dqkv.float()).all())
    assert float(lse[:2 * T].max()) < -1000.0


@pytest.mark.parametrize("T,H,dh", [(t, 2, 64) for t in (1, 5, 8, 9, 31, 32, 33, 64, 65, 96, 97, 145, 161, 197, 224, 225, 256)] + [(17, 3, 32), (256, 2, 48), (65, 1, 64)])
def test_attention_of_the_class_token(T, H, dh):
    # edges of a copy of 8 rows and of the waves, up to the 256 tokens that a block takes; other heads are for the general kernels
    B, D = 3, H * dh
    g = torch.Generator(device="cuda").manual_seed(1000 * T + D)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    q, kv, dout = rnd(B, D), rnd(B, T, 2 * D), rnd(B, D)
    f = P.lib().ppll_internal_attention_cls
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int] * 4 + [ctypes.c_void_p] * 8

    def run():
        bufs = [torch.full((n + GUARD,), 7.0, dtype=t, device="cuda")
                for n, t in ((B * D, torch.bfloat16), (B * H * T, torch.float32), (B * D, torch.bfloat16), (B * T * 2 * D, torch.bfloat16))]
        out, prob, dq, dkv = bufs
        status = f(B, T, H, dh, q.data_ptr(), kv.data_ptr(), out.data_ptr(), prob.data_ptr(), dout.data_ptr(), dq.data_ptr(), dkv.data_ptr(),
                   torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert status == 0
        return bufs

    bufs = run()
    sizes = (B * D, B * H * T, B * D, B * T * 2 * D)
    for t, n in zip(bufs, sizes):
        assert bool((t[n:] == 7.0).all())
    out, prob, dq, dkv = (t[:n].double() for t, n in zip(bufs, sizes))
    k, v = (t.reshape(B, T, H, dh).double() for t in kv.split(D, dim=2))
    qd, dod = q.view(B, 1, H, dh).double(), dout.view(B, 1, H, dh).double()
    s = (qd * k).sum(-1) / dh ** 0.5                            # [B, T, H]
    p = torch.softmax(s, 1)
    dp = (dod * v).sum(-1)
    delta = (p * dp).sum(1, keepdim=True)
    ds = p * (dp - delta)
    # every result is rounded to bf16 once; all else is fp32, with exponents and sums of 64 terms good to 2^-18 of the magnitudes
    mag = (p * dp.abs()).sum(1, keepdim=True) + (dod.abs() * v.abs()).sum(-1)
    eps = 2.0 ** -18 * (1 + (qd.abs() * k.abs()).sum(-1).max().item() / 16)
    ps, dss = p[..., None], ds[..., None]
    want = {"out": (out.view(B, H, dh), (ps * v).sum(1), (ps * v.abs()).sum(1)),
            "dq": (dq.view(B, H, dh), (dss * k).sum(1) / dh ** 0.5, ((p * mag)[..., None] * k.abs()).sum(1) / dh ** 0.5),
            "dk": (dkv.view(B, T, 2, H, dh)[:, :, 0], dss * qd / dh ** 0.5, (p * mag)[..., None] * qd.abs() / dh ** 0.5),
            "dv": (dkv.view(B, T, 2, H, dh)[:, :, 1], ps * dod, ps * dod.abs())}
    for name, (got, ref, size) in want.items():
        assert bool(((got - ref).abs() <= 2.0 ** -8 * ref.abs() + eps * size + 1e-30).all()), name
    assert bool(((prob.view(B, H, T).transpose(1, 2) - p).abs() <= eps * p + 1e-30).all())
    assert all(torch.equal(x, y) for x, y in zip(bufs, run()))
