"""The BatchNorm's apply pass, one piece of 8 channels a thread and several, against float64, at the edges of its workgroups."""
import ctypes

import pytest
import torch

from paper_2411_12780_amd import binding as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pieces", [1, 4])
@pytest.mark.parametrize("with_res,with_mask", [(0, 0), (1, 1)])
@pytest.mark.parametrize("rows,C", [(1, 8), (31, 64), (255, 8), (256, 8), (257, 8), (513, 16), (1023, 8), (128, 64), (129, 64), (700, 128), (4097, 32)])
def test_apply_pass(rows, C, with_res, with_mask, pieces):
    g = torch.Generator(device="cuda").manual_seed(rows + C)
    x, res = (torch.randn(rows, C, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    mean, shift = (torch.randn(C, generator=g, device="cuda") for _ in range(2))
    rstd, scale = (torch.rand(C, generator=g, device="cuda") + 0.5 for _ in range(2))
    y = torch.full((rows * C + 8192,), 7.0, dtype=torch.bfloat16, device="cuda")
    mask = torch.full((rows * C // 8 + 1024,), 7, dtype=torch.uint8, device="cuda")
    f = P.lib().ppll_internal_bn_apply
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int] * 3 + [ctypes.c_void_p] * 9
    status = f(pieces, rows, C, x.data_ptr(), mean.data_ptr(), rstd.data_ptr(), scale.data_ptr(), shift.data_ptr(), res.data_ptr() if with_res else None,
               y.data_ptr(), mask.data_ptr() if with_mask else None, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert status == 0 and bool((y[rows * C:] == 7.0).all())
    terms = [(x.double() - mean.double()) * (rstd.double() * scale.double()), shift.double().expand(rows, C)] + ([res.double()] if with_res else [])
    ref, size = sum(terms).clamp(min=0), sum(t.abs() for t in terms) + mean.double().abs() * rstd.double() * scale.double()
    got = y[:rows * C].view(rows, C).double()
    # one rounding to bf16, half a dozen fp32 operations
    assert bool(((got - ref).abs() <= ref * 2.0 ** -8 + size * 2.0 ** -21).all())
    bits = (got > 0).view(-1, 8).to(torch.int32) << torch.arange(8, device="cuda", dtype=torch.int32)
    n = rows * C // 8 if with_mask else 0
    assert torch.equal(mask[:n].to(torch.int32), bits.sum(1).to(torch.int32)[:n]) and bool((mask[n:] == 7).all())
