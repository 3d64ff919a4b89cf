"""The input gradient of a 3x3 convolution of stride 2 against a float64 sum, at the edges of its tiles of 128 gradient pixels."""
import ctypes

import pytest
import torch

from paper_2411_12780_amd import binding as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,W,Ci,Co", [
    (1, 2, 2, 16, 16), (3, 6, 10, 32, 64), (1, 2, 600, 16, 32), (5, 14, 14, 48, 48), (2, 128, 2, 64, 16),
    (2, 16, 16, 64, 64), (129, 16, 16, 64, 64),           # a tile of exactly one and two images; more tiles than half the places
    (700, 16, 16, 64, 64), (530, 24, 24, 16, 64), (400, 32, 32, 32, 32),     # several tiles a workgroup, the last ones ragged
])
def test_input_gradient_at_stride_2(B, H, W, Ci, Co):
    g = torch.Generator(device="cuda").manual_seed(B + H + W + Ci + Co)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    Ho, Wo = H // 2, W // 2
    dy, w = rnd(B, Ho, Wo, Co), rnd(9, Ci, Co)
    buf = torch.full((B * H * W * Ci + 4096,), 7.0, dtype=torch.bfloat16, device="cuda")
    f = P.lib().ppll_internal_conv_dgrad_s2
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int] * 5 + [ctypes.c_void_p] * 4
    status = f(B, H, W, Ci, Co, dy.data_ptr(), w.data_ptr(), buf.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert status == 0 and bool((buf[B * H * W * Ci:] == 7.0).all())
    ref, size = (torch.zeros(B, H + 2, W + 2, Ci, dtype=torch.float64, device="cuda") for _ in range(2))
    for ky in range(3):
        for kx in range(3):
            for out, a, b in ((ref, dy.double(), w[3 * ky + kx].double()), (size, dy.double().abs(), w[3 * ky + kx].double().abs())):
                out[:, ky:ky + 2 * Ho:2, kx:kx + 2 * Wo:2] += (a.reshape(-1, Co) @ b.t().contiguous()).view(B, Ho, Wo, Ci)
    ref, size = (t[:, 1:H + 1, 1:W + 1] for t in (ref, size))
    dx = buf[:B * H * W * Ci].view(B, H, W, Ci).double()
    # one rounding to bf16, fp32 sums of up to 4 Co terms
    assert bool(((dx - ref).abs() <= ref.abs() * 2.0 ** -8 + size * (4 * Co * 2.0 ** -24) + 1e-6).all())
