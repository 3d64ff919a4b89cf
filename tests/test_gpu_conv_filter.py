"""The weight gradient of a 3x3 convolution of 16 channels that leaves the backward launch of the BatchNorm behind it: against the launch
of its own on stored maps, and in whole blocks against the oracle."""
import ctypes

import pytest
import torch

from paper_2411_12780_amd import binding as P
from paper_2411_12780_amd import synth
from test_gpu_parity import _decisive_shifts, run_case

pytestmark = pytest.mark.gpu
C = 16


def conv_bn_bwd(filters, B, H, W, t, in_stored, with_dres):
    f = P.lib().ppll_internal_conv_bn_bwd
    f.restype = ctypes.c_int
    vp, i = ctypes.c_void_p, ctypes.c_int
    f.argtypes = [i] * 4 + [vp] * 25 + [ctypes.c_size_t, vp]
    out = {k: torch.full((B, H, W, C), 7.0, dtype=torch.bfloat16, device="cuda") for k in ("d", "dst", "y")}
    out.update(dgb=torch.zeros(2 * C, device="cuda"), stat=torch.zeros(1024, 2 * C, device="cuda"), dw=torch.full((9, C, C), 7.0, device="cuda"))
    arena = torch.full((1024 * (9 * C * C + 64),), float("nan"), device="cuda")
    rows = ctypes.c_int(0)
    p = lambda v: v.data_ptr()
    status = f(filters, B, H, W, p(t["x"]), p(t["dy"]), p(t["mask"]), p(t["sums"]), p(t["mean"]), p(t["rstd"]), p(t["g"]), p(out["dgb"]), p(t["w"]),
               p(out["d"]), p(t["dres"]) if with_dres else None, p(t["dmask"]) if with_dres else None, p(out["dst"]), p(t["nx"]), p(t["nmask"]),
               p(t["nmean"]), p(t["nrstd"]), p(t["ng"]), p(t["nb"]), p(out["stat"]), ctypes.addressof(rows), p(t["in"]) if in_stored else None,
               p(out["y"]), p(out["dw"]), p(arena), arena.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert status == 0
    return out, rows.value


@pytest.mark.parametrize("in_stored,with_dres", [(0, 0), (1, 1)])
@pytest.mark.parametrize("B,H,W", [
    # tiles of 256 pixels: rows of one image, one image, several, the last of them with one to three images; two tiles a workgroup and more
    (129, 32, 32), (515, 8, 32), (513, 32, 8), (517, 16, 16), (1027, 16, 8), (1031, 8, 16), (2053, 8, 8), (2055, 8, 8), (300, 32, 32), (1600, 16, 16),
])
def test_filter_from_the_backward_launch(B, H, W, in_stored, with_dres):
    g = torch.Generator(device="cuda").manual_seed(B + H + 100 * W)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    t = {k: rnd(B, H, W, C).to(torch.bfloat16) for k in ("x", "dy", "dres", "nx", "in")}
    t.update({k: torch.randint(0, 256, (B * H * W * C // 8,), generator=g, device="cuda", dtype=torch.uint8) for k in ("mask", "dmask", "nmask")})
    t.update(sums=rnd(2 * C) * 100, mean=rnd(C) * 0.1, rstd=1 + 0.1 * rnd(C), g=1 + 0.1 * rnd(C), w=(rnd(9, C, C) * 0.1).to(torch.bfloat16),
             nmean=rnd(C) * 0.1, nrstd=1 + 0.1 * rnd(C), ng=1 + 0.1 * rnd(C), nb=rnd(C))
    one, rows1 = conv_bn_bwd(1, B, H, W, t, in_stored, with_dres)
    two, rows2 = conv_bn_bwd(0, B, H, W, t, in_stored, with_dres)
    assert rows1 == rows2 and rows1 < B * H * W / 256       # several tiles a workgroup
    for k in ("dst", "dgb", "stat"):
        assert torch.equal(one[k], two[k]), k
    assert bool((one["d"] == 7.0).all())                    # not stored
    # the sums of both in float64, from the maps as they lie in memory
    y, d = (t["in"] if in_stored else two["y"]).double(), two["d"].double()
    pads = [torch.nn.functional.pad(v, (0, 0, 1, 1, 1, 1)) for v in (y, y.abs())]
    ref, size = (torch.stack([v[:, ky:ky + H, kx:kx + W].reshape(-1, C).t().contiguous() @ e.reshape(-1, C) for ky in range(3) for kx in range(3)])
                 for v, e in zip(pads, (d, d.abs())))
    # exact products; of the sum of magnitudes S, the last chain of 16 fp32 sums rounds at most 2^-24 k / 16 S at step k, evenly spread:
    # 2^-24 S sqrt(16 / 3 / 3) or 8e-8 S together, and the chains before it (workgroups, tiles, matrix steps) have smaller parts each
    e1, e2 = (float((o["dw"].double() - ref).norm() / size.norm()) for o in (one, two))
    print(f"filter errors against float64, of the sum of magnitudes: {e1:.2e} in one launch, {e2:.2e} in two")
    assert e1 <= 8e-8 and e2 <= 8e-8


@pytest.mark.parametrize("more", [
    dict(channels=16, height=32, width=32, batch=129, n_basic_blocks=1),                              # behind a stem
    dict(channels=16, height=16, width=16, batch=517, n_basic_blocks=2, act=True),                    # first block without an input gradient
    dict(channels=32, height=16, width=16, batch=129, n_basic_blocks=3, transition_block=2, act=True),  # a downsampling block behind one of 16
    dict(channels=16, height=8, width=8, batch=2055, n_basic_blocks=2, act=True),                     # last tile with three images of four
])
def test_blocks_that_take_their_filters_from_the_backward_launch(more):
    more = dict(more)
    act = more.pop("act", False)
    m = 2 if more.get("transition_block") else 1
    wl = synth.workload("resnet32_stage1_bf16", aux_channels=32, img_h=m * more["height"], img_w=m * more["width"], **more)
    if act:
        wl["input_kind"] = synth.ACTIVATION
    run_case(wl, steps=1, check_bn=True, tweak=_decisive_shifts)
