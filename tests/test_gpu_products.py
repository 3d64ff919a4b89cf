"""The bf16 product kernels against each other and against a float64 product, at the edges of their tiles.  The dispatch is passed
by, so that every kernel is reached whatever its rules say."""
import ctypes

import pytest
import torch

from paper_2411_12780_amd import binding as P

pytestmark = pytest.mark.gpu

FEW, TILED, COPYING, WIDE_128, WIDE_160, SPLIT, UNIT_256, UNIT_320 = 1, 2, 3, 4, 5, 6, 8, 10
NONE, GELU, DGELU = 0, 1, 2


def product(kernel, A, B, bt, bias, residual, epilogue, aux, C=None, C2=None):
    f = P.lib().ppll_internal_product
    f.restype = ctypes.c_int
    vp, i, l = ctypes.c_void_p, ctypes.c_int, ctypes.c_long
    f.argtypes = [i, i, i, i, vp, l, vp, l, i, vp, l, vp, vp, i, vp, vp, vp]
    M, K = A.shape
    N = B.shape[1 if bt else 0]
    if C is None:
        C, C2 = (torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    ptr = lambda t: None if t is None else t.data_ptr()
    status = f(kernel, M, N, K, ptr(A), A.stride(0), ptr(B), B.stride(0), bt, ptr(C), C.stride(0), ptr(bias), ptr(residual), epilogue,
               ptr(C2) if epilogue == GELU else None, ptr(aux) if epilogue == DGELU else None, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return status, C, C2


@pytest.mark.parametrize("epilogue", [NONE, GELU, DGELU])
@pytest.mark.parametrize("bt", [0, 1])
@pytest.mark.parametrize("M,N,K", [
    (1, 8, 128), (129, 264, 136), (161, 520, 200), (160, 256, 256), (127, 248, 1000), (320, 512, 160), (481, 776, 392), (33, 3072, 128),
])
def test_wide_tiles_give_what_the_tiled_kernel_gives(M, N, K, bt, epilogue):
    g = torch.Generator(device="cuda").manual_seed(M * 1000 + N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    A, B = rnd(M, K), rnd(K, N) if bt else rnd(N, K)
    bias = torch.randn(N, generator=g, device="cuda") if epilogue != DGELU else None
    residual = rnd(M, N) if epilogue == NONE else None
    aux = rnd(M, N)
    status, C, C2 = product(TILED, A, B, bt, bias, residual, epilogue, aux)
    assert status == 0
    v = A.double() @ (B.double() if bt else B.double().t().contiguous())
    if bias is not None:
        v = v + bias.double()
    if residual is not None:
        v = v + residual.double()
    ref = {NONE: v, DGELU: v * aux.double(), GELU: 0.5 * (1 + torch.erf(v / 2 ** 0.5)) + v * torch.exp(-0.5 * v * v) / (2 * torch.pi) ** 0.5}[epilogue]
    # one rounding to bf16 (2^-9 of a value at most), fp32 sums of up to 1000 terms far below it
    assert float((C.double() - ref).norm() / ref.norm()) <= 2.0 ** -8
    for kernel in (WIDE_128, WIDE_160):
        status, D, D2 = product(kernel, A, B, bt, bias, residual, epilogue, aux)
        assert status == 0
        assert torch.equal(C, D) and torch.equal(C2, D2), kernel


@pytest.mark.parametrize("epilogue", [NONE, GELU, DGELU])
@pytest.mark.parametrize("bt", [0, 1])
@pytest.mark.parametrize("M,N,K", [
    # edges of 256 x 256 and 320 x 256 tiles and of a stage of 64 k; two to sixteen stages, of which two are in LDS
    (1, 8, 128), (257, 264, 136), (321, 520, 200), (256, 256, 192), (320, 248, 1000), (639, 512, 328), (33, 776, 384),
])
def test_tiles_of_a_unit_give_what_the_tiled_kernel_gives(M, N, K, bt, epilogue):
    g = torch.Generator(device="cuda").manual_seed(M * 1000 + N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    wide = rnd(M, K + 40)                     # rows of A further apart than they are long
    A, B = wide[:, :K], rnd(K, N) if bt else rnd(N, K)
    bias = torch.randn(N, generator=g, device="cuda") if epilogue != DGELU else None
    residual = rnd(M, N) if epilogue == NONE else None
    aux = rnd(M, N)
    status, C, C2 = product(TILED, A, B, bt, bias, residual, epilogue, aux)
    assert status == 0
    for kernel in (UNIT_256, UNIT_320):
        status, D, D2 = product(kernel, A, B, bt, bias, residual, epilogue, aux)
        assert status == 0
        assert torch.equal(C, D) and torch.equal(C2, D2), kernel


def test_products_that_a_kernel_does_not_take_are_refused():
    A, B = torch.zeros(16, 120, dtype=torch.bfloat16, device="cuda"), torch.zeros(120, 16, dtype=torch.bfloat16, device="cuda")
    for kernel in (WIDE_128, WIDE_160, 3):
        status, C, _ = product(kernel, A, B, 1, None, None, NONE, None)
        assert status == 2 and bool((C == 7.0).all())


@pytest.mark.parametrize("epilogue", [NONE, GELU, DGELU])
@pytest.mark.parametrize("bt", [0, 1])
@pytest.mark.parametrize("M,N,K", [
    # edges of the 64 x 64 tile and of a stage of 64 k; one to five stages (four are in flight), odd and even numbers of them
    (1, 8, 128), (64, 64, 128), (65, 72, 136), (63, 56, 192), (129, 120, 200), (300, 264, 256), (640, 136, 264), (257, 384, 320), (33, 768, 3072),
])
def test_split_products(M, N, K, bt, epilogue):
    g = torch.Generator(device="cuda").manual_seed(M * 1000 + N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    wide = rnd(M, K + 24)                     # rows of A further apart than they are long
    A, B = wide[:, :K], rnd(K, N) if bt else rnd(N, K)
    bias = torch.randn(N, generator=g, device="cuda") if epilogue != DGELU else None
    residual = rnd(M, N) if epilogue == NONE else None
    aux = rnd(M, N)
    status, C, C2 = product(SPLIT, A, B, bt, bias, residual, epilogue, aux)
    assert status == 0
    v = A.double() @ (B.double() if bt else B.double().t().contiguous())
    if bias is not None:
        v = v + bias.double()
    if residual is not None:
        v = v + residual.double()
    ref = {NONE: v, DGELU: v * aux.double(), GELU: 0.5 * (1 + torch.erf(v / 2 ** 0.5)) + v * torch.exp(-0.5 * v * v) / (2 * torch.pi) ** 0.5}[epilogue]
    # per element: one rounding to bf16, and fp32 sums of K terms in any order on the scale of the sum of their magnitudes (GELU's
    # derivative has slope below 1.2; the factor of a saved derivative scales both)
    size = A.double().abs() @ (B.double() if bt else B.double().t().contiguous()).abs()
    if epilogue == DGELU:
        size = size * aux.double().abs()
    bound = ref.abs() * 2.0 ** -8 + size * (K * 2.0 ** -24) + 1e-6
    assert bool(((C.double() - ref).abs() <= bound).all())
    if epilogue == GELU:
        gelu = v * 0.5 * (1 + torch.erf(v / 2 ** 0.5))
        assert bool(((C2.double() - gelu).abs() <= gelu.abs() * 2.0 ** -8 + size * (K * 2.0 ** -23) + 1e-6).all())
    for kernel in (SPLIT, TILED):     # again, and on the kernel that takes the same products one tile of columns further: the same sums
        status, D, D2 = product(kernel, A, B, bt, bias, residual, epilogue, aux)
        assert status == 0 and torch.equal(C, D) and torch.equal(C2, D2), kernel


@pytest.mark.parametrize("epilogue", [NONE, GELU, DGELU])
@pytest.mark.parametrize("bt", [0, 1])
@pytest.mark.parametrize("M,N,K,apart", [(65, 72, 136, 80), (300, 264, 200, 5 * 264), (129, 120, 328, 128), (257, 384, 384, 17 * 384)])
def test_split_products_in_and_out_of_wider_buffers(M, N, K, apart, bt, epilogue):
    # As the class-token layer calls them: a slice of a weight for B, result rows further apart than they are long, of the query gradient
    # added to what is there.  Between the rows and behind the last one nothing changes.
    g = torch.Generator(device="cuda").manual_seed(M * 1000 + N + K + apart)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    A = rnd(M, K + 8)[:, :K]
    B = rnd(K, 3 * N)[:, N:2 * N] if bt else rnd(N, 2 * K)[:, K:]
    bias = torch.randn(N, generator=g, device="cuda") if epilogue != DGELU else None
    buf, buf2, aux = rnd(M * apart + 4096), rnd(M * apart + 4096), rnd(M, apart)[:, :N]
    rows = lambda t: t[:M * apart].view(M, apart)[:, :N]
    got = {}
    for kernel in (SPLIT, TILED):
        c, c2 = buf.clone(), buf2.clone()
        status, _, _ = product(kernel, A, B, bt, bias, rows(c) if epilogue == NONE else None, epilogue, aux, rows(c), rows(c2))
        assert status == 0
        for t, before in ((c, buf), (c2, buf2)):
            now, was = t.clone(), before.clone()
            rows(now).zero_(), rows(was).zero_()
            assert torch.equal(now, was)
        got[kernel] = rows(c), rows(c2)
    v = A.double() @ (B.double().contiguous() if bt else B.double().t().contiguous())
    size = A.double().abs() @ (B.double() if bt else B.double().t()).abs().contiguous()
    if bias is not None:
        v = v + bias.double()
    if epilogue == NONE:
        v, size = v + rows(buf).double(), size + rows(buf).double().abs()
    if epilogue == DGELU:
        v, size = v * aux.double(), size * aux.double().abs()
    if epilogue == GELU:
        gelu = v * 0.5 * (1 + torch.erf(v / 2 ** 0.5))
        assert bool(((got[SPLIT][1].double() - gelu).abs() <= gelu.abs() * 2.0 ** -8 + size * (K * 2.0 ** -23) + 1e-6).all())
    else:   # one rounding to bf16, fp32 sums of K terms
        assert bool(((got[SPLIT][0].double() - v).abs() <= v.abs() * 2.0 ** -8 + size * (K * 2.0 ** -24) + 1e-6).all())
        assert torch.equal(rows(buf2), got[SPLIT][1])
    assert torch.equal(got[SPLIT][0], got[TILED][0]) and torch.equal(got[SPLIT][1], got[TILED][1])


@pytest.mark.parametrize("epilogue", [NONE, GELU, DGELU])
@pytest.mark.parametrize("bt", [0, 1])
@pytest.mark.parametrize("M,N,K,apart", [
    # K in quarters of steps of 16: fewer quarters than waves, a part of a stage, two stages, a part of a third, more than four
    (1, 8, 8, 8), (31, 40, 72, 48), (33, 264, 136, 264), (64, 384, 384, 384), (65, 72, 520, 80), (128, 96, 3080, 17 * 96),
    (128, 3080, 200, 3080), (250, 2056, 1032, 2056),   # more than 256 tiles of 32 x 32: tiles of 32 x 64
    (255, 4104, 328, 4112), (256, 3072, 776, 3072),    # more of those than units as well
    (1000, 384, 1544, 384),                            # more rows than the first rule takes
])
def test_products_of_few_tiles(M, N, K, apart, bt, epilogue):
    g = torch.Generator(device="cuda").manual_seed(M * 1000 + N + K + apart)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    A = rnd(M, K + 8)[:, :K]                      # what lies behind a row is not part of the sum
    B = rnd(K, N + 8)[:, :N] if bt else rnd(N, K + 8)[:, :K]
    bias = torch.randn(N, generator=g, device="cuda") if epilogue != DGELU else None
    buf, buf2, aux = rnd(M * apart + 4096), rnd(M * apart + 4096), rnd(M, apart)[:, :N]
    rows = lambda t: t[:M * apart].view(M, apart)[:, :N]
    c, c2 = buf.clone(), buf2.clone()
    status, _, _ = product(FEW, A, B, bt, bias, rows(c) if epilogue == NONE else None, epilogue, aux, rows(c), rows(c2))
    assert status == 0
    for t, before in ((c, buf), (c2, buf2)):
        now, was = t.clone(), before.clone()
        rows(now).zero_(), rows(was).zero_()
        assert torch.equal(now, was)
    Bd = B.double().contiguous() if bt else B.double().t().contiguous()
    v, size = A.double().contiguous() @ Bd, A.double().abs().contiguous() @ Bd.abs()
    if bias is not None:
        v = v + bias.double()
    if epilogue == NONE:
        v, size = v + rows(buf).double(), size + rows(buf).double().abs()
    if epilogue == DGELU:
        v, size = v * aux.double(), size * aux.double().abs()
    # one rounding to bf16, fp32 sums of K terms (GELU: its slope is at most 1.13, its argument has the same error)
    if epilogue == GELU:
        gelu = v * 0.5 * (1 + torch.erf(v / 2 ** 0.5))
        assert bool(((rows(c2).double() - gelu).abs() <= gelu.abs() * 2.0 ** -8 + size * (K * 2.0 ** -23) + 1e-6).all())
    else:
        assert bool(((rows(c).double() - v).abs() <= v.abs() * 2.0 ** -8 + size * (K * 2.0 ** -24) + 1e-6).all())
        assert torch.equal(rows(buf2), rows(c2))


def test_products_that_the_split_kernel_does_not_take_are_refused():
    rnd = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)
    A, B, side = rnd(16, 128), rnd(128, 16), rnd(16, 16)
    for status, C, C2 in (product(SPLIT, A[:, :120], B[:120], 1, None, None, NONE, None),     # a reduction below 128
                          product(SPLIT, A, B, 1, None, side, DGELU, side)):                  # residual and saved derivative at once
        assert status == 2 and bool((C == 7.0).all()) and bool((C2 == 7.0).all())


@pytest.mark.parametrize("cuts,whole,shapes", [
    # M, N, K (and how much further apart the rows of A, B and C are): edges of the 384 x 192 tile, of a stage of 32 k, of the four
    # stages in flight; parts of unequal length, and one of none; long and short reductions in a set, in either order
    (1, 0, [(8, 8, 1, 0, 0, 0), (384, 192, 32, 0, 0, 0), (48, 200, 33, 8, 0, 8), (392, 184, 97, 0, 16, 0)]),
    (3, 0, [(384, 192, 520, 0, 0, 0), (200, 400, 1000, 8, 8, 4)]),
    (4, 2, [(768, 384, 449, 0, 0, 0), (136, 72, 128, 0, 0, 0), (400, 200, 640, 0, 8, 8)]),
    (16, 0, [(48, 64, 4500, 0, 0, 0)]),
    (12, 0, [(56, 8, 520, 0, 0, 0)]),
])
def test_weight_gradients_on_big_tiles(cuts, whole, shapes):
    g = torch.Generator(device="cuda").manual_seed(cuts * 100 + len(shapes))
    n = len(shapes)
    rnd = lambda r, c, pad: torch.randn(r, c + pad, generator=g, device="cuda").to(torch.bfloat16)
    A = [rnd(K, M, pa) for M, N, K, pa, pb, pc in shapes]
    B = [rnd(K, N, pb) for M, N, K, pa, pb, pc in shapes]
    C = [torch.full((M, N + pc), 7.0, device="cuda") for M, N, K, pa, pb, pc in shapes]
    sums = [torch.full((N,), 7.0, device="cuda") if j != 1 else None for j, (M, N, K, pa, pb, pc) in enumerate(shapes)]
    ws = torch.full((384 * 192 * 40,), float("nan"), device="cuda")
    f = P.lib().ppll_internal_weight_grads
    f.restype = ctypes.c_int
    flat = (ctypes.c_int * (6 * n))(*[v for M, N, K, pa, pb, pc in shapes for v in (M, N, K, M + pa, N + pb, N + pc)])
    ptrs = lambda ts: (ctypes.c_void_p * n)(*[None if t is None else t.data_ptr() for t in ts])
    f.argtypes = [ctypes.c_int] + [ctypes.c_void_p] * 6 + [ctypes.c_size_t, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    call = lambda: f(n, flat, ptrs(A), ptrs(B), ptrs(C), ptrs(sums), ws.data_ptr(), ws.numel(), cuts, whole, torch.cuda.current_stream().cuda_stream)
    assert call() == 0
    torch.cuda.synchronize()
    for (M, N, K, pa, pb, pc), a, b, c, s in zip(shapes, A, B, C, sums):
        a, b = a[:, :M].double(), b[:, :N].double()
        # fp32 sums of K terms in any order, on the scale of the sum of their magnitudes
        ref, size = a.t().contiguous() @ b, a.t().contiguous().abs() @ b.abs()
        assert bool(((c[:, :N].double() - ref).abs() <= size * (K * 2.0 ** -24) + 1e-6).all())
        assert bool((c[:, N:] == 7.0).all())
        if s is not None:
            assert bool(((s.double() - b.sum(0)).abs() <= b.abs().sum(0) * (K * 2.0 ** -24) + 1e-6).all())
    first = [c.clone() for c in C]
    assert call() == 0 and all(torch.equal(x, c) for x, c in zip(first, C))
    no_room = f(n, flat, ptrs(A), ptrs(B), ptrs(C), ptrs(sums), ws.data_ptr(), 0, 2, 0, torch.cuda.current_stream().cuda_stream)
    assert no_room == (4 if any(s[2] > 448 for s in shapes) else 0)
    torch.cuda.synchronize()


@pytest.mark.parametrize("K,cuts", [(25216, 1), (4501, 1), (9000, 3), (1000, 4)])
def test_column_sums_on_big_tiles_are_sixteen_chains_a_column(K, cuts):
    # what the other weight-gradient kernels sum: one chain for each k % 16, then the chains of a half of eight in pairs and the halves;
    # parts of whole stages of 32 k, added in ascending k.  Values around 1, where the length of a chain shows in its error
    g = torch.Generator(device="cuda").manual_seed(K)
    N = 200
    A = torch.randn(K, 48, generator=g, device="cuda").to(torch.bfloat16)
    B = (torch.randn(K, N, generator=g, device="cuda") + 1).to(torch.bfloat16)
    C, sums = torch.empty(48, N, device="cuda"), torch.empty(N, device="cuda")
    ws = torch.empty(384 * 192 * 2 * 2 * cuts, device="cuda")
    f = P.lib().ppll_internal_weight_grads
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int] + [ctypes.c_void_p] * 6 + [ctypes.c_size_t, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    one = lambda t: (ctypes.c_void_p * 1)(t.data_ptr())
    assert f(1, (ctypes.c_int * 6)(48, N, K, 48, N, N), one(A), one(B), one(C), one(sums), ws.data_ptr(), ws.numel(), cuts, 0,
             torch.cuda.current_stream().cuda_stream) == 0
    stages = -(-K // 32)
    per = 32 * -(-stages // cuts)
    want = None
    for k0 in range(0, K, per):
        part = B[k0:k0 + per].float()
        part = torch.cat([part, part.new_zeros(-len(part) % 16, N)]).view(-1, 2, 8, N)
        chains = torch.zeros(2, 8, N, device="cuda")
        for step in part:
            chains = chains + step
        pairs = chains[:, 0::2] + chains[:, 1::2]
        halves = (pairs[:, 0] + pairs[:, 1]) + (pairs[:, 2] + pairs[:, 3])
        want = halves[0] + halves[1] if want is None else want + (halves[0] + halves[1])
    assert torch.equal(sums, want)


@pytest.mark.parametrize("epilogue", [NONE, GELU, DGELU])
@pytest.mark.parametrize("bt", [0, 1])
@pytest.mark.parametrize("M,N,K", [
    # edges of 128 x 128 tiles and of a stage of 64 k; one to sixteen stages, of which four are in LDS; more rows than columns of tiles and
    # the other way round; tiles on some XCDs alone; 224 tiles, which leave four units an XCD over, and 232, which leave fewer
    (1, 8, 128), (129, 136, 136), (127, 520, 200), (257, 128, 256), (640, 248, 1000), (130, 1160, 392), (128 * 16, 128 * 14, 192),
    (128 * 29, 128 * 8, 136),
])
def test_tiles_with_copying_waves_give_what_the_tiled_kernel_gives(M, N, K, bt, epilogue):
    g = torch.Generator(device="cuda").manual_seed(M * 1000 + N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    A, B = rnd(M, K + 40)[:, :K], rnd(K, N + 8)[:, :N] if bt else rnd(N, K + 16)[:, :K]     # rows further apart than they are long
    bias = torch.randn(N, generator=g, device="cuda") if epilogue != DGELU else None
    residual = rnd(M, N) if epilogue == NONE else None
    aux = rnd(M, N)
    wide = [torch.full((M, N + 24), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    status, C, C2 = product(TILED, A, B, bt, bias, None, epilogue, None if epilogue != DGELU else aux)
    assert status == 0
    status, D, D2 = product(COPYING, A, B, bt, bias, None, epilogue, None if epilogue != DGELU else aux)
    assert status == 0
    assert torch.equal(C, D) and torch.equal(C2, D2)
    if residual is not None:                                  # its rows are brought ahead as well
        a, b = (product(kernel, A, B, bt, bias, residual, epilogue, aux)[1] for kernel in (TILED, COPYING))
        assert torch.equal(a, b)
    # into a buffer wider than the result
    if epilogue != DGELU:
        for kernel, into in ((TILED, wide[0]), (COPYING, wide[1])):
            assert product(kernel, A, B, bt, bias, None, NONE, None, C=into[:, :N], C2=into[:, :N])[0] == 0
        assert torch.equal(wide[0], wide[1]) and bool((wide[1][:, N:] == 7.0).all())


@pytest.mark.parametrize("bt", [0, 1])
@pytest.mark.parametrize("M,N,K", [
    # tiles of 64 x 64 in blocks per XCD (the last ones ragged or empty) and in stretches; K in and out of whole stages
    (640, 768, 384), (577, 712, 200), (300, 768, 136), (1105, 768, 128), (1000, 968, 264), (65, 960, 192), (705, 136, 392),
])
def test_maps_of_few_tiles_give_what_the_tiled_kernel_gives(M, N, K, bt):
    g = torch.Generator(device="cuda").manual_seed(M * 1000 + N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    A, B = rnd(M, K + 40)[:, :K], rnd(K, N + 8)[:, :N] if bt else rnd(N, K + 16)[:, :K]
    bias, residual = torch.randn(N, generator=g, device="cuda"), rnd(M, N)
    status, C, _ = product(TILED, A, B, bt, bias, residual, NONE, None)
    assert status == 0
    for kernel in (SPLIT, COPYING):
        status, D, _ = product(kernel, A, B, bt, bias, residual, NONE, None)
        assert status == 0
        assert torch.equal(C, D), kernel
