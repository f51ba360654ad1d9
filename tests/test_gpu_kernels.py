"""GPU tests of the MFMA GEMM and implicit-GEMM convolution passes in
isolation, through the kernel-level C entry points, against plain fp64
references (a matrix product; the oracle's convolution forward, input
gradient and weight gradient).  Shapes cover several tiles, ragged edges in
every dimension, both operand layouts, compensated products and split-K."""
import numpy as np
import pytest

import fo_synth as S
from oracle import layers as OL
from tests.gpu_util import announce, normwise, to_dev, torch_cuda

pytestmark = pytest.mark.gpu
A = pytest.importorskip("paper_2504_13850_amd.api")


def _bf16(rng, shape, scale=1.0):
    x = (rng.standard_normal(shape) * scale).astype(np.float32)
    h = S.bf16_bits_from_f32(x)
    return h, S.f32_from_bf16_bits(h).astype(np.float64)


def _split(rng, shape):
    """A value with exact (hi, lo) bf16 parts: x = hi + lo."""
    hi, hv = _bf16(rng, shape)
    lo, lv = _bf16(rng, shape, 2.0 ** -9)
    return hi, lo, hv + lv


def _dev16(h):
    return to_dev(h.view(np.int16))


@pytest.mark.parametrize("M,N,K,la,lb", [
    (256, 256, 256, 0, 0), (200, 130, 96, 0, 0), (129, 257, 70, 0, 1), (64, 10, 512, 0, 1),
    (512, 768, 3072, 0, 0), (300, 200, 1000, 1, 1), (10, 512, 64, 1, 1), (3, 5, 7, 0, 0), (1, 1, 1, 1, 0),
    # k-major, rows in whole chunks of 8 (the weight-gradient kernel with copies
    # into LDS): ragged row tiles and K tails of every depth
    (264, 136, 1000, 1, 1), (776, 392, 70, 1, 1), (8, 8, 5, 1, 1), (128, 1152, 4097, 1, 1),
    # row-major A times k-major B with every dimension in chunks of 8 (the
    # input-gradient kernel with copies into LDS)
    (264, 136, 1000, 0, 1), (776, 392, 72, 0, 1), (8, 8, 8, 0, 1), (2496, 768, 2304, 0, 1)])
def test_gemm_plain(M, N, K, la, lb):
    torch = torch_cuda()
    announce(f"gemm {M}x{N}x{K} layouts {la}{lb}")
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    a, av = _bf16(rng, (M, K))
    b, bv = _bf16(rng, (N, K))
    Ad = _dev16(a if la == 0 else np.ascontiguousarray(a.T))
    Bd = _dev16(b if lb == 0 else np.ascontiguousarray(b.T))
    C = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    A.fo_gemm_bf16(M, N, K, la, Ad, None, K if la == 0 else M, lb, Bd, None, K if lb == 0 else N, C, N)
    ref = av @ bv.T
    assert normwise(C.cpu().numpy(), ref) <= 1e-5


@pytest.mark.parametrize("M,N,K,splits,la", [(256, 384, 1024, 4, 1), (100, 70, 333, 3, 1), (768, 768, 4096, 8, 1),
                                             (2496, 768, 3072, 2, 0), (264, 136, 1000, 3, 0)])
def test_gemm_split_k(M, N, K, splits, la):
    torch = torch_cuda()
    announce(f"gemm split-K {M}x{N}x{K} s={splits} A layout {la}")
    rng = np.random.default_rng(K)
    a, av = _bf16(rng, (K, M))      # k-major B (and A when la = 1), as in weight and input gradients
    b, bv = _bf16(rng, (K, N))
    Ad = _dev16(a) if la == 1 else _dev16(np.ascontiguousarray(a.T))
    C = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    ws = torch.empty(splits * M * N, dtype=torch.float32, device="cuda")
    A.fo_gemm_bf16(M, N, K, la, Ad, None, M if la == 1 else K, 1, _dev16(b), None, N, C, N, splits, ws)
    assert normwise(C.cpu().numpy(), av.T @ bv) <= 1e-5


@pytest.mark.parametrize("M,N,K,with_alo", [(256, 256, 768, True), (130, 300, 96, True), (64, 512, 512, False)])
def test_gemm_compensated(M, N, K, with_alo):
    """hi.hi + hi.lo + lo.hi reproduces the product of the unrounded values
    to about 16 significant bits (the omitted lo.lo term is ~2^-18)."""
    torch = torch_cuda()
    announce(f"gemm compensated {M}x{N}x{K}")
    rng = np.random.default_rng(N)
    if with_alo:
        ah, al, av = _split(rng, (M, K))
    else:
        ah, av = _bf16(rng, (M, K))
        al = None
    bh, bl, bv = _split(rng, (N, K))
    C = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    A.fo_gemm_bf16(M, N, K, 0, _dev16(ah), None if al is None else _dev16(al), K, 0, _dev16(bh), _dev16(bl), K, C, N)
    assert normwise(C.cpu().numpy(), av @ bv.T) <= 2e-5


@pytest.mark.parametrize("M,N,K,splits,with_alo", [(300, 200, 1000, 3, True), (129, 640, 2048, 4, True),
                                                    (256, 130, 512, 2, False)])
def test_gemm_compensated_split_k(M, N, K, splits, with_alo):
    """The single-pass compensated product with K slices (fp32 partials, reduction pass)."""
    torch = torch_cuda()
    announce(f"gemm compensated split-K {M}x{N}x{K} s={splits}")
    rng = np.random.default_rng(M + K)
    if with_alo:
        ah, al, av = _split(rng, (M, K))
    else:
        ah, av = _bf16(rng, (M, K))
        al = None
    bh, bl, bv = _split(rng, (N, K))
    C = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    ws = torch.empty(splits * M * N, dtype=torch.float32, device="cuda")
    A.fo_gemm_bf16(M, N, K, 0, _dev16(ah), None if al is None else _dev16(al), K, 0, _dev16(bh), _dev16(bl), K, C, N,
                   splits, ws)
    assert normwise(C.cpu().numpy(), av @ bv.T) <= 2e-5


@pytest.mark.parametrize("M,N,K,form,splits", [
    # 64 x 64 tiles with K dealt to the waves: one tile and its remainders, K
    # shorter than a step, than one step per wave, ragged in a step, more slices
    # than K tiles; then the last sizes on this side of the 128 x 128 tiles
    (64, 64, 512, 3, 1), (65, 68, 520, 3, 1), (1, 4, 8, 3, 1), (63, 60, 40, 2, 1), (130, 200, 264, 3, 3),
    (64, 64, 64, 2, 4), (64, 64, 512, 1, 1), (65, 72, 520, 1, 1), (1, 8, 8, 1, 1), (63, 56, 40, 1, 1),
    (130, 200, 328, 1, 3), (64, 64, 64, 1, 4), (2048, 2048, 128, 3, 1), (2048, 2048, 128, 1, 1),
    (4104, 64, 192, 1, 1)])
def test_gemm_small_tiles(M, N, K, form, splits):
    """form 3 and 2: compensated with and without A's low part; 1: k-major B.  fp32 sums of at most
    3 x 520 products: bounds as in the tests above."""
    torch = torch_cuda()
    announce(f"gemm small tiles {M}x{N}x{K} form {form} s={splits}")
    rng = np.random.default_rng(M + 3 * N + 7 * K + form)
    al = bl = None
    if form == 3:
        ah, al, av = _split(rng, (M, K))
    else:
        ah, av = _bf16(rng, (M, K))
    if form == 1:
        bh, bv = _bf16(rng, (N, K))
        bh = np.ascontiguousarray(bh.T)
    else:
        bh, bl, bv = _split(rng, (N, K))
    C = torch.full((M + 1, N), 7.0, dtype=torch.float32, device="cuda")
    ws = torch.empty(splits * M * N, dtype=torch.float32, device="cuda")
    A.fo_gemm_bf16(M, N, K, 0, _dev16(ah), None if al is None else _dev16(al), K, int(form == 1), _dev16(bh),
                   None if bl is None else _dev16(bl), N if form == 1 else K, C, N, splits, ws)
    got = C.cpu().numpy()
    assert normwise(got[:M], av @ bv.T) <= (1e-5 if form == 1 else 2e-5)
    assert (got[M] == 7.0).all()  # nothing past the last row


CONVS = [  # (Bn, H, Ci, Co, k, stride, pad)
    (2, 16, 64, 128, 3, 1, 1), (3, 8, 128, 256, 3, 1, 1), (2, 4, 256, 512, 3, 1, 1), (2, 2, 512, 512, 3, 1, 1),
    (32, 2, 512, 512, 3, 1, 1), (2, 16, 64, 128, 3, 2, 1), (4, 4, 256, 512, 3, 2, 1), (2, 16, 64, 128, 1, 2, 0),
    (3, 4, 256, 512, 1, 2, 0), (1, 2, 512, 512, 3, 1, 1)]


def _conv_case(case, seed):
    Bn, H, Ci, Co, k, st, pad = case
    rng = np.random.default_rng(seed)
    x, xv = _bf16(rng, (Bn, H, H, Ci))
    w, wv = _bf16(rng, (Co, k, k, Ci), 0.05)
    Ho = (H + 2 * pad - k) // st + 1
    dy, dyv = _bf16(rng, (Bn, Ho, Ho, Co))
    conv = OL.Conv2d(wv.transpose(0, 3, 1, 2), None, st, pad)
    y = conv.fwd(xv.transpose(0, 3, 1, 2))
    dx = conv.bwd(dyv.transpose(0, 3, 1, 2))
    return (x, w, dy), (y.transpose(0, 2, 3, 1), dx.transpose(0, 2, 3, 1), conv.dw.transpose(0, 2, 3, 1)), Ho


@pytest.mark.parametrize("case", CONVS)
def test_conv_passes(case):
    torch = torch_cuda()
    Bn, H, Ci, Co, k, st, pad = case
    announce(f"conv {case}")
    (x, w, dy), (y_ref, dx_ref, dw_ref), Ho = _conv_case(case, sum(case))
    xd, wd, dyd = _dev16(x), _dev16(w), _dev16(dy)
    for splits in (1, 4):  # split-K forward and input gradient: fp32 partials, epilogue in the reduction
        ws = torch.empty(splits * Bn * H * H * max(Ci, Co), dtype=torch.float32, device="cuda")
        y = torch.zeros((Bn, Ho, Ho, Co), dtype=torch.float32, device="cuda")
        A.fo_conv2d_bf16(0, Bn, H, H, Ci, Co, k, st, pad, xd, None, None, wd, None, y, splits, ws)
        assert normwise(y.cpu().numpy(), y_ref) <= 1e-5, splits
        dx = torch.zeros((Bn, H, H, Ci), dtype=torch.float32, device="cuda")
        A.fo_conv2d_bf16(1, Bn, H, H, Ci, Co, k, st, pad, dyd, None, None, wd, None, dx, splits, ws)
        assert normwise(dx.cpu().numpy(), dx_ref) <= 1e-5, splits
    for splits in (1, 4):
        dw = torch.zeros((Co, k, k, Ci), dtype=torch.float32, device="cuda")
        rows, cols = Co, k * k * Ci
        ws = torch.empty(splits * rows * cols, dtype=torch.float32, device="cuda")
        if Bn * Ho * Ho < splits * 32:
            continue
        A.fo_conv2d_bf16(2, Bn, H, H, Ci, Co, k, st, pad, dyd, None, xd, None, None, dw, splits, ws)
        assert normwise(dw.cpu().numpy(), dw_ref) <= 1e-5, splits


ORDERED = [  # (pass, Bn, H, Ci, Co, k, stride, low parts of the activations, slices)
    (0, 64, 8, 256, 256, 3, 1, True, 4), (0, 64, 8, 128, 256, 3, 1, False, 5), (0, 64, 8, 256, 256, 3, 1, True, 7),
    (0, 64, 8, 128, 256, 3, 1, False, 8), (0, 40, 9, 64, 256, 3, 1, True, 6), (0, 64, 8, 64, 256, 1, 1, True, 5),
    (0, 64, 16, 64, 256, 3, 2, True, 8),
    (1, 64, 8, 256, 256, 3, 1, False, 4), (1, 40, 9, 256, 192, 3, 1, False, 5), (1, 16, 16, 256, 128, 3, 2, False, 7),
    (1, 64, 8, 256, 256, 3, 1, False, 8), (1, 64, 8, 256, 64, 1, 1, False, 6)]


@pytest.mark.parametrize("case", ORDERED)
def test_conv_ordered_slices(case):
    """The same bits from the kernel that holds all slices of its 64 x 64 tile and from 128 x 128
    tiles with a slice per workgroup, which a quarter of the images runs on: both where the
    library adds the slices and where they are left to the caller, who adds them one by one."""
    torch = torch_cuda()
    pass_, Bn, H, Ci, Co, k, st, low, splits = case
    announce(f"ordered conv {case}")
    rng = np.random.default_rng(sum(case))
    pad, Ho = k // 2, (H + 2 * (k // 2) - k) // st + 1
    shape = (Bn, H, H, Ci) if pass_ == 0 else (Bn, Ho, Ho, Co)
    xh, xl, _ = _split(rng, shape)
    wh, wl, _ = _split(rng, (Co, k, k, Ci))
    x, w = _dev16(xh), _dev16(wh)
    xlo, wlo = _dev16(xl) if low else None, _dev16(wl) if pass_ == 0 else None
    side, N = (Ho, Co) if pass_ == 0 else (H, Ci)

    def run(i0, n, keep):
        out = torch.full((n * side * side, N), 7.0, dtype=torch.float32, device="cuda")
        ws = torch.zeros((splits, n * side * side, N), dtype=torch.float32, device="cuda")
        part = slice(i0, i0 + n)
        left = A.fo_conv2d_bf16_ordered(pass_, n, H, H, Ci, Co, k, st, pad, x[part], None if xlo is None else xlo[part],
                                        w, wlo, out, splits, ws, keep)
        if left > 1:
            assert left == splits
            out = ws[0].clone()
            for z in range(1, splits):
                out += ws[z]
        return out.cpu().numpy(), left

    for keep in (False, True):
        got, left = run(0, Bn, keep)
        quarters = [run(i, Bn // 4, keep) for i in range(0, Bn, Bn // 4)]
        if keep:
            assert left == 1 and all(q[1] == splits for q in quarters)  # both kernels ran
        assert np.array_equal(got.view(np.uint32), np.concatenate([q[0] for q in quarters]).view(np.uint32)), keep


GEOMETRIES = [  # (Bn, H, W, Ci, Co, k, stride, pad): odd maps, even and wide filters, no and wide padding, strides
    (3, 7, 10, 64, 72, 3, 1, 1), (2, 9, 5, 64, 64, 5, 1, 2), (2, 8, 11, 128, 64, 2, 2, 0), (3, 11, 7, 64, 128, 3, 2, 1),
    (1, 13, 6, 192, 64, 5, 2, 3), (2, 12, 9, 64, 64, 3, 3, 1), (5, 3, 3, 64, 64, 1, 1, 0), (2, 5, 8, 64, 64, 3, 1, 3),
    (1, 4, 4, 64, 64, 4, 1, 0)]


@pytest.mark.parametrize("case", GEOMETRIES)
def test_conv_geometries(case):
    """Compensated forward, with and without the activations' low parts, and input gradient,
    unsplit and in slices, on 64 x 64 tiles (strides 1 and 2) and 128 x 128 ones."""
    torch = torch_cuda()
    Bn, H, W, Ci, Co, k, st, pad = case
    announce(f"conv geometry {case}")
    rng = np.random.default_rng(sum(case))
    Ho, Wo = (H + 2 * pad - k) // st + 1, (W + 2 * pad - k) // st + 1
    xh, xl, xv = _split(rng, (Bn, H, W, Ci))
    wh, wl, wv = _split(rng, (Co, k, k, Ci))
    dy, dyv = _bf16(rng, (Bn, Ho, Wo, Co))
    for low in (True, False):
        x = xv if low else S.f32_from_bf16_bits(xh).astype(np.float64)
        conv = OL.Conv2d(wv.transpose(0, 3, 1, 2), None, st, pad)
        ref = conv.fwd(x.transpose(0, 3, 1, 2)).transpose(0, 2, 3, 1)
        for splits in (1, 3):
            ws = torch.empty(splits * ref.size, dtype=torch.float32, device="cuda")
            y = torch.zeros(ref.shape, dtype=torch.float32, device="cuda")
            A.fo_conv2d_bf16(0, Bn, H, W, Ci, Co, k, st, pad, _dev16(xh), _dev16(xl) if low else None, None, _dev16(wh),
                             _dev16(wl), y, splits, ws)
            assert normwise(y.cpu().numpy(), ref) <= 2e-5, (low, splits)
    if Co % 64:
        return
    conv = OL.Conv2d(S.f32_from_bf16_bits(wh).astype(np.float64).transpose(0, 3, 1, 2), None, st, pad)
    conv.fwd(xv.transpose(0, 3, 1, 2))
    ref = conv.bwd(dyv.transpose(0, 3, 1, 2)).transpose(0, 2, 3, 1)
    for splits in (1, 3):
        ws = torch.empty(splits * ref.size, dtype=torch.float32, device="cuda")
        dx = torch.zeros(ref.shape, dtype=torch.float32, device="cuda")
        A.fo_conv2d_bf16(1, Bn, H, W, Ci, Co, k, st, pad, _dev16(dy), None, None, _dev16(wh), None, dx, splits, ws)
        assert normwise(dx.cpu().numpy(), ref) <= 1e-5, splits
