"""hbfp_gemm_conv2d: the convolution whose activation operand is gathered from the image converted once (Sec. 5.1:
convolutions are executed like matrix products), against the oracle - which lowers the image explicitly - and against
the library's own product on the lowered operand of hbfp_encode_im2col (bit for bit: a block of 32 channels of a pixel
is the same block in the image and in every window that contains the pixel).  hbfp_gemm_conv2d_dgrad: the data gradient
of a convolution of any stride, gathered from the output gradient converted once."""
import numpy as np
import pytest
import torch

from oracle import ref
from tests.util import random_cases, rel_fro

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def hb():
    from paper_1804_01526_amd import hbfp
    assert torch.cuda.is_available(), "these tests need the GPU"
    return hbfp


def _conv_case(hb, n, h, w, c, f, r, s, pad_h, pad_w, sh, sw, seed, beta=0.0, against_lowered=True):
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((n, h, w, c)) * np.exp2(rng.integers(-3, 4, size=(n, h, w, 1)))).astype(np.float32)
    wm = (rng.standard_normal((r * s * c, f)) * 0.1).astype(np.float32)
    conv = hb.Conv2d(n, h, w, c, r, s, pad_h, pad_w, sh, sw, 0, 0)
    ho, wo = conv.out_hw()
    print(f"[conv] n={n} h={h} w={w} c={c} f={f} r={r} s={s} pad=({pad_h},{pad_w}) stride=({sh},{sw}) -> {n * ho * wo} x {f}", flush=True)
    img = hb.encode(torch.from_numpy(x.reshape(n * h * w, c)).cuda(), 1, hb.make_format(8, 1, 32))
    flt = hb.encode(torch.from_numpy(wm).cuda(), 0, hb.make_format(8, 32, 1))
    y0 = None
    if beta:
        y0 = rng.standard_normal((n * ho * wo, f)).astype(np.float32)
        y = hb.gemm_conv2d(img, conv, flt, out=torch.from_numpy(y0).cuda(), beta=1.0)
    else:
        y = hb.gemm_conv2d(img, conv, flt)
    torch.cuda.synchronize()
    y = y.cpu().numpy()
    # the oracle: convert the image (blocks of 32 channels), lower the decoded values tap by tap, multiply in FP64
    xq = ref.decode(ref.encode(x.reshape(n * h * w, c), 1, 32, 8)).reshape(n, h, w, c)
    low = ref.im2col(xq, r, s, pad_h, pad_w, sh, sw)
    # converting the lowered matrix instead gives the same operand (pinned here on the CPU side of the test)
    np.testing.assert_array_equal(ref.decode(ref.encode(ref.im2col(x, r, s, pad_h, pad_w, sh, sw), 1, 32, 8)), low)
    want = ref.gemm(low, ref.decode(ref.encode(wm, 32, 1, 8)))
    if y0 is not None:
        want = want + y0.astype(np.float64)
    err = rel_fro(y, want)
    print(f"        rel fro err = {err:.3e}", flush=True)
    assert err <= TOL
    if against_lowered and not beta:
        ta = hb.encode_im2col(torch.from_numpy(x).cuda(), conv, hb.make_format(8, 1, 32))
        yl = hb.gemm(ta, flt, kernel=hb.KERNEL_INT8)
        torch.cuda.synchronize()
        assert np.array_equal(y, yl.cpu().numpy()), "differs from the product on the lowered operand"


@pytest.mark.parametrize("geom", [
    # n, h, w, c, f, r, s, pad_h, pad_w, stride_h, stride_w
    (2, 12, 13, 64, 40, 3, 3, 1, 1, 1, 1),
    (3, 9, 9, 128, 130, 3, 3, 1, 1, 1, 1),
    (2, 10, 11, 64, 24, 1, 1, 0, 0, 1, 1),          # a 1 x 1 convolution: a plain product, k = 64 stored as 128
    (2, 14, 9, 64, 50, 5, 3, 2, 1, 1, 1),
    (2, 15, 16, 128, 64, 3, 3, 1, 1, 2, 2),          # strided
    (1, 8, 8, 192, 33, 3, 3, 0, 0, 1, 1),            # no padding, three 64-channel stages per tap (27 stages: odd)
    (2, 7, 7, 64, 20, 3, 3, 2, 2, 1, 3),             # padding wider than the usual, mixed strides
    (5, 6, 6, 64, 16, 2, 2, 0, 1, 2, 1),
])
def test_conv_geometries(hb, geom):
    _conv_case(hb, *geom, seed=sum(geom))


def test_conv_accumulates_and_splits_k(hb):
    _conv_case(hb, 2, 12, 13, 64, 40, 3, 3, 1, 1, 1, 1, seed=5, beta=1.0)
    _conv_case(hb, 1, 6, 6, 1024, 100, 3, 3, 1, 1, 1, 1, seed=6)            # few tiles, k = 9216: split along k
    _conv_case(hb, 1, 6, 6, 1024, 100, 3, 3, 1, 1, 1, 1, seed=7, beta=1.0)


def test_conv_random_geometries(hb):
    for seed in random_cases(12):
        rng = np.random.default_rng(9000 + seed)
        r, s = int(rng.integers(1, 5)), int(rng.integers(1, 5))
        h, w = int(rng.integers(r, 14)), int(rng.integers(s, 14))
        geom = (int(rng.integers(1, 4)), h, w, 64 * int(rng.integers(1, 4)), int(rng.integers(1, 150)), r, s,
                int(rng.integers(0, r)), int(rng.integers(0, s)), int(rng.integers(1, 3)), int(rng.integers(1, 3)))
        _conv_case(hb, *geom, seed=seed)


def test_conv_data_gradient_of_a_stride_one_convolution(hb):
    """dX of y = conv(x, w) with padding 1: the same call on dY with padding r - 1 - pad = 1 and the mirrored filter with
    its channel axes exchanged, against the adjoint of the convolution sum taken in FP64 from the decoded operands."""
    rng = np.random.default_rng(44)
    n, h, w, c, f = 2, 9, 10, 64, 128
    w4 = (rng.standard_normal((3, 3, c, f)) * 0.1).astype(np.float32)
    dy = (rng.standard_normal((n, h, w, f)) * 1e-2).astype(np.float32)
    wd = ref.filter_matrix_dgrad(w4)                                       # [3*3*f, c]
    conv = hb.Conv2d(n, h, w, f, 3, 3, 1, 1, 1, 1, 0, 0)
    img = hb.encode(torch.from_numpy(dy.reshape(n * h * w, f)).cuda(), 1, hb.make_format(8, 1, 32))
    flt = hb.encode(torch.from_numpy(np.ascontiguousarray(wd)).cuda(), 0, hb.make_format(8, 32, 1))
    dx = hb.gemm_conv2d(img, conv, flt)
    torch.cuda.synchronize()
    dyq = ref.decode(ref.encode(dy.reshape(n * h * w, f), 1, 32, 8)).reshape(n, h, w, f).astype(np.float64)
    wq = ref.decode(ref.encode(np.ascontiguousarray(wd), 32, 1, 8)).astype(np.float64).reshape(3, 3, f, c)   # mirrored, [fr][fs][f][c]
    # adjoint, written out: dx[img, y, x, ch] = sum_{fr, fs, f} dy[img, y + 1 - fr, x + 1 - fs, f] * w4[fr, fs, ch, f]
    # where wq[2 - fr, 2 - fs, f, ch] is the quantised w4[fr, fs, ch, f]
    want = np.zeros((n, h, w, c))
    dyp = np.zeros((n, h + 2, w + 2, f))
    dyp[:, 1:-1, 1:-1] = dyq
    for fr in range(3):
        for fs in range(3):
            want += dyp[:, 2 - fr:2 - fr + h, 2 - fs:2 - fs + w, :] @ wq[2 - fr, 2 - fs]
    assert rel_fro(dx.cpu().numpy(), want.reshape(n * h * w, c)) <= TOL


def _slot_case(hb, n, h, w, c, f, r, s, pad_h, pad_w, sh, sw, kb, by_block, per_image, tiles, seed, beta=0.0):
    """The general gather: channels in blocks of kb (stored padded to 32), window entries tap by tap or channel block by
    channel block (by_block), the image with one exponent per pixel and block or one per training input (per_image), the
    filter with one exponent per column and block or in tiles (tiles: kb x kb tap by tap, the whole window x kb channels
    x 24 filters by block - the tiling of the two outer filter dimensions of Sec. 5.1)."""
    rng = np.random.default_rng(seed)
    x = (np.maximum(rng.standard_normal((n, h, w, c)), -0.5) * np.exp2(rng.integers(-3, 4, size=(n, 1, 1, 1)))).astype(np.float32)
    w4 = (rng.standard_normal((r, s, c, f)) * np.exp2(rng.integers(-4, 5, size=(1, 1, c, 1))) * 0.1).astype(np.float32)
    cb = kb if by_block else 0
    wmat = np.ascontiguousarray(ref.filter_matrix(w4, cb))
    conv = hb.Conv2d(n, h, w, c, r, s, pad_h, pad_w, sh, sw, cb, 0)
    ho, wo = conv.out_hw()
    print(f"[slots] n={n} h={h} w={w} c={c} f={f} r={r} s={s} pad=({pad_h},{pad_w}) stride=({sh},{sw}) blocks of {kb} "
          f"{'by block' if by_block else 'by tap'} {'per image' if per_image else 'per pixel'} {'tiles' if tiles else 'columns'}", flush=True)
    x2 = x.reshape(n * h * w, c)
    if per_image:
        img = hb.encode(torch.from_numpy(x2).cuda(), 1, hb.make_format(8, h * w, 0, k_slot=kb))
        xq = ref.decode(ref.encode(x.reshape(n, -1), 1, 0, 8)).reshape(n, h, w, c)
        low_fmt = hb.make_format(8, ho * wo, 0, k_slot=kb)
    else:
        img = hb.encode(torch.from_numpy(x2).cuda(), 1, hb.make_format(8, 1, kb))
        xq = ref.decode(ref.encode(x2, 1, kb, 8)).reshape(n, h, w, c)
        low_fmt = hb.make_format(8, 1, kb)
    if tiles and by_block:
        flt = hb.encode(torch.from_numpy(wmat).cuda(), 0, hb.make_format(8, r * s * kb, 24, k_slot=kb))
        wq = ref.decode(ref.encode(wmat, r * s * kb, 24, 8))
    elif tiles:
        flt = hb.encode(torch.from_numpy(wmat).cuda(), 0, hb.make_format(8, kb, kb))
        wq = ref.decode(ref.encode(wmat, kb, kb, 8))
    else:
        flt = hb.encode(torch.from_numpy(wmat).cuda(), 0, hb.make_format(8, kb, 1))
        wq = ref.decode(ref.encode(wmat, kb, 1, 8))
    y0 = None
    if beta:
        y0 = rng.standard_normal((n * ho * wo, f)).astype(np.float32)
        y = hb.gemm_conv2d(img, conv, flt, out=torch.from_numpy(y0).cuda(), beta=1.0)
    else:
        y = hb.gemm_conv2d(img, conv, flt)
    torch.cuda.synchronize()
    y = y.cpu().numpy()
    want = ref.gemm(ref.im2col(xq, r, s, pad_h, pad_w, sh, sw, cb), wq)
    if y0 is not None:
        want = want + y0.astype(np.float64)
    err = rel_fro(y, want)
    print(f"        rel fro err = {err:.3e}", flush=True)
    assert np.linalg.norm(want) > 0 and err <= TOL
    if not beta and not (per_image and ho * wo == 1):     # hbfp_encode_im2col has no one-exponent-per-row form with k_slot
        ta = hb.encode_im2col(torch.from_numpy(x).cuda(), conv, low_fmt)
        yl = hb.gemm(ta, flt, kernel=hb.KERNEL_INT8)
        torch.cuda.synchronize()
        if by_block and per_image and tiles and r * s > 1:
            # both operands repeat their exponents over the taps of a channel block: the gather scales such a run once,
            # the product on the lowered operand block by block - the same sum with fewer roundings
            assert rel_fro(y, yl.cpu().numpy()) <= 2e-6
        else:
            assert np.array_equal(y, yl.cpu().numpy()), "differs from the product on the lowered operand"


@pytest.mark.parametrize("geom", [
    # n, h, w, c, f, r, s, pad_h, pad_w, stride_h, stride_w, block, by block, per image, filter tiles
    (3, 9, 9, 48, 50, 3, 3, 1, 1, 1, 1, 24, True, True, True),          # the format of Sec. 5.1 in full
    (2, 10, 8, 72, 30, 3, 3, 1, 1, 1, 1, 24, True, True, True),         # 27 slots: an odd number, the last stage half empty
    (2, 10, 8, 72, 30, 3, 3, 1, 1, 2, 2, 24, True, False, False),
    (2, 9, 11, 48, 70, 3, 3, 1, 1, 1, 1, 24, False, True, True),        # tap by tap, 24 x 24 filter tiles
    (2, 9, 11, 96, 40, 3, 3, 1, 1, 1, 1, 32, False, False, False),      # blocks of 32 but 96 channels: three slots per tap
    (2, 8, 8, 32, 20, 5, 3, 2, 1, 1, 1, 32, False, False, False),       # one slot per tap
    (2, 8, 8, 32, 20, 3, 3, 1, 1, 1, 1, 16, True, False, False),        # blocks of 16
    (3, 7, 9, 24, 24, 1, 1, 0, 0, 1, 1, 8, False, False, False),        # blocks of 8, a 1 x 1 convolution
    (2, 12, 12, 24, 40, 2, 2, 0, 0, 2, 2, 24, True, True, True),        # a single channel block
    (1, 6, 6, 960, 100, 3, 3, 1, 1, 1, 1, 24, True, True, True),        # few tiles, 360 slots: split along k
    (1, 2, 1, 8, 128, 1, 1, 0, 0, 1, 1, 8, True, True, False),          # two pixels, one slot
    (2, 9, 9, 64, 40, 3, 3, 1, 1, 1, 1, 32, True, True, True),          # runs of 9 blocks of 32: scaled after 8 and after 1
    (2, 8, 10, 48, 30, 5, 5, 2, 2, 1, 1, 24, True, True, True),         # runs of 25
    (2, 11, 7, 16, 30, 2, 1, 0, 0, 1, 1, 8, True, True, True),          # runs of 2 blocks of 8
])
def test_conv_general_gather(hb, geom):
    _slot_case(hb, *geom, seed=sum(int(g) for g in geom))


def test_conv_general_gather_accumulates(hb):
    _slot_case(hb, 3, 9, 9, 48, 50, 3, 3, 1, 1, 1, 1, 24, True, True, True, seed=3, beta=1.0)
    _slot_case(hb, 1, 6, 6, 960, 100, 3, 3, 1, 1, 1, 1, 24, True, True, True, seed=4, beta=1.0)


def test_conv_general_gather_random(hb):
    for seed in random_cases(12):
        rng = np.random.default_rng(9700 + seed)
        r, s = int(rng.integers(1, 5)), int(rng.integers(1, 5))
        h, w = int(rng.integers(r, 13)), int(rng.integers(s, 13))
        kb = int(rng.choice([8, 16, 24, 32]))
        geom = (int(rng.integers(1, 4)), h, w, kb * int(rng.integers(1, 6)), int(rng.integers(1, 150)), r, s,
                int(rng.integers(0, r)), int(rng.integers(0, s)), int(rng.integers(1, 3)), int(rng.integers(1, 3)),
                kb, bool(rng.integers(0, 2)), bool(rng.integers(0, 2)), bool(rng.integers(0, 2)))
        _slot_case(hb, *geom, seed=seed)


def _conv_bfp_case(hb, n, h, w, c, f, r, s, pad, st, kb, by_block, per_image, tiles, out_fmt, relu, seed):
    """hbfp_gemm_conv2d_bfp against the oracle's conversion of the library's own FP32 convolution (bit for bit: the same
    product, converted in the kernel or behind it), whose parity with the oracle the tests above establish."""
    from tests.util import unpack
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((n, h, w, c)) * np.exp2(rng.integers(-3, 4, size=(n, 1, 1, 1)))).astype(np.float32)
    w4 = (rng.standard_normal((r, s, c, f)) * 0.1).astype(np.float32)
    cb = kb if by_block else 0
    wmat = np.ascontiguousarray(ref.filter_matrix(w4, cb))
    conv = hb.Conv2d(n, h, w, c, r, s, pad, pad, st, st, cb, 0)
    ho, wo = conv.out_hw()
    f_img = hb.make_format(8, h * w, 0, k_slot=kb) if per_image else hb.make_format(8, 1, kb)
    f_flt = (hb.make_format(8, r * s * kb, 24, k_slot=kb) if by_block else hb.make_format(8, kb, kb)) if tiles else hb.make_format(8, kb, 1)
    img = hb.encode(torch.from_numpy(x.reshape(n * h * w, c)).cuda(), 1, f_img)
    flt = hb.encode(torch.from_numpy(wmat).cuda(), 0, f_flt)
    print(f"[conv bfp] n={n} h={h} w={w} c={c} f={f} r={r} s={s} pad={pad} stride={st} blocks of {kb} by_block={by_block} "
          f"per_image={per_image} tiles={tiles} out={out_fmt} relu={relu}", flush=True)
    m, br, bc, rounding, sd = out_fmt
    out = hb.gemm_conv2d_bfp(img, conv, flt, hb.make_format(m, br, bc, rounding, sd), relu=relu)
    y = hb.gemm_conv2d(img, conv, flt)
    torch.cuda.synchronize()
    y = y.cpu().numpy()
    if relu:
        y = np.maximum(y, 0.0)
    want = ref.encode(y, br, bc, m, rounding, sd)
    mant, exps = unpack(out)
    np.testing.assert_array_equal(exps, want.exps)
    np.testing.assert_array_equal(mant, want.mant)
    assert np.abs(mant).max() > 0


@pytest.mark.parametrize("case", [
    # n, h, w, c, f, r, s, pad, stride, block, by block, per image, tiles, (m, block rows, block cols, rounding, seed), relu
    (2, 12, 13, 64, 40, 3, 3, 1, 1, 32, False, False, False, (8, 1, 32, 0, 0), True),       # 64 channels per stage; 40 filters: a ragged block
    (3, 9, 9, 128, 130, 3, 3, 1, 1, 32, False, False, False, (8, 1, 32, 1, 77), False),      # stochastic rounding, two column tiles
    (2, 15, 16, 128, 64, 3, 3, 1, 2, 32, False, False, False, (6, 1, 32, 0, 0), True),       # strided, 6-bit output
    (3, 9, 9, 48, 50, 3, 3, 1, 1, 24, True, True, True, (8, 1, 32, 0, 0), True),             # Sec. 5.1's pairing, runs scaled once
    (2, 10, 8, 72, 96, 3, 3, 1, 1, 24, False, False, False, (8, 1, 32, 1, 5), True),         # slot by slot
    (2, 12, 13, 64, 40, 3, 3, 1, 1, 32, False, False, False, (8, 1, 24, 0, 0), True),        # blocks of 24: converted behind the product
    (2, 12, 13, 64, 40, 3, 3, 1, 1, 32, False, False, False, (12, 1, 32, 0, 0), False),      # 12 bits: behind the product
    (1, 6, 6, 1024, 100, 3, 3, 1, 1, 32, False, False, False, (8, 1, 32, 0, 0), True),       # split along k: behind the product
    (2, 12, 12, 24, 40, 2, 2, 0, 2, 24, True, True, True, (8, 144 // 4, 0, 0, 0), False),    # one exponent per training input out: behind
])
def test_conv_delivered_as_an_encoded_operand(hb, case):
    _conv_bfp_case(hb, *case, seed=sum(int(v) for v in case[:9]))


def test_conv_delivered_as_an_encoded_operand_random(hb):
    for seed in random_cases(10):
        rng = np.random.default_rng(9800 + seed)
        r, s = int(rng.integers(1, 4)), int(rng.integers(1, 4))
        h, w = int(rng.integers(max(r, s), 14)), int(rng.integers(max(r, s), 14))
        kb = int(rng.choice([8, 16, 24, 32]))
        by_block = bool(rng.integers(0, 2))
        per_image = bool(rng.integers(0, 2))
        _conv_bfp_case(hb, int(rng.integers(1, 4)), h, w, kb * int(rng.integers(1, 6)), int(rng.integers(1, 200)), r, s,
                       int(rng.integers(0, min(r, s))), int(rng.integers(1, 3)), kb, by_block, per_image, by_block and per_image,
                       (int(rng.integers(4, 9)), 1, 32, int(rng.integers(0, 2)), seed), bool(rng.integers(0, 2)), seed)


def test_conv_data_gradient_of_a_stride_one_convolution_in_the_format_of_the_experiments(hb):
    """Stride 1: the data gradient is hbfp_gemm_conv2d itself on dY (padding r - 1 - pad) in any format the gather takes;
    here dY with one exponent per training input in blocks of 24 filters, the mirrored filter in tiles over the whole
    window, 24 filters and 24 channels, against the oracle's lowered dY times its decoded filter."""
    rng = np.random.default_rng(52)
    n, h, w, c, f, r, s, pad = 3, 9, 10, 50, 72, 3, 3, 1
    dy = (rng.standard_normal((n, h, w, f)) * 1e-2 * np.exp2(rng.integers(-3, 4, size=(n, 1, 1, 1)))).astype(np.float32)
    w4 = (rng.standard_normal((r, s, c, f)) * np.exp2(rng.integers(-3, 4, size=(1, 1, 1, f))) * 0.1).astype(np.float32)
    wd = np.ascontiguousarray(ref.filter_matrix_dgrad(w4, 24))                                  # [(f block, tap, f in block), c]
    conv = hb.Conv2d(n, h, w, f, r, s, r - 1 - pad, s - 1 - pad, 1, 1, 24, 0)
    img = hb.encode(torch.from_numpy(dy.reshape(n * h * w, f)).cuda(), 1, hb.make_format(8, h * w, 0, k_slot=24))
    flt = hb.encode(torch.from_numpy(wd).cuda(), 0, hb.make_format(8, r * s * 24, 24, k_slot=24))
    dx = hb.gemm_conv2d(img, conv, flt)
    torch.cuda.synchronize()
    dyq = ref.decode(ref.encode(dy.reshape(n, -1), 1, 0, 8)).reshape(n, h, w, f)
    low = ref.im2col_dgrad(dyq, h, w, r, s, pad, pad)                                             # columns (tap, f)
    low = low.reshape(n * h * w, r * s, f // 24, 24).transpose(0, 2, 1, 3).reshape(n * h * w, -1)  # -> (f block, tap, f in block)
    want = ref.gemm(low, ref.decode(ref.encode(wd, r * s * 24, 24, 8)))
    assert np.linalg.norm(want) > 0 and rel_fro(dx.cpu().numpy(), want) <= TOL


def _dgrad_case(hb, n, h, w, c, f, r, s, pad_h, pad_w, sh, sw, seed, beta=0.0, kb=32, by_block=False, per_image=False, tiles=False):
    """hbfp_gemm_conv2d_dgrad against the oracle (dY converted, spread out and lowered explicitly, FP64 product with the
    converted mirrored filter) and, bit for bit, against hbfp_gemm_conv2d on a dY whose zeros are really stored.
    kb / by_block / per_image / tiles: the formats of _slot_case, with the filters of dY in the place of the channels."""
    rng = np.random.default_rng(seed)
    ho, wo = (h + 2 * pad_h - r) // sh + 1, (w + 2 * pad_w - s) // sw + 1
    print(f"[dgrad] n={n} h={h} w={w} c={c} f={f} r={r} s={s} pad=({pad_h},{pad_w}) stride=({sh},{sw}) dy {ho}x{wo} blocks of {kb} "
          f"{'by block' if by_block else 'by tap'} {'per image' if per_image else 'per pixel'} {'tiles' if tiles else 'columns'}", flush=True)
    dy = (rng.standard_normal((n, ho, wo, f)) * 1e-2 * np.exp2(rng.integers(-3, 4, size=(n, 1 if per_image else ho, 1 if per_image else wo, 1)))).astype(np.float32)
    w4 = (rng.standard_normal((r, s, c, f)) * 0.1).astype(np.float32)
    cb = kb if by_block else 0
    wd = np.ascontiguousarray(ref.filter_matrix_dgrad(w4, cb))             # [r*s*f, c]
    conv = hb.Conv2d(n, h, w, c, r, s, pad_h, pad_w, sh, sw, cb, 0)
    assert conv.out_hw() == (ho, wo)
    f_img = (lambda rows: hb.make_format(8, rows, 0, k_slot=kb)) if per_image else (lambda rows: hb.make_format(8, 1, kb))
    f_flt = (hb.make_format(8, r * s * kb, 24, k_slot=kb) if by_block else hb.make_format(8, kb, kb)) if tiles else hb.make_format(8, kb, 1)
    o_flt = ((r * s * kb, 24) if by_block else (kb, kb)) if tiles else (kb, 1)
    img = hb.encode(torch.from_numpy(dy.reshape(n * ho * wo, f)).cuda(), 1, f_img(ho * wo))
    flt = hb.encode(torch.from_numpy(wd).cuda(), 0, f_flt)
    x0 = None
    if beta:
        x0 = rng.standard_normal((n * h * w, c)).astype(np.float32)
        dx = hb.gemm_conv2d_dgrad(img, conv, flt, out=torch.from_numpy(x0).cuda(), beta=1.0)
    else:
        dx = hb.gemm_conv2d_dgrad(img, conv, flt)
    torch.cuda.synchronize()
    dx = dx.cpu().numpy()
    dyq = (ref.decode(ref.encode(dy.reshape(n, -1), 1, 0, 8)) if per_image else ref.decode(ref.encode(dy.reshape(n * ho * wo, f), 1, kb, 8))).reshape(n, ho, wo, f)
    low = ref.im2col_dgrad(dyq, h, w, r, s, pad_h, pad_w, sh, sw)          # columns (tap, filter)
    if by_block:                                                           # -> (filter block, tap, filter in block)
        low = low.reshape(n * h * w, r * s, f // kb, kb).transpose(0, 2, 1, 3).reshape(n * h * w, -1)
    want = ref.gemm(low, ref.decode(ref.encode(wd, o_flt[0], o_flt[1], 8)))
    if x0 is not None:
        want = want + x0.astype(np.float64)
    err = rel_fro(dx, want)
    print(f"        rel fro err = {err:.3e}", flush=True)
    assert err <= TOL
    ph, pw = r - 1 - pad_h, s - 1 - pad_w
    if ph >= 0 and pw >= 0 and not beta:
        hc, wc = h + r - 1 - 2 * ph, w + s - 1 - 2 * pw                 # the spread-out dY, with the rows no window reaches
        spread = np.zeros((n, hc, wc, f), dtype=np.float32)
        spread[:, 0:(ho - 1) * sh + 1:sh, 0:(wo - 1) * sw + 1:sw, :] = dy
        simg = hb.encode(torch.from_numpy(spread.reshape(n * hc * wc, f)).cuda(), 1, f_img(hc * wc))
        sconv = hb.Conv2d(n, hc, wc, f, r, s, ph, pw, 1, 1, cb, 0)
        assert sconv.out_hw() == (h, w)
        ds = hb.gemm_conv2d(simg, sconv, flt)
        torch.cuda.synchronize()
        assert np.array_equal(dx, ds.cpu().numpy()), "differs from the convolution of the stored spread-out gradient"


@pytest.mark.parametrize("geom", [
    # n, h, w, c, f, r, s, pad_h, pad_w, stride_h, stride_w   (of the forward convolution)
    (2, 12, 12, 40, 64, 3, 3, 1, 1, 2, 2),           # the last row and column of x are reached by part of a window only
    (2, 13, 11, 128, 128, 3, 3, 1, 1, 2, 2),
    (3, 9, 10, 64, 64, 3, 3, 1, 1, 1, 1),            # stride 1: the plain gather
    (2, 14, 14, 130, 64, 1, 1, 0, 0, 2, 2),          # a strided 1 x 1 convolution: three quarters of dx are zero
    (1, 17, 15, 24, 192, 5, 3, 2, 1, 3, 2),
    (2, 10, 9, 64, 64, 2, 2, 0, 0, 2, 2),            # windows that tile the image
    (2, 9, 9, 33, 64, 3, 3, 0, 0, 4, 4),             # stride beyond the window: rows of x that no window touches
    (2, 6, 7, 20, 64, 2, 2, 3, 2, 2, 2),             # padding wider than the window
])
def test_conv_data_gradient_geometries(hb, geom):
    _dgrad_case(hb, *geom, seed=sum(geom) + 1)


@pytest.mark.parametrize("geom", [
    # n, h, w, c, f, r, s, pad_h, pad_w, stride_h, stride_w, block, by block, per image, filter tiles
    (2, 12, 12, 40, 48, 3, 3, 1, 1, 2, 2, 24, True, True, True),       # the format of Sec. 5.1, strided
    (2, 11, 9, 30, 72, 3, 3, 1, 1, 2, 1, 24, False, True, True),
    (2, 10, 10, 50, 96, 3, 3, 1, 1, 2, 2, 32, False, False, False),    # 96 filters in blocks of 32: three slots per tap
    (2, 9, 9, 20, 32, 2, 2, 0, 0, 3, 3, 16, True, False, False),
    (3, 8, 8, 24, 48, 3, 3, 1, 1, 1, 1, 24, True, True, True),         # stride 1 in that format
    (1, 7, 7, 100, 960, 3, 3, 1, 1, 2, 2, 24, True, True, True),       # few tiles, 360 slots: split along k
])
def test_conv_data_gradient_general_formats(hb, geom):
    n, h, w, c, f, r, s, ph, pw, sh, sw, kb, by_block, per_image, tiles = geom
    _dgrad_case(hb, n, h, w, c, f, r, s, ph, pw, sh, sw, seed=sum(int(g) for g in geom), kb=kb, by_block=by_block, per_image=per_image, tiles=tiles)


@pytest.mark.parametrize("geom", [
    # n, h, w, c, f, r, s, pad_h, pad_w, beta   (stride 1, blocks of 24, by block, per image, filter tiles)
    (3, 8, 8, 24, 48, 3, 3, 1, 1, 0.0),
    (1, 7, 7, 100, 960, 3, 3, 1, 1, 0.0),            # 360 slots in runs of 9, split along k: ranges begin inside a run
    (1, 7, 7, 100, 960, 3, 3, 1, 1, 1.0),
    (2, 6, 7, 30, 48, 2, 3, 2, 1, 0.0),              # padding as wide as the window: positions that no window of dY reaches
    (1, 9, 5, 20, 72, 1, 4, 1, 4, 0.0),              # ... in both directions, windows of one row
    (2, 5, 12, 130, 48, 4, 2, 0, 1, 1.0),
])
def test_conv_data_gradient_scales_runs_once(hb, geom):
    """Stride 1 in the format of Sec. 5.1: dY is read without gaps, so runs of blocks with one exponent are scaled once, as in the
    forward call; against the oracle and the forward call, and by the kernel that does so."""
    from tests.util import launched_kernels
    n, h, w, c, f, r, s, ph, pw, beta = geom
    _dgrad_case(hb, n, h, w, c, f, r, s, ph, pw, 1, 1, seed=n + h + c + f, beta=beta, kb=24, by_block=True, per_image=True, tiles=True)
    conv = hb.Conv2d(n, h, w, c, r, s, ph, pw, 1, 1, 24, 0)
    ho, wo = conv.out_hw()
    dy = hb.encode(torch.randn((n * ho * wo, f), device="cuda"), 1, hb.make_format(8, ho * wo, 0, k_slot=24))
    flt = hb.encode(torch.randn((r * s * f, c), device="cuda"), 0, hb.make_format(8, r * s * 24, 24, k_slot=24))
    names = launched_kernels(lambda: hb.gemm_conv2d_dgrad(dy, conv, flt))
    assert any(k.startswith("gemm_i8_w8_kernel<3, true") for k in names), names


def test_conv_data_gradient_general_formats_random(hb):
    for seed in random_cases(12):
        rng = np.random.default_rng(9900 + seed)
        r, s = int(rng.integers(1, 5)), int(rng.integers(1, 5))
        h, w = int(rng.integers(r, 14)), int(rng.integers(s, 14))
        kb = int(rng.choice([8, 16, 24, 32]))
        _dgrad_case(hb, int(rng.integers(1, 4)), h, w, int(rng.integers(1, 150)), kb * int(rng.integers(1, 6)), r, s,
                    int(rng.integers(0, r + 1)), int(rng.integers(0, s + 1)), int(rng.integers(1, 4)), int(rng.integers(1, 4)), seed=seed,
                    kb=kb, by_block=bool(rng.integers(0, 2)), per_image=bool(rng.integers(0, 2)), tiles=bool(rng.integers(0, 2)))


def test_conv_data_gradient_accumulates_and_splits_k(hb):
    _dgrad_case(hb, 2, 12, 12, 40, 64, 3, 3, 1, 1, 2, 2, seed=15, beta=1.0)
    _dgrad_case(hb, 1, 8, 8, 100, 1024, 3, 3, 1, 1, 2, 2, seed=16)         # few tiles, k = 9216: split along k
    _dgrad_case(hb, 1, 8, 8, 100, 1024, 3, 3, 1, 1, 2, 2, seed=17, beta=1.0)


def test_conv_data_gradient_random_geometries(hb):
    for seed in random_cases(12):
        rng = np.random.default_rng(9500 + seed)
        r, s = int(rng.integers(1, 5)), int(rng.integers(1, 5))
        h, w = int(rng.integers(r, 16)), int(rng.integers(s, 16))
        geom = (int(rng.integers(1, 4)), h, w, int(rng.integers(1, 150)), 64 * int(rng.integers(1, 4)), r, s,
                int(rng.integers(0, r + 1)), int(rng.integers(0, s + 1)), int(rng.integers(1, 4)), int(rng.integers(1, 4)))
        _dgrad_case(hb, *geom, seed=seed)


def test_conv_data_gradient_under_graph_replay(hb):
    """Conversion of dY + hbfp_gemm_conv2d_dgrad (phase by phase) captured in a HIP graph and replayed on new gradients in
    the same buffers, with eager work in between; every replay against the eager result (bit for bit) and the oracle."""
    n, h, w, c, f, r, s, pad, st = 2, 11, 12, 48, 64, 3, 3, 1, 2
    conv = hb.Conv2d(n, h, w, c, r, s, pad, pad, st, st, 0, 0)
    ho, wo = conv.out_hw()
    rng = np.random.default_rng(71)
    w4 = (rng.standard_normal((r, s, c, f)) * 0.1).astype(np.float32)
    wd = np.ascontiguousarray(ref.filter_matrix_dgrad(w4))
    flt = hb.encode(torch.from_numpy(wd).cuda(), 0, hb.make_format(8, 32, 1))
    fmt = hb.make_format(8, 1, 32)
    dy = torch.zeros((n * ho * wo, f), device="cuda")
    td = hb.encode(dy, 1, fmt)
    dx = torch.empty((n * h * w, c), device="cuda")
    ws = torch.empty(hb.gemm_conv2d_dgrad_workspace(td.desc, conv, flt.desc), dtype=torch.uint8, device="cuda")
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        hb.encode(dy, 1, fmt, out=td, stream=stream)
        hb.gemm_conv2d_dgrad(td, conv, flt, out=dx, workspace=ws, stream=stream)
        stream.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            hb.encode(dy, 1, fmt, out=td, stream=stream)
            hb.gemm_conv2d_dgrad(td, conv, flt, out=dx, workspace=ws, stream=stream)
    for i, scale in enumerate([1e-2, 3.0, 2.0 ** -100, 1e-3]):
        g = (rng.standard_normal((n, ho, wo, f)) * scale).astype(np.float32)
        dy.copy_(torch.from_numpy(g.reshape(n * ho * wo, f)).cuda())
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = dx.cpu().numpy().copy()
        eager = hb.gemm_conv2d_dgrad(hb.encode(dy, 1, fmt), conv, flt)
        torch.cuda.synchronize()
        print(f"[case] dgrad graph replay {i} scale={scale}", flush=True)
        assert np.array_equal(got, eager.cpu().numpy())
        gq = ref.decode(ref.encode(g.reshape(n * ho * wo, f), 1, 32, 8)).reshape(n, ho, wo, f)
        want = ref.gemm(ref.im2col_dgrad(gq, h, w, r, s, pad, pad, st, st), ref.decode(ref.encode(wd, 32, 1, 8)))
        assert np.linalg.norm(want) > 0 and rel_fro(got, want) <= TOL


def test_conv_data_gradient_rejects_what_it_does_not_cover(hb):
    import ctypes
    conv = hb.Conv2d(2, 8, 8, 48, 3, 3, 1, 1, 2, 2, 0, 0)                  # dy 4 x 4
    dy = hb.encode(torch.zeros((2 * 4 * 4, 64), device="cuda"), 1, hb.make_format(8, 1, 32))
    flt = hb.encode(torch.zeros((9 * 64, 48), device="cuda"), 0, hb.make_format(8, 32, 1))
    dx = torch.empty((128, 48), device="cuda")
    ws = torch.empty(hb.gemm_conv2d_dgrad_workspace(dy.desc, conv, flt.desc), dtype=torch.uint8, device="cuda")
    call = lambda d, c, f_, ldx=48, beta=0.0, w=ws: hb._lib.hbfp_gemm_conv2d_dgrad(
        ctypes.byref(d.desc), ctypes.byref(c), ctypes.byref(f_.desc), dx.data_ptr(), ldx, beta, w.data_ptr(), w.numel(), None)
    assert call(dy, conv, flt) == hb.OK
    assert call(dy, conv, flt, ldx=40) == hb.ERR_ARG
    assert call(dy, conv, flt, beta=2.0) == hb.ERR_ARG
    assert call(dy, hb.Conv2d(2, 8, 8, 48, 3, 3, 1, 1, 1, 1, 0, 0), flt) == hb.ERR_LAYOUT              # dy of another stride
    assert call(dy, hb.Conv2d(2, 8, 8, 40, 3, 3, 1, 1, 2, 2, 0, 0), flt) == hb.ERR_LAYOUT              # filter of other channels
    assert call(dy, hb.Conv2d(2, 8, 8, 48, 3, 3, 1, 1, 2, 2, 16, 0), flt) == hb.ERR_FORMAT             # channel-block order
    dy24 = hb.encode(torch.zeros((2 * 4 * 4, 64), device="cuda"), 1, hb.make_format(8, 1, 16))
    assert call(dy24, conv, flt) == hb.ERR_FORMAT                                                      # blocks of 16 filters
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    assert call(dy, conv, flt, w=small) == hb.ERR_WORKSPACE
    torch.cuda.synchronize()


def test_conv_rejects_what_it_does_not_cover(hb):
    import ctypes
    x = torch.zeros((2 * 8 * 8, 64), device="cuda")
    img = hb.encode(x, 1, hb.make_format(8, 1, 32))
    flt = hb.encode(torch.zeros((9 * 64, 16), device="cuda"), 0, hb.make_format(8, 32, 1))
    conv = hb.Conv2d(2, 8, 8, 64, 3, 3, 1, 1, 1, 1, 0, 0)
    y = torch.empty((128, 16), device="cuda")
    ws = torch.empty(hb.gemm_conv2d_workspace(img.desc, conv, flt.desc), dtype=torch.uint8, device="cuda")
    call = lambda i, c, f_, ldy=16, beta=0.0, w=ws: hb._lib.hbfp_gemm_conv2d(
        ctypes.byref(i.desc), ctypes.byref(c), ctypes.byref(f_.desc), y.data_ptr(), ldy, beta, w.data_ptr(), w.numel(), None)
    assert call(img, conv, flt) == hb.OK
    assert call(img, conv, flt, ldy=8) == hb.ERR_ARG
    assert call(img, conv, flt, beta=0.5) == hb.ERR_ARG
    assert call(img, hb.Conv2d(2, 8, 8, 64, 3, 3, 1, 1, 1, 1, 16, 0), flt) == hb.ERR_FORMAT            # channel blocks that are not the stored blocks
    assert call(img, hb.Conv2d(2, 8, 9, 64, 3, 3, 1, 1, 1, 1, 0, 0), flt) == hb.ERR_LAYOUT             # not this image
    img24 = hb.encode(x, 1, hb.make_format(8, 1, 24))
    assert call(img24, conv, flt) == hb.ERR_FORMAT                                                       # blocks of 24: 64 channels are no multiple, and the filter has 32
    img16 = hb.encode(x, 1, hb.make_format(8, 1, 16))
    assert call(img16, conv, flt) == hb.ERR_FORMAT                                                       # blocks of 16 against a filter in blocks of 32
    flt5 = hb.encode(torch.zeros((25 * 64, 16), device="cuda"), 0, hb.make_format(8, 32, 1))
    assert call(img, conv, flt5) == hb.ERR_LAYOUT
    assert hb._lib.hbfp_gemm_conv2d(ctypes.byref(img.desc), ctypes.byref(conv), ctypes.byref(flt.desc), y.data_ptr(), 16, 0.0,
                                    None, 0, None) == hb.ERR_WORKSPACE
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,h,w,c,r", [(1, 7, 9, 32, 3), (2, 20, 20, 64, 3), (16, 28, 28, 64, 3), (4, 14, 14, 128, 1)])
def test_conv_bfp_over_its_own_image(hb, n, h, w, c, r):
    """The encoded convolution stored over the image it reads (a residual block's layer in place): same bytes as into buffers
    of its own.  The workspace query sees the overlap."""
    print(f"[conv bfp in place] {n}x{h}x{w}x{c} r={r}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + c)
    conv = hb.Conv2d(n, h, w, c, r, r, r // 2, r // 2, 1, 1, 0, 0)
    act = hb.make_format(8, 1, 32)
    img = hb.encode(torch.randn((n * h * w, c), generator=gen, device="cuda"), 1, act)
    flt = hb.encode(torch.randn((r * r * c, c), generator=gen, device="cuda") * 0.1, 0, hb.make_format(8, 32, 1))
    want = hb.gemm_conv2d_bfp(img, conv, flt, act, relu=True)
    assert hb.gemm_conv2d_bfp_workspace(img.desc, conv, flt.desc, img.desc) >= 4 * n * h * w * c
    hb.gemm_conv2d_bfp(img, conv, flt, act, relu=True, out=img)
    torch.cuda.synchronize()
    assert torch.equal(img.mant, want.mant) and torch.equal(img.exps, want.exps)


@pytest.mark.parametrize("n,h,w,c,f,r,s,pad,sh,sw,kb", [
    (64, 23, 23, 64, 40, 3, 3, 1, 1, 1, 32),         # two column tiles of one wave
    (50, 26, 26, 48, 100, 3, 3, 1, 1, 1, 24),        # blocks of 24, block by block along k
    (54, 25, 25, 96, 160, 3, 3, 1, 1, 1, 32),        # tiles of 192 filters, an odd number of channel blocks
    (34, 33, 32, 72, 192, 3, 3, 1, 1, 1, 24),        # whole tiles of 192
    (40, 30, 60, 48, 128, 3, 3, 1, 1, 2, 24),        # strided along the rows (in both directions no strip fits)
    (520, 16, 8, 32, 128, 3, 3, 1, 2, 1, 32),        # strided down the image, a single channel block
    (2100, 4, 4, 24, 33, 3, 3, 1, 1, 1, 24),         # several images in a unit of 64 positions
    (60, 25, 25, 64, 30, 2, 2, 0, 1, 1, 32),         # no padding, fewer filters than a column tile
    (52, 28, 27, 32, 128, 1, 5, 0, 1, 1, 32),        # a window of one row
    (130, 28, 28, 72, 100, 3, 3, 1, 1, 1, 24),       # three and four units of positions, blocks of 24
    (100, 28, 28, 64, 160, 3, 3, 1, 1, 1, 32),       # two and three units on tiles of 192
    (100, 28, 28, 48, 192, 3, 3, 1, 1, 1, 24),
    (130, 28, 28, 64, 32, 3, 3, 1, 1, 1, 32),        # one column tile in all, three and four units
    (130, 28, 28, 48, 50, 3, 3, 1, 1, 1, 24),        # ... one of each wave
])
def test_conv_strips_against_the_lowered_product(hb, n, h, w, c, f, r, s, pad, sh, sw, kb):
    """Sizes at which the product runs from strips of the image on the bf16 instruction, against the int8 product on the lowered operand.
    Values are small integers, so that every sum is exact in FP32 whatever its order: equal to the bit, delivered encoded too."""
    from tests.util import launched_kernels
    g = torch.Generator(device="cuda").manual_seed(n + f)
    x = torch.randint(-7, 8, (n, h, w, c), device="cuda", generator=g) * torch.randint(0, 3, (n, h, w, 1), device="cuda", generator=g)
    wm = torch.randint(-7, 8, (r * s * c, f), device="cuda", generator=g).float()
    conv = hb.Conv2d(n, h, w, c, r, s, pad, pad, sh, sw, kb if kb < 32 else 0, 0)
    print(f"[conv] n={n} h={h} w={w} c={c} f={f} window {r}x{s} pad={pad} stride=({sh},{sw}) blocks of {kb}", flush=True)
    img = hb.encode(x.float().view(n * h * w, c), 1, hb.make_format(8, 1, kb))
    flt = hb.encode(wm, 0, hb.make_format(8, kb, 1))
    low = hb.encode_im2col(x.float(), conv, hb.make_format(8, 1, kb))
    y = hb.gemm_conv2d(img, conv, flt)
    assert torch.equal(y, hb.gemm(low, flt, kernel=hb.KERNEL_INT8))
    fmt = hb.make_format(8, 1, 32)
    enc, want = hb.gemm_conv2d_bfp(img, conv, flt, fmt, relu=True), hb.encode(torch.relu(y), 1, fmt)
    assert torch.equal(enc.mant, want.mant) and torch.equal(enc.exps, want.exps)
    names = launched_kernels(lambda: hb.gemm_conv2d(img, conv, flt, out=y))
    assert any(k.startswith("gemm_strip_kernel") for k in names), names


@pytest.mark.parametrize("n,f,kb,per_image", [
    (54, 24, 32, False), (54, 32, 24, True),                             # one column tile: the first wave's
    (54, 40, 32, False),             # one of 32 and one of 8: a wave each
    (54, 64, 32, False), (54, 64, 24, True), (80, 320, 32, False),       # two whole ones alone in the last 128 columns
    (54, 96, 32, False), (54, 80, 24, False),                            # three: two and one
    (54, 100, 24, False),            # three and a part
    (54, 160, 32, False), (54, 192, 24, True),                           # tiles of 192: a second wave of two and of three
])
def test_conv_strips_add_to_c_once(hb, n, f, kb, per_image):
    """beta = 1 from strips: no column belongs to two waves, which would both add to it.  Small integers: equal to the bit to the int8
    product on the lowered operand added in FP32, forward and as the data gradient of stride 1."""
    from tests.util import launched_kernels
    c, h = 2 * kb, 25
    g = torch.Generator(device="cuda").manual_seed(n + f)
    whole = dict(k_slot=kb) if per_image else {}
    cb = kb if kb < 32 else 0
    x = torch.randint(-7, 8, (n, h, h, c), device="cuda", generator=g).float()
    wm = torch.randint(-7, 8, (9 * c, f), device="cuda", generator=g).float()
    y0 = torch.randint(-99, 100, (n * h * h, f), device="cuda", generator=g).float()
    img = hb.encode(x.view(-1, c), 1, hb.make_format(8, h * h, 0, k_slot=kb) if per_image else hb.make_format(8, 1, kb))
    flt = hb.encode(wm, 0, hb.make_format(8, 9 * kb, kb, k_slot=kb) if per_image else hb.make_format(8, kb, 1))
    conv = hb.Conv2d(n, h, h, c, 3, 3, 1, 1, 1, 1, cb, 0)
    low = hb.encode_im2col(hb.decode(img).view(n, h, h, c), conv, hb.make_format(8, 1, kb))
    want = y0 + hb.gemm(low, flt, kernel=hb.KERNEL_INT8)
    fw = hb.Conv2d(n, h, h, f, 3, 3, 1, 1, 1, 1, cb, 0)                  # dY has c columns, dX f: the same product
    for call in (lambda out, beta: hb.gemm_conv2d(img, conv, flt, out=out, beta=beta),
                 lambda out, beta: hb.gemm_conv2d_dgrad(img, fw, flt, out=out, beta=beta)):
        print(f"[conv strips, beta] n={n} f={f} blocks of {kb}", flush=True)
        got = call(y0.clone(), 1.0)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        names = launched_kernels(lambda: call(got, 0.0))
        assert any(k.startswith("gemm_strip_kernel") for k in names), names


@pytest.mark.parametrize("n,h,w,c,f,kb,bits,sr", [
    (2, 160, 160, 64, 192, 32, 8, 0),        # rows so long that a strip of 192 positions fits, one of 256 does not
    (2, 156, 158, 96, 129, 32, 8, 1),        # ... ragged, an odd number of channel blocks, stochastic
    (4, 170, 170, 48, 144, 24, 8, 0),        # three and four units of positions, the FP32 product on tiles of 192 filters
    (130, 28, 28, 64, 128, 32, 4, 1),        # three and four units on tiles of 128 both
    (100, 20, 20, 72, 60, 24, 8, 1),         # one wave of columns only
    (130, 28, 28, 64, 32, 32, 8, 0), (130, 28, 28, 72, 20, 24, 8, 1),    # one column tile in all
    (130, 28, 28, 64, 96, 32, 4, 1), (100, 20, 20, 48, 75, 24, 8, 0),    # the second wave has one
])
def test_conv_strips_delivered_encoded_are_the_conversion_of_the_product(hb, n, h, w, c, f, kb, bits, sr):
    """Sums that round (exponents far apart): the encoded result has the bytes of the FP32 result's conversion, so both come from strips
    and add in one order, whatever the tiles."""
    from tests.util import launched_kernels
    g = torch.Generator(device="cuda").manual_seed(n + f)
    x = torch.randn((n * h * w, c), device="cuda", generator=g) * torch.exp2(torch.rand((n * h * w, 1), device="cuda", generator=g) * 24.0)
    wm = torch.randn((9 * c, f), device="cuda", generator=g) * torch.exp(torch.randn((9 * c, f), device="cuda", generator=g) * 3.0)
    conv = hb.Conv2d(n, h, w, c, 3, 3, 1, 1, 1, 1, kb if kb < 32 else 0, 0)
    img, flt = hb.encode(x, 1, hb.make_format(8, 1, kb)), hb.encode(wm, 0, hb.make_format(8, kb, 1))
    fmt = hb.make_format(bits, 1, 32, hb.STOCHASTIC if sr else hb.RNE, 77)
    print(f"[conv strips, encoded] n={n} {h}x{w}x{c} f={f} blocks of {kb} bits={bits} sr={sr}", flush=True)
    for relu in (False, True):
        y = hb.gemm_conv2d(img, conv, flt)
        enc, want = hb.gemm_conv2d_bfp(img, conv, flt, fmt, relu=relu), hb.encode(torch.relu(y) if relu else y, 1, fmt)
        torch.cuda.synchronize()
        assert torch.equal(enc.mant, want.mant) and torch.equal(enc.exps, want.exps)
    for call in (lambda: hb.gemm_conv2d(img, conv, flt), lambda: hb.gemm_conv2d_bfp(img, conv, flt, fmt)):
        names = launched_kernels(call)
        assert sum(k.startswith("gemm_strip_kernel") for k in names) == 1, names


@pytest.mark.parametrize("n,h,w,c,f,pad,sw,kb,bits,per_image,log2_x,log2_w", [
    (60, 25, 25, 64, 128, 1, 1, 32, 8, False, 0, 0),
    (64, 25, 25, 96, 60, 0, 1, 32, 4, False, 0, 0),          # an odd number of channel blocks, narrow mantissas
    (60, 25, 25, 72, 144, 1, 1, 24, 8, True, 0, 0),          # the tiling of Sec. 5.1
    (40, 30, 60, 48, 100, 1, 2, 24, 8, False, 0, 0),         # strided
    (60, 25, 25, 64, 128, 1, 1, 32, 8, False, -70, -62),     # sums below the normal range
    (60, 25, 25, 64, 128, 1, 1, 32, 8, False, -127, 60),     # blocks whose last bits lie below the normal range
    (60, 25, 25, 48, 40, 1, 1, 24, 6, True, -126, 80),
    (60, 25, 25, 64, 128, 1, 1, 32, 8, False, 124, -60),     # the largest exponent bytes
    (60, 25, 25, 72, 192, 1, 1, 24, 8, True, -60, 124),
])
def test_conv_strips_are_fp32_sums_of_exact_products(hb, n, h, w, c, f, pad, sw, kb, bits, per_image, log2_x, log2_w):
    """Exponents far apart and at both ends of their range, forward and (stride 1) as the data gradient, against 64 bits.  Every product is
    exact and each of the K additions rounds by at most 2^-23 of a partial sum, which is at most sum |a||b| (2^-149 where that is
    subnormal); over the whole result the roundings do not conspire: sqrt(K) 2^-24 of its norm."""
    from tests.util import launched_kernels
    g = torch.Generator(device="cuda").manual_seed(n + c + f + bits)
    spread = 0.0 if log2_x or log2_w else 24.0
    x = torch.randn((n, h, w, c), device="cuda", generator=g) * torch.exp2(torch.rand((n, h, w, 1), device="cuda", generator=g) * spread)
    x = (x.double() * 2.0 ** log2_x).clamp(-3.4e38, 3.4e38).float()
    wm = (torch.randn((9 * c, f), device="cuda", generator=g).double() * 2.0 ** log2_w).clamp(-3.4e38, 3.4e38).float()
    cb = kb if kb < 32 else 0
    conv = hb.Conv2d(n, h, w, c, 3, 3, pad, pad, 1, sw, cb, 0)
    ho, wo = conv.out_hw()
    print(f"[conv strips, fp64] n={n} {h}x{w}x{c} f={f} pad={pad} stride (1,{sw}) blocks of {kb} bits={bits} per image={per_image} "
          f"2^{log2_x} 2^{log2_w}", flush=True)
    img = hb.encode(x.view(-1, c), 1, hb.make_format(bits, h * w, 0, k_slot=kb) if per_image else hb.make_format(bits, 1, kb))
    flt = hb.encode(wm, 0, hb.make_format(bits, 9 * kb, kb, k_slot=kb) if per_image else hb.make_format(bits, kb, 1))
    # the lowered image and the filter matrix in 64 bits, window entries tap by tap
    xd = torch.nn.functional.pad(hb.decode(img).double().view(n, h, w, c), (0, 0, pad, pad, pad, pad))
    low = torch.cat([xd[:, a:a + ho, b:b + (wo - 1) * sw + 1:sw] for a in range(3) for b in range(3)], 3).reshape(n * ho * wo, 9 * c)
    wd = hb.decode(flt).double()
    if cb:
        wd = wd.view(c // kb, 9, kb, f).transpose(0, 1).reshape(9 * c, f)
    want, K = low @ wd, 9 * c
    bound = K * (2.0 ** -23 * (low.abs() @ wd.abs()) + 2.0 ** -149)
    calls = [lambda: hb.gemm_conv2d(img, conv, flt)]
    if sw == 1 and pad == 1:                                # dY has c columns, dX f: the same sum
        calls.append(lambda: hb.gemm_conv2d_dgrad(img, hb.Conv2d(n, h, w, f, 3, 3, 1, 1, 1, 1, cb, 0), flt))
    for call in calls:
        y = call().double()
        assert bool(torch.isfinite(y).all()) and float(want.norm()) > 0
        err = (y - want).abs()
        print(f"        largest error / bound = {float((err / bound).max()):.3e}, rel. norm {float(err.norm() / want.norm()):.3e}", flush=True)
        assert bool((err <= bound).all()) and float(err.norm()) <= K ** 0.5 * 2.0 ** -24 * float(want.norm())
        names = launched_kernels(call)
        assert any(k.startswith("gemm_strip_kernel") for k in names), names
