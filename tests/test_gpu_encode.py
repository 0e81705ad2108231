"""GPU parity of FP32 -> BFP -> FP32 against the CPU oracle, through the C ABI.
Mantissas, exponent bytes and decoded values must match bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import ref
from tests.util import launched_kernels, random_cases, unpack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_1804_01526_amd import hbfp
    assert torch.cuda.is_available(), "these tests need the GPU"
    return hbfp


def _data(shape, seed, spread=8):
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal(shape) * np.exp2(rng.integers(-spread, spread + 1, size=shape))).astype(np.float32)
    x[rng.random(shape) < 0.03] = 0.0
    return x


def _check(hb, x, axis, br, bc, m, rounding, seed=0, src=None):
    """Encode x on the GPU (optionally from a strided view `src`) and compare with the oracle."""
    print(f"[case] shape={x.shape} axis={axis} block=({br},{bc}) m={m} rounding={rounding} seed={seed}", flush=True)
    fmt = hb.make_format(m, br, bc, rounding, seed)
    xs = torch.from_numpy(x).cuda() if src is None else src
    bt = hb.encode(xs, axis, fmt)
    torch.cuda.synchronize()
    want = ref.encode(x, br, bc, m, rounding, seed)
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, want.exps)
    np.testing.assert_array_equal(mant, want.mant)
    back = hb.decode(bt)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(back.cpu().numpy(), ref.decode(want))
    return bt


ROW_CASES = [
    # rows, cols, block along k, m, rounding
    (37, 1000, 32, 8, 0), (64, 4096, 32, 8, 1), (5, 100, 24, 8, 0), (128, 128, 32, 12, 1),
    (3, 7000, 64, 12, 0), (129, 520, 128, 8, 0), (16, 96, 20, 8, 1), (7, 1001, 32, 8, 0),
    (1, 100000, 32, 8, 1), (300, 40, 8, 4, 0), (33, 4096, 24, 8, 0), (2, 333, 64, 16, 1),
    (70, 128, 32, 2, 0), (1, 5, 32, 8, 0), (50, 72, 24, 12, 1),
]


@pytest.mark.parametrize("rows,cols,B,m,rounding", ROW_CASES)
def test_encode_rowwise_blocks(hb, rows, cols, B, m, rounding):
    _check(hb, _data((rows, cols), rows * 7 + cols), 1, 1, B, m, rounding, seed=0xC0FFEE + rows)


COL_CASES = [
    (1000, 37, 32, 8, 0), (4096, 64, 32, 8, 1), (100, 5, 24, 8, 0), (128, 128, 32, 12, 1),
    (7000, 3, 64, 12, 0), (96, 200, 20, 8, 1), (1001, 70, 32, 8, 0), (333, 130, 64, 16, 1),
    (40, 300, 8, 4, 0), (4096, 33, 24, 8, 0), (5, 1, 32, 8, 0), (260, 257, 64, 8, 1),
]


@pytest.mark.parametrize("rows,cols,B,m,rounding", COL_CASES)
def test_encode_colwise_blocks(hb, rows, cols, B, m, rounding):
    _check(hb, _data((rows, cols), rows * 3 + cols), 0, B, 1, m, rounding, seed=0xBEEF + cols)


TILE_CASES = [
    # rows, cols, axis, br, bc, m, rounding
    (100, 100, 0, 24, 24, 8, 0), (100, 100, 1, 24, 24, 8, 0), (130, 70, 0, 24, 24, 8, 1), (70, 130, 1, 64, 64, 12, 1),
    (50, 3000, 1, 1, 0, 8, 0), (3000, 50, 0, 0, 1, 8, 0), (64, 64, 1, 0, 0, 8, 0), (200, 300, 0, 0, 0, 12, 1),
    (129, 1030, 1, 1, 200, 8, 0), (1030, 129, 0, 200, 1, 8, 1), (33, 65, 1, 2, 32, 8, 0), (65, 33, 0, 32, 2, 8, 0),
    (48, 4100, 1, 24, 24, 8, 0), (4100, 48, 0, 24, 24, 8, 1), (300, 200, 0, 100, 100, 8, 0), (200, 300, 1, 100, 100, 8, 1),
    (150, 150, 0, 64, 64, 12, 0), (130, 2100, 1, 1100, 128, 8, 0), (64, 200, 0, 16, 3, 8, 0), (200, 64, 1, 3, 16, 8, 1),
    # several row strips of the maximum pass, blocks that cross them, widths that are no multiple of 4
    (700, 2100, 0, 0, 1, 8, 0), (700, 2100, 1, 1, 0, 8, 1), (520, 1300, 0, 256, 1, 12, 0), (520, 1300, 1, 1, 256, 12, 1),
    (300, 1100, 0, 64, 64, 8, 0), (300, 1100, 1, 64, 64, 8, 1), (131, 1029, 1, 1, 0, 8, 0), (1029, 131, 0, 0, 1, 8, 1),
    (400, 1500, 0, 0, 0, 8, 0), (400, 1500, 1, 0, 0, 12, 1), (257, 515, 0, 130, 70, 8, 0), (257, 515, 1, 70, 130, 8, 0),
]


@pytest.mark.parametrize("rows,cols,axis,br,bc,m,rounding", TILE_CASES)
def test_encode_tiles_and_long_blocks(hb, rows, cols, axis, br, bc, m, rounding):
    _check(hb, _data((rows, cols), rows + 13 * cols), axis, br, bc, m, rounding, seed=0xABCD)


SLOT_CASES = [
    # rows, cols, axis, br, bc, k_slot, m, rounding: exponent blocks longer than the stored blocks
    (70, 1000, 1, 1, 0, 24, 8, 0), (1000, 70, 0, 0, 1, 24, 8, 1), (130, 2000, 1, 1, 96, 24, 8, 1), (2000, 130, 0, 96, 1, 24, 12, 0),
    (200, 1030, 1, 64, 64, 32, 8, 0), (1030, 200, 0, 64, 64, 32, 8, 1), (300, 520, 1, 0, 0, 64, 12, 0), (520, 300, 0, 0, 0, 24, 8, 0),
    (33, 4100, 1, 1, 0, 32, 8, 0), (4100, 33, 0, 0, 1, 128, 8, 0), (90, 777, 1, 3, 0, 20, 8, 1), (777, 90, 0, 0, 3, 20, 8, 0),
]


@pytest.mark.parametrize("rows,cols,axis,br,bc,slot,m,rounding", SLOT_CASES)
def test_encode_exponent_blocks_longer_than_stored_blocks(hb, rows, cols, axis, br, bc, slot, m, rounding):
    """hbfp_format.k_slot: mantissas and exponents are those of the br x bc blocks (the oracle knows nothing of the
    stored blocks); the stored blocks repeat the exponent (checked by unpack)."""
    x = _data((rows, cols), rows + 7 * cols + slot)
    print(f"[case] shape={x.shape} axis={axis} block=({br},{bc}) k_slot={slot} m={m} rounding={rounding}", flush=True)
    fmt = hb.make_format(m, br, bc, rounding, 0x51075, k_slot=slot)
    bt = hb.encode(torch.from_numpy(x).cuda(), axis, fmt)
    torch.cuda.synchronize()
    assert bt.desc.kblock == slot and bt.desc.kshare > 1
    want = ref.encode(x, br, bc, m, rounding, 0x51075)
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, want.exps)
    np.testing.assert_array_equal(mant, want.mant)
    back = hb.decode(bt)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(back.cpu().numpy(), ref.decode(want))


CONV_CASES = [
    # n, h, w, c, r, s, pad_h, pad_w, stride_h, stride_w, block, m, rounding
    (2, 9, 10, 16, 3, 3, 1, 1, 1, 1, 32, 8, 0), (3, 8, 7, 8, 3, 3, 1, 1, 1, 1, 24, 8, 1), (2, 12, 11, 40, 1, 1, 0, 0, 1, 1, 8, 8, 0),
    (2, 11, 13, 24, 5, 3, 2, 1, 2, 1, 64, 12, 0), (1, 14, 14, 32, 3, 3, 0, 0, 2, 2, 128, 8, 1), (5, 6, 6, 16, 3, 3, 1, 1, 1, 1, 16, 4, 0),
    (2, 7, 9, 48, 2, 4, 1, 2, 1, 3, 40, 12, 1), (1, 28, 28, 128, 3, 3, 1, 1, 1, 1, 32, 8, 0),
]


@pytest.mark.parametrize("n,h,w,c,r,s,ph,pw,sh,sw,B,m,rounding", CONV_CASES)
def test_encode_im2col_equals_encoding_the_lowered_matrix(hb, n, h, w, c, r, s, ph, pw, sh, sw, B, m, rounding):
    """hbfp_encode_im2col against the oracle's encode of the oracle's lowered matrix, bit for bit."""
    print(f"[case] conv n={n} h={h} w={w} c={c} filter={r}x{s} pad=({ph},{pw}) stride=({sh},{sw}) block={B} m={m} rounding={rounding}", flush=True)
    x = _data((n, h, w, c), n + 3 * h + 5 * w + c)
    conv = hb.Conv2d(n, h, w, c, r, s, ph, pw, sh, sw, 0, 0)
    bt = hb.encode_im2col(torch.from_numpy(x).cuda(), conv, hb.make_format(m, 1, B, rounding, 0xC0DE))
    torch.cuda.synchronize()
    low = ref.im2col(x, r, s, ph, pw, sh, sw)
    assert (bt.desc.src_rows, bt.desc.src_cols) == low.shape
    want = ref.encode(low, 1, B, m, rounding, 0xC0DE)
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, want.exps)
    np.testing.assert_array_equal(mant, want.mant)


CONV_WGRAD_CASES = [
    # n, h, w, c, r, s, pad_h, pad_w, stride_h, stride_w, block (output positions), m, rounding
    (2, 9, 10, 16, 3, 3, 1, 1, 1, 1, 32, 8, 0), (3, 8, 7, 5, 3, 3, 1, 1, 1, 1, 24, 8, 1), (2, 12, 11, 40, 1, 1, 0, 0, 1, 1, 8, 8, 0),
    (2, 11, 13, 24, 5, 3, 2, 1, 2, 1, 64, 12, 0), (1, 14, 14, 33, 3, 3, 0, 0, 2, 2, 20, 8, 1), (4, 28, 28, 16, 3, 3, 1, 1, 1, 1, 32, 8, 0),
]


@pytest.mark.parametrize("n,h,w,c,r,s,ph,pw,sh,sw,B,m,rounding", CONV_WGRAD_CASES)
def test_encode_im2col_weight_gradient_orientation(hb, n, h, w, c, r, s, ph, pw, sh, sw, B, m, rounding):
    """contract_axis 0: operand rows = window entries, k = output positions in blocks of B; bit for bit the oracle's
    encode of the oracle's lowered matrix with B x 1 blocks."""
    print(f"[case] conv wgrad n={n} h={h} w={w} c={c} filter={r}x{s} pad=({ph},{pw}) stride=({sh},{sw}) block={B} m={m} rounding={rounding}", flush=True)
    x = _data((n, h, w, c), 2 * n + 3 * h + 5 * w + c)
    conv = hb.Conv2d(n, h, w, c, r, s, ph, pw, sh, sw, 0, 0)
    bt = hb.encode_im2col(torch.from_numpy(x).cuda(), conv, hb.make_format(m, B, 1, rounding, 0xFACE), contract_axis=0)
    torch.cuda.synchronize()
    low = ref.im2col(x, r, s, ph, pw, sh, sw)
    want = ref.encode(low, B, 1, m, rounding, 0xFACE)
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, want.exps)
    np.testing.assert_array_equal(mant, want.mant)


@pytest.mark.parametrize("B,m,rounding", [(24, 8, 0), (32, 8, 0), (32, 8, 1), (24, 12, 0), (20, 8, 0)])
@pytest.mark.parametrize("n,h,w,c,r,s,ph,pw,sh,sw", [
    (5, 9, 7, 20, 3, 3, 1, 1, 1, 1),        # several rows and images in a piece of 24 or 32 positions
    (3, 28, 28, 7, 3, 3, 1, 1, 1, 1),       # at most two rows in a piece
    (2, 5, 70, 30, 3, 5, 1, 2, 1, 1),       # rows longer than two pieces
    (4, 15, 16, 33, 3, 3, 1, 1, 2, 2),      # strided
    (4, 9, 13, 18, 2, 3, 0, 1, 1, 3),       # strides that differ
    (40, 3, 3, 11, 3, 3, 0, 0, 1, 1),       # a position per image
    (6, 4, 4, 16, 3, 3, 3, 3, 1, 1),        # more padding than the window: corners move back
    (3, 6, 6, 9, 2, 2, 0, 0, 3, 3),         # a stride beyond the window
])
def test_encode_im2col_pieces_inside_the_tensor(hb, n, h, w, c, r, s, ph, pw, sh, sw, B, m, rounding):
    """The weight-gradient orientation at sizes small enough for loads with a check per value, in the geometries that decide where whole
    pieces of positions can do without (the next test), bit for bit against the oracle's encode of the lowered matrix."""
    rng = np.random.default_rng(n * h * w + c)
    x = rng.standard_normal((n, h, w, c)).astype(np.float32)
    conv = hb.Conv2d(n, h, w, c, r, s, ph, pw, sh, sw, 0, 0)
    print(f"[case] im2col {n}x{h}x{w}x{c} window {r}x{s} pad ({ph},{pw}) stride ({sh},{sw}) B={B} m={m}", flush=True)
    bt = hb.encode_im2col(torch.from_numpy(x).cuda(), conv, hb.make_format(m, B, 1, rounding, 0xBEEF), contract_axis=0)
    torch.cuda.synchronize()
    want = ref.encode(ref.im2col(x, r, s, ph, pw, sh, sw), B, 1, m, rounding, 0xBEEF)
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, want.exps)
    np.testing.assert_array_equal(mant, want.mant)


@pytest.mark.parametrize("B,m,rounding", [(32, 8, 0), (24, 8, 1), (24, 12, 0)])
@pytest.mark.parametrize("n,h,w,c,r,s,ph,pw,sh,sw,unchecked", [
    (600, 9, 7, 20, 3, 3, 1, 1, 1, 1, True),
    (50, 28, 28, 21, 3, 3, 1, 1, 1, 1, True),
    (42, 5, 70, 30, 3, 5, 1, 2, 1, 1, True),
    (360, 15, 16, 33, 3, 3, 1, 1, 2, 2, True),
    (560, 9, 13, 50, 2, 3, 0, 1, 1, 3, True),
    (12500, 3, 3, 60, 3, 3, 0, 0, 1, 1, True),
    (600, 4, 4, 16, 3, 3, 3, 3, 1, 1, False),        # corners move back
    (7000, 6, 6, 64, 2, 2, 0, 0, 3, 3, True),
    (3, 9, 10, 300, 3, 3, 1, 1, 1, 1, False),        # few pieces
    (30, 100, 100, 64, 1, 1, 0, 0, 1, 1, False),     # one pixel, whole waves: 18.3 Mi values
    (15, 100, 100, 64, 1, 1, 0, 0, 1, 1, True), (30, 100, 100, 66, 1, 1, 0, 0, 1, 1, True),
])
def test_encode_im2col_weight_gradient_of_many_pieces(hb, n, h, w, c, r, s, ph, pw, sh, sw, unchecked, B, m, rounding):
    """The geometries above at sizes from which pieces inside the tensor are loaded without a check and workgroups are dealt to the XCDs
    by position, against the oracle, and by the instance that the sizes call for."""
    from tests.util import launched_kernels
    rng = np.random.default_rng(n + c)
    x = rng.standard_normal((n, h, w, c)).astype(np.float32)
    xd = torch.from_numpy(x).cuda()
    conv, fmt = hb.Conv2d(n, h, w, c, r, s, ph, pw, sh, sw, 0, 0), hb.make_format(m, B, 1, rounding, 0xBEEF)
    print(f"[case] im2col {n}x{h}x{w}x{c} window {r}x{s} pad ({ph},{pw}) stride ({sh},{sw}) B={B} m={m}", flush=True)
    bt = hb.encode_im2col(xd, conv, fmt, contract_axis=0)
    torch.cuda.synchronize()
    want = ref.encode(ref.im2col(x, r, s, ph, pw, sh, sw), B, 1, m, rounding, 0xBEEF)
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, want.exps)
    np.testing.assert_array_equal(mant, want.mant)
    names = launched_kernels(lambda: hb.encode_im2col(xd, conv, fmt, contract_axis=0, out=bt))
    kernel = f"enc_col_kernel<32, {str(m > 8).lower()}, {rounding}, false, true, {str(unchecked).lower()}>"
    assert names == [kernel], (names, kernel)


@pytest.mark.parametrize("n,h,w,c,r,s,ph,pw,sh,sw,slot,m,rounding", [
    (3, 9, 10, 16, 3, 3, 1, 1, 1, 1, 24, 8, 0), (2, 8, 7, 8, 3, 3, 1, 1, 1, 1, 24, 8, 1), (4, 12, 11, 40, 1, 1, 0, 0, 1, 1, 8, 12, 1),
    (2, 11, 13, 24, 5, 3, 2, 1, 2, 1, 64, 8, 0), (2, 15, 15, 32, 2, 2, 0, 0, 3, 3, 32, 8, 1), (70, 6, 6, 16, 3, 3, 1, 1, 1, 1, 16, 8, 0),
])
def test_encode_im2col_one_exponent_per_training_input(hb, n, h, w, c, r, s, ph, pw, sh, sw, slot, m, rounding):
    """Sec. 5.1: the x tensor gets one exponent per training input.  The oracle converts the image tensor as a matrix
    [n][h*w*c] with one block per row and lowers the mantissas afterwards; the library gathers and converts in one go
    (with stride 3 and a 2 x 2 filter some pixels lie in no window: they still count for the exponent)."""
    print(f"[case] conv per-image n={n} h={h} w={w} c={c} filter={r}x{s} pad=({ph},{pw}) stride=({sh},{sw}) slot={slot} m={m} rounding={rounding}", flush=True)
    x = _data((n, h, w, c), 5 * n + 3 * h + w + c, spread=3)
    x *= np.exp2(np.random.default_rng(n).integers(-6, 7, size=(n, 1, 1, 1))).astype(np.float32)      # images of different scale
    conv = hb.Conv2d(n, h, w, c, r, s, ph, pw, sh, sw, 0, 0)
    ho, wo = conv.out_hw()
    fmt = hb.make_format(m, ho * wo, 0, rounding, 0x1A6E, k_slot=slot)
    bt = hb.encode_im2col(torch.from_numpy(x).cuda(), conv, fmt)
    torch.cuda.synchronize()
    img = ref.encode(x.reshape(n, h * w * c), 1, 0, m, rounding, 0x1A6E)
    want_mant = ref.im2col(img.mant.reshape(n, h, w, c), r, s, ph, pw, sh, sw)
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, img.exps)
    np.testing.assert_array_equal(mant, want_mant)
    with pytest.raises(hb.HbfpError) as e:                          # the table of image maxima needs its workspace
        hb._check(hb._lib.hbfp_encode_im2col(bt.mant.data_ptr(), ctypes.byref(conv), ctypes.byref(bt.desc), None, 0, None),
                  "hbfp_encode_im2col")
    assert e.value.status == hb.ERR_WORKSPACE


@pytest.mark.parametrize("n,h,w,c,r,s,ph,pw,sh,sw,cb,B,m,rounding,axis", [
    (2, 9, 10, 48, 3, 3, 1, 1, 1, 1, 24, 24, 8, 0, 1), (2, 8, 7, 40, 3, 3, 1, 1, 1, 1, 16, 16, 8, 1, 1), (3, 7, 7, 128, 3, 3, 1, 1, 1, 1, 24, 24, 8, 0, 1),
    (2, 11, 9, 56, 5, 3, 2, 1, 2, 1, 32, 32, 12, 1, 1), (2, 9, 10, 48, 3, 3, 1, 1, 1, 1, 24, 32, 8, 0, 0), (2, 8, 7, 21, 3, 3, 1, 1, 1, 1, 5, 24, 8, 1, 0),
])
def test_encode_im2col_channel_block_order(hb, n, h, w, c, r, s, ph, pw, sh, sw, cb, B, m, rounding, axis):
    """hbfp_conv2d.c_block: the window entries run channel block by channel block (the last block may be shorter:
    40 = 16 + 16 + 8, 128 = 5 * 24 + 8); both operand orientations, against the oracle's lowering in the same order."""
    print(f"[case] conv c_block n={n} h={h} w={w} c={c} filter={r}x{s} c_block={cb} block={B} m={m} rounding={rounding} axis={axis}", flush=True)
    x = _data((n, h, w, c), n + 7 * h + 3 * w + c + cb)
    conv = hb.Conv2d(n, h, w, c, r, s, ph, pw, sh, sw, cb, 0)
    fmt = hb.make_format(m, 1, B, rounding, 0xB10C) if axis == 1 else hb.make_format(m, B, 1, rounding, 0xB10C)
    bt = hb.encode_im2col(torch.from_numpy(x).cuda(), conv, fmt, contract_axis=axis)
    torch.cuda.synchronize()
    low = ref.im2col(x, r, s, ph, pw, sh, sw, cb)
    want = ref.encode(low, 1, B, m, rounding, 0xB10C) if axis == 1 else ref.encode(low, B, 1, m, rounding, 0xB10C)
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, want.exps)
    np.testing.assert_array_equal(mant, want.mant)


@pytest.mark.parametrize("case", random_cases(40))
def test_encode_im2col_random_geometries(hb, case):
    """Random images, windows, paddings, strides, channel blocks, block lengths and modes (blocks along the window,
    blocks over the output positions, one exponent per image) against the oracle's lowering + conversion."""
    rng = np.random.default_rng(8000 + case)
    mode = ("fwd", "wgrad", "per_image")[case % 3]
    n, h, w = int(rng.integers(1, 5)), int(rng.integers(3, 13)), int(rng.integers(3, 13))
    r, s_ = int(rng.integers(1, min(h, 5) + 1)), int(rng.integers(1, min(w, 5) + 1))
    ph, pw = int(rng.integers(0, r)), int(rng.integers(0, s_))
    sh, sw = int(rng.integers(1, 4)), int(rng.integers(1, 4))
    c = int(rng.integers(1, 9)) * 8 if mode != "wgrad" else int(rng.integers(1, 50))
    cb = 0
    if rng.random() < 0.5:
        cb = int(rng.choice([8, 16, 24])) if mode != "wgrad" else int(rng.integers(1, c + 1))
    m, rounding = int(rng.choice([4, 8, 12])), int(rng.integers(0, 2))
    x = _data((n, h, w, c), 8500 + case, spread=4)
    conv = hb.Conv2d(n, h, w, c, r, s_, ph, pw, sh, sw, cb, 0)
    ho, wo = conv.out_hw()
    low = ref.im2col(x, r, s_, ph, pw, sh, sw, cb)
    print(f"[case] {case}: {mode} n={n} h={h} w={w} c={c} window={r}x{s_} pad=({ph},{pw}) stride=({sh},{sw}) c_block={cb} m={m} rounding={rounding}", flush=True)
    xg = torch.from_numpy(x).cuda()
    if mode == "fwd":
        B = int(rng.choice([8, 16, 24, 32, 64, 128]))
        bt = hb.encode_im2col(xg, conv, hb.make_format(m, 1, B, rounding, 77 + case))
        want = ref.encode(low, 1, B, m, rounding, 77 + case)
        want_mant, want_exps = want.mant, want.exps
    elif mode == "wgrad":
        B = int(rng.choice([8, 20, 24, 32, 64]))
        bt = hb.encode_im2col(xg, conv, hb.make_format(m, B, 1, rounding, 77 + case), contract_axis=0)
        want = ref.encode(low, B, 1, m, rounding, 77 + case)
        want_mant, want_exps = want.mant, want.exps
    else:
        slot = int(rng.choice([8, 16, 24, 32]))
        if slot >= r * s_ * c:
            slot = 8
        if r * s_ * c <= 8:
            pytest.skip("window of 8 entries: nothing to cut into stored blocks")
        if ho * wo == 1:
            with pytest.raises(hb.HbfpError):      # one output position per image: not the per-image format
                hb.encode_im2col(xg, conv, hb.make_format(m, 1, 0, rounding, 77 + case, k_slot=slot))
            return
        bt = hb.encode_im2col(xg, conv, hb.make_format(m, ho * wo, 0, rounding, 77 + case, k_slot=slot))
        img = ref.encode(x.reshape(n, -1), 1, 0, m, rounding, 77 + case)
        want_mant, want_exps = ref.im2col(img.mant.reshape(n, h, w, c), r, s_, ph, pw, sh, sw, cb), img.exps
    torch.cuda.synchronize()
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, want_exps)
    np.testing.assert_array_equal(mant, want_mant)


def test_encode_im2col_argument_checks(hb):
    x = torch.zeros((2, 8, 8, 16), device="cuda")
    conv = hb.Conv2d(2, 8, 8, 16, 3, 3, 1, 1, 1, 1, 0, 0)
    for fmt, status in ((hb.make_format(8, 1, 20), hb.ERR_FORMAT), (hb.make_format(8, 1, 0), hb.ERR_FORMAT),
                        (hb.make_format(8, 2, 32), hb.ERR_FORMAT)):
        with pytest.raises(hb.HbfpError) as e:
            hb.encode_im2col(x, conv, fmt)
        assert e.value.status == status
    with pytest.raises(hb.HbfpError) as e:                          # descriptor of another shape
        hb.encode_im2col(x, conv, hb.make_format(8, 1, 32), out=hb.alloc(hb.make_format(8, 1, 32), 100, 144, 1))
    assert e.value.status == hb.ERR_LAYOUT
    with pytest.raises(hb.HbfpError) as e:                          # channels not a multiple of 8
        hb.encode_im2col(torch.zeros((1, 8, 8, 12), device="cuda"), hb.Conv2d(1, 8, 8, 12, 3, 3, 1, 1, 1, 1, 0, 0), hb.make_format(8, 1, 24))
    assert e.value.status == hb.ERR_FORMAT


@pytest.mark.parametrize("axis,br,bc,slot", [(1, 1, 0, 0), (0, 0, 1, 0), (0, 0, 0, 0), (1, 64, 64, 0), (0, 64, 64, 0), (1, 1, 0, 24), (1, 1, 256, 0)])
def test_paper_block_shapes_at_layer_size_bit_exact(hb, axis, br, bc, slot):
    """2048 x 4096 (the launch shapes of a layer-sized conversion: several strips and column groups of the maximum
    pass, whole rows in the registers of a wave) in the block shapes of Sec. 4 and Sec. 6: one exponent per row,
    per column, for the matrix, 64 x 64 tiles, one exponent per row stored in blocks of 24; compared in full,
    decode included."""
    rng = np.random.default_rng(axis * 100 + br + bc + slot)
    x = (rng.standard_normal((2048, 4096)) * np.exp2(rng.integers(-6, 7, size=(2048, 1)))).astype(np.float32)
    print(f"[case] 2048x4096 axis={axis} block=({br},{bc}) k_slot={slot}", flush=True)
    fmt = hb.make_format(8, br, bc, 0, 0, k_slot=slot)
    bt = hb.encode(torch.from_numpy(x).cuda(), axis, fmt)
    torch.cuda.synchronize()
    want = ref.encode(x, br, bc, 8)
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, want.exps)
    np.testing.assert_array_equal(mant, want.mant)
    back = hb.decode(bt)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(back.cpu().numpy(), ref.decode(want))


def test_config3_activation_operand_from_the_image_tensor_full_size(hb):
    """Config 3's forward operand (128 x 28 x 28 x 128 image, 3 x 3 window, padding 1 -> 100352 x 1152, blocks of 32) in the
    launch shape the benchmark times, against the oracle's encode of its own lowered matrix, in full."""
    rng = np.random.default_rng(303)
    x = np.maximum(rng.standard_normal((128, 28, 28, 128)), 0).astype(np.float32)
    conv = hb.Conv2d(128, 28, 28, 128, 3, 3, 1, 1, 1, 1, 0, 0)
    bt = hb.encode_im2col(torch.from_numpy(x).cuda(), conv, hb.make_format(8, 1, 32))
    torch.cuda.synchronize()
    want = ref.encode(ref.im2col(x, 3, 3, 1, 1), 1, 32, 8)
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, want.exps)
    np.testing.assert_array_equal(mant, want.mant)


def test_two_pass_conversions_in_a_replayed_graph(hb):
    """The two-pass conversions (table of block maxima cleared by a fill kernel, not a memset) and the convolution
    gather with one exponent per image, captured in a HIP graph and replayed on new inputs in the same buffers, with
    eager work and synchronisation between the replays; every replay must equal the eager conversion."""
    rows, cols = 300, 1100
    x = torch.zeros((rows, cols), device="cuda")
    img = torch.zeros((3, 10, 10, 16), device="cuda")
    conv = hb.Conv2d(3, 10, 10, 16, 3, 3, 1, 1, 1, 1, 0, 0)
    jobs = [(hb.make_format(8, 0, 1), 0), (hb.make_format(8, 0, 0), 1), (hb.make_format(8, 64, 64), 1), (hb.make_format(8, 1, 0, k_slot=24), 1)]
    outs = [hb.alloc(f, rows, cols, ax) for f, ax in jobs]
    wss = [torch.empty(max(hb.encode_workspace(o.desc), 256), dtype=torch.uint8, device="cuda") for o in outs]
    f_img = hb.make_format(8, 100, 0, k_slot=24)
    o_img = hb.alloc(f_img, 300, 144, 1)
    ws_img = torch.empty(max(hb.encode_workspace(o_img.desc), 256), dtype=torch.uint8, device="cuda")
    stream = torch.cuda.Stream()

    def run():
        for (f, ax), o, ws in zip(jobs, outs, wss):
            hb.encode(x, ax, f, out=o, workspace=ws, stream=stream)
        hb.encode_im2col(img, conv, f_img, out=o_img, workspace=ws_img, stream=stream)

    with torch.cuda.stream(stream):
        run()
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            run()
    rng = np.random.default_rng(5)
    for step in range(4):
        print(f"[case] two-pass graph replay {step}", flush=True)
        x.copy_(torch.from_numpy((rng.standard_normal((rows, cols)) * 2.0 ** (3 * step - 4)).astype(np.float32)))
        img.copy_(torch.from_numpy(rng.standard_normal((3, 10, 10, 16)).astype(np.float32) * (step + 1)))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = [(o.mant.clone(), o.exps.clone()) for o in outs + [o_img]]
        eager = [hb.encode(x, ax, f) for f, ax in jobs] + [hb.encode_im2col(img, conv, f_img)]
        torch.cuda.synchronize()
        for (gm, ge), e in zip(got, eager):
            assert torch.equal(gm, e.mant) and torch.equal(ge, e.exps)


def _random_format_case(case):
    rng = np.random.default_rng(7000 + case)
    rows, cols = int(rng.integers(1, 400)), int(rng.integers(1, 1400))
    if rng.random() < 0.3:
        cols = int(rng.integers(1, 350)) * 4                         # aligned widths take the vector paths
    axis = int(rng.integers(0, 2))
    pick = lambda n: int(rng.choice([0, 1, 2, 3, 8, 20, 24, 32, 33, 64, 100, 128, 200, 256, n]))
    br, bc = pick(rows), pick(cols)
    m = int(rng.choice([2, 4, 8, 8, 8, 12, 16]))
    rounding = int(rng.integers(0, 2))
    slot = 0
    kext = (bc if bc and bc < cols else cols) if axis == 1 else (br if br and br < rows else rows)
    whole = kext == (cols if axis == 1 else rows)
    if rng.random() < 0.4:
        divs = [d for d in (4, 8, 12, 20, 24, 32, 50, 64) if d < kext and (whole or kext % d == 0)]
        if divs:
            slot = int(rng.choice(divs))
    return rows, cols, axis, br, bc, m, rounding, slot


@pytest.mark.parametrize("case", random_cases(60))
def test_encode_random_shapes_and_formats(hb, case):
    """Random shapes, block shapes, widths, rounding modes and stored-block lengths: every conversion path (row, column,
    register tile, one wave per row, two passes in either orientation) against the oracle, decode included."""
    rows, cols, axis, br, bc, m, rounding, slot = _random_format_case(case)
    print(f"[case] {case}: shape=({rows},{cols}) axis={axis} block=({br},{bc}) m={m} rounding={rounding} k_slot={slot}", flush=True)
    x = _data((rows, cols), 9000 + case, spread=10)
    fmt = hb.make_format(m, br, bc, rounding, 0xF00D + case, k_slot=slot)
    bt = hb.encode(torch.from_numpy(x).cuda(), axis, fmt)
    torch.cuda.synchronize()
    want = ref.encode(x, br, bc, m, rounding, 0xF00D + case)
    mant, exps = unpack(bt)
    np.testing.assert_array_equal(exps, want.exps)
    np.testing.assert_array_equal(mant, want.mant)
    back = hb.decode(bt)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(back.cpu().numpy(), ref.decode(want))


REGISTER_TILE_CASES = [
    # tiles of at most 32 x 32 with column counts and tile widths that are multiples of 4: the register-tile kernel
    # rows, cols, br, bc, m, rounding
    (100, 100, 24, 24, 8, 0), (130, 72, 24, 24, 8, 1), (97, 1060, 32, 32, 8, 0), (33, 44, 3, 8, 8, 0), (64, 64, 8, 4, 8, 1),
    (260, 200, 17, 20, 12, 0), (50, 96, 24, 12, 16, 0), (75, 132, 32, 28, 16, 1), (1, 8, 24, 24, 8, 0), (500, 36, 9, 32, 12, 1),
]


@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("rows,cols,br,bc,m,rounding", REGISTER_TILE_CASES)
def test_encode_small_tiles_both_orientations(hb, rows, cols, br, bc, m, rounding, axis):
    _check(hb, _data((rows, cols), rows + 17 * cols + axis), axis, br, bc, m, rounding, seed=0x5EED + br)


def test_encode_small_tiles_from_misaligned_source(hb):
    """Leading dimensions and starts that rule out 16-byte loads take the other tile path; same bytes."""
    big = _data((60, 1100), 6)
    g = torch.from_numpy(big).cuda()
    for c0, cols in ((0, 1000), (4, 1024), (3, 1000), (0, 998)):
        view = g[:, c0:c0 + cols]
        for axis in (0, 1):
            _check(hb, big[:, c0:c0 + cols].copy(), axis, 24, 24, 8, 0, src=view)


def test_encode_from_strided_source(hb):
    big = _data((70, 1100), 5)
    g = torch.from_numpy(big).cuda()
    for c0, cols in ((0, 1000), (4, 1024), (3, 999)):            # leading dimension 1100; aligned and misaligned starts
        view = g[:, c0:c0 + cols]
        x = np.ascontiguousarray(big[:, c0:c0 + cols])
        _check(hb, x, 1, 1, 32, 8, 1, seed=77, src=view)
        _check(hb, x, 0, 32, 1, 8, 0, src=view)
        _check(hb, x, 0, 24, 24, 8, 0, src=view)


def test_encode_special_values(hb):
    rng = np.random.default_rng(9)
    x = _data((64, 256), 10)
    x[0, :] = 0.0                                                 # all-zero blocks
    x[1, :32] = -0.0
    x[2, :] = (rng.integers(-50, 50, size=256) * 2.0 ** -149).astype(np.float32)     # subnormal-only blocks
    x[3, :] = (rng.standard_normal(256) * 2.0 ** -126).astype(np.float32)            # around the smallest normal
    x[4, :] = (rng.standard_normal(256) * 2.0 ** 120).astype(np.float32)             # large
    x[5, ::32] = np.nextafter(np.float32(2.0), np.float32(0))                        # maxima just below a power of two
    x[6, ::32] = np.float32(1.9921875)                                               # 255/128: ties at the top for m=8
    x[7, :] = np.float32(3.0e38) * rng.choice([-1, 1], size=256)                     # near FLT_MAX
    x[8, :32] = np.float32(2.0 ** -149)
    x[9, ::2] = np.float32(2.0 ** 100)
    x[9, 1::2] = np.float32(2.0 ** -100)                                             # huge spread inside a block
    for m in (8, 12, 16):
        for rounding in (0, 1):
            _check(hb, x, 1, 1, 32, m, rounding, seed=5)
            _check(hb, x, 0, 32, 1, m, rounding, seed=5)
            _check(hb, x, 1, 8, 64, m, rounding, seed=5)


def test_encode_is_deterministic_and_reuses_buffers(hb):
    x = _data((256, 2048), 21)
    g = torch.from_numpy(x).cuda()
    fmt = hb.make_format(8, 1, 32, hb.STOCHASTIC, 99)
    a = hb.encode(g, 1, fmt)
    m1, e1 = a.mant.clone(), a.exps.clone()
    a.mant.fill_(7)
    a.exps.fill_(7)
    hb.encode(g, 1, fmt, out=a)                                  # same buffers, fully overwritten
    torch.cuda.synchronize()
    assert torch.equal(a.mant, m1) and torch.equal(a.exps, e1)


@pytest.mark.parametrize("m,rounding", [(8, 0), (8, 1), (12, 0), (12, 1)])
def test_config2_full_size_bit_exact(hb, m, rounding):
    """64M log-normal values, blocks of 32 contiguous elements: every mantissa and exponent byte."""
    import synth
    n = 1 << 26
    x = synth.c2_lognormal(n).reshape(1, n)
    print(f"[case] config 2 full size m={m} rounding={rounding}", flush=True)
    fmt = hb.make_format(m, 1, 32, rounding, 20180401)
    g = torch.from_numpy(x).cuda()
    bt = hb.encode(g, 1, fmt)
    back = hb.decode(bt)
    torch.cuda.synchronize()
    want = ref.encode(x, 1, 32, m, rounding, 20180401)
    got_m = bt.mant.cpu().numpy().reshape(-1)
    assert np.array_equal(got_m, want.mant.reshape(-1).astype(got_m.dtype))
    assert np.array_equal(bt.exps.cpu().numpy().reshape(-1), want.exps.reshape(-1))
    assert np.array_equal(back.cpu().numpy(), ref.decode(want))


MULTI_CASES = [
    # rows, cols, [(axis, br, bc, m)], rounding
    (100, 120, [(1, 1, 24, 8), (0, 24, 1, 8)], 0),                       # an activation: along its rows and down its columns
    (4100, 48, [(1, 1, 24, 8), (0, 24, 1, 8)], 1),
    (130, 264, [(0, 24, 24, 8), (1, 24, 24, 8)], 0),                     # a weight matrix: both orientations of its tiles
    (96, 96, [(1, 24, 24, 16), (0, 24, 24, 8), (1, 24, 24, 8)], 0),      # wide copy + two narrow copies
    (70, 200, [(1, 1, 32, 12), (0, 16, 1, 8), (1, 16, 32, 8)], 1),       # rows, columns and whole tiles of a 16 x 32 tile
    (64, 100, [(1, 1, 24, 8), (0, 24, 1, 8)], 0),                        # 100 columns: not a whole number of blocks
    (50, 90, [(1, 1, 24, 8), (0, 24, 1, 8)], 0),                         # 90 columns: not a multiple of 4 -> one launch per output
    (80, 128, [(1, 1, 64, 8), (0, 64, 1, 8)], 0),                        # blocks longer than 32 -> one launch per output
]


@pytest.mark.parametrize("rows,cols,outs,rounding", MULTI_CASES)
def test_encode_multi_matches_single_encodes(hb, rows, cols, outs, rounding):
    x = _data((rows, cols), rows * 5 + cols)
    print(f"[case] shape={x.shape} outs={outs} rounding={rounding}", flush=True)
    g = torch.from_numpy(x).cuda()
    fmts = [hb.make_format(m, br, bc, rounding, 100 + i) for i, (axis, br, bc, m) in enumerate(outs)]
    tensors = [hb.alloc(f, rows, cols, axis) for f, (axis, _, _, _) in zip(fmts, outs)]
    for t in tensors:                                  # poison the outputs: padding must be rewritten too
        t.mant.fill_(0x55)
        t.exps.fill_(0x55)
    hb.encode_multi(g, tensors)
    torch.cuda.synchronize()
    for i, (t, (axis, br, bc, m)) in enumerate(zip(tensors, outs)):
        want = ref.encode(x, br, bc, m, rounding, 100 + i)
        mant, exps = unpack(t)
        np.testing.assert_array_equal(exps, want.exps)
        np.testing.assert_array_equal(mant, want.mant)


@pytest.mark.parametrize("m,rounding", [(8, 0), (12, 0), (8, 1), (13, 1)])
@pytest.mark.parametrize("rows,cols,br,bc,slot", [
    (70, 17, 0, 1, 0),             # one exponent per column, one strip and a column
    (65, 16, 0, 1, 0),             # the shortest block that the column kernel leaves over
    (5120, 36, 0, 1, 0),           # the longest strip with aligned rows, and the same from unaligned ones
    (5121, 36, 0, 1, 0),           # one element more: two passes from aligned rows
    (10241, 33, 0, 1, 0),          # two passes from unaligned rows
    (1000, 333, 70, 3, 0),         # tiles across 3 columns, 14 whole blocks and a short one
    (777, 50, 200, 64, 0),         # the widest tile
    (129, 63, 128, 48, 0),         # a block of one element behind a whole one
    (1396, 150, 216, 24, 24),      # filter tiles: stored blocks of 24 that repeat an exponent over 9 of them
    (2000, 1100, 72, 2, 24),       # enough blocks for strips of twice the width
    (4200, 515, 128, 24, 0),       # the same with tiles of 24 columns
    (90, 5, 0, 0, 30),             # one exponent for the matrix, stored blocks of 30
])
def test_long_blocks_down_the_rows(hb, rows, cols, br, bc, slot, m, rounding):
    """Long exponent blocks down the source rows against the oracle, bit for bit: the strip kernel at the edges of its strips,
    blocks and rule, and the two-pass conversion next to it.  Some columns are zero, some blocks tiny."""
    print(f"[case] {rows}x{cols} blocks {br}x{bc} slot {slot} m={m} rounding={rounding}", flush=True)
    rng = np.random.default_rng(rows + cols)
    X = (rng.standard_normal((rows, cols)) * np.exp2(rng.integers(-20, 21, size=(rows, cols)))).astype(np.float32)
    X[:, cols // 2] = 0.0
    X[: rows // 3, cols // 3] *= np.float32(2.0 ** -100)
    pad = torch.full((rows, cols + 3), 3.0e38, device="cuda")
    pad[:, :cols] = torch.from_numpy(X).cuda()
    for src in (torch.from_numpy(X).cuda(), pad[:, :cols]):          # rows back to back, and 3 elements apart
        fmt = hb.make_format(m, br, bc, rounding, 1234567, k_slot=slot)
        out = hb.alloc(fmt, rows, cols, 0)
        out.mant.fill_(85)
        out.exps.fill_(85)
        hb.encode(src, 0, fmt, out=out)
        torch.cuda.synchronize()
        want = ref.encode(X, br, bc, m, rounding, 1234567)
        mant, exps = unpack(out)
        np.testing.assert_array_equal(mant, want.mant)
        np.testing.assert_array_equal(exps, want.exps)


@pytest.mark.parametrize("rows,cols,blk,m", [(700, 6000, 24, 8), (256, 256, 32, 8), (1000, 70, 16, 12), (129, 1000, 64, 8), (8200, 1024, 32, 8)])
def test_column_conversion_of_few_and_many_workgroups(hb, rows, cols, blk, m):
    """The column kernel with whole, halved and quartered shares per workgroup, against the oracle bit for bit."""
    print(f"[case] {rows}x{cols} blocks {blk}x1 m={m}", flush=True)
    X = np.random.default_rng(rows).standard_normal((rows, cols)).astype(np.float32)
    out = hb.encode(torch.from_numpy(X).cuda(), 0, hb.make_format(m, blk, 1))
    torch.cuda.synchronize()
    want = ref.encode(X, blk, 1, m)
    mant, exps = unpack(out)
    np.testing.assert_array_equal(mant, want.mant)
    np.testing.assert_array_equal(exps, want.exps)


@pytest.mark.parametrize("rows,cols,bc,rounding,where", [
    (500, 300, 1, 0, "strip held"), (4500, 2999, 1, 0, "strip held"), (2560, 200, 1, 0, "strip held"), (5120, 200, 1, 0, "two passes"),
    (1280, 64, 1, 1, "strip held"), (2560, 200, 1, 1, "two passes"), (5120, 1000, 1, 1, "two passes"), (4096, 4096, 1, 1, "strip held"),
    (2000, 38, 1, 1, "strip held"), (5000, 33, 1, 1, "two passes"), (10000, 501, 1, 0, "two passes"), (10000, 3001, 1, 0, "strip"),
    (8191, 6001, 1, 1, "two passes"), (861, 559, 64, 1, "strip held"),
    (5000, 1, 1, 0, "strip held"), (7261, 3, 1, 1, "strip held"), (11040, 4, 4, 1, "two passes")])
def test_where_long_blocks_down_the_rows_are_converted(hb, rows, cols, bc, rounding, where):
    """One exponent per `bc` columns: strips, held in registers or read twice, or two passes where few strips would be too long; each
    case on the side that was measured faster."""
    x = torch.randn((rows, cols), device="cuda")
    fmt = hb.make_format(8, 0, bc, rounding, 3)
    out = hb.alloc(fmt, rows, cols, 0)
    names = launched_kernels(lambda: hb.encode(x, 0, fmt, out=out))
    strips = [n.split("<")[0] for n in names if n.startswith("enc_strip_")]
    assert strips == {"strip": ["enc_strip_kernel"], "strip held": ["enc_strip_held_kernel"], "two passes": []}[where], names


@pytest.mark.parametrize("rows,cols,br,bc,pieces", [(270, 30, 256, 1, 1), (512, 300, 0, 1, 1), (520, 300, 0, 1, 3), (1536, 300, 0, 1, 3), (1540, 300, 0, 1, 5),
                                                    (2600, 1300, 0, 1, 5), (2100, 4, 0, 8, 3)])
@pytest.mark.parametrize("rounding", [0, 1])
def test_held_strips_run_no_more_code_than_they_have_pieces(hb, rows, cols, br, bc, pieces, rounding):
    """A short strip takes the instance that is unrolled for its own number of pieces, not the one for five."""
    x = torch.randn((rows, cols), device="cuda")
    fmt = hb.make_format(8, br, bc, rounding, 3)
    out = hb.alloc(fmt, rows, cols, 0)
    names = launched_kernels(lambda: hb.encode(x, 0, fmt, out=out))
    assert names == [f"enc_strip_held_kernel<false, {rounding}, {pieces}>"], names


@pytest.mark.parametrize("rows,cols,br,held", [(5120, 1035, 0, True), (5121, 1035, 0, False), (1024, 1024, 128, True), (1024, 1040, 128, False),
                                               (4096, 4096, 240, True), (4096, 4096, 128, False), (4096, 4096, 512, True)])
def test_which_strips_are_held_in_registers(hb, rows, cols, br, held):
    """What fits the registers; blocks that give half of the threads nothing only in at most 512 workgroups."""
    x = torch.randn((rows, cols), device="cuda")
    fmt = hb.make_format(8, br, 1)
    out = hb.alloc(fmt, rows, cols, 0)
    names = launched_kernels(lambda: hb.encode(x, 0, fmt, out=out))
    assert len(names) == 1 and names[0].startswith("enc_strip_held_kernel<" if held else "enc_strip_kernel<"), names


@pytest.mark.parametrize("m,rounding", [(8, 0), (12, 1)])
@pytest.mark.parametrize("rows,cols", [(33, 4096), (33, 4104), (9, 5119), (9, 5121), (7, 6144), (7, 6150), (5, 8192)])
def test_rows_held_by_a_wave(hb, rows, cols, m, rounding):
    """One exponent per row at the edges of what a wave's register budgets (8, 10, 12 and 16 chunks per lane) hold."""
    rng = np.random.default_rng(rows + cols)
    X = (rng.standard_normal((rows, cols)) * np.exp2(rng.integers(-20, 21, size=(rows, cols)))).astype(np.float32)
    X[0], X[1, -1], X[2] = 0.0, 3e38, 1e-42
    src = torch.from_numpy(X).cuda()
    fmt = hb.make_format(m, 1, 0, rounding, 99)
    out = hb.alloc(fmt, rows, cols, 1)
    out.mant.fill_(85)
    out.exps.fill_(85)
    hb.encode(src, 1, fmt, out=out)
    want = ref.encode(X, 1, 0, m, rounding, 99)
    mant, exps = unpack(out)
    np.testing.assert_array_equal(mant, want.mant)
    np.testing.assert_array_equal(exps, want.exps)


@pytest.mark.parametrize("m,rounding", [(8, 0), (12, 1)])
@pytest.mark.parametrize("rows,cols,br,bc", [(1023, 1035, 0, 1), (1030, 1035, 0, 1), (2560, 1035, 0, 1), (2570, 1035, 0, 1), (5120, 1024, 0, 1), (5130, 1035, 0, 1),
                                             (4200, 1100, 2048, 3), (2900, 1300, 0, 40), (3000, 13, 0, 1), (500, 140, 0, 1), (512, 70, 0, 1), (513, 70, 0, 1),
                                             (1530, 100, 0, 1), (1540, 100, 0, 1), (270, 30, 256, 1), (671, 281, 128, 24), (2058, 4, 0, 8)])
def test_strips_held_in_registers(hb, rows, cols, br, bc, m, rounding):
    """Strips at the edges of what 512 and 1024 threads hold (one, three and five pieces: 512, 1536 and 2560 values of 16 columns; 5120)
    and past it, where they are read twice; several exponent blocks down the rows, tiles of columns.  Denormal, non-finite and empty blocks among the values."""
    rng = np.random.default_rng(rows + cols)
    X = (rng.standard_normal((rows, cols)) * np.exp2(rng.integers(-20, 21, size=(1, cols)))).astype(np.float32)
    X[:, 0], X[:, 5 % cols] = 0.0, 1e-42
    X[rows - 1, 7 % cols] = 3e38
    src = torch.from_numpy(X).cuda()
    fmt = hb.make_format(m, br, bc, rounding, 99)
    out = hb.alloc(fmt, rows, cols, 0)
    out.mant.fill_(85)
    out.exps.fill_(85)
    hb.encode(src, 0, fmt, out=out)
    want = ref.encode(X, br, bc, m, rounding, 99)
    mant, exps = unpack(out)
    np.testing.assert_array_equal(mant, want.mant)
    np.testing.assert_array_equal(exps, want.exps)


@pytest.mark.parametrize("m,rounding", [(8, 0), (12, 1)])
@pytest.mark.parametrize("rows,cols,br,bc,slot", [(5000, 1, 0, 1, 0), (300, 3, 0, 1, 0), (700, 7, 0, 2, 0), (513, 5, 200, 3, 0), (640, 15, 128, 4, 0),
                                                  (1000, 9, 216, 9, 24), (400, 15, 0, 15, 0), (129, 2, 128, 1, 0)])
def test_strips_narrower_than_sixteen_columns(hb, rows, cols, br, bc, slot, m, rounding):
    """A strip has no more columns than the matrix: against the oracle bit for bit."""
    rng = np.random.default_rng(rows + cols)
    X = (rng.standard_normal((rows, cols)) * np.exp2(rng.integers(-20, 21, size=(rows, cols)))).astype(np.float32)
    src = torch.from_numpy(X).cuda()
    fmt = hb.make_format(m, br, bc, rounding, 99, k_slot=slot)
    out = hb.alloc(fmt, rows, cols, 0)
    out.mant.fill_(85)
    out.exps.fill_(85)
    assert any(n.startswith("enc_strip_") for n in launched_kernels(lambda: hb.encode(src, 0, fmt, out=out)))
    want = ref.encode(X, br, bc, m, rounding, 99)
    mant, exps = unpack(out)
    np.testing.assert_array_equal(mant, want.mant)
    np.testing.assert_array_equal(exps, want.exps)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, np.finfo(np.float32).max])
@pytest.mark.parametrize("rows,cols,br,bc,slot", [(500, 33, 0, 1, 0), (700, 40, 128, 1, 0), (432, 50, 216, 24, 24), (6001, 40, 0, 1, 0)])
def test_one_value_out_of_range_spoils_its_own_block_only(hb, rows, cols, br, bc, slot, bad):
    """Inputs have to be finite and nothing traps the others: an infinity or NaN leaves its own exponent block unspecified, every
    other block is as if it were not there (strips, and two passes for the last size)."""
    rng = np.random.default_rng(rows)
    X = rng.standard_normal((rows, cols)).astype(np.float32)
    want = ref.encode(X, br, bc, 8)
    r, c = rows // 2, cols // 2
    X[r, c] = bad
    fmt = hb.make_format(8, br, bc, k_slot=slot)
    mant, exps = unpack(hb.encode(torch.from_numpy(X).cuda(), 0, fmt))
    kr, kc = br or rows, bc or cols
    keep = np.ones((rows, cols), dtype=bool)
    keep[r // kr * kr:(r // kr + 1) * kr, c // kc * kc:(c // kc + 1) * kc] = False
    np.testing.assert_array_equal(mant[keep], want.mant[keep])
    other = np.ones(exps.shape, dtype=bool)
    other[r // kr, c // kc] = False
    np.testing.assert_array_equal(exps[other], want.exps[other])
    if np.isfinite(bad):                                       # the largest finite value is an ordinary one
        full = ref.encode(X, br, bc, 8)
        np.testing.assert_array_equal(mant, full.mant)
        np.testing.assert_array_equal(exps, full.exps)


@pytest.mark.parametrize("rows,cols,pad,aligned16", [(64, 256, 0, False), (4095, 4096, 0, False), (4096, 4096, 0, True), (3000, 5600, 0, True), (3001, 5599, 0, False),
                                                     (3000, 5600, 2, False), (4096, 4096, 4, True)])
@pytest.mark.parametrize("rounding,unroll", [(0, 4), (1, 2)])
def test_which_loads_rows_are_read_with(hb, rows, cols, pad, aligned16, rounding, unroll):
    """Rows that start on 16 bytes and hold at least 16 Mi values have the instance that reads nothing else to themselves; the bytes are
    those of the oracle either way."""
    x = torch.randn((rows, cols + pad), device="cuda", generator=torch.Generator(device="cuda").manual_seed(cols))[:, :cols]
    fmt = hb.make_format(8, 1, 24, rounding, 5)
    out = hb.alloc(fmt, rows, cols, 1)
    names = launched_kernels(lambda: hb.encode(x, 1, fmt, out=out))
    assert names == [f"enc_row_kernel<4, false, {rounding}, {unroll}, false, {str(not aligned16).lower()}>"], names
    want = ref.encode(x.cpu().numpy(), 1, 24, 8, rounding, 5)
    mant, exps = unpack(out)
    np.testing.assert_array_equal(mant, want.mant)
    np.testing.assert_array_equal(exps, want.exps)
