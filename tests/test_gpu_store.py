"""Where the product kernels store C: whole tiles, edges of one row or column more or less, a row pitch, and C += .

The inputs are integers, scaled by a power of two per row and per column, whose blocks all hold a 1 in the top bit: every sum is exact
in FP32, C must equal the FP64 product of the operands, and an exponent taken from another row or column shows.  The bytes of the
buffer around C must stay as they were.
"""
import pytest
import torch

from tests.util import launched_kernels

pytestmark = pytest.mark.gpu

INT8, SCALED, WIDE, FP16, BF16, F16P = 1, 2, 3, 4, 5, 6


def _operands(M, K, N, bits, block):
    from paper_1804_01526_amd import hbfp
    g = torch.Generator(device="cuda").manual_seed(M * 1009 + N)
    top = 2 ** (bits - 1) - 1
    A = torch.randint(-3, 4, (M, K), device="cuda", generator=g).float()
    B = torch.randint(-3, 4, (K, N), device="cuda", generator=g).float()
    A[:, ::block or K] = top
    B[::block or K, :] = top
    A *= 2.0 ** torch.randint(-3, 4, (M, 1), device="cuda", generator=g)
    B *= 2.0 ** torch.randint(-3, 4, (1, N), device="cuda", generator=g)
    return (hbfp.encode(A, 1, hbfp.make_format(bits, 1, block, hbfp.RNE)), hbfp.encode(B, 0, hbfp.make_format(bits, block, 1, hbfp.RNE)),
            A.double() @ B.double())


@pytest.mark.parametrize("beta", [0.0, 1.0])
@pytest.mark.parametrize("kernel,bits,block,edge", [(INT8, 8, 32, 128), (INT8, 8, 0, 128), (BF16, 8, 32, 256), (BF16, 8, 24, 128), (F16P, 12, 64, 256),
                                                    (FP16, 12, 64, 128), (SCALED, 4, 32, 256), (WIDE, 8, 0, 256)])
@pytest.mark.parametrize("dm,dn", [(0, 0), (1, -1), (-1, 33), (-31, 0), (0, 1)])
def test_edges_pitch_and_accumulation(kernel, bits, block, edge, dm, dn, beta):
    from paper_1804_01526_amd import hbfp
    M, N, K, pad = edge + dm, 2 * edge + dn, 192, 5
    print(f"[store] kernel={kernel} bits={bits} block={block} {M}x{N} beta={beta}", flush=True)
    a, b, want = _operands(M, K, N, bits, block)
    buf = torch.full((M + 2, N + pad), 7.0, device="cuda")
    C = buf[1:M + 1, 2:N + 2]
    if beta:
        C.copy_(torch.arange(N, device="cuda").float().expand(M, N))
        want = (want + torch.arange(N, device="cuda").double()).float().double()
    hbfp.gemm(a, b, out=C, beta=beta, kernel=kernel)
    assert torch.equal(C.double(), want)
    buf[1:M + 1, 2:N + 2] = 7.0
    assert bool((buf == 7.0).all())


# Large outputs whose rows are not whole lines leave by ordinary stores, others past the caches: rows off 32 bytes from 6 Mi outputs on,
# rows off 128 from 10 Mi on; the base of C counts like its pitch; with one exponent per row up to 1024 of k
@pytest.mark.parametrize("kernel,bits,block,K", [(BF16, 8, 24, 192), (F16P, 12, 64, 192), (SCALED, 4, 32, 192), (WIDE, 8, 0, 192), (WIDE, 8, 0, 1100),
                                                 (INT8, 12, 128, 192), (INT8, 12, 64, 192)])
@pytest.mark.parametrize("M,N,pad,at,stream", [(2419, 2601, 0, 0, False), (2420, 2600, 1, 0, False), (2432, 2592, 0, 1, False), (2430, 2600, 0, 0, True),
                                               (2417, 2601, 0, 0, True), (2560, 2560, 32, 0, True), (2600, 4040, 0, 0, False)])
def test_how_large_outputs_leave(kernel, bits, block, K, M, N, pad, at, stream):
    from paper_1804_01526_amd import hbfp
    print(f"[store] kernel={kernel} bits={bits} block={block} {M}x{N}x{K} pitch {N + pad}", flush=True)
    stream = stream or (kernel == WIDE and K > 1024)
    a, b, want = _operands(M, K, N, bits, block)
    buf = torch.full((M * (N + pad) + 32,), 7.0, device="cuda")
    C = buf[at:at + M * (N + pad)].view(M, N + pad)[:, :N]
    names = launched_kernels(lambda: hbfp.gemm(a, b, out=C, kernel=kernel))
    assert torch.equal(C.double(), want)
    C.fill_(7.0)
    assert bool((buf == 7.0).all())
    product = [n for n in names if n.startswith("gemm_")][0]
    assert product.endswith(f"{str(stream).lower()}>"), names


def _fastest(call):
    """us of a call among others, replayed from a graph"""
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(20):
            call()
    times = []
    for _ in range(10):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        graph.replay()
        t1.record()
        torch.cuda.synchronize()
        times.append(t0.elapsed_time(t1) * 50)
    return min(times)


@pytest.mark.parametrize("M,K,N", [(4995, 104, 3043), (4037, 55, 4663)])
def test_ragged_rows_are_not_far_behind_whole_lines(M, K, N):
    """A large product whose rows end inside cache lines against the same one with a pitch of whole lines: streaming stores took it to
    1.8 times, ordinary ones leave it within a third."""
    from paper_1804_01526_amd import hbfp
    a = hbfp.encode(torch.randn((M, K), device="cuda"), 1, hbfp.make_format(8, 1, 24))
    b = hbfp.encode(torch.randn((K, N), device="cuda"), 0, hbfp.make_format(8, 24, 1))
    pa, pb = hbfp.pack(a), hbfp.pack(b)

    whole, own = torch.empty((M, (N + 31) // 32 * 32), device="cuda")[:, :N], torch.empty((M, N), device="cuda")
    lines = _fastest(lambda: hbfp.gemm_packed(a, pa, b, pb, out=whole))
    ragged = _fastest(lambda: hbfp.gemm_packed(a, pa, b, pb, out=own))
    print(f"[store] {M}x{K}x{N}: rows of whole lines {lines:.1f} us, ragged {ragged:.1f} us", flush=True)
    assert ragged <= lines * 4 / 3


@pytest.mark.parametrize("M,K,N", [(4092, 78, 3748), (1000, 512, 1000)])
def test_factors_of_rows_and_columns_cost_little(M, K, N):
    """FP16 planes against bf16 planes of the same size: the same matrix instructions and bytes, and a factor per row and column before
    the stores (applied as part of every store they took half as long again)."""
    from paper_1804_01526_amd import hbfp
    out, times = torch.empty((M, N), device="cuda"), []
    for bits in (8, 12):
        a = hbfp.encode(torch.randn((M, K), device="cuda"), 1, hbfp.make_format(bits, 1, 32))
        b = hbfp.encode(torch.randn((K, N), device="cuda"), 0, hbfp.make_format(bits, 32, 1))
        pa, pb = hbfp.pack(a), hbfp.pack(b)
        times.append(_fastest(lambda: hbfp.gemm_packed(a, pa, b, pb, out=out)))
    print(f"[store] {M}x{K}x{N}: bf16 planes {times[0]:.1f} us, FP16 planes {times[1]:.1f} us", flush=True)
    assert times[1] <= times[0] * 4 / 3


@pytest.mark.parametrize("M,N", [(128, 128), (127, 130), (64, 257)])
def test_slices_of_a_split_product(M, N):
    from paper_1804_01526_amd import hbfp
    a, b, want = _operands(M, 16384, N, 8, 32)
    buf = torch.full((M + 1, N + 3), 7.0, device="cuda")
    hbfp.gemm(a, b, out=buf[:M, 1:N + 1], kernel=INT8)
    assert torch.equal(buf[:M, 1:N + 1].double(), want.float().double())
    buf[:M, 1:N + 1] = 7.0
    assert bool((buf == 7.0).all())


# one exponent per row and column: tiles of 128 (2; alone, split along k over 2 .. 7 and over 8 and more ranges), 192 (3) and 256 (4),
# those with 4 stages and with so many that every buffer of the ring is filled again
@pytest.mark.parametrize("M,K,N,tile,splits", [(200, 1000, 300, 2, 1), (1, 130, 1, 2, 1), (128, 128, 129, 2, 1), (300, 4100, 520, 2, 7), (640, 3000, 641, 2, 4),
                                               (300, 4000, 260, 2, 8), (130, 20000, 70, 2, 32), (65, 40001, 64, 2, 64), (3001, 129, 2999, 3, 1),
                                               (2900, 1000, 2901, 3, 1), (4096, 129, 4095, 4, 1), (3700, 1100, 3651, 4, 1)])
@pytest.mark.parametrize("beta", [0.0, 1.0])
def test_one_exponent_per_row(M, K, N, tile, splits, beta):
    from paper_1804_01526_amd import hbfp
    print(f"[one exponent] {M}x{K}x{N} beta={beta}", flush=True)
    a, b, want = _operands(M, K, N, 8, 0)
    C = torch.full((M, N + 3), 5.0, device="cuda")
    hbfp.gemm(a, b, out=C[:, :N], beta=beta)
    assert torch.equal(C[:, :N], (want + (5.0 if beta else 0.0)).float())
    assert bool((C[:, N:] == 5.0).all())
    names = launched_kernels(lambda: hbfp.gemm(a, b, out=C[:, :N], beta=beta))
    assert names[0].startswith(f"gemm_i8_wide_kernel<{tile}, ") and names[1:] == (["wide_sum_kernel"] if splits > 1 else []), names
    if splits > 1:
        assert hbfp.gemm_select_workspace(a.desc, b.desc, 0) == splits * 4 * M * N


# 12-bit operands as FP16 planes: a row's factor comes from its largest exponent byte, wherever that lies (16 lanes read four
# blocks each, the last word of a row may hold 1 to 4 of them); the other kernel prepares planes and words in one launch
@pytest.mark.parametrize("kernel", [F16P, FP16])
@pytest.mark.parametrize("blocks,at", [(1, 0), (5, 4), (63, 62), (64, 0), (257, 256), (301, 299)])
def test_largest_exponent_of_a_row(kernel, blocks, at):
    from paper_1804_01526_amd import hbfp
    M, N, K = 33, 40, 64 * blocks
    g = torch.Generator(device="cuda").manual_seed(blocks)
    A = torch.randint(-3, 4, (M, K), device="cuda", generator=g).float()
    B = torch.randint(-3, 4, (K, N), device="cuda", generator=g).float()
    A[:, ::64] = 2047.0
    B[::64, :] = 2047.0
    A[:, 64 * at:64 * at + 64] *= 1024.0
    A[::2] = A[::2].flip(1)
    a, b = hbfp.encode(A, 1, hbfp.make_format(12, 1, 64, hbfp.RNE)), hbfp.encode(B, 0, hbfp.make_format(12, 64, 1, hbfp.RNE))
    want = hbfp.decode(a).double() @ hbfp.decode(b).double()
    C = hbfp.gemm(a, b, kernel=kernel).double()
    # FP32 sums of exact products, one rounding per product at the worst
    bound = 2.0 ** -24 * (K + 2) * (hbfp.decode(a).double().abs() @ hbfp.decode(b).double().abs())
    assert bool(((C - want).abs() <= bound).all())


# a product of one exponent per row that is split along k: a workspace without its slices is as good as ever, the product then runs
# unsplit with the same bits; less than the words is refused
@pytest.mark.parametrize("call", ["gemm", "int8", "wide", "partials", "batch", "bfp", "f32", "packed", "packed batch"])
def test_split_product_without_room_for_its_slices(call):
    from paper_1804_01526_amd import hbfp
    M, K, N = 130, 20000, 70
    mixed = call.startswith("packed")
    g = torch.Generator(device="cuda").manual_seed(1)
    A = torch.randn((M, K), device="cuda", generator=g) * 2.0 ** torch.randint(-4, 5, (M, 1), device="cuda", generator=g)
    B = torch.randn((K, N), device="cuda", generator=g) * 2.0 ** torch.randint(-4, 5, (1, N), device="cuda", generator=g)
    fa, fb, fo = hbfp.make_format(4 if mixed else 8, 1, 0), hbfp.make_format(8, 0, 1), hbfp.make_format(8, 1, 32)
    a, b = hbfp.encode(A, 1, fa), hbfp.encode(B, 0, fb)
    slices = (hbfp.gemm_select_workspace(a.desc, b.desc, INT8) + 255) // 256 * 256
    words = 4 * a.desc.exp_ld * (256 + 128)
    assert slices > words and words % 256 == 0
    C, C2 = torch.empty((M, N), device="cuda"), torch.empty((M, N), device="cuda")
    if call in ("gemm", "int8", "wide"):
        kernel = {"gemm": 0, "int8": INT8, "wide": WIDE}[call]
        full, run = hbfp.gemm_select_workspace(a.desc, b.desc, kernel), lambda ws: hbfp.gemm(a, b, out=C, kernel=kernel, workspace=ws)
    elif call == "partials":
        full, run = slices, lambda ws: hbfp.gemm_partials(a, b, workspace=ws)
    elif call == "batch":
        full, run = 2 * slices, lambda ws: hbfp.gemm_batch([(a, b), (a, b)], [C, C2], kernel=INT8, workspace=ws)[1]
    elif call == "bfp":
        out = hbfp.alloc(fo, M, N, 1)
        full, run = hbfp.gemm_bfp_workspace(a.desc, b.desc, out.desc, 0), lambda ws: hbfp.gemm_bfp(a, b, fo, 1, out=out, workspace=ws).mant
    elif call == "f32":
        full = hbfp.gemm_f32_workspace(0, 0, M, N, K, fa, fb)
        run = lambda ws: hbfp.gemm_f32(0, 0, A, B, fa, fb, out=C, workspace=ws)
    elif call == "packed":
        full, run = hbfp.gemm_packed_workspace(a.desc, b.desc), lambda ws: hbfp.gemm_packed(a, hbfp.pack(a), b, hbfp.pack(b), out=C, workspace=ws)
    else:
        pa, pb = hbfp.pack(a), hbfp.pack(b)
        full, run = 2 * slices, lambda ws: hbfp.gemm_packed_batch([(a, pa, b, pb)] * 2, [C, C2], workspace=ws)[1]
    full = (full + 255) // 256 * 256
    least = full - (slices - words) * (2 if "batch" in call else 1)
    print(f"[store] {call}: {least} of {full} bytes", flush=True)
    want = run(torch.empty(full, dtype=torch.uint8, device="cuda")).clone()
    C.fill_(-1.0), C2.fill_(-1.0)
    guarded = torch.full((least + 4096,), 85, dtype=torch.uint8, device="cuda")
    assert torch.equal(run(guarded[:least]), want)
    assert bool((guarded[least:] == 85).all())
    with pytest.raises(hbfp.HbfpError):
        run(guarded[:least - 256])

