"""Products of FP32 matrices that convert their operands inside the product (small sizes), against the conversions and the product
as calls of their own: the same bits, at the edges of the tiles, of the contraction and of the rule."""
import pytest
import torch

from tests.util import launched_kernels

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_1804_01526_amd import hbfp
    return hbfp


def _operands(hb, M, N, K, block, pad, trans_a, trans_b):
    gen = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)

    def source(rows, cols):
        x = torch.randn((rows, cols + pad), generator=gen, device="cuda")
        x *= torch.exp2(torch.randint(-30, 30, (rows, 1), generator=gen, device="cuda").float())
        x = x[:, :cols]
        if rows * cols > 64:                                     # denormal and non-finite blocks beside ordinary ones
            x[0, 0], x[-1, -1], x[rows // 2, 0] = 1e-42, float("inf"), float("nan")
        return x

    A, B = source(*((K, M) if trans_a else (M, K))), source(*((N, K) if trans_b else (K, N)))
    fa = hb.make_format(8, *((block, 1) if trans_a else (1, block)))
    fb = hb.make_format(6, *((1, block) if trans_b else (block, 1)))
    return A, B, fa, fb


@pytest.mark.parametrize("M,N,K,block,pad,inside", [(1, 1, 1, 32, 0, "tt"), (33, 31, 255, 32, 0, "tt"), (64, 97, 256, 32, 1, "tt"),
                                                    (32, 32, 257, 32, 3, "tt"), (100, 130, 512, 32, 0, "tt"), (45, 70, 380, 24, 4, "tf"),
                                                    (511, 65, 511, 32, 0, "tt"), (40, 64, 513, 32, 3, "ff"),
                                                    (5, 8192, 61, 17, 3, "tt"), (5, 8193, 61, 32, 0, "ff"), (84, 48, 192, 24, 0, "tt"),
                                                    (33, 65, 250, 24, 1, "tf"), (26, 40, 211, 16, 0, "tf"), (40, 33, 127, 19, 2, "tt"), (31, 33, 93, 8, 0, "tf")])
@pytest.mark.parametrize("trans_a,trans_b", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_products_that_convert_their_operands(hb, M, N, K, block, pad, inside, trans_a, trans_b):
    """`inside`: whether one launch does it (t), for any direction of the operands but, and for, both along the rows."""
    print(f"[case] gemm_f32 {M}x{N}x{K} block {block} pad {pad} {trans_a}{trans_b}", flush=True)
    A, B, fa, fb = _operands(hb, M, N, K, block, pad, trans_a, trans_b)
    got = hb.gemm_f32(trans_a, trans_b, A, B, fa, fb)
    want = hb.gemm(hb.encode(A, 0 if trans_a else 1, fa), hb.encode(B, 1 if trans_b else 0, fb))
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    names = launched_kernels(lambda: hb.gemm_f32(trans_a, trans_b, A, B, fa, fb))
    both_rows = trans_a == 0 and trans_b == 1
    assert (len(names) == 1 and names[0].startswith("gemm_convert_kernel")) == (inside[1 if both_rows else 0] == "t"), names


@pytest.mark.parametrize("M,N,K,block,kernel", [(64, 64, 256, 32, "<1, false>"), (64, 64, 96, 24, "<1, false>"), (84, 48, 192, 24, "<1, true>"),
                                                (134, 829, 248, 24, "<2, true>"), (26, 40, 208, 16, "<2, true>"), (64, 64, 100, 8, "<2, false>"),
                                                (64, 64, 500, 32, "<2, false>")])
def test_where_short_blocks_are_read_by_quadruples(hb, M, N, K, block, kernel):
    A, B, fa, fb = _operands(hb, M, N, K, block, 0, 0, 0)
    names = launched_kernels(lambda: hb.gemm_f32(0, 0, A, B, fa, fb))
    assert names == ["gemm_convert_kernel" + kernel], names


@pytest.mark.parametrize("M,N,K,ta,tb", [(84, 48, 192, 0, 1), (134, 829, 248, 0, 0), (6, 58, 362, 1, 1)])
def test_converting_inside_is_no_slower_than_converting_first(hb, M, N, K, ta, tb):
    """Blocks of 24, replayed from graphs: one launch against one of the two conversions and the product, a tenth of margin
    (value by value 84 x 48 x 192 was a fifth behind even the two launches)."""
    A, B, fa, fb = _operands(hb, M, N, K, 24, 0, ta, tb)
    C, ws = torch.empty((M, N), device="cuda"), torch.empty(hb.gemm_f32_workspace(ta, tb, M, N, K, fa, fb), dtype=torch.uint8, device="cuda")
    a, b = hb.encode(A, 1 - ta, fa), hb.encode(B, tb, fb)

    def separate():
        hb.encode(A, 1 - ta, fa, out=a)
        hb.gemm(a, b, out=C, workspace=ws)

    def fastest(call):
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

    first, inside = fastest(separate), fastest(lambda: hb.gemm_f32(ta, tb, A, B, fa, fb, out=C, workspace=ws))
    print(f"[case] {M}x{N}x{K}: one conversion and the product {first:.1f} us, one launch {inside:.1f} us", flush=True)
    assert inside <= first * 1.1


@pytest.mark.parametrize("over", ["A", "B"])
def test_converting_product_over_its_own_operand(hb, over):
    """A square product stored over a source: the operands are converted whole before the first store."""
    A, B, fa, fb = _operands(hb, 160, 160, 160, 32, 0, 0, 0)
    want = hb.gemm_f32(0, 0, A, B, fa, fb)
    out = A if over == "A" else B
    hb.gemm_f32(0, 0, A, B, fa, fb, out=out)
    assert torch.equal(out.view(torch.int32), want.view(torch.int32))
