// Small BFP matrix products: inference on a few rows, layers of a few hundred columns (Eq. (2) of Sec. 4, blocks stored as 32,
// 8-bit class).  What counts is latency: the 128 x 128-tile kernels behind a launch for scale words, and before one that sums
// slices where few tiles split the contraction, start at 9 us.  Here a workgroup of 8 waves owns 32 columns and 32 or 64 rows
// of C; its waves deal the contraction out among themselves in groups of four blocks (128 bytes of a row), load operands
// and exponent bytes straight into registers, a group ahead, and meet in LDS: one launch, no workspace touched.  Per block the
// arithmetic is that of the int8 kernels: an integer sum started from the row constants, one subtraction and one
// multiply-add.  The result leaves as FP32 or, with ReLU if asked for, as an encoded operand.
// 256^3: 3.3 us (the tile kernel 7.8, 9.8 with a launch for its scale words); 16 x 4096 x 4096: 11.8 us (14.7 and 17.2 in two
// and three launches), bound by its vector instructions and load latency in turn (two waves per SIMD), not by the 17 MB of B.
#include <atomic>

#include "bfp_device.h"
#include "gemm_common.h"

namespace hbfp {
namespace {

constexpr int kSmallWaves = 8;
constexpr int kSmallThreads = kSmallWaves * 64;

struct SmallParams {
    const uint8_t *A, *B;        // int8 mantissas [rows][kpad]
    const uint8_t *eA, *eB;      // exponent bytes [rows][exp_ld]
    float *C;                    // [M][ldc]; unused with an encoded output
    int64_t M, N, kpad, eA_ld, eB_ld, ldc;
    int32_t groups;              // kpad / 128
    int32_t beta;
    float final_scale;
    // encoded output (ENC): blocks of 32 along the columns of C
    uint8_t *mant, *exps;
    int64_t okpad, oexp_ld;
    int32_t onblk, om, orounding, orelu;
    uint32_t s0, s1;
};

// MT: row tiles of 32; ENC: the product leaves as an encoded operand
template <int MT, bool ENC>
__global__ __launch_bounds__(kSmallThreads, 2) void gemm_small_kernel(const SmallParams p) {
    __shared__ __attribute__((aligned(16))) float part[kSmallWaves][MT * 32][32];
    const int t = threadIdx.x, lane = t & 63, l32 = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t col0 = (int64_t)blockIdx.x * 32, row0 = (int64_t)blockIdx.y * (32 * MT);
    const int64_t col = col0 + l32 < p.N ? col0 + l32 : p.N - 1;      // columns and rows behind the last read it again
    const uint8_t *b_src = p.B + col * p.kpad + lh * 16, *eb_src = p.eB + col * p.eB_ld;
    const uint8_t *a_src[MT], *ea_src[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int64_t row = row0 + i * 32 + l32 < p.M ? row0 + i * 32 + l32 : p.M - 1;
        a_src[i] = p.A + row * p.kpad + lh * 16;
        ea_src[i] = p.eA + row * p.eA_ld;
    }
    const v2i one_hot = {lh ? 0 : 0x3F80, 0};
    float acc[MT][16];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.0f;

    // a group of four blocks: operands and exponent bytes; the next group is under way while one is multiplied
    struct Group {
        v4i b[4], a[MT][4];
        uint32_t eb, ea[MT];
    };
    auto load = [&](Group &x, int g) {
        g = g < p.groups ? g : p.groups - 1;                   // behind the end: something that exists, not used
#pragma unroll
        for (int k = 0; k < 4; ++k) x.b[k] = *reinterpret_cast<const v4i *>(b_src + (int64_t)g * 128 + k * 32);
        x.eb = *reinterpret_cast<const uint32_t *>(eb_src + (int64_t)g * 4);
#pragma unroll
        for (int i = 0; i < MT; ++i) {
#pragma unroll
            for (int k = 0; k < 4; ++k) x.a[i][k] = *reinterpret_cast<const v4i *>(a_src[i] + (int64_t)g * 128 + k * 32);
            x.ea[i] = *reinterpret_cast<const uint32_t *>(ea_src[i] + (int64_t)g * 4);
        }
    };
    Group cur;
    load(cur, wave);
    // not unrolled: the loop body is small on purpose, because a kernel this short pays for every line of instructions that
    // it fetches (four groups unrolled took 16 x 4096 x 4096 from 10.8 to 16.4 us)
#pragma unroll 1
    for (int g = wave; g < p.groups; g += kSmallWaves) {
        Group next;
        load(next, g + kSmallWaves);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t e = (cur.eb >> (8 * k)) & 0xffu;
            const float scale = __uint_as_float((e > 254u ? 254u : e) << 23);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                e = (cur.ea[i] >> (8 * k)) & 0xffu;
                const v16i rows = row_constants(((e > 254u ? 254u : e) << 7) | 0x40u, one_hot);
                const v16i sum = __builtin_amdgcn_mfma_i32_32x32x32_i8(cur.a[i][k], cur.b[k], rows, 0, 0, 0);
                float x[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) x[v] = __int_as_float(sum[v]) - __int_as_float(rows[v]);
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][v] = fmaf(x[v], scale, acc[i][v]);
            }
            if (MT > 1 || (k & 1)) __builtin_amdgcn_sched_barrier(0);      // no pile-up of block sums beyond two
        }
        cur = next;
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) part[wave][i * 32 + 8 * (v >> 2) + 4 * lh + (v & 3)][l32] = acc[i][v];
    __syncthreads();
    // a thread sums four columns of a row over the waves, in their order; the 8 lanes of a row stay together
    if (t >= MT * 256) return;
    const int r = t >> 3, c4 = (t & 7) * 4;
    const int64_t row = row0 + r;
    if (row >= p.M) return;
    float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) {
        const float4 d = *reinterpret_cast<const float4 *>(&part[w][r][c4]);
        x[0] += d.x, x[1] += d.y, x[2] += d.z, x[3] += d.w;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] *= p.final_scale;
    if (!ENC) {
        float *dst = p.C + row * p.ldc + col0 + c4;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (col0 + c4 + i < p.N) dst[i] = p.beta ? dst[i] + x[i] : x[i];
        return;
    }
    uint32_t amax = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (col0 + c4 + i >= p.N || (p.orelu && x[i] < 0.0f)) x[i] = 0.0f;
        amax = max(amax, __float_as_uint(x[i]) & 0x7fffffffu);
    }
    amax = max(amax, (uint32_t)__shfl_xor((int)amax, 1));
    amax = max(amax, (uint32_t)__shfl_xor((int)amax, 2));
    amax = max(amax, (uint32_t)__shfl_xor((int)amax, 4));
    const uint32_t Eb = p.orounding ? block_exponent<1>(amax, p.om) : block_exponent<0>(amax, p.om);
    uint32_t w = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint64_t idx = (uint64_t)row * (uint64_t)p.N + (uint64_t)(col0 + c4 + i);
        const int q = p.orounding ? quantise<1>(x[i], Eb, p.om, (uint32_t)idx, (uint32_t)(idx >> 32), p.s0, p.s1)
                                  : quantise<0>(x[i], Eb, p.om, 0u, 0u, 0u, 0u);
        w |= ((uint32_t)q & 0xffu) << (8 * i);
    }
    *reinterpret_cast<uint32_t *>(p.mant + row * p.okpad + col0 + c4) = w;
    if (c4 == 0) {
        const int64_t blk = (int64_t)blockIdx.x;
        if (blk < p.oexp_ld) p.exps[row * p.oexp_ld + blk] = blk < p.onblk ? (uint8_t)Eb : (uint8_t)1;
    }
}

template <int MT>
int launch_small(const SmallParams &p, bool enc, unsigned workgroups, hipStream_t s) {
    const dim3 grid(workgroups, (unsigned)ceil_div(p.M, 32 * MT));
    if (enc) hipLaunchKernelGGL((gemm_small_kernel<MT, true>), grid, dim3(kSmallThreads), 0, s, p);
    else hipLaunchKernelGGL((gemm_small_kernel<MT, false>), grid, dim3(kSmallThreads), 0, s, p);
    return launch_status();
}

}  // namespace

// The faster of the two tile heights (1 or 2 row tiles of 32) and its estimate.  One workgroup is resident per compute unit; a
// round of them costs a start and, per group of four blocks, what was measured up to one group per wave and beyond.
static int small_row_tiles(const GemmArgs &a, double *us) {
    const double g = (double)(a.kpad / 128), g8 = g < 8 ? g : 8;
    const int64_t cols = ceil_div(a.N, 32);
    const double t1 = 1.3 + (double)ceil_div(ceil_div(a.M, 32) * cols, 256) * (1.3 + 0.45 * g8 + 0.26 * (g - g8));
    const double t2 = 1.3 + (double)ceil_div(ceil_div(a.M, 64) * cols, 256) * (1.6 + 0.75 * g8 + 0.47 * (g - g8));
    if (us) *us = t1 <= t2 ? t1 : t2;
    return t1 <= t2 ? 1 : 2;
}

// Whether the product runs here: its estimate against that of the 128 x 128-tile kernels, which make their scale words inside the
// kernel at these sizes.  Measured, tile kernels -> here: 256^3 7.8 -> 3.3 us, 512^3 10.2 -> 4.6, 300 x 300 x 2000 12.4 -> 8.9,
// 128 x 4096 x 1024 14.9 -> 9.5, 512 x 512 x 4096 16.5 -> 14.2, 16 x 4096 x 4096 14.7 -> 11.8; behind at 1024 x 1024 x 512
// (10.5, 11.0), 1000^3 (15.8, 18.7), 2048 x 1024 x 256 (8.8, 14.2), 32 x 2048 x 8192 (16.7, 22.3), 16 x 64 x 8192 (10.1, 17.8).
// Of 175 shapes the rule is more than 3 % from the faster side at 11, nine of them left to the tile kernels (2 x 4623 x 8192
// 21.3 against 16.0 us: the estimate knows nothing of rows that are all one).
bool gemm_small_ok(const GemmArgs &a) {
    if (a.P || a.mA > 8 || a.mB > 8 || a.kbp != 32 || a.M > (1 << 20) || a.N > (1 << 20)) return false;
    double us;
    small_row_tiles(a, &us);
    return us < gemm_i8_estimate(a);
}

int launch_gemm_small(const GemmArgs &a, hipStream_t s, const hbfp_tensor *enc, int relu) {
    if (!gemm_small_ok(a)) return HBFP_ERR_FORMAT;
    SmallParams p = {};
    p.A = (const uint8_t *)a.mantA;
    p.B = (const uint8_t *)a.mantB;
    p.eA = a.expA;
    p.eB = a.expB;
    p.C = a.C;
    p.M = a.M;
    p.N = a.N;
    p.kpad = a.kpad;
    p.eA_ld = a.expA_ld;
    p.eB_ld = a.expB_ld;
    p.ldc = a.ldc;
    p.groups = (int32_t)(a.kpad / 128);
    p.beta = a.beta != 0.0f;
    p.final_scale = ldexpf(1.0f, 27 - a.mA - a.mB);
    int64_t cols = a.N;
    if (enc) {
        p.mant = (uint8_t *)enc->mant;
        p.exps = enc->exps;
        p.okpad = enc->kpad;
        p.oexp_ld = enc->exp_ld;
        p.onblk = (int32_t)enc->nblk;
        p.om = enc->mant_bits;
        p.orounding = enc->rounding;
        p.orelu = relu;
        p.s0 = (uint32_t)enc->seed;
        p.s1 = (uint32_t)(enc->seed >> 32);
        cols = enc->kpad;                                      // the padding of the rows too
    }
    const unsigned workgroups = (unsigned)ceil_div(cols, 32);
    return small_row_tiles(a, nullptr) == 1 ? launch_small<1>(p, enc != nullptr, workgroups, s) : launch_small<2>(p, enc != nullptr, workgroups, s);
}

}  // namespace hbfp
