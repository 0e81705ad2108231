// Small BFP matrix products: inference on a few rows, layers of a few hundred columns (Eq. (2) of Sec. 4, blocks stored as 32,
// 8-bit class).  What counts is latency: the 128 x 128-tile kernels behind a launch for scale words, and before one that sums
// slices where few tiles split the contraction, start at 9 us.  Here a workgroup of 8 waves owns 32 columns and 32 or 64 rows
// of C; its waves deal the contraction out among themselves in groups of four blocks (128 bytes of a row), load operands
// and exponent bytes straight into registers, a group ahead, and meet in LDS: one launch, no workspace touched.  Per block the
// arithmetic is that of the int8 kernels: an integer sum started from the row constants, one subtraction and one
// multiply-add.  The result leaves as FP32 or, with ReLU if asked for, as an encoded operand.
// 256^3: 3.3 us (the tile kernel 7.8, 9.8 with a launch for its scale words).  At most 32 rows have a kernel of their own below:
// 16 x 4096 x 4096 7.5 us (11.7 on this one, 14.7 and 17.2 on the tile kernel in two and three launches).
#include <atomic>

#include "bfp_device.h"
#include "gemm_common.h"

namespace hbfp {
namespace {

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

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

// four columns of a row as part of an encoded operand: 8 neighbouring lanes hold block `blk`, the 32 columns from col0 on
template <int ROUND>
__device__ __forceinline__ uint32_t small_quantise(const SmallParams &p, const float4 &x, uint32_t Eb, uint64_t idx) {
    const int q0 = quantise<ROUND>(x.x, Eb, p.om, (uint32_t)idx, (uint32_t)(idx >> 32), p.s0, p.s1);
    const int q1 = quantise<ROUND>(x.y, Eb, p.om, (uint32_t)(idx + 1), (uint32_t)((idx + 1) >> 32), p.s0, p.s1);
    const int q2 = quantise<ROUND>(x.z, Eb, p.om, (uint32_t)(idx + 2), (uint32_t)((idx + 2) >> 32), p.s0, p.s1);
    const int q3 = quantise<ROUND>(x.w, Eb, p.om, (uint32_t)(idx + 3), (uint32_t)((idx + 3) >> 32), p.s0, p.s1);
    return ((uint32_t)q0 & 0xffu) | (((uint32_t)q1 & 0xffu) << 8) | (((uint32_t)q2 & 0xffu) << 16) | ((uint32_t)q3 << 24);
}
__device__ __forceinline__ void small_encode(const SmallParams &p, float4 x, int64_t row, int64_t col0, int c4, int64_t blk) {
    const int64_t left = p.N - (col0 + c4);
    x.x = left < 1 || (p.orelu && x.x < 0.0f) ? 0.0f : x.x;
    x.y = left < 2 || (p.orelu && x.y < 0.0f) ? 0.0f : x.y;
    x.z = left < 3 || (p.orelu && x.z < 0.0f) ? 0.0f : x.z;
    x.w = left < 4 || (p.orelu && x.w < 0.0f) ? 0.0f : x.w;
    uint32_t amax = max(max(__float_as_uint(x.x) & 0x7fffffffu, __float_as_uint(x.y) & 0x7fffffffu),
                        max(__float_as_uint(x.z) & 0x7fffffffu, __float_as_uint(x.w) & 0x7fffffffu));
    amax = max(amax, (uint32_t)__shfl_xor((int)amax, 1));
    amax = max(amax, (uint32_t)__shfl_xor((int)amax, 2));
    amax = max(amax, (uint32_t)__shfl_xor((int)amax, 4));
    const uint64_t idx = (uint64_t)row * (uint64_t)p.N + (uint64_t)(col0 + c4);
    uint32_t Eb, w;
    if (p.orounding) {
        Eb = block_exponent<1>(amax, p.om);
        w = small_quantise<1>(p, x, Eb, idx);
    } else {
        Eb = block_exponent<0>(amax, p.om);
        w = small_quantise<0>(p, x, Eb, idx);
    }
    *reinterpret_cast<uint32_t *>(p.mant + row * p.okpad + col0 + c4) = w;
    if (c4 == 0 && blk < p.oexp_ld) p.exps[row * p.oexp_ld + blk] = blk < p.onblk ? (uint8_t)Eb : (uint8_t)1;
}

// a group of four blocks of 32 columns and MT row tiles: operands (row lane % 32, 16 bytes by lane / 32) and exponent bytes
template <int MT>
struct SmallGroup {
    v4i b[4], a[MT][4];
    uint32_t eb, ea[MT];
};
template <int MT>
__device__ __forceinline__ void small_multiply(const SmallGroup<MT> &x, const v2i &one_hot, float (&acc)[MT][16]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t e = (x.eb >> (8 * k)) & 0xffu;
        const float scale = __uint_as_float((e > 254u ? 254u : e) << 23);
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            e = (x.ea[i] >> (8 * k)) & 0xffu;
            const v16i rows = row_constants(((e > 254u ? 254u : e) << 7) | 0x40u, one_hot);
            const v16i sum = __builtin_amdgcn_mfma_i32_32x32x32_i8(x.a[i][k], x.b[k], rows, 0, 0, 0);
            float y[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) y[v] = __int_as_float(sum[v]) - __int_as_float(rows[v]);
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][v] = fmaf(y[v], scale, acc[i][v]);
        }
        if (MT > 1 || (k & 1)) __builtin_amdgcn_sched_barrier(0);      // no pile-up of block sums beyond two
    }
}

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

    SmallGroup<MT> cur;
    // a group ahead of the one that is multiplied
    auto load = [&](SmallGroup<MT> &x, int g) {
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
    load(cur, wave);
    // not unrolled: the loop body is small on purpose, because a kernel this short pays for every line of instructions that
    // it fetches (four groups unrolled took 16 x 4096 x 4096 from 10.8 to 16.4 us)
#pragma unroll 1
    for (int g = wave; g < p.groups; g += kSmallWaves) {
        SmallGroup<MT> next;
        load(next, g + kSmallWaves);
        __builtin_amdgcn_sched_barrier(0);
        small_multiply<MT>(cur, one_hot, acc);
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
    small_encode(p, make_float4(x[0], x[1], x[2], x[3]), row, col0, c4, (int64_t)blockIdx.x);
}

// The sum over the waves and what leaves: thread t of the first 64 MT NT adds four columns of a row over the waves, in their
// order (part: [wave][16 MT][16 NT]); the 4 NT lanes of a row stay together, and with NT = 2 they hold one block of 32.
template <int MT, int NT, bool ENC>
__device__ __forceinline__ void few_finish(const SmallParams &p, const float *part, int t, int64_t row0, int64_t col0) {
    if (t >= 64 * MT * NT) return;
    const int r = t / (4 * NT), c4 = (t % (4 * NT)) * 4;
    const int64_t row = row0 + r;
    if (row >= p.M) return;
    float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) {
        const float4 d = *reinterpret_cast<const float4 *>(part + (w * 16 * MT + r) * 16 * NT + c4);
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
    small_encode(p, make_float4(x[0], x[1], x[2], x[3]), row, col0, c4, (int64_t)blockIdx.x);
}

// Few rows (at most 32): inference of a layer on a small batch.  What bounds it is how many bytes of B are on their way: a
// contraction of 4096 left a wave of the kernel above four groups of blocks, two of them in flight, half of each matrix
// instruction's 32 rows empty.  Here a wave owns 16 MT rows and 16 columns (32 where the output is converted: a block) and keeps
// its part of the contraction in flight as asynchronous copies into LDS of its own, up to four chunks of 128 k ahead, no
// barrier before the waves' sums meet; v_mfma_i32_16x16x32_i8 fits the rows.  As many chunks ahead as the workgroups that share
// a compute unit leave room for: what is in flight per compute unit counts, not how many workgroups asked for it.  The
// arithmetic per block, its order over the chunks and over the waves are those of the kernel above, so are the bits.
// The kernel above -> this one: 16 x 4096 x 4096 11.7 -> 7.5 us (2.2 TB/s of B; converted 12.1 -> 8.7), 32 rows 13.7 -> 9.6,
// 12 x 5586 x 435 11.9 -> 6.4, 31 x 4277 x 15967 28.5 -> 26.8, 1 x 512 x 512 3.5 -> 3.05.
// LDS of a chunk: rows of 128 bytes, A's 16 MT, then B's, 16-byte pieces XORed with row % 8 (copies of 8 rows and fragment
// reads of 16 rows by 8 bytes then cover the banks evenly), behind them the exponent bytes of the chunk's four blocks: rows
// 0 .. 31, columns 0 .. 31, a word each.
struct FewParams : SmallParams {
    int32_t ahead;               // chunks in flight per wave, 1 to 4
};
template <int MT, bool ENC>
struct Few {
    static constexpr int NT = ENC ? 2 : 1;
    static constexpr int kChunk = (MT + NT) * 2048 + 256;
    static constexpr int kCopies = 2 * (MT + NT) + 1;
};
template <int MT, bool ENC>
__global__ __launch_bounds__(kSmallThreads, 2) void gemm_few_kernel(const FewParams p) {
    typedef Few<MT, ENC> R;
    constexpr int NT = R::NT;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int t = threadIdx.x, lane = t & 63, l16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t col0 = (int64_t)blockIdx.x * (16 * NT);
    // the columns that exist; a workgroup of nothing but padding (encoded outputs) reads the last one
    const int64_t bcol0 = col0 < p.N ? col0 : p.N - 1;
    const int rows = (int)p.M, cols = (int)(p.N - bcol0 < 16 * NT ? p.N - bcol0 : 16 * NT);       // both at least 1
    const uint32_t base = wave * (uint32_t)(p.ahead * R::kChunk);
    // a copy moves 8 rows of 128 bytes; rows and columns behind the last read it again
    const int r8 = lane >> 3, piece = ((lane & 7) ^ r8) * 16;
    uint32_t voff[2 * (MT + NT)];
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) voff[i] = (uint32_t)(8 * i + r8 < rows ? 8 * i + r8 : rows - 1) * (uint32_t)p.kpad + piece;
#pragma unroll
    for (int i = 0; i < 2 * NT; ++i) voff[2 * MT + i] = (uint32_t)(8 * i + r8 < cols ? 8 * i + r8 : cols - 1) * (uint32_t)p.kpad + piece;
    const int er = lane & 31;
    const uint8_t *esrc = lane < 32 ? p.eA + (int64_t)(er < rows ? er : rows - 1) * p.eA_ld : p.eB + (bcol0 + (er < cols ? er : cols - 1)) * p.eB_ld;
    const uint8_t *a0 = p.A, *b0 = p.B + bcol0 * p.kpad;
    auto request = [&](int chunk, int buf) {
        const uint32_t to = base + buf * R::kChunk;
        const int64_t k = (int64_t)chunk * 128;
#pragma unroll
        for (int i = 0; i < 2 * MT; ++i) async_copy16(a0 + k, voff[i], to + i * 1024);
#pragma unroll
        for (int i = 0; i < 2 * NT; ++i) async_copy16(b0 + k, voff[2 * MT + i], to + (2 * MT + i) * 1024);
        async_copy4_at(esrc + 4 * (int64_t)chunk, to + (MT + NT) * 2048);
    };
    float acc[MT][NT][4] = {};
    const int mine = p.groups > wave ? (p.groups - wave + kSmallWaves - 1) / kSmallWaves : 0;     // chunks wave, wave + 8, ...
    const int ahead = mine < p.ahead ? mine : p.ahead;
    for (int i = 0; i < ahead; ++i) request(wave + i * kSmallWaves, i);
    const uint32_t frag = l16 * 128 + (q & 1) * 8, sw = l16 & 7;
    int buf = 0;
#pragma unroll 1
    for (int i = 0; i < mine; ++i) {
        // chunk i has landed when only those behind it are under way
        const int behind = mine - 1 - i < p.ahead - 1 ? mine - 1 - i : p.ahead - 1;
        if (behind >= 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * R::kCopies) : "memory");
        else if (behind == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * R::kCopies) : "memory");
        else if (behind == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(R::kCopies) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const uint8_t *c = lds + base + buf * R::kChunk;
        v2i a[MT][4], b[NT][4];
        v4u ea[MT];
        uint32_t eb[NT];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t off = frag + (((2 * k + (q >> 1)) ^ sw) * 16);
#pragma unroll
            for (int m = 0; m < MT; ++m) a[m][k] = *reinterpret_cast<const v2i *>(c + off + m * 2048);
#pragma unroll
            for (int n = 0; n < NT; ++n) b[n][k] = *reinterpret_cast<const v2i *>(c + off + (MT + n) * 2048);
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) ea[m] = *reinterpret_cast<const v4u *>(c + (MT + NT) * 2048 + (m * 16 + 4 * q) * 4);
#pragma unroll
        for (int n = 0; n < NT; ++n) eb[n] = *reinterpret_cast<const uint32_t *>(c + (MT + NT) * 2048 + 128 + (n * 16 + l16) * 4);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                     // read: the buffer may be filled again
        if (i + p.ahead < mine) request(wave + (i + p.ahead) * kSmallWaves, buf);
        buf = buf + 1 == p.ahead ? 0 : buf + 1;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float scale[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const uint32_t e = (eb[n] >> (8 * k)) & 0xffu;
                scale[n] = __uint_as_float((e > 254u ? 254u : e) << 23);
            }
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                v4i from;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const uint32_t e = (ea[m][v] >> (8 * k)) & 0xffu;
                    from[v] = (int)(((e > 254u ? 254u : e) << 23) | 0x400000u);          // 1.5 * 2^(E - 127)
                }
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    const v4i sum = __builtin_amdgcn_mfma_i32_16x16x32_i8(__builtin_bit_cast(long, a[m][k]), __builtin_bit_cast(long, b[n][k]), from, 0, 0, 0);
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[m][n][v] = fmaf(__int_as_float(sum[v]) - __int_as_float(from[v]), scale[n], acc[m][n][v]);
                }
            }
        }
    }
    __syncthreads();
    float *part = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[(wave * 16 * MT + m * 16 + 4 * q + v) * 16 * NT + n * 16 + l16] = acc[m][n][v];
    __syncthreads();
    few_finish<MT, NT, ENC>(p, part, t, 0, col0);
}

constexpr int kFewLds = 160 * 1024;
template <int MT, bool ENC>
int launch_few_t(const SmallParams &p, int64_t cols, hipStream_t s) {
    static std::atomic<bool> configured{false};
    void (*kernel)(FewParams) = &gemm_few_kernel<MT, ENC>;
    if (allow_dynamic_lds(configured, reinterpret_cast<const void *>(kernel), kFewLds) != HBFP_OK) return HBFP_ERR_LAUNCH;
    const int64_t wgs = ceil_div(cols, 16 * Few<MT, ENC>::NT), per_cu = ceil_div(wgs, 256);
    const int chunk = kSmallWaves * Few<MT, ENC>::kChunk;                  // of all waves
    FewParams f;
    static_cast<SmallParams &>(f) = p;
    int64_t room = kFewLds / per_cu / chunk;
    const int64_t most = ceil_div(p.groups, kSmallWaves);
    room = room > most ? most : room;
    f.ahead = (int32_t)(room > 4 ? 4 : room < 1 ? 1 : room);
    int bytes = f.ahead * chunk;
    const int sums = kSmallWaves * 16 * MT * 16 * Few<MT, ENC>::NT * 4;
    bytes = bytes > sums ? bytes : sums;
    hipLaunchKernelGGL(kernel, dim3((unsigned)wgs), dim3(kSmallThreads), bytes, s, f);
    return launch_status();
}
int launch_few(const SmallParams &p, bool enc, int64_t cols, hipStream_t s) {
    const bool two = p.M > 16;
    if (enc) return two ? launch_few_t<2, true>(p, cols, s) : launch_few_t<1, true>(p, cols, s);
    return two ? launch_few_t<2, false>(p, cols, s) : launch_few_t<1, false>(p, cols, s);
}
// Whether a product that runs here takes the kernel for few rows.  Up to three chunks of k per product (four where it is
// converted) the start of a workgroup with that much LDS is what counts, and the other kernel is ahead.
bool few_rows_ok(int64_t M, int64_t kpad, bool enc) { return M <= 32 && kpad / 128 >= (enc ? 5 : 4) && kpad <= (1 << 26); }

// A product of two FP32 matrices in one launch (hbfp_gemm_f32 at small sizes): the workgroup converts its 32 rows of A and its 32
// columns of B itself.  What bounds these calls is launches and latency: a launch that converts both operands (5.1 us at 256^3)
// and one that multiplies (3.7 us) have their starts and the gap between them to pay.  A block of 32 x 32 values is one wave's:
// its lanes hold 16 values of a row or column each, in the order in which the matrix instruction takes them, so what is
// handed from the converting wave to the multiplying one is 16 bytes per lane.  All of a wave's loads are requested before the
// first conversion, from lanes that own them: by whole lines, 8 lanes to a row, the loads are fewer and the instructions more
// (512^3 6.6 us both ways, 128 x 2000 x 500 9.0 against 9.6).  Blocks go round over the waves to be converted, but a wave multiplies the four blocks of its group, as in
// the kernels above: the same order of sums, the same bits.
struct ConvertSource {
    const float *src;
    int64_t ld;
    int32_t rows, m;             // rows or columns of the operand
    int32_t down;                // the contraction runs down the source rows
};
struct ConvertParams {
    ConvertSource x[2];
    float *C;
    int64_t ldc;
    int32_t K, kblock, nblk, groups;
    float final_scale;
};
// 16 values of block `blk` of row `r`: those from 16 lh on, zeros behind the block's and the matrix's end.  QUADS: what is left of a
// block by whole quadruples (launch_gemm_convert)
template <bool QUADS>
__device__ __forceinline__ void convert_load(const ConvertSource &x, const ConvertParams &p, int64_t r, int lh, int blk, float (&v)[16]) {
    int len = 0;
    if (blk < p.nblk) len = p.K - blk * p.kblock < p.kblock ? p.K - blk * p.kblock : p.kblock;
    const int left = len - 16 * lh;
    const int64_t k0 = (int64_t)(len ? blk : 0) * p.kblock;
    if (x.down) {
        const float *s = x.src + (left > 0 ? 16 * lh : 0) * x.ld + r;
        if (len == 32) {
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = s[(k0 + j) * x.ld];
        } else if (QUADS) {
#pragma unroll
            for (int j = 0; j < 16; j += 4) {
                if (j + 4 <= left) {
#pragma unroll
                    for (int e = j; e < j + 4; ++e) v[e] = s[(k0 + e) * x.ld];
                } else {
#pragma unroll
                    for (int e = j; e < j + 4; ++e) v[e] = e < left ? s[(k0 + e) * x.ld] : 0.0f;
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = j < left ? s[(k0 + j) * x.ld] : 0.0f;
        }
    } else {
        const float *s = x.src + r * x.ld + k0 + (left > 0 ? 16 * lh : 0);
        if (len == 32) {
#pragma unroll
            for (int j = 0; j < 16; j += 4) {
                const v4f_any d = *reinterpret_cast<const v4f_any *>(s + j);
                v[j] = d[0], v[j + 1] = d[1], v[j + 2] = d[2], v[j + 3] = d[3];
            }
        } else if (QUADS) {
#pragma unroll
            for (int j = 0; j < 16; j += 4) {
                if (j + 4 <= left) {
                    const v4f_any d = *reinterpret_cast<const v4f_any *>(s + j);
                    v[j] = d[0], v[j + 1] = d[1], v[j + 2] = d[2], v[j + 3] = d[3];
                } else {
#pragma unroll
                    for (int e = j; e < j + 4; ++e) v[e] = e < left ? s[e] : 0.0f;
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = j < left ? s[j] : 0.0f;
        }
    }
}
__device__ __forceinline__ uint32_t convert_word(const float *v, uint32_t Eb, int m) {
    return pack4_i8(quantise<0>(v[0], Eb, m, 0, 0, 0, 0), quantise<0>(v[1], Eb, m, 0, 0, 0, 0),
                    quantise<0>(v[2], Eb, m, 0, 0, 0, 0), quantise<0>(v[3], Eb, m, 0, 0, 0, 0));
}
// the block's mantissas, 16 bytes per lane of the matrix instruction, and its exponents, a byte per row `pitch` bytes apart
__device__ __forceinline__ void convert_store(const ConvertSource &x, int lane, const float (&v)[16], uint8_t *mant, uint8_t *exps, int pitch) {
    uint32_t amax = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) amax = max(amax, __float_as_uint(v[j]) & 0x7fffffffu);
    amax = max(amax, (uint32_t)__shfl_xor((int)amax, 32));
    const uint32_t Eb = block_exponent<0>(amax, x.m);
    v4u w;
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = convert_word(v + 4 * j, Eb, x.m);
    *reinterpret_cast<v4u *>(mant + lane * 16) = w;
    if (lane < 32) exps[lane * pitch] = (uint8_t)Eb;
}
// PER: blocks that a wave converts of each operand
template <int PER>
struct Convert {
    static constexpr int kBlocks = PER * kSmallWaves, kExpRow = kBlocks + 4;
    static constexpr int kMant = kBlocks * 1024, kPart = kSmallWaves * 32 * 32 * 4;      // bytes: one operand's, the waves' sums
    static constexpr int kExps = 2 * kMant > kPart ? 2 * kMant : kPart;
    static constexpr int kLds = kExps + 2 * 32 * kExpRow;
};
template <int PER, bool QUADS>
__global__ __launch_bounds__(kSmallThreads, 2) void gemm_convert_kernel(const ConvertParams p) {
    typedef Convert<PER> R;
    __shared__ __attribute__((aligned(16))) uint8_t lds[R::kLds];
    const int t = threadIdx.x, lane = t & 63, l32 = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t origin[2] = {(int64_t)blockIdx.y * 32, (int64_t)blockIdx.x * 32};
    float v[2][PER][16];
#pragma unroll
    for (int i = 0; i < PER; ++i)
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            const int64_t r = origin[o] + l32 < p.x[o].rows ? origin[o] + l32 : p.x[o].rows - 1;   // behind the last: that one again
            convert_load<QUADS>(p.x[o], p, r, lh, wave + i * kSmallWaves, v[o][i]);
        }
#pragma unroll
    for (int i = 0; i < PER; ++i)
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            const int blk = wave + i * kSmallWaves;
            convert_store(p.x[o], lane, v[o][i], lds + o * R::kMant + blk * 1024, lds + R::kExps + o * 32 * R::kExpRow + blk, R::kExpRow);
        }
    __syncthreads();
    const v2i one_hot = {lh ? 0 : 0x3F80, 0};
    float acc[1][16];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[0][j] = 0.0f;
    if (wave < p.groups) {
        SmallGroup<1> g;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            g.a[0][k] = *reinterpret_cast<const v4i *>(lds + (4 * wave + k) * 1024 + lane * 16);
            g.b[k] = *reinterpret_cast<const v4i *>(lds + R::kMant + (4 * wave + k) * 1024 + lane * 16);
        }
        g.ea[0] = *reinterpret_cast<const uint32_t *>(lds + R::kExps + l32 * R::kExpRow + 4 * wave);
        g.eb = *reinterpret_cast<const uint32_t *>(lds + R::kExps + (32 + l32) * R::kExpRow + 4 * wave);
        small_multiply<1>(g, one_hot, acc);
    }
    __syncthreads();                                             // the sums lie where the mantissas were
    float *part = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int j = 0; j < 16; ++j) part[(wave * 32 + 8 * (j >> 2) + 4 * lh + (j & 3)) * 32 + l32] = acc[0][j];
    __syncthreads();
    if (t >= 256) return;
    const int r = t >> 3, c4 = (t & 7) * 4;
    const int64_t row = origin[0] + r, col = origin[1] + c4;
    if (row >= p.x[0].rows) return;
    float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) {
        const float4 d = *reinterpret_cast<const float4 *>(part + (w * 32 + r) * 32 + c4);
        x[0] += d.x, x[1] += d.y, x[2] += d.z, x[3] += d.w;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (col + i < p.x[1].rows) p.C[row * p.ldc + col + i] = x[i] * p.final_scale;
}

template <int PER, bool QUADS>
int launch_convert(const ConvertParams &p, hipStream_t s) {
    const dim3 grid((unsigned)ceil_div(p.x[1].rows, 32), (unsigned)ceil_div(p.x[0].rows, 32));
    hipLaunchKernelGGL((gemm_convert_kernel<PER, QUADS>), grid, dim3(kSmallThreads), 0, s, p);
    return launch_status();
}

template <int MT>
int launch_small(const SmallParams &p, bool enc, unsigned workgroups, hipStream_t s) {
    const dim3 grid(workgroups, (unsigned)ceil_div(p.M, 32 * MT));
    void (*fp32)(SmallParams) = &gemm_small_kernel<MT, false>, (*encoded)(SmallParams) = &gemm_small_kernel<MT, true>;
    hipLaunchKernelGGL(enc ? encoded : fp32, grid, dim3(kSmallThreads), 0, s, p);
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

// What the kernel for few rows takes: a start, and for every 1024 of k and every workgroup of a compute unit what was measured with
// one workgroup on the chip and with all of it busy (fitted to 345 shapes of 1 to 32 rows, 16 to 20 000 columns and 1024 to 20 000 of
// k, and to 240 with an encoded output, whose workgroups have twice the columns).
static double few_rows_us(const GemmArgs &a, bool enc) {
    const int64_t wgs = ceil_div(a.N, enc ? 32 : 16);
    const double busy = wgs < 256 ? (double)wgs / 256.0 : 1.0;
    const double step = a.M <= 16 ? (enc ? 0.82 + 0.5 * busy : 0.6 + 0.2 * busy) : (enc ? 1.3 + 0.5 * busy : 0.95 + 0.15 * busy);
    return (enc ? 3.3 : 2.7) + (double)a.kpad / 1024.0 * (double)ceil_div(wgs, 256) * step;
}

// Whether the product runs here: its estimate against that of the 128 x 128-tile kernels, which make their scale words inside the
// kernel at these sizes.  Measured, tile kernels -> here: 256^3 7.8 -> 3.3 us, 512^3 10.2 -> 4.6, 300 x 300 x 2000 12.4 -> 8.9,
// 128 x 4096 x 1024 14.9 -> 9.5, 512 x 512 x 4096 16.5 -> 14.2; behind at 1024 x 1024 x 512 (10.5, 11.0), 1000^3 (15.8, 18.7),
// 2048 x 1024 x 256 (8.8, 14.2).
// At most 32 rows are weighed by the kernel that they run on; the tile kernels' estimate is 2 to 5 us too high where few columns
// are split along k.  Tile kernels -> here: 16 x 4096 x 4096 14.3 -> 7.5, 1 x 4096 x 8192 18.5 -> 10.5, 16 x 1024 x 8192 12.2 -> 8.9,
// 32 x 2048 x 8192 15.1 -> 12.9, 17 x 16384 x 16384 92.6 -> 73.0; behind at 16 x 64 x 16384 (10.3, 12.6), 32 x 64 x 8192 (9.3, 11.4),
// 32 x 1024 x 12288 (14.4, 16.8).  Of the 345 shapes 8 are more than 3 % from the faster side, all together 0.3 % behind it (11 %
// by the estimate of the kernel above, which left most contractions from 6144 on to the tile kernels).
bool gemm_small_ok(const GemmArgs &a, bool enc) {
    if (a.P || a.mA > 8 || a.mB > 8 || a.kbp != 32 || a.M > (1 << 20) || a.N > (1 << 20)) return false;
    if (few_rows_ok(a.M, a.kpad, enc)) return few_rows_us(a, enc) < gemm_i8_estimate(a) - (a.N <= 512 ? 3.5 : 0.0);
    double us;
    small_row_tiles(a, &us);
    return us < gemm_i8_estimate(a);
}

int launch_gemm_small(const GemmArgs &a, hipStream_t s, const hbfp_tensor *enc, int relu) {
    if (!gemm_small_ok(a, enc != nullptr)) return HBFP_ERR_FORMAT;
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
    if (few_rows_ok(p.M, p.kpad, enc != nullptr)) return launch_few(p, enc != nullptr, cols, s);
    const unsigned workgroups = (unsigned)ceil_div(cols, 32);
    return small_row_tiles(a, nullptr) == 1 ? launch_small<1>(p, enc != nullptr, workgroups, s) : launch_small<2>(p, enc != nullptr, workgroups, s);
}

// Whether the product converts its own operands: one round of workgroups, at most two blocks of each operand per wave, and the
// products that the kernels above would take.  Every workgroup converts for itself and one of few blocks is mostly the fetch of
// its own instructions: with four blocks per wave the two launches are ahead or level (512 x 512 x 1024 10.9 us against 12.9
// here).  So they are from 257 of k on where both operands lie along the rows in blocks that are not 32 long and are read value
// by value (511^3 read so: 10.8 against 13.5; one such operand 10.8, 10.5).  Measured in a graph, two launches -> here: 256^3
// 7.0 -> 4.7 us, both operands down the rows 7.0 -> 4.2, 512^3 8.4 -> 6.6, 511^3 10.8 -> 8.0, 128 x 2000 x 500 9.25 -> 9.0,
// 33 x 2047 x 499 10.2 -> 6.6, 16 x 4096 x 512 8.6 -> 5.7, 33 x 2048 x 64 6.8 -> 4.5; call by call, where the host's two launches
// are the bound, 13.0 -> 9.5 at all of them.
bool gemm_convert_ok(const GemmArgs &a, const EncodeGeom *geom) {
    if (!encode_pair_ok(geom[0], geom[1]) || !gemm_small_ok(a)) return false;
    if (a.kpad > 512 || ceil_div(a.M, 32) * ceil_div(a.N, 32) > 256) return false;
    return a.kpad <= 256 || a.kblock == 32 || geom[0].axis == 0 || geom[1].axis == 0;
}

int launch_gemm_convert(const GemmArgs &a, const float *const *src, const EncodeGeom *geom, hipStream_t s) {
    if (!gemm_convert_ok(a, geom)) return HBFP_ERR_FORMAT;
    ConvertParams p = {};
    for (int o = 0; o < 2; ++o) {
        const EncodeGeom &g = geom[o];
        p.x[o].src = src[o];
        p.x[o].ld = g.ld;
        p.x[o].rows = (int32_t)g.R;
        p.x[o].m = g.m;
        p.x[o].down = g.axis == 0;
    }
    p.C = a.C;
    p.ldc = a.ldc;
    p.K = (int32_t)geom[0].K;
    p.kblock = (int32_t)a.kblock;
    p.nblk = (int32_t)a.nblk;
    p.groups = (int32_t)(a.kpad / 128);
    p.final_scale = ldexpf(1.0f, 27 - a.mA - a.mB);
    const int64_t blocks = a.kpad / 32;
    // Blocks of 16 to 31 in contractions beyond 128 are read by quadruples: value by value they were up to 23 % behind the two launches
    // (two launches, value by value, quadruples: 134 x 829 x 248 in blocks of 24 8.5, 9.4, 7.0 us, 84 x 48 x 192 7.5, 8.9, 5.4).
    // Shorter blocks and contractions stay ahead without and pay for the longer code with 2 to 10 %.
    const bool quads = a.kblock >= 16 && a.kblock < 32 && a.kpad > 128;
    if (blocks <= 8) return quads ? launch_convert<1, true>(p, s) : launch_convert<1, false>(p, s);
    return quads ? launch_convert<2, true>(p, s) : launch_convert<2, false>(p, s);
}

}  // namespace hbfp
