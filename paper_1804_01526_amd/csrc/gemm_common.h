// Pieces shared by the matrix-product kernels (each translation unit gets its own copy).
#pragma once
#include "hbfp_internal.h"

namespace hbfp {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

// Workgroup -> tile.  Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.  XCD x gets
// a contiguous eighth of the tiles, walked in bands of 8 tile rows column by column, so that the 64
// tiles an XCD works on at any time are an 8 x 8 patch: 8 row panels and 8 column panels of the current
// k range stay in that XCD's L2 and each is used 8 times.  Returns false for the padding workgroups.
__device__ __forceinline__ bool tile_of_workgroup(int wg, int tiles_m, int tiles_n, int &tm, int &tn) {
    const int ntiles = tiles_m * tiles_n;
    const int per_xcd = (ntiles + 7) >> 3;
    const int t = (wg & 7) * per_xcd + (wg >> 3);
    if ((wg >> 3) >= per_xcd || t >= ntiles) return false;
    const int band = t / (8 * tiles_n);
    const int rows_in_band = tiles_m - band * 8 < 8 ? tiles_m - band * 8 : 8;
    const int r = t - band * 8 * tiles_n;
    tn = r / rows_in_band;
    tm = band * 8 + r % rows_in_band;
    return true;
}

// Split-K launches with at least 8 k ranges (few tiles, very long k): a one-dimensional grid of
// 8 * tiles * ceil(splits / 8) workgroups.
// XCD x takes the k ranges x, x + 8, ... and, for each, every tile: the tiles of one k range share their operand
// panels in that XCD's L2, and the work is spread over all 8 XCDs however few tiles there are (dealing tiles to
// XCDs as above would leave XCDs idle when there are fewer than 8 tiles).  Returns false for padding workgroups.
__device__ __forceinline__ bool tile_and_split_of_workgroup(int wg, int tiles_m, int tiles_n, int splits, int &tm, int &tn,
                                                            int &split) {
    const int ntiles = tiles_m * tiles_n;
    const int slot = wg >> 3;
    split = (slot / ntiles) * 8 + (wg & 7);
    if (split >= splits) return false;
    const int t = slot % ntiles;
    tn = t / tiles_m;
    tm = t - tn * tiles_m;
    return true;
}

__device__ __forceinline__ void async_copy16(const void *gbase, uint32_t voff, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(gbase) : "memory");
}
// the same copies from a full 64-bit address per lane (gathers whose sources do not share one base)
__device__ __forceinline__ void async_copy16_at(const void *addr, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(addr) : "memory");
}
__device__ __forceinline__ void async_copy4_at(const void *addr, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_addr), "v"(addr) : "memory");
}
__device__ __forceinline__ void async_copy4(const void *gbase, uint32_t voff, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_addr), "v"(voff), "s"(gbase) : "memory");
}

// Whether rows of C go past the caches.  They are written once and not read again by the call, so streaming stores leave the caches to
// the operands: 2 to 6 Mi outputs are 3 to 11 % faster than with ordinary stores, larger ones in whole lines 2 %.  But where a row ends
// inside a line the next row writes the rest of it, and once C no longer fits the L2 caches (32 MB) such a line leaves them as two
// partial writes: packed 4995 x 3043 x 104 29.7 us streaming, 17.8 with ordinary stores, 4037 x 4663 x 55 41.1 and 24.1.  Ordinary
// stores are ahead from 6 Mi outputs on for rows off 32 bytes (6 to 8 Mi 9 %, 14 to 20 Mi 34 %), from 10 Mi on for rows off 128 (7 %).
// A group of products shares one launch: the larger part of its outputs decides.  The choice is the host's: in one kernel the compiler
// makes ordinary stores of two branches that differ in this alone.
inline bool stores_stream(const GemmArgs *args, int n = 1) {
    int64_t count = 0, balance = 0;
    for (int i = 0; i < n; ++i) count += args[i].M * args[i].N;
    for (int i = 0; i < n; ++i) {
        const uint64_t off = (uint64_t)(uintptr_t)args[i].C | (uint64_t)args[i].ldc * 4;
        const bool stream = (off & 127) == 0 || count < ((int64_t)((off & 31) ? 6 : 10) << 20);
        balance += stream ? args[i].M * args[i].N : -args[i].M * args[i].N;
    }
    return balance >= 0;
}

// Stores a wave's TI x TJ results of 32 x 32 (lane l: column l % 32, register v: row 8 (v / 4) + 4 (l / 32) + v % 4); dst is
// their first element, rows and cols what is left of the product from there, value(i, j, v) the output.  STREAM: past the caches
// (stores_stream).
// Bound by its instructions: with a 64-bit product for every row, and two tests and a branch around every store, the 128
// stores of a lane of the 256 x 256-tile kernels were 2500 instructions of straight code that the waves fetched once each,
// and a kernel of a few k-steps spent most of its time there.  Here a whole tile is stores and one addition per row; only
// the edges of the product and C += take the tests.  One-exponent product 3001 x 4500 x 2999 70 -> 64 us, a step of three
// packed 4096^3 products 431 -> 413, two of 1337 x 2052 x 1500 and their conversions 80.5 -> 73.4, 12-bit 8192^3 1035 -> 984.
template <int TI, int TJ, bool STREAM, class V>
__device__ __forceinline__ void store_result(float *dst, int64_t ld, int64_t rows, int64_t cols, bool add, int lane, const V &value) {
    const int lh = lane >> 5, l32 = lane & 31;
    if (rows <= 0 || cols <= 0) return;
    float *p = dst + 4 * lh * ld + l32;
    if (rows >= 32 * TI && cols >= 32 * TJ && !add) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    if (STREAM) __builtin_nontemporal_store(value(i, j, v), p + 32 * j);
                    else p[32 * j] = value(i, j, v);
                }
                p += (v & 3) == 3 ? 5 * ld : ld;
            }
        return;
    }
    const int r_end = (int)(rows < 32 * TI ? rows : 32 * TI) - 4 * lh, c_end = (int)(cols < 32 * TJ ? cols : 32 * TJ) - l32;
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            if (32 * i + 8 * (v >> 2) + (v & 3) < r_end) {
#pragma unroll
                for (int j = 0; j < TJ; ++j)
                    if (32 * j < c_end) {
                        float x = value(i, j, v);
                        if (add) x = p[32 * j] + x;
                        if (STREAM) __builtin_nontemporal_store(x, p + 32 * j);
                        else p[32 * j] = x;
                    }
            }
            p += (v & 3) == 3 ? 5 * ld : ld;
        }
}

// A kernel queued behind the block-scaled product kernel as its stand-in runs only when one of the two packed
// operands is marked out of range (the first two words of its header are equal); without headers it always runs.
__device__ __forceinline__ bool stands_down(const int *run_a, const int *run_b) {
    return run_a && run_a[0] != run_a[1] && run_b[0] != run_b[1];
}

typedef short v4s __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));

// rowc holds, in its low half, the bf16 pattern of 1.5 * 2^(Ea - 127) of row (lane % 32); every other
// 16-bit element of the first operand meets a zero of one_hot (a bf16 one at k = 0 of lanes 0..31) and
// only has to be finite.  The product is exact, so the result is the FP32 constant in every column.
__device__ __forceinline__ v16i row_constants(uint32_t rowc, const v2i &one_hot) {
    const v2i a2 = {(int)rowc, 0};
    const v16f zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    const v16f c = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(v4s, a2), __builtin_bit_cast(v4s, one_hot), zero, 0, 0, 0);
    return __builtin_bit_cast(v16i, c);
}

// exponent bytes [rows][ld] -> scale words [slots][rows_pad] for both operands in one launch (blockIdx.z
// picks the operand); rows past the end get the smallest scale.  A thread turns four consecutive blocks
// of one row (one 32-bit load: ld and slots are multiples of 4) into four words; consecutive lanes take
// consecutive rows, so the stores are contiguous.
struct WordParams {
    const uint8_t *exps[2];
    uint32_t *words[2];
    int64_t ld[2], rows[2], rows_pad[2];
    int slots, row_blocks;
    uint32_t a_or;               // 0x40: row words are 1.5 * 2^(E - 127) as bf16; 0: 2^(E - 127) as bf16
    const int *run_a, *run_b;
};
// one block of 256 threads of that job: block index, operand, thread
__device__ __forceinline__ void scale_words_block(const WordParams &w, uint32_t block, int z, int thread) {
    const int64_t row = (int64_t)(block % (uint32_t)w.row_blocks) * 256 + thread;
    if (row >= w.rows_pad[z]) return;
    const int s0 = (int)(block / (uint32_t)w.row_blocks) * 4;
    const uint32_t e4 = row < w.rows[z] ? *reinterpret_cast<const uint32_t *>(w.exps[z] + row * w.ld[z] + s0) : 0x01010101u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t e = (e4 >> (8 * i)) & 0xffu;
        e = e > 254u ? 254u : e;
        w.words[z][(int64_t)(s0 + i) * w.rows_pad[z] + row] = z == 0 ? ((e << 7) | w.a_or) : (e << 23);
    }
}
__global__ __launch_bounds__(256) void scale_words_t_kernel(const WordParams w) {
    if (stands_down(w.run_a, w.run_b)) return;
    scale_words_block(w, blockIdx.x, (int)blockIdx.z, (int)threadIdx.x);
}

// bytes of one operand's scale words: [slots][rows rounded up to 128]
inline size_t word_bytes(int64_t rows, int64_t slots) { return (size_t)slots * (size_t)(ceil_div(rows, 128) * 128) * 4; }

// slots must be a multiple of 4 and at most the exponent row pitch of either operand
inline WordParams scale_word_params(const uint8_t *eA, int64_t ldA, int64_t M, const uint8_t *eB, int64_t ldB, int64_t N, int slots,
                                    uint32_t a_or, uint32_t *wA, uint32_t *wB, const int *run_a, const int *run_b) {
    WordParams wp;
    wp.exps[0] = eA; wp.exps[1] = eB;
    wp.words[0] = wA; wp.words[1] = wB;
    wp.ld[0] = ldA; wp.ld[1] = ldB;
    wp.rows[0] = M; wp.rows[1] = N;
    wp.rows_pad[0] = ceil_div(M, 128) * 128; wp.rows_pad[1] = ceil_div(N, 128) * 128;
    wp.slots = slots;
    wp.a_or = a_or;
    wp.run_a = run_a;
    wp.run_b = run_b;
    const int64_t maxpad = wp.rows_pad[0] > wp.rows_pad[1] ? wp.rows_pad[0] : wp.rows_pad[1];
    wp.row_blocks = (int)ceil_div(maxpad, 256);
    return wp;
}
// blocks of 256 threads per operand that the job consists of
inline int64_t scale_word_blocks(const WordParams &wp) { return (int64_t)wp.row_blocks * (wp.slots / 4); }
inline int launch_scale_words(const uint8_t *eA, int64_t ldA, int64_t M, const uint8_t *eB, int64_t ldB, int64_t N, int slots,
                              uint32_t a_or, uint32_t *wA, uint32_t *wB, const int *run_a, const int *run_b,
                              hipStream_t s) {
    const WordParams wp = scale_word_params(eA, ldA, M, eB, ldB, N, slots, a_or, wA, wB, run_a, run_b);
    if (scale_word_blocks(wp) > 0x7fffffff) return HBFP_ERR_ARG;
    hipLaunchKernelGGL(scale_words_t_kernel, dim3((unsigned)scale_word_blocks(wp), 1, 2), dim3(256), 0, s, wp);
    return launch_status();
}

}  // namespace
}  // namespace hbfp
