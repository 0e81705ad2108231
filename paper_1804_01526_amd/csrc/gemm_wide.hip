// BFP matrix product with one exponent per operand row (the basic scheme of Sec. 4: "one exponent per row
// of A and per column of B", Eq. (2) with a single block):
//     C[i][j] = 2^(eA[i] + eB[j]) * sum_k mA[i][k] * mB[j][k]
// Here nothing happens between the matrix instructions of a tile: the whole contraction is one chain of
// v_mfma_i32_32x32x32_i8 into int32 accumulators and the two exponents are applied once, when C is stored.
// The kernel is therefore built for the matrix core alone: four waves of 32 T x 32 T, T = 4 (a tile of 256 x 256 of C
// per workgroup, 256 int32 accumulators per lane at one wave per SIMD, a pair of matrix instructions needs one 16-byte
// LDS read per lane: 64 B/clk per CU at the full matrix rate, where a 64 x 128 wave tile would need 94 of the 128 the
// LDS can deliver), 3 or 2 (128 x 128, two workgroups per CU).  Large products are bound by the chip's power (3001 x 4500 x
// 2999 on T = 3: matrix instructions 70 % of the loop's clocks at 1.7 GHz; 2.3 us until the first stage is there, 34 us of
// loop, 10 us in which all compute units store C at once) and go furthest on the largest tile; the smaller ones fill the chip
// where those are too few, and long contractions of few tiles are split (wide_plan).  Operands are read as they are stored
// (int8 [rows][kpad]): 128 bytes of k of the tile's rows per stage, whole cache lines, or 64 where those do not pay (launch_gemm_wide),
// copied global -> LDS asynchronously into a ring of two to four stages, rows of 128 (64) bytes with the 16-byte chunk index XORed with
// (row >> 1) & 7 ((row >> 2) & 3), so that copies and the fragment reads of 16 rows cover all banks.  Fragments are read one k-step (32)
// ahead, between the matrix instructions, and the hand-over of a ring buffer (one barrier per stage) sits in the stage's last
// k-step.
#include "gemm_common.h"

namespace hbfp {
namespace {

constexpr int kWideThreads = 256;
// T: 32 x 32 tiles along a side of a wave's part of C; the workgroup's tile is 64 T x 64 T.  K: bytes of k per stage and operand row,
// RING: stages in LDS.
template <int T, int K, int RING>
struct Wide {
    static constexpr int kRows = 64 * T;
    static constexpr int kChunks = K / 16, kSteps = K / 32;
    static constexpr int kOperand = kRows * K;           // 32 KB for T = 4
    static constexpr int kStage = 2 * kOperand;
    static constexpr int kLds = RING * kStage;
    static constexpr int kCopies = kStage / 1024 / 4;    // copies of 1 KB per wave and stage
    // Stages ahead of the one multiplied from.  Of 128 bytes: RING, the hand-over waits for the wave's last fragments and frees the
    // stage's own buffer.  Of 64, whose last k-step has too little left to hide that wait behind: RING - 1, the hand-over comes a row
    // earlier and frees the buffer of the stage before (1704 x 2914 x 811 13.6 -> 12.8 us).
    static constexpr bool kOwn = K == 128;
    static constexpr int kAhead = kOwn ? RING : RING - 1;
    // rows of K bytes whose 16-byte chunks are exchanged so that the reads of 16 consecutive rows at one k cover all banks
    static __device__ __forceinline__ int swizzle(int row) { return K == 128 ? (row >> 1) & 7 : (row >> 2) & 3; }
};

struct WideParams {
    const uint8_t *A, *B;        // int8 mantissas [rows][kpad]
    const uint8_t *eA, *eB;      // exponent bytes [rows][exp_ld], block 0
    float *C;
    int64_t M, N, kpad, eA_ld, eB_ld, ldc;
    int32_t *partial;            // split along k: int32 sums [splits][M][N]
    int32_t nstage;              // kpad / K
    int32_t splits, stages_per_split;
    int32_t tiles_m, tiles_n, beta;
    int32_t exp_offset;          // C = acc * 2^(Ea + Eb + exp_offset)
    const int *run_a, *run_b;
};

// STREAM: how C leaves (stores_stream)
template <int T, int K, int RING, bool STREAM>
__global__ __launch_bounds__(kWideThreads, T == 4 ? 1 : 2) void gemm_i8_wide_kernel(const WideParams p) {
    typedef Wide<T, K, RING> W;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    if (stands_down(p.run_a, p.run_b)) return;
    int tm, tn, split = blockIdx.y;
    if (p.splits >= 8 ? !tile_and_split_of_workgroup(blockIdx.x, p.tiles_m, p.tiles_n, p.splits, tm, tn, split)
                      : !tile_of_workgroup(blockIdx.x, p.tiles_m, p.tiles_n, tm, tn))
        return;                                                                 // whole workgroup, before any barrier
    const int st_begin = split * p.stages_per_split;
    const int nstage = p.nstage - st_begin < p.stages_per_split ? p.nstage - st_begin : p.stages_per_split;   // at least 1

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int l32 = lane & 31, lh = lane >> 5;
    const int64_t row0 = (int64_t)tm * W::kRows, col0 = (int64_t)tn * W::kRows;

    // ---- exponents: thread t keeps row t's and column t's until C is stored
    const int64_t row_t = row0 + (t < W::kRows ? t : 0), col_t = col0 + (t < W::kRows ? t : 0);
    const int ea_t = p.eA[(row_t < p.M ? row_t : p.M - 1) * p.eA_ld], eb_t = p.eB[(col_t < p.N ? col_t : p.N - 1) * p.eB_ld];

    // ---- copies: piece c of a stage is 1 KB, 8 rows x 128 or 16 rows x 64 bytes; the first half are pieces of A, the others of B; wave w
    // moves pieces w, w + 4, ...  A lane copies 16 bytes: LDS chunk lane % kChunks of its row, which holds source chunk
    // (lane % kChunks) ^ swizzle(row).  Rows past the edge re-read the last row (their results are never stored).
    constexpr int kPieces = W::kOperand / 1024;
    const uint8_t *cbase[W::kCopies];
    uint32_t cvoff[W::kCopies], coff[W::kCopies];
#pragma unroll
    for (int i = 0; i < W::kCopies; ++i) {
        const int c = wave + 4 * i;
        const bool is_a = c < kPieces;
        const int r = (is_a ? c : c - kPieces) * (1024 / K) + lane / W::kChunks;
        const int64_t lim = is_a ? p.M - row0 : p.N - col0;
        const int rr = r < lim ? r : (int)lim - 1;
        const int chunk = (lane % W::kChunks) ^ W::swizzle(r);
        cbase[i] = (is_a ? p.A + row0 * p.kpad : p.B + col0 * p.kpad) + (int64_t)st_begin * K;
        cvoff[i] = (uint32_t)rr * (uint32_t)p.kpad + chunk * 16;
        coff[i] = c * 1024;
    }
#define HBFP_WIDE_COPY(i, ring_)                                                                    \
    {                                                                                              \
        async_copy16(cbase[i], cvoff[i], (uint32_t)((ring_) * W::kStage) + coff[i]);              \
        cbase[i] += K;                                                                         \
    }
#define HBFP_WIDE_COPY_STAGE(ring_)                                                                 \
    {                                                                                              \
        _Pragma("unroll") for (int i = 0; i < W::kCopies; ++i) HBFP_WIDE_COPY(i, ring_);          \
    }

    // ---- fragment addresses inside a stage: row tile i of A is rows 32 T wm + 32 i + l32, k-step s the chunks 2 s + lh
    int fa[W::kSteps], fb[W::kSteps];                 // per k-step: byte offset of (row tile 0, this lane); tiles are 32 rows apart
    {
        const int ra = 32 * T * wm + l32, rb = 32 * T * wn + l32;
#pragma unroll
        for (int s = 0; s < W::kSteps; ++s) {
            fa[s] = ra * K + (((2 * s + lh) ^ W::swizzle(ra)) * 16);
            fb[s] = W::kOperand + rb * K + (((2 * s + lh) ^ W::swizzle(rb)) * 16);
        }
    }

    v16i acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    v4i a[2][T], b[2][T];                               // [buffer][tile]
#define HBFP_WIDE_FENCE                 \
    asm volatile("" ::: "memory");      \
    __builtin_amdgcn_sched_barrier(0)
#define HBFP_WIDE_READ(buf, base_, s, i)                                                                       \
    {                                                                                                         \
        a[buf][i] = *reinterpret_cast<const v4i *>((base_) + fa[s] + (i) * 32 * K);                        \
        b[buf][i] = *reinterpret_cast<const v4i *>((base_) + fb[s] + (i) * 32 * K);                        \
    }
#define HBFP_WIDE_ROW(buf, i)                                                                                  \
    {                                                                                                         \
        _Pragma("unroll") for (int j = 0; j < T; ++j)                                                         \
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[buf][i], b[buf][j], acc[i][j], 0, 0, 0);      \
    }
    // one k-step of 32: T x T matrix instructions on buffer `buf`; after each row of them, one row tile and one column
    // tile of the next k-step are requested into the other buffer.  HAND: the hand-over sits behind the first row, or in front
    // of it; COPY: the copies into the ring buffer that it frees ride along
#define HBFP_WIDE_KSTEP(buf, NEXT, nbase_, ns, HAND, COPY)                                                      \
    {                                                                                                         \
        _Pragma("unroll") for (int i_ = 0; i_ < T; ++i_) {                                                    \
            if (i_ == 0 && !W::kOwn) { HAND; }                                                                \
            HBFP_WIDE_ROW(buf, i_);                                                                           \
            if (i_ == 0 && W::kOwn) { HAND; }                                                                 \
            if (NEXT) HBFP_WIDE_READ(1 - (buf), nbase_, ns, i_);                                              \
            if (COPY) { _Pragma("unroll") for (int c_ = 0; c_ < W::kCopies / T; ++c_) HBFP_WIDE_COPY(W::kCopies / T * i_ + c_, taken); } \
            HBFP_WIDE_FENCE;                                                                                  \
        }                                                                                                     \
    }
    // A stage is kSteps k-steps; the fragments of its first were requested during the stage before.  The hand-over, in its last: this
    // wave has its last fragments of the stage (kOwn; otherwise those of the stage before, which it has multiplied), and its copies of
    // the next stage have landed when only those of the AFTER stages behind it are in flight; after the barrier that holds for
    // everybody, and the buffer of the stage (or of the one before) takes the copies of stage st + kAhead (COPY).  LAST: nothing follows.
#define HBFP_WIDE_STAGE(AFTER, COPY, LAST)                                                                     \
    {                                                                                                         \
        const uint8_t *base = lds + ring * W::kStage;                                                        \
        const int next = ring + 1 == RING ? 0 : ring + 1, taken = W::kOwn ? ring : ring == 0 ? RING - 1 : ring - 1; \
        _Pragma("unroll") for (int s_ = 0; s_ < W::kSteps - 1; ++s_)                                          \
            HBFP_WIDE_KSTEP(s_ & 1, true, base, s_ + 1, {}, false);                                           \
        HBFP_WIDE_KSTEP(1, !(LAST), lds + next * W::kStage, 0, {                                              \
            if (!(LAST)) {                                                                                    \
                if (W::kOwn) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((AFTER) * W::kCopies) : "memory"); \
                else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AFTER) * W::kCopies) : "memory");              \
                __builtin_amdgcn_s_barrier();                                                                 \
                asm volatile("" ::: "memory");                                                                \
            }                                                                                                 \
        }, COPY);                                                                                             \
        ring = next;                                                                                          \
    }

    // prologue: up to three stages on their way (with two, contractions of 2 to 20 stages on 192 x 192 tiles take 1 % longer), the
    // fragments of k-step 0 when the first has landed, then the fourth stage
    HBFP_WIDE_COPY_STAGE(0);
    if (W::kAhead > 2 && nstage > 2) {
        HBFP_WIDE_COPY_STAGE(1);
        HBFP_WIDE_COPY_STAGE(2);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * W::kCopies) : "memory");
    } else if (nstage > 1) {
        HBFP_WIDE_COPY_STAGE(1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(W::kCopies) : "memory");
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < T; ++i) HBFP_WIDE_READ(0, lds, 0, i);
    __builtin_amdgcn_sched_barrier(0);                            // (the copies in front of the reads: 1 % more)
    if (W::kAhead > 3 && nstage > 3) HBFP_WIDE_COPY_STAGE(3);
    int ring = 0;
    int st = 0;
    for (; st + W::kAhead < nstage; ++st) HBFP_WIDE_STAGE(W::kAhead - 2, true, false);
    if (W::kAhead > 3 && nstage - st == 4) {
        HBFP_WIDE_STAGE(2, false, false);
        ++st;
    }
    if (W::kAhead > 2 && nstage - st == 3) {
        HBFP_WIDE_STAGE(1, false, false);
        ++st;
    }
    if (nstage - st == 2) HBFP_WIDE_STAGE(0, false, false);
    HBFP_WIDE_STAGE(0, false, true);
#undef HBFP_WIDE_STAGE
#undef HBFP_WIDE_KSTEP
#undef HBFP_WIDE_ROW
#undef HBFP_WIDE_READ
#undef HBFP_WIDE_FENCE
#undef HBFP_WIDE_COPY_STAGE
#undef HBFP_WIDE_COPY

    // ---- C = acc * 2^(Ea + Eb + offset): int32 -> FP32 rounds to nearest even above 2^24, the scaling is exact.  The exponent
    // bytes come through LDS: loaded here, between stores that they could alias, every row waited for its own.
    __syncthreads();                                        // everybody has read the last stage
    int *exps = reinterpret_cast<int *>(lds);               // of the rows, then of the columns
    if (t < W::kRows) {
        exps[t] = ea_t > 254 ? 254 : ea_t;
        exps[W::kRows + t] = (eb_t > 254 ? 254 : eb_t) + p.exp_offset;
    }
    __syncthreads();
    int eb[T];
#pragma unroll
    for (int j = 0; j < T; ++j) eb[j] = exps[W::kRows + 32 * T * wn + 32 * j + l32];
    const int *ea = exps + 32 * T * wm + 4 * lh;
    const int64_t i0 = row0 + 32 * T * wm, j0 = col0 + 32 * T * wn;
    if (T == 2 && p.splits > 1) {                           // bit patterns of the int32 sums
        store_result<T, T, false>(reinterpret_cast<float *>(p.partial) + ((int64_t)split * p.M + i0) * p.N + j0, p.N, p.M - i0, p.N - j0, false,
                                  lane, [&](int i, int j, int v) { return __int_as_float(acc[i][j][v]); });
        return;
    }
    store_result<T, T, STREAM>(p.C + i0 * p.ldc + j0, p.ldc, p.M - i0, p.N - j0, p.beta != 0, lane, [&](int i, int j, int v) {
        return __builtin_amdgcn_ldexpf((float)acc[i][j][v], ea[32 * i + 8 * (v >> 2) + (v & 3)] + eb[j]);
    });
}

// The sum of the slices of a product split along k: int32, so any order gives the same bits, those of the unsplit product.
// A thread sums four outputs 256 apart, eight slices in flight each.
__global__ __launch_bounds__(256) void wide_sum_kernel(const WideParams p) {
    if (stands_down(p.run_a, p.run_b)) return;
    const int64_t n = p.M * p.N;
    const int64_t e0 = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    int sum[4] = {0, 0, 0, 0};
    for (int z = 0; z < p.splits; z += 8) {
        int v[4][8];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < 8; ++k) v[u][k] = e0 + u * 256 < n && z + k < p.splits ? p.partial[(int64_t)(z + k) * n + e0 + u * 256] : 0;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < 8; ++k) sum[u] += v[u][k];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t e = e0 + u * 256;
        if (e >= n) return;
        const int64_t row = n < ((int64_t)1 << 31) ? (int64_t)((uint32_t)e / (uint32_t)p.N) : e / p.N, col = e - row * p.N;
        const int ea = p.eA[row * p.eA_ld], eb = p.eB[col * p.eB_ld];
        const float val = __builtin_amdgcn_ldexpf((float)sum[u], (ea > 254 ? 254 : ea) + (eb > 254 ? 254 : eb) + p.exp_offset);
        float *dst = p.C + row * p.ldc + col;
        *dst = p.beta ? *dst + val : val;
    }
}

template <int T, int K, int RING>
int launch_wide_t(WideParams p, bool stream, hipStream_t s) {
    static std::atomic<bool> configured[2];
    constexpr int lds_bytes = Wide<T, K, RING>::kLds;
    void (*const kernel)(WideParams) = stream ? &gemm_i8_wide_kernel<T, K, RING, true> : &gemm_i8_wide_kernel<T, K, RING, false>;
    if (allow_dynamic_lds(configured[stream], reinterpret_cast<const void *>(kernel), lds_bytes) != HBFP_OK) return HBFP_ERR_LAUNCH;
    p.nstage *= 128 / K;
    p.stages_per_split *= 128 / K;
    const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n;
    const dim3 grid = p.splits >= 8 ? dim3((unsigned)(8 * tiles * ceil_div(p.splits, 8))) : dim3((unsigned)(ceil_div(tiles, 8) * 8), (unsigned)p.splits);
    hipLaunchKernelGGL(kernel, grid, dim3(kWideThreads), lds_bytes, s, p);
    return launch_status();
}

// Tile and split of a product: the smallest estimate in us.  A launch costs `base`; a workgroup `step` per 64 bytes of k, more
// the more of the chip is busy (power and L2), and `tail` for filling the ring and storing its tile.  Tiles of 256 and 192 have
// a compute unit to themselves and go in rounds, of 128 two share one.  Fitted to 99 shapes of 1 to 8192 rows and contractions
// of 64 to 59 635: 0.7 % behind the best of the three on average, 19 % at the worst (1069 x 5990 x 3765).  Against the kernel of
// blocks of 128 and more on 128 x 128 tiles, which all products of fewer than 128 tiles of 256 x 256 took before, 32 % ahead on
// average: 2048 x 4096 x 2048 34.6 -> 24.6 us, 1024 x 2048 x 1024 16.1 -> 10.0, 16 x 4096 x 4096 26.2 -> 15.8; 256 x 256 ->
// 192 x 192 tiles 3001 x 4500 x 2999 (144 -> 256 tiles) 64.6 -> 51.9 us, 1826 x 3178 x 3145 41.3 -> 32.4.
struct WidePlan {
    int T, splits;
};
WidePlan wide_plan(int64_t M, int64_t N, int64_t nstage, bool may_split) {
    static const double base[3] = {3.1, 1.6, 5.1}, lone[3] = {0.17, 0.30, 0.48}, full[3] = {0.32, 0.50, 0.86}, tail[3] = {3.0, 8.4, 10.9};
    WidePlan best = {2, 1};
    double least = 0.0;
    for (int t = 0; t < 3; ++t) {
        const int64_t tiles = ceil_div(M, 64 * (t + 2)) * ceil_div(N, 64 * (t + 2));
        for (int s = 1; s <= 64; ++s) {
            if (s > 1 && (t > 0 || !may_split || nstage / s < 8 || tiles * s > 512)) break;
            if (s > 8 && s % 8) continue;                       // the k ranges are dealt to the 8 XCDs in turn: keep them level
            const double wgs = (double)(tiles * s), per_cu = (double)(s < 8 ? ceil_div(tiles, 8) * s : tiles * ceil_div(s, 8)) / 32.0;
            const double busy = wgs < 256.0 ? wgs / 256.0 : 1.0, step = lone[t] + busy * (full[t] - lone[t]);
            const double load = t == 0 ? (per_cu > 1.0 ? per_cu : 1.0) : (double)ceil_div((int64_t)(per_cu * 32.0), 32);
            double us = base[t] + load * ((double)(ceil_div(nstage / 2, s) * 2) * step + tail[t]);
            if (s > 1) us += 3.0 + (double)(s + 1) * (double)(M * N) * 4e-6 / 3.0;
            if ((t == 0 && s == 1) || us < least) least = us, best = {t + 2, s};
        }
    }
    return best;
}

}  // namespace

// One exponent per operand row, 8-bit mantissas, rows of the stored operands addressable with 32-bit offsets
bool gemm_wide_possible(const GemmArgs &a) {
    return !a.P && a.nblk == 1 && a.mA <= 8 && a.mB <= 8 && (uint64_t)255 * (uint64_t)a.kpad + 64 < ((uint64_t)1 << 32) &&
           ceil_div(a.M, 128) * ceil_div(a.N, 128) <= 0x7ffffff0 && a.kpad / 64 <= 0x7fffffff;
}

// ... and a contraction longer than 64, or enough full tiles of 256 x 256 to fill the chip (below, the kernels of short blocks
// scale once per workgroup too)
bool gemm_wide_ok(const GemmArgs &a) {
    if (!gemm_wide_possible(a)) return false;
    if (a.kbp >= 128) return true;
    const int64_t tiles = ceil_div(a.M, 256) * ceil_div(a.N, 256);
    return tiles >= 128 && (double)a.M * (double)a.N >= 0.75 * 65536.0 * (double)tiles;
}

// slices of a product split along k; a stand-by launch is not split, nor one whose caller brought no room for them
size_t gemm_wide_workspace(const GemmArgs &a) {
    const WidePlan plan = wide_plan(a.M, a.N, a.kpad / 64, !a.run_a && !a.unsplit);
    return plan.splits > 1 ? (size_t)plan.splits * (size_t)a.M * (size_t)a.N * 4 : 0;
}

int launch_gemm_wide(const GemmArgs &a, void *workspace, hipStream_t s) {
    const WidePlan plan = wide_plan(a.M, a.N, a.kpad / 64, !a.run_a && !a.unsplit);
    if (plan.splits > 1 && !workspace) return HBFP_ERR_WORKSPACE;
    WideParams p = {};
    p.A = (const uint8_t *)a.mantA;
    p.B = (const uint8_t *)a.mantB;
    p.eA = a.expA;
    p.eB = a.expB;
    p.C = a.C;
    p.partial = (int32_t *)workspace;
    p.M = a.M;
    p.N = a.N;
    p.kpad = a.kpad;
    p.eA_ld = a.expA_ld;
    p.eB_ld = a.expB_ld;
    p.ldc = a.ldc;
    p.nstage = (int32_t)(a.kpad / 128);                          // in stages of 128 bytes here
    p.stages_per_split = (int32_t)ceil_div(p.nstage, plan.splits);
    p.splits = (int32_t)ceil_div(p.nstage, p.stages_per_split);
    p.tiles_m = (int32_t)ceil_div(a.M, 64 * plan.T);
    p.tiles_n = (int32_t)ceil_div(a.N, 64 * plan.T);
    p.beta = a.beta != 0.0f;
    p.exp_offset = -250 - a.mA - a.mB;
    p.run_a = a.run_a;
    p.run_b = a.run_b;
    // Only contractions up to 1024 end in so much of a burst that ordinary stores pay for what C takes of the last-level cache from the
    // conversions beside the product (conversions and product, streaming -> ordinary: 3001 x 600 x 2999 29.3 -> 26.9 us, 5000 x 1024 x
    // 4001 54.6 -> 54.1, 4100 x 1024 x 2501 38.9 -> 34.7, but 5000 x 1200 x 4001 60.5 -> 63.7, 3001 x 4500 x 2999 86.9 -> 88.4)
    const bool stream = a.kpad > 1024 || stores_stream(&a);
    // Stages of whole cache lines (128 bytes a row) halve the requests of 64, but the first is twice as much to wait for, and the chip
    // asks for all first stages at once: they pay where a workgroup has enough of them, or a compute unit another workgroup to turn
    // to.  64 -> 128, in stages of 128:
    //   128 x 128, two workgroups on a compute unit (a ring of two is enough): up to 512 from 10, or 6 with more than 400, 1826 x 3178 x
    //   3145 31.8 -> 27.5 us, 535 x 6827 x 2014 19.3 -> 17.6, 1947 x 3347 x 718 14.6 -> 13.6; 2254 x 2228 x 917 14.8 -> 15.5.  More
    //   than 512: 7 and 8, and from 20 on, 4265 x 2872 x 920 27.5 -> 25.1, 3320 x 5698 x 4356 120 -> 106; 7445 x 1553 x 468 17.4 ->
    //   18.2, 2657 x 3534 x 2002 36.6 -> 38.4
    //   128 x 128, one (a ring of four): from 25, 2709 x 848 x 3095 17.4 -> 16.6, 600 x 6000 x 5000 27.5 -> 26.2, 365 x 4670 x 6800
    //   32.8 -> 27.9; 224 x 4343 x 2613 13.8 -> 15.2, 1000^3 9.8 -> 10.5.  At most four rows of tiles, one column or fewer than 64
    //   tiles: from 33, 256 x 5120 x 5120 27.2 -> 20.8; 256 x 4096 x 4096 14.9 -> 16.7, 326 x 3601 x 3843 16.7 -> 18.0
    //   192 x 192 (a ring of three): from 9 with most of the chip busy, 1661 x 5106 x 10233 92 -> 86, 3001 x 2999 x 3001 38.2 -> 36.4,
    //   6000^3 230 -> 209; 1543 x 4809 x 423 14.2 -> 14.5; with less of it 1283 x 4381 x 3908 32.8 -> 35.2, 3673 x 2042 x 4843 45 both
    //   256 x 256 (two): 8192^3 468 -> 451, 8192 x 8192 x 512 98.8 -> 95; with less of the chip busy fewer than 20, 4580 x 2944 x 880
    //   29.8 -> 28.7; 3543 x 3523 x 3371 59.2 -> 61.5, 1704 x 5736 x 5564 69 -> 76
    const int64_t wgs_all = (int64_t)p.tiles_m * p.tiles_n * p.splits;
    const int stages = p.stages_per_split;
    const bool few = p.tiles_m <= 4 || p.tiles_n == 1 || wgs_all < 64;
    const int rc = plan.T == 4   ? (wgs_all >= 240 || stages < 20 ? launch_wide_t<4, 128, 2>(p, stream, s) : launch_wide_t<4, 64, 4>(p, stream, s))
                   : plan.T == 3 ? (wgs_all >= 228 && stages >= 9 ? launch_wide_t<3, 128, 3>(p, stream, s) : launch_wide_t<3, 64, 4>(p, stream, s))
                   : wgs_all > 256
                       ? (stages >= 20 || (wgs_all > 512 ? stages == 7 || stages == 8 : stages >= (wgs_all > 400 ? 6 : 10))
                              ? launch_wide_t<2, 128, 2>(p, stream, s)
                              : launch_wide_t<2, 64, 4>(p, stream, s))
                       : (stages >= (few ? 33 : 25) ? launch_wide_t<2, 128, 4>(p, stream, s) : launch_wide_t<2, 64, 4>(p, stream, s));
    if (rc != HBFP_OK || p.splits == 1) return rc;
    const int64_t wgs = ceil_div(a.M * a.N, 1024);
    if (wgs > 0x7fffffff) return HBFP_ERR_ARG;
    hipLaunchKernelGGL(wide_sum_kernel, dim3((unsigned)wgs), dim3(256), 0, s, p);
    return launch_status();
}

}  // namespace hbfp
