// Convolution as a matrix product whose activation operand stays in LDS over the filter taps, on the bf16 matrix
// instruction (the operands of Sec. 5.1: an image converted once, 8-bit mantissas and less).
//
// The int8 kernel that gathers the image tap by tap (gemm.hip) spends two vector instructions on every output and exponent
// block, 328 of the 520 clocks that a k-step of 32 costs a SIMD (vector and matrix instructions of a SIMD do not overlap
// on this chip), and a mantissa times its block's power of two is a bf16 number, which needs none of them: 256 clocks.  What keeps
// plain products on int8 - converting an operand inside the product costs as much as it saves - does not hold for a convolution:
// consecutive output positions and all taps of the window read the same pixels, so a workgroup converts the strip of image
// that its 256 output positions meet once per 64 channels, and the r * s taps multiply from it.
//
// A workgroup of four waves computes up to 256 positions x 128 filters, or 192 x 192 (each wave half of either).  Per chunk of two stored channel blocks
// it reads the strip - pixels are consecutive in memory, whole rows of the image with what lies left and right of the window -
// converts it to bf16 (3 instructions an element) and stores it in LDS as [pixel][channels] at a pitch of an odd number of 16 bytes, where the
// fragments of 16 consecutive pixels cover all banks whatever the tap.  Fragments of positions whose tap lies outside the image
// are read from a pixel of zeros.  The filters come as bf16 panels that a small kernel has laid out in the order in which they
// are used; each wave loads its fragments straight from the caches (every one serves four matrix instructions), a tap
// ahead.  One barrier before and one behind each strip; two workgroups per compute unit cover each other's conversions.
// The int8 kernel -> this one, each with its launch in front, on the same operands again and again: 128 x 28 x 28 x 128, 128 filters of
// 3 x 3 52.4 -> 31.3 us (delivered encoded 55.2 -> 35.8), 64 x 28 x 28 x 144, 144 filters, blocks of 24 59.8 -> 30.7; with other inputs
// in turn the kernels take 30.5 + 5.1 us (36.3 + 5.1) and 31.5 + 3.9.  The matrix instructions alone would take 13 and 11 us: all
// workgroups start together, store together (51 MB, 10 us) and wait for their first strip together.  Panels that go through a ring in
// LDS, where two waves share a fragment, cost a barrier per tap and more than they save (38 and 40 us); a higher priority for one of
// the two workgroups of a compute unit changes nothing.  Blocks of other lengths than
// 24 and 32 have no instance here and run on the int8 kernel.
#include <atomic>

#include "bf_pack.h"
#include "hbfp_internal.h"
#include "mx_out.h"

namespace hbfp {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int kStripThreads = 256;
constexpr int kStripUnit = 64;                   // output positions: 32 for each of the two waves along them
constexpr int kStripLds = 80 * 1024;             // two workgroups per compute unit
constexpr int strip_units_most(int nt) { return nt == 2 ? 4 : 3; }

struct StripParams {
    const uint8_t *img, *eimg;   // int8 mantissas [pixels][pix_bytes], exponent bytes [pixels][eimg_ld], a stored block of 32 bytes each
    const uint8_t *panels;       // filters as bf16: [32 filters][step][lane][8 values]
    float *C;
    int64_t pix_bytes, eimg_ld, ldc, M, N;
    float inv_wo, inv_ho;        // 1 / Wo, 1 / Ho
    int32_t H, W, Ho, Wo, S, taps, pad_h, pad_w, str_h, str_w, pixels;
    int32_t ncb;                 // stored blocks per pixel
    int32_t steps;               // matrix instructions' steps of 16 of a whole contraction
    int32_t tail;                // pixels of the strip behind the last position's corner
    int32_t zero_at;             // LDS offset of the pixel of zeros
    int32_t units, slots, tiles_n;   // units of 64 positions; workgroups per XCD along them and, times tiles_n, in all
    int32_t beta, m;
    MxOut enc;                   // ENC only
};

// Filters -> panels.  A lane makes 8 values: filter 32 tile + lane % 32, channels 16 step + 8 (lane / 32) of the chunk.  A workgroup has
// one tap of a chunk and one column tile, a wave each of its steps: what it reads is known after one division of scalars.  Bound by
// its latency; with four 64-bit divisions per lane, from a running number of the piece, 1296 x 144 in blocks of 24 took 4.1 us
// (3.0 now), 1152 x 128 as long as now (5.0).
struct StripPanels {
    const uint8_t *mant, *exps;
    uint8_t *out;
    int64_t kpad, exp_ld, N;
    int32_t ncb, taps, by_block, m, steps;
};
template <int KS>
__global__ __launch_bounds__(64 * KS) void strip_panels_kernel(const StripPanels p) {
    const int lane = threadIdx.x & 63, step = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const uint32_t g = blockIdx.x, tile = blockIdx.y, chunk = g / (uint32_t)p.taps, tap = g - chunk * (uint32_t)p.taps;
    const int oct = 2 * step + (lane >> 5), cb = 2 * (int)chunk + (oct >= KS ? 1 : 0), in_block = oct >= KS ? oct - KS : oct;
    const int64_t f = (int64_t)tile * 32 + (lane & 31);
    v4u v = {0, 0, 0, 0};
    if (f < p.N && cb < p.ncb) {                                                  // (an odd number of blocks is filled up with zeros)
        const int64_t slot = p.by_block ? (int64_t)cb * p.taps + tap : (int64_t)tap * p.ncb + cb;
        const int e = p.exps[f * p.exp_ld + slot];
        v = bf_octet_i8(*reinterpret_cast<const v2i *>(p.mant + f * p.kpad + slot * 32 + in_block * 8), e > 254 ? 254 : e, p.m);
    }
    *reinterpret_cast<v4u *>(p.out + ((int64_t)tile * p.steps + (int64_t)g * KS + step) * 1024 + lane * 16) = v;
}

// 2^(biased - 127), subnormal for biased <= 0 (-22 at the least)
__device__ __forceinline__ float strip_unit(int biased) { return __uint_as_float(biased > 0 ? (uint32_t)biased << 23 : 1u << (22 + biased)); }
// an octet of int8 mantissas times the unit of their block as bf16 numbers (exact: at most 7 significant bits)
__device__ __forceinline__ v4u strip_octet(int w0, int w1, float unit) {
    v4u out;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int w = (i < 2 ? w0 : w1) >> (16 * (i & 1));
        const float lo = (float)(int8_t)w * unit, hi = (float)(int8_t)(w >> 8) * unit;
        out[i] = __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
    }
    return out;
}

// One wave's part of a workgroup: MT x NT results of 32 x 32 (MT: the workgroup's units, NT: column tiles of this wave).
// row0: the workgroup's first position, i0: this wave's, tile0: its first column tile.
template <int KS, int MT, int NT, bool ENC, bool STREAM>
__device__ __forceinline__ void strip_wave(const StripParams &p, uint8_t *lds, int64_t row0, int wm, int tile0, bool idle) {
    constexpr int kPitch = KS * 32 + 16;
    const int t = threadIdx.x, lane = t & 63;
    const int l32 = lane & 31, lh = lane >> 5;

    // the input pixel under filter tap (0, 0) of the output position `d` behind the workgroup's first, and its row and column (which may
    // lie outside).  Divisions of small numbers in FP32: exact, the host keeps Wo and Ho below 2^20.
    const uint32_t per_img = (uint32_t)(p.Ho * p.Wo), img0 = (uint32_t)row0 / per_img, rem0 = (uint32_t)row0 - img0 * per_img;
    const int oy0 = (int)(rem0 / (uint32_t)p.Wo), ox0 = (int)rem0 - oy0 * p.Wo;
    const auto corner = [&](int d, int &cy, int &cx) {
        const int dy = (int)(((float)(ox0 + d) + 0.5f) * p.inv_wo), y = oy0 + dy, di = (int)(((float)y + 0.5f) * p.inv_ho);
        cy = (y - di * p.Ho) * p.str_h - p.pad_h;
        cx = (ox0 + d - dy * p.Wo) * p.str_w - p.pad_w;
        return (((int)img0 + di) * p.H + cy) * p.W + cx;
    };
    const int rows = (int)(p.M - row0 < MT * kStripUnit ? p.M - row0 : MT * kStripUnit);
    int y_, x_;
    const int first = __builtin_amdgcn_readfirstlane(corner(0, y_, x_));
    const int units = 4 * (__builtin_amdgcn_readfirstlane(corner(rows - 1, y_, x_)) - first + p.tail);

    // ---- strip: a unit is 16 bytes of a pixel, half a stored block; a thread has kUnits of them in flight
    constexpr int kUnits = 5;
    v4i raw[kUnits];
    int e[kUnits];
    const auto request = [&](int chunk, int u0) {
#pragma unroll
        for (int i = 0; i < kUnits; ++i) {
            const int at = u0 + i * kStripThreads, u = at < units ? at : units - 1;   // (no branch: the loads leave together)
            int px = first + (u >> 2);
            px = px < 0 ? 0 : px >= p.pixels ? p.pixels - 1 : px;
            raw[i] = *reinterpret_cast<const v4i *>(p.img + px * p.pix_bytes + chunk * 64 + (u & 3) * 16);
            e[i] = p.eimg[px * p.eimg_ld + 2 * chunk + ((u >> 1) & 1)];
        }
    };
    const auto convert = [&](int u0) {
#pragma unroll
        for (int i = 0; i < kUnits; ++i) {
            const int u = u0 + i * kStripThreads, oct = 2 * (u & 1);             // of the block
            uint8_t *dst = lds + (u >> 2) * kPitch + (((u >> 1) & 1) * KS + oct) * 16;
            const float unit = strip_unit((e[i] > 254 ? 254 : e[i]) + 2 - p.m);
            const v4u lo = strip_octet(raw[i][0], raw[i][1], unit), hi = strip_octet(raw[i][2], raw[i][3], unit);
            if (u < units && oct < KS) *reinterpret_cast<v4u *>(dst) = lo;
            if (u < units && oct + 1 < KS) *reinterpret_cast<v4u *>(dst + 16) = hi;
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    request(0, t);

    // this lane's rows: where they sit in the strip, and which taps meet the image there (while the first loads are on their way)
    int abase[MT];
    uint32_t amask[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int d = wm * 32 * MT + 32 * i + l32;
        int cy, cx;
        abase[i] = (corner(d < rows ? d : rows - 1, cy, cx) - first) * kPitch + lh * 16;
        const int lo = cx < 0 ? -cx : 0, hi = p.W - cx < p.S ? p.W - cx : p.S;   // columns lo .. hi - 1 of the window
        const uint32_t cols = hi > lo ? (0xffffffffu >> (32 - hi)) & ~((1u << lo) - 1u) : 0;
        amask[i] = 0;
        for (int fr = 0, at = 0; at < p.taps; ++fr, at += p.S)
            if ((unsigned)(cy + fr) < (unsigned)p.H) amask[i] |= cols << at;
    }
    const int zero = p.zero_at + lh * 16;
    if (t < kPitch / 16) *reinterpret_cast<v4u *>(lds + p.zero_at + t * 16) = v4u{0, 0, 0, 0};

    // filters: a tile past the last column re-reads the last one (its products are not stored); the loads are bounded by the buffer
    const int tiles32 = (int)((p.N + 31) / 32), taps = idle ? 0 : p.taps;
    const __amdgpu_buffer_rsrc_t panels = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.panels), 0, (tiles32 * p.steps + 4) * 1024, 0x00020000);
    int pb[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) pb[j] = (tile0 + j < tiles32 ? tile0 + j : tiles32 - 1) * p.steps * 1024;
    const auto filters = [&](int at) { return __builtin_bit_cast(v8bf, __builtin_amdgcn_raw_buffer_load_b128(panels, lane * 16, at, 0)); };

    constexpr int kAcc = ENC ? (MT + 1) / 2 * 2 : MT;                            // (the encoding takes two row tiles at a time)
    v16f acc[kAcc][NT];
#pragma unroll
    for (int i = 0; i < kAcc; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    const int chunks = (p.ncb + 1) / 2;
    for (int chunk = 0; chunk < chunks; ++chunk) {
        if (chunk) {
            request(chunk, t);
            __syncthreads();                                                     // everybody has read the chunk before
        }
        convert(t);
        for (int u0 = t + kUnits * kStripThreads; u0 - t < units; u0 += kUnits * kStripThreads) {
            request(chunk, u0);
            convert(u0);
        }
        // ---- the taps of the window
        v8bf b[KS][NT];
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int j = 0; j < NT; ++j) b[s][j] = filters(pb[j] + s * 1024);
        __syncthreads();
        // Fragments of A are requested one step ahead, each into the registers that its matrix instructions have just read: the
        // others of the step pass before it is used.  The compiler would request it right in front of its use.
        int fr = 0, fs = 0, off = 0;
        int pa[MT];
        v8bf a[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            pa[i] = amask[i] & 1 ? abase[i] : zero;
            a[i] = *reinterpret_cast<const v8bf *>(lds + pa[i]);
        }
        for (int tap = 0; tap < taps; ++tap) {
            off += kPitch;
            if (++fs == p.S) fs = 0, ++fr, off = fr * p.W * kPitch;
            const uint32_t bit = tap + 1 < taps ? 2u << tap : 0u;                // of the next tap
#pragma unroll
            for (int j = 0; j < NT; ++j) pb[j] += KS * 1024;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
#pragma unroll
                for (int i = 0; i < MT; ++i) {
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[i][j] = ENC ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[s][j], a[i], acc[i][j], 0, 0, 0)
                                        : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[s][j], acc[i][j], 0, 0, 0);
                    if (s == KS - 1) pa[i] = amask[i] & bit ? abase[i] + off : zero;
                    a[i] = *reinterpret_cast<const v8bf *>(lds + pa[i] + (s + 1) % KS * 32);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int j = 0; j < NT; ++j) b[s][j] = filters(pb[j] + s * 1024);   // of the next tap; behind the last one not used
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    const int64_t i0 = row0 + wm * 32 * MT, j0 = (int64_t)tile0 * 32;
    const int64_t end = p.M < i0 + 32 * MT ? p.M : i0 + 32 * MT;
    if constexpr (ENC) {
        static_assert(NT <= 2, "two column tiles at a time, the second one of zeros if there is none");
#pragma unroll
        for (int h = 0; h < MT; h += 2) {
            v16f two[2][2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) two[i][j][v] = j < NT ? acc[h + i][j < NT ? j : 0][v] : 0.0f;
            if (p.enc.rounding) mx_store_encoded<1, 2>(p.enc, two, i0 + 32 * h, j0, end, p.N, lane);
            else mx_store_encoded<0, 2>(p.enc, two, i0 + 32 * h, j0, end, p.N, lane);
        }
    } else if (!idle) {
        store_result<MT, NT, STREAM>(p.C + i0 * p.ldc + j0, p.ldc, end - i0, p.N - j0, p.beta != 0, lane, [&](int i, int j, int v) { return acc[i][j][v]; });
    }
}

// KS: steps of 16 per tap of a chunk (two blocks of 8 KS channels); NT: column tiles of a wave at most; ENC: the product leaves as the
// next layer's image.  The code of every number of units and of column tiles is its own: with tests inside the loops the
// accumulators did not stay in their registers.
template <int KS, int NT, bool ENC, bool STREAM>
__global__ __launch_bounds__(kStripThreads, 2) void gemm_strip_kernel(const StripParams p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    // Every XCD gets an eighth of the units and deals them to its slots; two workgroups that meet on a compute unit are 32 places
    // apart, so that the larger shares, which come first, meet smaller ones.
    const int xcd = blockIdx.x & 7, place = blockIdx.x >> 3;
    const int slot = place / p.tiles_n, tn = place - slot * p.tiles_n;
    const int from = (int)((int64_t)p.units * xcd / 8), share = (int)((int64_t)p.units * (xcd + 1) / 8) - from;
    const int base = share / p.slots, more = share - base * p.slots;
    const int mt = base + (slot < more ? 1 : 0);                                 // this workgroup's units
    const int64_t row0 = (int64_t)(from + base * slot + (slot < more ? slot : more)) * kStripUnit;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wm = wave & 1, wn = (wave >> 1) ^ ((place >> 5) & 1);              // (the other way round 32 places on: the same SIMDs)
    // The column tiles that hold filters, half of them for either wave (ENC: NT for the first, which encodes two together).  A wave
    // computes and stores its own ones alone: no column belongs to two waves (with beta both would add to it), and a tile without
    // filters costs as much as one with (128 x 28 x 28 x 128 with two tiles for every wave that has one -> now: 32 filters 26.7 ->
    // 16.8 us, delivered encoded 32.7 -> 22.5, 64 filters 25.9 -> 20.3, 96 32.8 -> 27.8, encoded 36.6 -> 34.0, 128 level).
    const int tiles32 = (int)((p.N + 31) / 32), here = tiles32 - 2 * NT * tn < 2 * NT ? tiles32 - 2 * NT * tn : 2 * NT;
    const int split = ENC || NT == 3 ? NT : (here + 1) / 2, own = wn ? here - split : here < split ? here : split;
    const int tile0 = 2 * NT * tn + wn * split;
    const bool idle = own <= 0;                                                  // this wave has no column to compute
    if constexpr (NT == 2) {
        const bool narrow = own == 1;                                            // (the barriers of both kinds of wave are the same)
        if (mt == 4) {
            if (narrow) strip_wave<KS, 4, 1, ENC, STREAM>(p, lds, row0, wm, tile0, idle);
            else strip_wave<KS, 4, NT, ENC, STREAM>(p, lds, row0, wm, tile0, idle);
        } else if (mt == 3) {
            if (narrow) strip_wave<KS, 3, 1, ENC, STREAM>(p, lds, row0, wm, tile0, idle);
            else strip_wave<KS, 3, NT, ENC, STREAM>(p, lds, row0, wm, tile0, idle);
        } else if (mt == 2) {
            if (narrow) strip_wave<KS, 2, 1, ENC, STREAM>(p, lds, row0, wm, tile0, idle);
            else strip_wave<KS, 2, NT, ENC, STREAM>(p, lds, row0, wm, tile0, idle);
        } else if (mt == 1) {
            if (narrow) strip_wave<KS, 1, 1, ENC, STREAM>(p, lds, row0, wm, tile0, idle);
            else strip_wave<KS, 1, NT, ENC, STREAM>(p, lds, row0, wm, tile0, idle);
        }
    } else {
        const bool narrow = own < NT;                                            // (tiles of 192 filters have five column tiles at least)
        if (mt == 3) {
            if (narrow) strip_wave<KS, 3, NT - 1, false, STREAM>(p, lds, row0, wm, tile0, idle);
            else strip_wave<KS, 3, NT, false, STREAM>(p, lds, row0, wm, tile0, idle);
        } else if (mt == 2) {
            if (narrow) strip_wave<KS, 2, NT - 1, false, STREAM>(p, lds, row0, wm, tile0, idle);
            else strip_wave<KS, 2, NT, false, STREAM>(p, lds, row0, wm, tile0, idle);
        } else if (mt == 1) {
            if (narrow) strip_wave<KS, 1, NT - 1, false, STREAM>(p, lds, row0, wm, tile0, idle);
            else strip_wave<KS, 1, NT, false, STREAM>(p, lds, row0, wm, tile0, idle);
        }
    }
}

// pixels that the strip of any workgroup holds at most: from the corner of its first position to the far corner of its last.
// Between neighbouring positions the corner moves by the stride, by more at the end of a row and of an image.
int64_t strip_pixels(const hbfp_conv2d &c, int64_t ho, int64_t wo, int64_t rows) {
    const int64_t per_row = c.stride_h * (int64_t)c.w - wo * c.stride_w, per_img = (c.h - ho * c.stride_h) * c.w;
    return (rows - 1) * (int64_t)c.stride_w + ceil_div(rows - 1, wo) * (per_row > 0 ? per_row : 0) +
           ceil_div(rows - 1, ho * wo) * (per_img > 0 ? per_img : 0) + (int64_t)(c.r - 1) * c.w + c.s;
}

// bytes of LDS: the strip of that many units of positions and the pixel of zeros
int64_t strip_lds(const hbfp_conv2d &c, int64_t ho, int64_t wo, int kblock, int units) {
    return (strip_pixels(c, ho, wo, kStripUnit * units) + 1) * (kblock / 8 * 32 + 16);
}

template <int KS, int NT, bool ENC>
int launch_strip_t(const StripParams &p, bool stream, int lds_bytes, hipStream_t s) {
    static std::atomic<bool> configured[2];
    void (*const kernel)(StripParams) = stream ? &gemm_strip_kernel<KS, NT, ENC, true> : &gemm_strip_kernel<KS, NT, ENC, ENC>;
    if (allow_dynamic_lds(configured[stream], reinterpret_cast<const void *>(kernel), kStripLds) != HBFP_OK) return HBFP_ERR_LAUNCH;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(8 * p.slots * p.tiles_n)), dim3(kStripThreads), lds_bytes, s, p);
    return launch_status();
}

// How the output is dealt: column tiles of 128 or 192 filters, whichever computes fewer columns that do not exist, and as many
// workgroups as fill 2 x 32 places of every XCD, once or as often as it takes with at most 256 (192) positions each.
int strip_nt(int64_t N) { return ceil_div(N, 128) * 128 <= ceil_div(N, 192) * 192 ? 2 : 3; }
struct StripPlan {
    int nt, tiles_n, units, slots;
};
StripPlan strip_plan(int64_t M, int64_t N, bool enc, int units_most) {
    StripPlan q;
    q.nt = enc ? 2 : strip_nt(N);
    q.tiles_n = (int)ceil_div(N, 64 * q.nt);
    q.units = (int)ceil_div(M, kStripUnit);
    const int64_t share = ceil_div(q.units, 8);
    for (int64_t rounds = 1;; ++rounds) {
        const int64_t slots = 64 * rounds / q.tiles_n;
        if (slots < 1 || ceil_div(share, slots) > units_most) continue;
        q.slots = (int)(slots < share ? slots : share);
        return q;
    }
}

// steps of 16: kblock / 8 per tap of two blocks
int strip_steps(int64_t ncb, int64_t kblock, int64_t taps) { return (int)(taps * ((ncb + 1) / 2) * (kblock / 8)); }

}  // namespace

// Whether the convolution runs on this kernel (a: as for launch_gemm_conv_i8; room: bytes of workspace, which holds the panels).  The
// answer is the same for a result delivered encoded, whose bytes are those of the FP32 result's conversion.
bool gemm_strip_ok(const GemmArgs &a, const hbfp_conv2d &c, int64_t ho, int64_t wo, int kblock, size_t room) {
    const int64_t taps = (int64_t)c.r * c.s;
    if ((kblock != 24 && kblock != 32) || c.c % kblock || taps > 32 || taps < 2) return false;
    // corners in increasing order, positions within one window of their input
    if (ho >= (1 << 20) || wo >= (1 << 20)) return false;
    if (2 * c.pad_h > c.r - 1 || 2 * c.pad_w > c.s - 1) return false;
    if (a.M > 0x7fffffff || a.N > 32 * 65535) return false;        // (column tiles are the panel launch's blockIdx.y)
    if (c.n * c.h * c.w > (1 << 30)) return false;                 // pixel numbers behind the last one, of a strip's end, fit an int
    if (strip_lds(c, ho, wo, kblock, strip_units_most(strip_nt(a.N))) > kStripLds) return false;
    const int64_t steps = strip_steps(c.c / kblock, kblock, taps);
    const size_t panels = ((size_t)ceil_div(a.N, 32) * steps + 4) * 1024;         // (addressed with 31 bits)
    if (panels > room || panels > 0x7fffffff) return false;
    // Below 128 tiles the start of a workgroup and its first strip count, and the int8 kernel splits long contractions.  int8 -> here with 129
    // tiles 27.6 -> 18.1 and 15.4 -> 12.7 us, 147 22.6 -> 16.6, 154 19.9 -> 12.6, 196 28.3 -> 20.5, 784 41.5 -> 36.0; with fewer it gains at
    // some and loses at others: 62 tiles 23.2 -> 17.7 and 19.0 -> 19.1, 74 17.0 -> 15.3 and, 2304 of k, 26.6 -> 28.0, 98 30.1 -> 30.7.
    // (Slots are at most an XCD's units, which with the column tiles bounds the grid.)
    return ceil_div(a.M, 256) * ceil_div(a.N, 128) >= 128 && ceil_div(a.M, 8 * kStripUnit) * ceil_div(a.N, 128) <= 0x7ffffff;
}

int launch_gemm_strip(const GemmArgs &a, const hbfp_conv2d &c, int64_t ho, int64_t wo, int64_t pix_bytes, bool by_block, int kblock, void *workspace,
                      hipStream_t s, const hbfp_tensor *enc, int relu) {
    StripPanels q = {};
    q.mant = (const uint8_t *)a.mantB;
    q.exps = a.expB;
    q.out = (uint8_t *)workspace;
    q.kpad = a.kpad;
    q.exp_ld = a.expB_ld;
    q.N = a.N;
    q.ncb = (int32_t)(c.c / kblock);
    q.taps = c.r * c.s;
    q.by_block = by_block;
    q.m = a.mB;
    q.steps = strip_steps(q.ncb, kblock, q.taps);
    const dim3 pieces((unsigned)(q.steps / (kblock / 8)), (unsigned)ceil_div(a.N, 32));
    if (kblock == 24) hipLaunchKernelGGL(strip_panels_kernel<3>, pieces, dim3(192), 0, s, q);
    else hipLaunchKernelGGL(strip_panels_kernel<4>, pieces, dim3(256), 0, s, q);
    if (launch_status() != HBFP_OK) return HBFP_ERR_LAUNCH;

    // An encoded result is computed on tiles of 128 filters, whose shares of four units need a longer strip than the three of tiles of
    // 192: three units there too where the fourth does not fit.
    const int most = !enc ? strip_units_most(strip_nt(a.N)) : strip_lds(c, ho, wo, kblock, 4) <= kStripLds ? 4 : 3;
    const StripPlan plan = strip_plan(a.M, a.N, enc != nullptr, most);
    const int lds_bytes = (int)strip_lds(c, ho, wo, kblock, most);
    StripParams p = {};
    p.img = (const uint8_t *)a.mantA;
    p.eimg = a.expA;
    p.panels = (const uint8_t *)workspace;
    p.C = a.C;
    p.pix_bytes = pix_bytes;
    p.eimg_ld = a.expA_ld;
    p.ldc = a.ldc;
    p.M = a.M;
    p.N = a.N;
    p.H = (int32_t)c.h;
    p.W = (int32_t)c.w;
    p.Ho = (int32_t)ho;
    p.Wo = (int32_t)wo;
    p.S = c.s;
    p.inv_wo = 1.0f / (float)wo;
    p.inv_ho = 1.0f / (float)ho;
    p.taps = q.taps;
    p.pad_h = c.pad_h;
    p.pad_w = c.pad_w;
    p.str_h = c.stride_h;
    p.str_w = c.stride_w;
    p.pixels = (int32_t)(c.n * c.h * c.w);
    p.ncb = q.ncb;
    p.steps = q.steps;
    p.tail = (int32_t)((c.r - 1) * c.w + c.s);
    p.zero_at = lds_bytes - (kblock / 8 * 32 + 16);
    p.units = plan.units;
    p.slots = plan.slots;
    p.tiles_n = plan.tiles_n;
    p.beta = a.beta != 0.0f;
    p.m = a.mA;
    if (enc) {
        p.enc = mx_out_of(*enc, relu);
        return kblock == 24 ? launch_strip_t<3, 2, true>(p, true, lds_bytes, s) : launch_strip_t<4, 2, true>(p, true, lds_bytes, s);
    }
    const bool stream = stores_stream(&a);
    if (plan.nt == 3) return kblock == 24 ? launch_strip_t<3, 3, false>(p, stream, lds_bytes, s) : launch_strip_t<4, 3, false>(p, stream, lds_bytes, s);
    return kblock == 24 ? launch_strip_t<3, 2, false>(p, stream, lds_bytes, s) : launch_strip_t<4, 2, false>(p, stream, lds_bytes, s);
}

}  // namespace hbfp
