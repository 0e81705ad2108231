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
// A workgroup of four waves computes 256 positions x 128 filters (each wave 128 x 64).  Per chunk of two stored channel blocks
// it reads the strip - pixels are consecutive in memory, whole rows of the image with what lies left and right of the window -
// converts it to bf16 (3 instructions an element) and stores it in LDS as [pixel][channels] at a pitch of an odd number of 16 bytes, where the
// fragments of 16 consecutive pixels cover all banks whatever the tap.  Fragments of positions whose tap lies outside the image
// are read from a pixel of zeros.  The filters come as bf16 panels that a small kernel has laid out in the order in which they
// are used; each wave loads its fragments straight from the caches (every one serves four matrix instructions), a tap
// ahead.  One barrier before and one behind each strip; two workgroups per compute unit cover each other's conversions.
#include <atomic>

#include "bf_pack.h"
#include "hbfp_internal.h"
#include "mx_out.h"

namespace hbfp {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int kStripThreads = 256;
constexpr int kStripRows = 256;                  // output positions of a workgroup
constexpr int kStripCols = 128;                  // filters of a workgroup
constexpr int kStripLds = 80 * 1024;             // two workgroups per compute unit

struct StripParams {
    const uint8_t *img, *eimg;   // int8 mantissas [pixels][pix_bytes], exponent bytes [pixels][eimg_ld], a stored block of 32 bytes each
    const uint8_t *panels;       // filters as bf16: [32 filters][step][lane][8 values]
    float *C;
    int64_t pix_bytes, eimg_ld, ldc, M, N;
    int32_t H, W, Ho, Wo, S, taps, pad_h, pad_w, str_h, str_w, pixels;
    int32_t ncb, octets;         // stored blocks per pixel, 8-channel pieces of a block
    int32_t steps;               // matrix instructions' steps of 16 of a whole contraction
    int32_t tail;                // pixels of the strip behind the last position's corner
    int32_t zero_at;             // LDS offset of the pixel of zeros
    int32_t tiles_m, tiles_n, beta, m;
    MxOut enc;                   // ENC only
};

// filters -> panels.  A lane makes 8 values: filter 32 nt + lane % 32, channels 16 step + 8 (lane / 32) of the chunk.
struct StripPanels {
    const uint8_t *mant, *exps;
    uint8_t *out;
    int64_t kpad, exp_ld, N;
    int32_t ncb, octets, taps, by_block, m, steps, full, last;   // full, last: steps per tap of a chunk of two blocks, of the last chunk
    int32_t tiles;
};
__global__ __launch_bounds__(256) void strip_panels_kernel(const StripPanels p) {
    const int lane = threadIdx.x & 63;
    const int64_t piece = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int nt = (int)(piece / p.steps), step = (int)(piece % p.steps);
    if (nt >= p.tiles) return;
    const int per_chunk = p.taps * p.full;
    int chunk = step / per_chunk, rest = step % per_chunk, per_tap = p.full;
    if (2 * chunk + 1 >= p.ncb || chunk * 2 >= p.ncb) {                          // the last chunk holds one block
        chunk = p.ncb / 2;
        rest = step - chunk * per_chunk;
        per_tap = p.last;
    }
    const int tap = rest / per_tap, oct = 2 * (rest % per_tap) + (lane >> 5);
    const int cb = 2 * chunk + oct / p.octets, in_block = oct % p.octets;
    const int64_t f = (int64_t)nt * 32 + (lane & 31);
    v4u v = {0, 0, 0, 0};
    if (f < p.N && oct < 2 * p.octets && cb < p.ncb) {
        const int64_t slot = p.by_block ? (int64_t)cb * p.taps + tap : (int64_t)tap * p.ncb + cb;
        const int e = p.exps[f * p.exp_ld + slot];
        v = bf_octet_i8(*reinterpret_cast<const v2i *>(p.mant + f * p.kpad + slot * 32 + in_block * 8), e > 254 ? 254 : e, p.m);
    }
    *reinterpret_cast<v4u *>(p.out + piece * 1024 + lane * 16) = v;
}

// KS: steps of 16 per tap of a chunk (two blocks of 8 KS channels); ENC: the product leaves as the next layer's image
template <int KS, bool ENC, bool STREAM>
__global__ __launch_bounds__(kStripThreads, 2) void gemm_strip_kernel(const StripParams p) {
    constexpr int MT = 4, NT = 2;
    constexpr int kPitch = KS * 32 + 16, kHalf = (KS + 1) / 2;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    int tm, tn;
    if (!tile_of_workgroup(blockIdx.x, p.tiles_m, p.tiles_n, tm, tn)) return;    // whole workgroup, before any barrier
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int l32 = lane & 31, lh = lane >> 5;
    const int64_t row0 = (int64_t)tm * kStripRows, col0 = (int64_t)tn * kStripCols;

    // the input pixel under filter tap (0, 0) of an output position, and its row and column (which may lie outside)
    const auto corner = [&](int64_t pos, int &cy, int &cx) {
        const uint32_t per_img = (uint32_t)(p.Ho * p.Wo), i = (uint32_t)pos / per_img, rem = (uint32_t)pos % per_img;
        cy = (int)(rem / (uint32_t)p.Wo) * p.str_h - p.pad_h;
        cx = (int)(rem % (uint32_t)p.Wo) * p.str_w - p.pad_w;
        return ((int)i * p.H + cy) * p.W + cx;
    };
    const int64_t last_row = (p.M < row0 + kStripRows ? p.M : row0 + kStripRows) - 1;
    int y_, x_;
    const int first = corner(row0, y_, x_), length = corner(last_row, y_, x_) - first + p.tail;

    // this lane's rows: where they sit in the strip, and which taps meet the image there
    int abase[MT];
    uint32_t amask[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        int64_t r = row0 + wm * 32 * MT + 32 * i + l32;
        if (r > last_row) r = last_row;
        int cy, cx;
        abase[i] = (corner(r, cy, cx) - first) * kPitch + lh * 16;
        amask[i] = 0;
        for (int tap = 0, fr = 0, fs = 0; tap < p.taps; ++tap) {
            if ((unsigned)(cy + fr) < (unsigned)p.H && (unsigned)(cx + fs) < (unsigned)p.W) amask[i] |= 1u << tap;
            if (++fs == p.S) fs = 0, ++fr;
        }
    }
    const int zero = p.zero_at + lh * 16;
    if (t < kPitch / 16) *reinterpret_cast<v4u *>(lds + p.zero_at + t * 16) = v4u{0, 0, 0, 0};

    v16f acc[MT / 2][2][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i / 2][i % 2][j][v] = 0.0f;

    // filters: tiles 4 tn + 2 wn and the next; a tile past the last column re-reads the last one (never stored)
    const int tiles32 = (int)((p.N + 31) / 32);
    const uint8_t *pb[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int nt = 4 * tn + NT * wn + j;
        pb[j] = p.panels + (int64_t)(nt < tiles32 ? nt : tiles32 - 1) * p.steps * 1024;
    }
    const uint32_t lane16 = lane * 16;
    const int taps = col0 + 64 * wn < p.N ? p.taps : 0;                          // uniform; 0: this wave has no column to compute

    const int chunks = (p.ncb + 1) / 2;
    const int units = length * 4;
    for (int chunk = 0; chunk < chunks; ++chunk) {
        // ---- strip: a unit is 16 bytes of a pixel, half a stored block
        for (int u0 = t; u0 - t < units; u0 += 4 * kStripThreads) {
            v4i raw[4];
            int e[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int u = u0 + i * kStripThreads;
                int px = first + (u >> 2);
                px = px < 0 ? 0 : px >= p.pixels ? p.pixels - 1 : px;
                if (u < units) {
                    raw[i] = *reinterpret_cast<const v4i *>(p.img + px * p.pix_bytes + chunk * 64 + (u & 3) * 16);
                    e[i] = p.eimg[px * p.eimg_ld + 2 * chunk + ((u >> 1) & 1)];
                }
            }
            if (u0 == t && chunk) __syncthreads();                               // everybody has read the chunk before
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int u = u0 + i * kStripThreads;
                if (u < units) {
                    const int oct = 2 * (u & 1);                                 // of the block
                    uint8_t *dst = lds + (u >> 2) * kPitch + (((u >> 1) & 1) * p.octets + oct) * 16;
                    const int eb = e[i] > 254 ? 254 : e[i];
                    if (oct < p.octets) *reinterpret_cast<v4u *>(dst) = bf_octet_i8(v2i{raw[i][0], raw[i][1]}, eb, p.m);
                    if (oct + 1 < p.octets) *reinterpret_cast<v4u *>(dst + 16) = bf_octet_i8(v2i{raw[i][2], raw[i][3]}, eb, p.m);
                }
            }
        }
        // ---- the taps of the window
        const bool full = 2 * chunk + 1 < p.ncb;                                 // two blocks, or the last one alone
        const int bytes = (full ? KS : kHalf) * 1024;                            // of a filter tile and tap
        v8bf b[KS][NT];
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int j = 0; j < NT; ++j) b[s][j] = *reinterpret_cast<const v8bf *>(pb[j] + s * 1024 + lane16);
        __syncthreads();
        int fr = 0, fs = 0;
        for (int tap = 0; tap < taps; ++tap) {
            const int off = (fr * p.W + fs) * kPitch;
            if (++fs == p.S) fs = 0, ++fr;
            int pa[MT];
#pragma unroll
            for (int i = 0; i < MT; ++i) pa[i] = (amask[i] >> tap) & 1 ? abase[i] + off : zero;
#pragma unroll
            for (int j = 0; j < NT; ++j) pb[j] += bytes;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (s >= kHalf && !full) break;
                v8bf a[MT];
#pragma unroll
                for (int i = 0; i < MT; ++i) a[i] = *reinterpret_cast<const v8bf *>(lds + pa[i] + s * 32);
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[i / 2][i % 2][j] = ENC ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[s][j], a[i], acc[i / 2][i % 2][j], 0, 0, 0)
                                                   : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[s][j], acc[i / 2][i % 2][j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < NT; ++j)                                     // of the next tap; behind the last one not used
                    b[s][j] = *reinterpret_cast<const v8bf *>(pb[j] + s * 1024 + lane16);
            }
        }
    }

    const int64_t i0 = row0 + wm * 32 * MT, j0 = col0 + wn * 32 * NT;
    if (ENC) {
#pragma unroll
        for (int h = 0; h < MT / 2; ++h) {
            if (p.enc.rounding) mx_store_encoded<1, NT>(p.enc, acc[h], i0 + 64 * h, j0, p.M, p.N, lane);
            else mx_store_encoded<0, NT>(p.enc, acc[h], i0 + 64 * h, j0, p.M, p.N, lane);
        }
        return;
    }
    store_result<MT, NT, STREAM>(p.C + i0 * p.ldc + j0, p.ldc, p.M - i0, p.N - j0, p.beta != 0, lane,
                                 [&](int i, int j, int v) { return acc[i / 2][i % 2][j][v]; });
}

// pixels that the strip of any workgroup holds at most: from the corner of its first position to the far corner of its last.
// Between neighbouring positions the corner moves by the stride, by more at the end of a row and of an image.
int64_t strip_pixels(const hbfp_conv2d &c, int64_t ho, int64_t wo) {
    const int64_t per_row = c.stride_h * (int64_t)c.w - wo * c.stride_w, per_img = (c.h - ho * c.stride_h) * c.w;
    return (kStripRows - 1) * (int64_t)c.stride_w + ceil_div(kStripRows - 1, wo) * (per_row > 0 ? per_row : 0) +
           ceil_div(kStripRows - 1, ho * wo) * (per_img > 0 ? per_img : 0) + (int64_t)(c.r - 1) * c.w + c.s;
}

template <int KS, bool ENC>
int launch_strip_t(const StripParams &p, bool stream, int lds_bytes, hipStream_t s) {
    static std::atomic<bool> configured[2];
    void (*const kernel)(StripParams) = stream ? &gemm_strip_kernel<KS, ENC, true> : &gemm_strip_kernel<KS, ENC, false>;
    if (allow_dynamic_lds(configured[stream], reinterpret_cast<const void *>(kernel), kStripLds) != HBFP_OK) return HBFP_ERR_LAUNCH;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(ceil_div((int64_t)p.tiles_m * p.tiles_n, 8) * 8)), dim3(kStripThreads), lds_bytes, s, p);
    return launch_status();
}

int strip_steps(int64_t ncb, int64_t kblock, int64_t taps) {
    const int64_t full = kblock / 8, last = (full + 1) / 2;      // steps of 16 per tap of two blocks, of one
    return (int)(taps * (ncb / 2 * full + ncb % 2 * last));
}

}  // namespace

// Whether the convolution runs on this kernel (a: as for launch_gemm_conv_i8; room: bytes of workspace, which holds the panels)
bool gemm_strip_ok(const GemmArgs &a, const hbfp_conv2d &c, int64_t ho, int64_t wo, int kblock, size_t room) {
    const int64_t taps = (int64_t)c.r * c.s;
    if (kblock % 8 || kblock > 32 || c.c % kblock || taps > 32 || taps < 2) return false;
    // corners in increasing order, positions within one window of their input
    if (2 * c.pad_h > c.r - 1 || 2 * c.pad_w > c.s - 1) return false;
    const int64_t pitch = kblock / 8 * 32 + 16, pixels = strip_pixels(c, ho, wo);
    if ((pixels + 1) * pitch > kStripLds) return false;
    const int64_t steps = strip_steps(c.c / kblock, kblock, taps);
    if (((size_t)ceil_div(a.N, 32) * steps + 4) * 1024 > room) return false;
    const int64_t tiles = ceil_div(a.M, kStripRows) * ceil_div(a.N, kStripCols);
    return tiles >= 128 && tiles <= 0x7ffffff0;
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
    q.octets = kblock / 8;
    q.taps = c.r * c.s;
    q.by_block = by_block;
    q.m = a.mB;
    q.full = kblock / 8;
    q.last = (q.full + 1) / 2;
    q.steps = strip_steps(q.ncb, kblock, q.taps);
    q.tiles = (int32_t)ceil_div(a.N, 32);
    hipLaunchKernelGGL(strip_panels_kernel, dim3((unsigned)ceil_div((int64_t)q.tiles * q.steps, 4)), dim3(256), 0, s, q);
    if (launch_status() != HBFP_OK) return HBFP_ERR_LAUNCH;

    const int64_t pitch = kblock / 8 * 32 + 16, strip = strip_pixels(c, ho, wo);
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
    p.taps = q.taps;
    p.pad_h = c.pad_h;
    p.pad_w = c.pad_w;
    p.str_h = c.stride_h;
    p.str_w = c.stride_w;
    p.pixels = (int32_t)(c.n * c.h * c.w);
    p.ncb = q.ncb;
    p.octets = q.octets;
    p.steps = q.steps;
    p.tail = (int32_t)((c.r - 1) * c.w + c.s);
    p.zero_at = (int32_t)(strip * pitch);
    p.tiles_m = (int32_t)ceil_div(a.M, kStripRows);
    p.tiles_n = (int32_t)ceil_div(a.N, kStripCols);
    p.beta = a.beta != 0.0f;
    p.m = a.mA;
    const int lds_bytes = (int)((strip + 1) * pitch);
    if (enc) {
        p.enc = mx_out_of(*enc, relu);
        switch (kblock) {
            case 8: return launch_strip_t<1, true>(p, true, lds_bytes, s);
            case 16: return launch_strip_t<2, true>(p, true, lds_bytes, s);
            case 24: return launch_strip_t<3, true>(p, true, lds_bytes, s);
            default: return launch_strip_t<4, true>(p, true, lds_bytes, s);
        }
    }
    const bool stream = stores_stream(&a);
    switch (kblock) {
        case 8: return launch_strip_t<1, false>(p, stream, lds_bytes, s);
        case 16: return launch_strip_t<2, false>(p, stream, lds_bytes, s);
        case 24: return launch_strip_t<3, false>(p, stream, lds_bytes, s);
        default: return launch_strip_t<4, false>(p, stream, lds_bytes, s);
    }
}

}  // namespace hbfp
