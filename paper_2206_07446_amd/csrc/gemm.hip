// Implicit im2col GEMM convolution on the matrix cores (the "sgemm" kernel family of
// Table 2 / Fig. 5, including 1x1 pointwise layers):
//     y[k, n] = sum_kk Wp[k, kk] * col[kk, n],  n = (img, p, q),  kk = (c, r, s)
// The col matrix is never materialised: every wavefront gathers its B fragments
// straight from x.
//
// float32: v_mfma_f32_16x16x4_f32.  One k-step = 4 channels at one filter tap (r,s);
//   lane l holds row/column l%16 and channel slot l/16, so the packed weight fragment
//   of a step is 64 consecutive floats (one coalesced 256 B load) and the B fragment is
//   x[c0 + l/16][ih][iw + l%16...] (contiguous along W for stride 1).
// float16: v_mfma_f32_16x16x32_f16.  One k-step = 32 channels at one tap; lane l holds
//   8 consecutive channels (slot group l/16).  For filters larger than 1x1, x is first copied
//   to a [N][Cpad32 / 8][H][W][8] half buffer in the workspace and both fragments are
//   16-byte loads.  For 1x1 filters (most layers of the bottleneck and inverted-residual
//   networks) that copy would cost a launch of its own, as long as the layer itself: there a
//   lane gathers its 8 channels straight from NCHW with eight 2-byte loads per fragment.
//   Layers large enough to fill workgroups (and float32 3x3 ones) run in items that share pixels through LDS instead (tile_gemm.h).
//
// Batch-1 layers put one or two wavefronts on a SIMD, and a lone wavefront issues one
// instruction every four cycles: the k-loop must be almost nothing but loads and MFMAs.
// So all addressing is hoisted: operands come through buffer loads whose hardware range
// check returns 0 for an out-of-range offset; each lane keeps one byte offset per filter
// tap, already set beyond the buffer where the tap falls into the zero padding; the
// channel advance is a scalar offset; fragments of consecutive steps use immediate
// offsets.  A chunk (one channel block x all taps, or 8 channel blocks for 1x1) is loaded
// one chunk ahead of the MFMAs (register ping-pong).  KS wavefronts of a workgroup share one
// output tile and split the channel blocks; partial sums meet in LDS, fixed order.
#include <algorithm>
#include <atomic>
#include <climits>
#include "nnv_internal.h"
#include "buf.h"
#include "depthwise.h"

namespace nnv {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef half8_t half8;

struct GemmParams {
    const void *x;       // float32 NCHW, or half copy in octets of channels
    const void *wp;      // packed panels
    const float *bias;
    void *y;
    int N, C, H, W, K, R, S, sh, sw, ph, pw, P, Q;
    int npix;            // N*P*Q
    int K16;             // 16-row panels in all: groups * kg16
    int kg16, Kg, Cg;    // per group: 16-row panels, output channels, input channels (groups == 1: the whole layer)
    int cblocks;         // channel blocks (of 4 float32 / 32 half channels) of one group
    int c_rem;           // float32: C % 4, float16 1x1: C % 32 (channels of the last, partial block; 0 = full)
    uint32_t plane_bytes;   // float16 1x1: bytes of one channel plane of x (H*W*2)
    int ks_shift;        // wavefronts sharing one output tile = 1 << ks_shift
    int cpad;            // channels of the half copy of x: a multiple of 32, or 8 (kModeTaps)
    uint32_t x_bytes, w_bytes;   // sizes of the x and wp buffers (range-checked loads)
    uint32_t cb_stride;  // bytes between channel blocks in x
    int half_out;
    int relu;              // outputs clamped at zero before the store
    int grid_nx, grid_ny;  // logical grid: tile groups along n, along m
    int m_major;           // 1: consecutive logical tiles walk n first (an XCD keeps few weight panels),
                           // 0: they walk m first (an XCD keeps a pixel range of x)
};

// Chunking mode of the work items of float16 1x1 layers whose pixels can be read in pairs
// (gemm_accumulate_pairs); the other modes are those of ModeT below.
constexpr int kModePairs = 2;
// ... and of float16 layers of at most 8 input channels with a filter larger than 1x1 (gemm_accumulate_taps).
constexpr int kModeTaps = 4, kTapsMaxChannels = 8;
// ... and of the work items of float16 1x1 layers of many channels whose pixels cannot be read in pairs
// (gemm_accumulate_octets); fewer channel blocks or output panels than this are gathered from NCHW.
constexpr int kModeOctets = 6, kOctetsMinBlocks = 16, kOctetsMinPanels = 32;
// ... and of float32 3x3 layers whose pixels go through LDS (gemm_accumulate_patch; single layers and those of a cold pass).
constexpr int kModePatch = 8;

// The parameters that follow from a layer's sizes, its storage type and its chunking mode.
__host__ __device__ inline void gemm_derived(GemmParams &g, const bool half, const int mode) {
    const bool gather = half && (mode == 1 || mode == kModePairs);   // float16 1x1: B fragments gathered from NCHW
    g.cpad = mode == kModeTaps ? 8 : (g.C + 31) / 32 * 32;
    g.cblocks = half ? (g.Cg + 31) / 32 : (g.Cg + 3) / 4;
    g.c_rem = gather ? g.Cg % 32 : half ? 0 : g.Cg % 4;
    g.plane_bytes = (uint32_t)g.H * (uint32_t)g.W * 2u;
    g.half_out = half;
    const uint32_t pix = (uint32_t)g.N * (uint32_t)g.H * (uint32_t)g.W;
    g.x_bytes = half ? pix * (uint32_t)(gather ? g.C : g.cpad) * 2u : pix * (uint32_t)g.C * 4u;
    g.w_bytes = (uint32_t)g.K16 * (uint32_t)g.cblocks * (uint32_t)(g.R * g.S) * (half ? 1024u : 256u);
    g.cb_stride = gather ? 32u * g.plane_bytes : half ? (uint32_t)g.H * (uint32_t)g.W * 64u : (uint32_t)g.H * (uint32_t)g.W * 16u;
}

template <bool HALF> struct FragT { typedef float type; };
template <> struct FragT<true> { typedef half8 type; };

// MODE: how the k-steps of a wavefront are grouped into chunks (a chunk is what is loaded ahead)
//   1  1x1 filter: a unit is a channel block, a chunk is 8 units (2 in half precision)
//   3  3x3 filter, float32: a unit = chunk = one channel block, 9 taps, tap offsets loop-invariant
//      3x3 filter, half: row mode (fragments are four registers wide, nine steps do not fit)
//   5,7  filters with S = 5 / 7 (float32): row mode, a unit = chunk = one filter row of a channel block
//   0  anything else: a unit = chunk = one k-step
template <bool HALF, int MODE> struct ModeT {
    static constexpr bool ROW = MODE == 5 || MODE == 7 || (MODE == 3 && HALF);
    static constexpr bool WHOLE3 = MODE == 3 && !HALF;
    static constexpr int UNITS = MODE == 1 ? (HALF ? 2 : 8) : 1;                           // units per chunk
    static constexpr int STEPS = MODE == 0 ? 1 : MODE == 1 ? UNITS : WHOLE3 ? 9 : MODE;    // k-steps per chunk
    static constexpr int NVOFF = (MODE == 0 || MODE == 1) ? 1 : STEPS;                     // tap offsets kept per lane
};

// Output pixels of a wavefront's tile columns: image, position in the P x Q plane, inside the problem or not.
template <int TN> struct PixState {
    int img[TN], pq[TN];
    bool valid[TN];
};

// The k-loop of one wavefront: TM x TN blocks of 16 x 16 outputs (panels mb0.., 16-pixel blocks
// nb0..), summed over the ks-th of nsplit equal ranges of the layer's units.
template <bool HALF, int TM, int TN, int MODE, int NBUF>
__device__ __forceinline__ void gemm_accumulate(const GemmParams &g, const int mb0, const int nb0, const int ks,
                                                const int nsplit, const int lane, floatx4 (&acc)[TM][TN],
                                                PixState<TN> &px) {
    typedef typename FragT<HALF>::type frag_t;
    typedef ModeT<HALF, MODE> MT;
    constexpr int STEPS = MT::STEPS, UNITS = MT::UNITS, NVOFF = MT::NVOFF;
    constexpr bool ROW = MT::ROW, WHOLE3 = MT::WHOLE3;
    constexpr uint32_t FB = sizeof(frag_t);            // bytes per lane of one fragment
    constexpr uint32_t FRAG = 64 * FB;                 // bytes of one fragment
    const int col = lane & 15, slot = lane >> 4;
    const int grp = mb0 / g.kg16;
    const int cbase = grp * g.Cg;                         // first input channel of the group
    const int PQ = g.P * g.Q, RS = g.R * g.S;

    // ---- per-lane pixel state: origin of the patch in x (bytes, may be negative) and tap offsets
    int xbase[TN], ih0[TN], iw0[TN];
    int (&pix_img)[TN] = px.img, (&pix_pq)[TN] = px.pq;
    bool (&pvalid)[TN] = px.valid;
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int n = (nb0 + t) * 16 + col;
        pvalid[t] = n < g.npix;
        const int nn = pvalid[t] ? n : 0;
        const int img = g.N == 1 ? 0 : nn / PQ;
        const int pq = nn - img * PQ;
        const int p = pq / g.Q, q = pq - p * g.Q;
        pix_img[t] = img; pix_pq[t] = pq;
        ih0[t] = p * g.sh - g.ph;
        iw0[t] = q * g.sw - g.pw;
        if (HALF && MODE == 1) xbase[t] = (((img * g.C + cbase + slot * 8) * g.H + ih0[t]) * g.W + iw0[t]) * 2;   // NCHW
        else if (HALF) xbase[t] = (((img * (g.cpad >> 3) + (cbase >> 3) + slot) * g.H + ih0[t]) * g.W + iw0[t]) * 16;   // copy in octets of channels
        else xbase[t] = (((img * g.C + cbase + slot) * g.H + ih0[t]) * g.W + iw0[t]) * 4;
    }
    const int tap_w = HALF ? 16 : 4;                     // bytes per step along s
    const int tap_h = g.W * tap_w;                       // bytes per step along r
    auto tap_off = [&](int t, int r, int s) -> uint32_t {
        const bool ok = pvalid[t] && (unsigned)(ih0[t] + r) < (unsigned)g.H && (unsigned)(iw0[t] + s) < (unsigned)g.W;
        return ok ? (uint32_t)(xbase[t] + r * tap_h + s * tap_w) : kOobOffset;
    };
    // row mode: the column part of the tap offsets (origin + s, or out of range) does not change
    // from chunk to chunk; a chunk's offsets are that plus its row, or out of range for a row in
    // the padding
    uint32_t colv[TN][ROW ? NVOFF : 1];
    if (ROW) {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int sx = 0; sx < NVOFF; ++sx)
                colv[t][sx] = (pvalid[t] && (unsigned)(iw0[t] + sx) < (unsigned)g.W) ? (uint32_t)(xbase[t] + sx * tap_w) : kOobOffset;
    }
    // byte offset per tap of the current chunk; loop-invariant for MODE 1 and 3
    uint32_t voff[TN][NVOFF];
    if (MODE == 1) {
#pragma unroll
        for (int t = 0; t < TN; ++t) voff[t][0] = tap_off(t, 0, 0);
    } else if (WHOLE3) {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int rs = 0; rs < NVOFF; ++rs) voff[t][rs] = tap_off(t, rs / 3, rs % 3);
    }
    // ---- this wavefront's range of units
    const int nunits = MODE == 0 ? g.cblocks * RS : ROW ? g.cblocks * g.R : g.cblocks;
    const int per_wave = (nunits + nsplit - 1) / nsplit;
    const int u_begin = min(nunits, ks * per_wave);
    const int u_end = min(nunits, u_begin + per_wave);
    const int steps_per_unit = MODE == 0 ? 1 : ROW ? MODE : RS;   // MODE 1: RS == 1
    const uint32_t nsteps_total = (uint32_t)g.cblocks * RS;

    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, g.x_bytes);
    const uint32_t a_lane = lane * FB;
    frag_t a[NBUF][STEPS][TM], b[NBUF][STEPS][TN];

    // Load the chunk starting at unit u (clamped into the range: a chunk past the end re-reads
    // valid data that is never used).  Straight-line code, no branches between the loads.
    // The weight fragments of a chunk are consecutive in memory: they are read through a
    // resource window that starts at the chunk (immediate offsets per step) and ends at the end
    // of the buffer, so a read past this wavefront's range or past the last panel returns
    // data that is not used, or zero, but never faults.
    auto load_chunk = [&](int buf, int u) {
        u = max(min(u, u_end - 1), 0);
#pragma unroll
        for (int m = 0; m < TM; ++m) {
            uint32_t off = ((uint32_t)(mb0 + m) * nsteps_total + (uint32_t)u * steps_per_unit) * FRAG;
            off = min(off, g.w_bytes);        // panels beyond K: empty window, all zeros
            const __amdgpu_buffer_rsrc_t win = make_rsrc(static_cast<const char *>(g.wp) + off, g.w_bytes - off);
#pragma unroll
            for (int j = 0; j < STEPS; ++j) a[buf][j][m] = buf_load<frag_t>(win, a_lane + j * FRAG, 0u);
        }
        if constexpr (MODE == 1 && HALF) {
            // x is NCHW: the lane's 8 channels are 8 planes apart; channels past C (last block)
            // read as zero through an out-of-range offset
#pragma unroll
            for (int j = 0; j < STEPS; ++j) {
                const int cb = min(u + j, u_end - 1);
                const bool part = g.c_rem != 0 && cb == g.cblocks - 1;   // uniform
#pragma unroll
                for (int t = 0; t < TN; ++t) {
                    half8 v;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        uint32_t vo = voff[t][0];
                        if (part) vo = slot * 8 + i < g.c_rem ? vo : kOobOffset;
                        const unsigned short h = __builtin_amdgcn_raw_buffer_load_b16(
                            xres, vo, (uint32_t)cb * g.cb_stride + (uint32_t)i * g.plane_bytes, 0);
                        v[i] = __builtin_bit_cast(_Float16, h);
                    }
                    b[buf][j][t] = v;
                }
            }
        } else if (MODE == 1) {
#pragma unroll
            for (int j = 0; j < STEPS; ++j) {
                const int cb = min(u + j, u_end - 1);
#pragma unroll
                for (int t = 0; t < TN; ++t) b[buf][j][t] = buf_load<frag_t>(xres, voff[t][0], (uint32_t)cb * g.cb_stride);
            }
        } else {
            int cb, r0 = 0, s0 = 0;
            if (WHOLE3) cb = u;
            else if (MODE == 0) { cb = u / RS; const int rs = u - cb * RS; r0 = rs / g.S; s0 = rs - r0 * g.S; }
            else { cb = u / g.R; r0 = u - cb * g.R; }
            if (ROW) {
#pragma unroll
                for (int t = 0; t < TN; ++t) {
                    const bool rok = (unsigned)(ih0[t] + r0) < (unsigned)g.H;
                    const uint32_t radd = (uint32_t)(r0 * tap_h);
#pragma unroll
                    for (int s = 0; s < NVOFF; ++s) voff[t][s] = rok ? colv[t][s] + radd : kOobOffset;   // 2^31 + anything below 2^31 stays out of range
                }
            } else if (MODE == 0) {
#pragma unroll
                for (int t = 0; t < TN; ++t) voff[t][0] = tap_off(t, r0, s0);
            }
            const bool partial = !HALF && g.c_rem != 0 && cb == g.cblocks - 1;   // uniform
            const uint32_t b_soff = (uint32_t)cb * g.cb_stride;
#pragma unroll
            for (int j = 0; j < STEPS; ++j) {
#pragma unroll
                for (int t = 0; t < TN; ++t) {
                    uint32_t vo = voff[t][j < NVOFF ? j : 0];
                    if (partial) vo = slot < g.c_rem ? vo : kOobOffset;
                    b[buf][j][t] = buf_load<frag_t>(xres, vo, b_soff);
                }
            }
        }
    };

#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[m][t] = floatx4{0.f, 0.f, 0.f, 0.f};

    auto mfma_step = [&](int buf, int j) {
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                if constexpr (HALF)
                    acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[buf][j][m], b[buf][j][t], acc[m][t], 0, 0, 0);
                else
                    acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[buf][j][m], b[buf][j][t], acc[m][t], 0, 0, 0);
            }
    };
    // MFMAs of the chunk starting at unit u: all of it, or (MODE 1 tail) only its valid units
    auto compute = [&](int buf, int u) {
        if (UNITS == 1 || u + UNITS <= u_end) {
#pragma unroll
            for (int j = 0; j < STEPS; ++j) mfma_step(buf, j);
        } else {
#pragma unroll
            for (int j = 0; j < STEPS; ++j)
                if (u + j < u_end) mfma_step(buf, j);
        }
    };

    // ring of NBUF register sets: loads run NBUF-1 chunks ahead of the MFMAs
    if (u_begin < u_end) {
#pragma unroll
        for (int i = 0; i < NBUF - 1; ++i) load_chunk(i, u_begin + i * UNITS);
        __builtin_amdgcn_s_setprio(0);
        // The scheduling barriers keep the loads of a later chunk in front of the MFMAs of the
        // current one: left alone, the compiler sinks them behind the MFMAs to save registers,
        // which puts every load's latency in front of the instruction that needs it.
        __builtin_amdgcn_sched_barrier(0);
        for (int u = u_begin; u < u_end; u += NBUF * UNITS) {
#pragma unroll
            for (int i = 0; i < NBUF; ++i) {
                load_chunk((i + NBUF - 1) % NBUF, u + (i + NBUF - 1) * UNITS);
                __builtin_amdgcn_sched_barrier(0);
                if (i == 0 || u + i * UNITS < u_end) compute(i, u + i * UNITS);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

}

// ---- the k-loops of the work-item kernel for float32 3x3 and 1x1 filters, TM = 1, 2 or 4 panels per tile.
// What bounds the 32 x 32 tile on a busy chip is the vector memory path of a CU (address unit and
// data return are 60-70 % busy, measured), not the matrix pipe: every MFMA needs one operand
// fragment through it.  A 64 x 32 tile needs 0.75.  To keep the register count where four
// wavefronts still fit on a SIMD, a chunk is one filter row (3 k-steps) and three chunks form the
// ring, so loads run two chunks (48 MFMAs) ahead; the buffer of a chunk is the filter row it
// belongs to, which makes every index in the unrolled loop a constant.
template <int TN>
__device__ __forceinline__ void gemm_pixels(const GemmParams &g, const int mb0, const int nb0, const int lane,
                                            PixState<TN> &px, int (&ih0)[TN], int (&iw0)[TN], int (&xbase)[TN]) {
    const int col = lane & 15, slot = lane >> 4;
    const int cbase = (mb0 / g.kg16) * g.Cg;              // first input channel of the tile's group
    const int PQ = g.P * g.Q;
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int n = (nb0 + t) * 16 + col;
        px.valid[t] = n < g.npix;
        const int nn = px.valid[t] ? n : 0;
        const int img = g.N == 1 ? 0 : nn / PQ;
        const int pq = nn - img * PQ;
        const int p = pq / g.Q, q = pq - p * g.Q;
        px.img[t] = img; px.pq[t] = pq;
        ih0[t] = p * g.sh - g.ph;
        iw0[t] = q * g.sw - g.pw;
        xbase[t] = (((img * g.C + cbase + slot) * g.H + ih0[t]) * g.W + iw0[t]) * 4;
    }
}

// The rows of a matrix block may be any output channels as long as the store agrees.  In the two functions
// below a lane takes TM consecutive floats of a weight fragment, one per block: row i of block m is row
// TM * (i % QM) + m of panel i / QM, QM = 16 / TM, so one load of 4 TM bytes replaces TM of them (9 loads per 24
// MFMAs with four panels, 18 before).  Measured, us a grouped call: VGG-16-shaped stack 289 -> 276, ResNet-50 98 -> 95,
// SqueezeNet 38 -> 34, MobileNetV1 44 -> 42.  The per-lane byte offset, out of range for panels beyond K:
template <int TM>
__device__ __forceinline__ uint32_t gemm_a_offset(const GemmParams &g, const int mb0, const int lane, const uint32_t panel_steps) {
    constexpr int QM = 16 / TM;
    const int col = lane & 15, slot = lane >> 4;
    const int panel = col / QM;
    return mb0 + panel < g.K16 ? (uint32_t)panel * panel_steps * 256u + (uint32_t)slot * 64u + (uint32_t)(col % QM) * (4u * TM) : kOobOffset;
}

// CHAINS = 2: the products go to two sets of sums in turn, added at the end.  Single layers and those of a cold pass take two: a sum of half as many products
// at a time is nearer to the exact one (64 channels at 56x56 -> 64, relative 2-norm of the error, one chain / two: 2.17e-7 / 1.60e-7), which is what lets a layer's reduction be cut
// into fewer wavefronts (plan_im2col).
template <int TM, int TN, int CHAINS>
__device__ __forceinline__ void gemm_accumulate_3x3(const GemmParams &g, const int mb0, const int nb0, const int ks,
                                                    const int nsplit, const int lane, floatx4 (&acc)[TM][TN],
                                                    PixState<TN> &px) {
    const int slot = lane >> 4;
    int ih0[TN], iw0[TN], xbase[TN];
    gemm_pixels<TN>(g, mb0, nb0, lane, px, ih0, iw0, xbase);
    uint32_t voff[TN][9];
    const int tap_h = g.W * 4;
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const bool rok = px.valid[t] && (unsigned)(ih0[t] + r) < (unsigned)g.H;
#pragma unroll
            for (int sx = 0; sx < 3; ++sx)
                voff[t][r * 3 + sx] = (rok && (unsigned)(iw0[t] + sx) < (unsigned)g.W) ? (uint32_t)(xbase[t] + r * tap_h + sx * 4) : kOobOffset;
        }
    const int cblocks = g.cblocks;
    const int per = (cblocks + nsplit - 1) / nsplit;
    const int cb_begin = min(cblocks, ks * per), cb_end = min(cblocks, cb_begin + per);
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, g.x_bytes);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, g.w_bytes);
    const uint32_t a_voff = gemm_a_offset<TM>(g, mb0, lane, (uint32_t)cblocks * 9u);
    const uint32_t a_base = (uint32_t)mb0 * (uint32_t)cblocks * 9u;
    typename FloatVec<TM>::type a[3][3];
    float b[3][3][TN];
    floatx4 sum[CHAINS][TM][TN];
    auto load_row = [&](const int r, int cb) __attribute__((always_inline)) {
        cb = max(min(cb, cb_end - 1), 0);          // past the range: re-read valid data that is not used
        const bool partial = g.c_rem != 0 && cb == cblocks - 1;     // uniform
        const uint32_t soff = (a_base + (uint32_t)cb * 9u + (uint32_t)r * 3u) * 256u;
#pragma unroll
        for (int sx = 0; sx < 3; ++sx) a[r][sx] = buf_load_floats<TM>(wres, a_voff + sx * 256u, soff);
        const uint32_t b_soff = (uint32_t)cb * g.cb_stride;
#pragma unroll
        for (int sx = 0; sx < 3; ++sx)
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                uint32_t vo = voff[t][r * 3 + sx];
                if (partial) vo = slot < g.c_rem ? vo : kOobOffset;
                b[r][sx][t] = buf_load<float>(xres, vo, b_soff);
            }
    };
    auto compute_row = [&](const int r) __attribute__((always_inline)) {
#pragma unroll
        for (int sx = 0; sx < 3; ++sx)
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int t = 0; t < TN; ++t) {
                    floatx4 &to = sum[(r * 3 + sx) % CHAINS][m][t];
                    to = __builtin_amdgcn_mfma_f32_16x16x4f32(float_of<TM>(a[r][sx], m), b[r][sx][t], to, 0, 0, 0);
                }
    };
#pragma unroll
    for (int c = 0; c < CHAINS; ++c)
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t) sum[c][m][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (cb_begin < cb_end) {
        load_row(0, cb_begin);
        load_row(1, cb_begin);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        for (int cb = cb_begin; cb < cb_end; ++cb) {
            load_row(2, cb);
            __builtin_amdgcn_sched_barrier(0);
            compute_row(0);
            __builtin_amdgcn_sched_barrier(0);
            load_row(0, cb + 1);
            __builtin_amdgcn_sched_barrier(0);
            compute_row(1);
            __builtin_amdgcn_sched_barrier(0);
            load_row(1, cb + 1);
            __builtin_amdgcn_sched_barrier(0);
            compute_row(2);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[m][t] = CHAINS == 2 ? sum[0][m][t] + sum[CHAINS - 1][m][t] : sum[0][m][t];
}

// The same sums, in the same order and the same two chains, for 3x3 filters at stride 1 with one column of padding: the pixels of a tile go through LDS.
// What bounds the smallest tile is the vector memory path of its CU: a product takes a fragment of weights and a gather of 16 pixels x 4 planes, and
// the nine taps gather the same pixels nine times.  Outputs n and n + 1 of a row lie over neighbouring inputs, so that the three rows of input under 16 outputs are
// 18 entries each, whatever the width of the image: a wavefront reads them with one load per channel, lays them down in a buffer of its own and takes the taps
// from there, 4 loads for four channels instead of 36.  Taps left and right of the image read an entry that is always zero.  Three channel blocks of
// weights and pixels are on their way.
constexpr int kPatchRow = 20, kPatchZero = 18;          // entries of a row; the one that is zero
constexpr int kPatchChannel = 80;                       // floats from channel to channel: neighbouring slots in different banks
constexpr int kPatchFloats = 2 * 4 * kPatchChannel;     // of a wavefront: two buffers of four channels
__device__ __forceinline__ void gemm_accumulate_patch(const GemmParams &g, const int mb0, const int nb0, const int ks, const int nsplit, const int lane,
                                                      float *lds, floatx4 (&acc)[1][1], PixState<1> &px) {
    constexpr int D = 3;
    const int slot = lane >> 4, j = lane & 15;
    uint32_t xo, at[3];             // the lane's entry of a channel, its taps of filter row 0
    {
        const int r = lane / kPatchRow, e = lane - r * kPatchRow, v = nb0 * 16 - 1 + e;
        const bool live = r < 3 && e < kPatchZero && v >= 0 && v < g.npix;
        const int n = live ? v : 0, PQ = g.P * g.Q;
        const int img = g.N == 1 ? 0 : n / PQ, pq = n - img * PQ, p = pq / g.Q, q = pq - p * g.Q, ih = p - g.ph + r;
        xo = live && (unsigned)ih < (unsigned)g.H ? (uint32_t)(((img * g.C + (mb0 / g.kg16) * g.Cg) * g.H + ih) * g.W + q) * 4u : kOobOffset;
        int ih0[1], iw0[1], xbase[1];
        gemm_pixels<1>(g, mb0, nb0, lane, px, ih0, iw0, xbase);
        at[0] = slot * kPatchChannel + (iw0[0] < 0 ? kPatchZero : j);
        at[1] = slot * kPatchChannel + j + 1;
        at[2] = slot * kPatchChannel + (iw0[0] + 2 >= g.W ? kPatchZero : j + 2);
    }
    const int cblocks = g.cblocks;
    const int per = (cblocks + nsplit - 1) / nsplit;
    const int cb_begin = min(cblocks, ks * per), cb_end = min(cblocks, cb_begin + per);
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, g.x_bytes), zres = make_rsrc(g.x, 0u);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, g.w_bytes);
    const uint32_t a_voff = gemm_a_offset<1>(g, mb0, lane, (uint32_t)cblocks * 9u);
    const uint32_t a_base = (uint32_t)mb0 * (uint32_t)cblocks * 9u;
    const uint32_t plane = g.cb_stride >> 2;
    float a[D][9], xr[D][4];
    // (blocks past the range: the last one again, not used)
    auto load_a = [&](const int d, int cb) __attribute__((always_inline)) {
        cb = min(cb, cb_end - 1);
#pragma unroll
        for (int i = 0; i < 9; ++i) a[d][i] = buf_load<float>(wres, a_voff + i % 3 * 256u, (a_base + (uint32_t)cb * 9u + i / 3 * 3) * 256u);
    };
    auto load_x = [&](const int d, int cb) __attribute__((always_inline)) {
        cb = min(cb, cb_end - 1);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool ok = cb * 4 + c < g.Cg;             // uniform
            xr[d][c] = buf_load<float>(ok ? xres : zres, xo, ok ? (uint32_t)cb * g.cb_stride + c * plane : 0u);
        }
    };
    // (lanes read what others of the wavefront wrote: everything before the fence in order before everything after it; no instruction)
    auto put = [&](const int d, const uint32_t buf) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < 4; ++c) lds[buf + c * kPatchChannel + lane] = xr[d][c];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    acc[0][0] = floatx4{0.f, 0.f, 0.f, 0.f};
    floatx4 odd = floatx4{0.f, 0.f, 0.f, 0.f};
    if (cb_begin >= cb_end) return;
    // The pixels of block b, in registers b % D, go to LDS one block ahead: the registers are free when block b begins.
    load_x(0, cb_begin);
#pragma unroll
    for (int d = 0; d < D - 1; ++d) {
        load_a(d, cb_begin + d);
        load_x(d + 1, cb_begin + d + 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    uint32_t cur = 0;
    put(0, 0);
    for (int cb = cb_begin; cb < cb_end; cb += D) {
#pragma unroll
        for (int i = 0; i < D; ++i) {
            if (i > 0 && cb + i >= cb_end) break;
            float b[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) b[k] = lds[cur + at[k % 3] + k / 3 * kPatchRow];
            load_a((i + D - 1) % D, cb + i + D - 1);
            load_x(i, cb + i + D);
            __builtin_amdgcn_sched_barrier(0);
            cur = cur ? 0 : 4 * kPatchChannel;
            put((i + 1) % D, cur);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                floatx4 &to = k % 2 ? odd : acc[0][0];
                to = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][k], b[k], to, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    acc[0][0] += odd;
}

// 1x1 filters: a chunk is four channel blocks, three chunks form the ring.
template <int TM, int TN>
__device__ __forceinline__ void gemm_accumulate_1x1(const GemmParams &g, const int mb0, const int nb0, const int ks,
                                                    const int nsplit, const int lane, floatx4 (&acc)[TM][TN],
                                                    PixState<TN> &px) {
    constexpr int CH = 4;
    int ih0[TN], iw0[TN], xbase[TN];
    gemm_pixels<TN>(g, mb0, nb0, lane, px, ih0, iw0, xbase);
    uint32_t voff[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t)
        voff[t] = (px.valid[t] && (unsigned)ih0[t] < (unsigned)g.H && (unsigned)iw0[t] < (unsigned)g.W) ? (uint32_t)xbase[t] : kOobOffset;
    const int cblocks = g.cblocks;
    const int nchunks = (cblocks + CH - 1) / CH;
    const int per = (nchunks + nsplit - 1) / nsplit;
    const int q_begin = min(nchunks, ks * per), q_end = min(nchunks, q_begin + per);
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, g.x_bytes);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, g.w_bytes);
    const uint32_t a_voff = gemm_a_offset<TM>(g, mb0, lane, (uint32_t)cblocks);
    const uint32_t a_base = (uint32_t)mb0 * (uint32_t)cblocks;
    // Chunks past the range and blocks past C are read through an empty resource (every load
    // returns 0), so the MFMAs need no condition and the unrolled loop keeps one accumulator set.
    const __amdgpu_buffer_rsrc_t zres = make_rsrc(g.x, 0u);
    typename FloatVec<TM>::type a[3][CH];
    float b[3][CH][TN];
    auto load_chunk = [&](const int buf, const int q) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int cbj = q * CH + j;
            const bool ok = q < q_end && cbj < cblocks;          // uniform
            const int cb = ok ? cbj : 0;
            const __amdgpu_buffer_rsrc_t wsel = ok ? wres : zres, xsel = ok ? xres : zres;
            a[buf][j] = buf_load_floats<TM>(wsel, a_voff, (a_base + (uint32_t)cb) * 256u);
#pragma unroll
            for (int t = 0; t < TN; ++t) b[buf][j][t] = buf_load<float>(xsel, voff[t], (uint32_t)cb * g.cb_stride);
        }
    };
    auto compute = [&](const int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < CH; ++j)
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(float_of<TM>(a[buf][j], m), b[buf][j][t], acc[m][t], 0, 0, 0);
    };
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[m][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (q_begin < q_end) {
        load_chunk(0, q_begin);
        load_chunk(1, q_begin + 1);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        for (int q = q_begin; q < q_end; q += 3) {
            load_chunk(2, q + 2);
            __builtin_amdgcn_sched_barrier(0);
            compute(0);
            __builtin_amdgcn_sched_barrier(0);
            load_chunk(0, q + 3);
            __builtin_amdgcn_sched_barrier(0);
            compute(1);
            __builtin_amdgcn_sched_barrier(0);
            load_chunk(1, q + 4);
            __builtin_amdgcn_sched_barrier(0);
            compute(2);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// float16 1x1 filters that cannot read pixels in pairs (odd planes, strides, padding), with 512 input and 512
// output channels or more:
// from the copy in octets of channels, as the larger filters.  Gathered from NCHW, two channel blocks take 36 loads
// and run one ahead, about 1 us each time: an item of 2048 channels was 30 us, half of its whole launch.  Here a
// block takes 6 loads and kRing - 1 blocks are in flight.  Measured, us a call: ResNet-50-shaped stack 64 -> 58, batch 2
// at 150 x 187 75 -> 63.  With fewer channels on either side the copy costs what the loads save: from 256 input channels
// and any number of outputs on, EfficientNet-B0 took 46 instead of 40.5, MobileNetV2 30.7 instead of 28.7; and one 1152 ->
// 320 layer alone does not pay for a copy launch (EfficientNet-B0 45 instead of 40).
template <int TM, int TN>
__device__ __forceinline__ void gemm_accumulate_octets(const GemmParams &g, const int mb0, const int nb0, const int ks,
                                                       const int nsplit, const int lane, floatx4 (&acc)[TM][TN],
                                                       PixState<TN> &px) {
    constexpr int kRing = 4;
    const int slot = lane >> 4;
    int ih0[TN], iw0[TN], xb32[TN];
    gemm_pixels<TN>(g, mb0, nb0, lane, px, ih0, iw0, xb32);          // (xb32: the float32 origin, not used)
    uint32_t voff[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const bool ok = px.valid[t] && (unsigned)ih0[t] < (unsigned)g.H && (unsigned)iw0[t] < (unsigned)g.W;
        voff[t] = ok ? (uint32_t)((((px.img[t] * (g.cpad >> 3) + slot) * g.H + ih0[t]) * g.W + iw0[t]) * 16) : kOobOffset;
    }
    const int cblocks = g.cblocks;
    const int per = (cblocks + nsplit - 1) / nsplit;
    const int u_begin = min(cblocks, ks * per), u_end = min(cblocks, u_begin + per);
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, g.x_bytes);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, g.w_bytes);
    const __amdgpu_buffer_rsrc_t zres = make_rsrc(g.x, 0u);        // blocks past the range read zeros
    uint32_t a_voff[TM], a_base[TM];
#pragma unroll
    for (int m = 0; m < TM; ++m) {
        const bool ok = mb0 + m < g.K16;
        a_voff[m] = ok ? (uint32_t)lane * 16u : kOobOffset;
        a_base[m] = ok ? (uint32_t)(mb0 + m) * (uint32_t)cblocks : 0u;
    }
    half8 a[kRing][TM], b[kRing][TN];
    auto load_unit = [&](const int buf, const int u) __attribute__((always_inline)) {
        const bool ok = u < u_end;                                  // uniform
        const uint32_t cb = ok ? (uint32_t)u : 0u;
        const __amdgpu_buffer_rsrc_t wsel = ok ? wres : zres, xsel = ok ? xres : zres;
#pragma unroll
        for (int m = 0; m < TM; ++m) a[buf][m] = buf_load<half8>(wsel, a_voff[m], (a_base[m] + cb) * 1024u);
#pragma unroll
        for (int t = 0; t < TN; ++t) b[buf][t] = buf_load<half8>(xsel, voff[t], cb * g.cb_stride);
    };
    auto compute = [&](const int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t)
                acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[buf][m], b[buf][t], acc[m][t], 0, 0, 0);
    };
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[m][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (u_begin >= u_end) return;
#pragma unroll
    for (int i = 0; i < kRing - 1; ++i) load_unit(i, u_begin + i);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    int u = u_begin;
    while (u + kRing - 1 < u_end) {
#pragma unroll
        for (int i = 0; i < kRing; ++i) {
            load_unit((i + kRing - 1) % kRing, u + i + kRing - 1);
            __builtin_amdgcn_sched_barrier(0);
            compute(i);
            __builtin_amdgcn_sched_barrier(0);
        }
        u += kRing;
    }
    if (u < u_end) {
#pragma unroll
        for (int i = 0; i < kRing - 1; ++i) compute(i);      // blocks past the range are zeros
    }
}

// float16 layers of at most 8 input channels (a network's first layer): a k-step of 32 channels at one tap
// would be three quarters zeros or more, and the 49 taps of a 7x7 filter 49 such steps.  The position
// of an element along k is free as long as both fragments agree, so here a step is 8 channels at four
// taps: lanes of slot s take tap 4 * u + s, from x's single octet and from the part of the weight fragment that
// holds channels 0..7 (its first sixteen lanes).  13 steps instead of 49, and a copy of x a quarter the size.
// Measured, us a call: ResNet-50-shaped stack 62 -> 54, SqueezeNet 35 -> 24, GoogLeNet 52 -> 40, ResNet-18 39 -> 33.
template <int TM, int TN>
__device__ __forceinline__ void gemm_accumulate_taps(const GemmParams &g, const int mb0, const int nb0, const int ks,
                                                     const int nsplit, const int lane, floatx4 (&acc)[TM][TN],
                                                     PixState<TN> &px) {
    constexpr int kRing = 3;
    const int col = lane & 15, slot = lane >> 4;
    const int PQ = g.P * g.Q, RS = g.R * g.S, S = g.S;
    int ih0[TN], iw0[TN], xbase[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int n = (nb0 + t) * 16 + col;
        px.valid[t] = n < g.npix;
        const int nn = px.valid[t] ? n : 0;
        const int img = g.N == 1 ? 0 : nn / PQ;
        const int pq = nn - img * PQ;
        const int p = pq / g.Q, q = pq - p * g.Q;
        px.img[t] = img; px.pq[t] = pq;
        ih0[t] = p * g.sh - g.ph;
        iw0[t] = q * g.sw - g.pw;
        xbase[t] = ((img * g.H + ih0[t]) * g.W + iw0[t]) * 16;
    }
    const uint32_t magic = 65536u / (uint32_t)S + 1u;      // (tap * magic) >> 16 == tap / S: taps stay below 2^7, S at most 32
    const int steps = (RS + 3) >> 2;
    const int per = (steps + nsplit - 1) / nsplit;
    const int u_begin = min(steps, ks * per), u_end = min(steps, u_begin + per);
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, g.x_bytes);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, g.w_bytes);
    const __amdgpu_buffer_rsrc_t zres = make_rsrc(g.x, 0u);        // panels beyond K read zeros
    half8 a[kRing][TM], b[kRing][TN];
    auto load_step = [&](const int buf, const int u) __attribute__((always_inline)) {
        const int tap = u * 4 + slot;
        const bool in = u < u_end && tap < RS;
        const int r = (int)(((uint32_t)tap * magic) >> 16), s = tap - r * S;
        const uint32_t avo = in ? (uint32_t)(tap * 64 + col) * 16u : kOobOffset;
#pragma unroll
        for (int m = 0; m < TM; ++m) {
            const bool ok = mb0 + m < g.K16;                        // uniform
            a[buf][m] = buf_load<half8>(ok ? wres : zres, avo, ok ? (uint32_t)(mb0 + m) * (uint32_t)RS * 1024u : 0u);
        }
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            const bool ok = in && px.valid[t] && (unsigned)(ih0[t] + r) < (unsigned)g.H && (unsigned)(iw0[t] + s) < (unsigned)g.W;
            b[buf][t] = buf_load<half8>(xres, ok ? (uint32_t)(xbase[t] + (r * g.W + s) * 16) : kOobOffset, 0u);
        }
    };
    auto compute = [&](const int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t)
                acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[buf][m], b[buf][t], acc[m][t], 0, 0, 0);
    };
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[m][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (u_begin >= u_end) return;
#pragma unroll
    for (int i = 0; i < kRing - 1; ++i) load_step(i, u_begin + i);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    int u = u_begin;
    while (u + kRing - 1 < u_end) {
#pragma unroll
        for (int i = 0; i < kRing; ++i) {
            load_step((i + kRing - 1) % kRing, u + i + kRing - 1);
            __builtin_amdgcn_sched_barrier(0);
            compute(i);
            __builtin_amdgcn_sched_barrier(0);
        }
        u += kRing;
    }
    if (u < u_end) {
#pragma unroll
        for (int i = 0; i < kRing - 1; ++i) compute(i);      // steps past the range are zeros
    }
}

// float16 1x1 filters, stride 1, no padding, planes of an even number of pixels: work items read x in
// pairs of pixels.  A matrix column may be any pixel as long as the store agrees, so column `col`
// of block t is pixel 2 * col + t of the tile's 32: one 4-byte load per channel carries both blocks'
// element, eight of them and eight v_perm make the two fragments.  What bounds the gather is the
// vector memory path: 16 two-byte loads and 2 of the weights for 4 MFMAs before, 8 and 4 for 8 MFMAs with
// four panels per tile now.  Measured (us, one call of the 1x1 layers of a stack): ResNet-50 41.7 -> 35.7,
// MobileNetV1 17.4 -> 14.6, MobileNetV2 17.6 -> 16.0, EfficientNet-B0 30.1 -> 26.8.
// A unit is a channel block; kRing units form the ring (3 and 4 of them measured the same or slower).
// The steady loop ends where a further load would lie past the range.
template <int TM>
__device__ __forceinline__ void gemm_accumulate_pairs(const GemmParams &g, const int mb0, const int nb0, const int ks,
                                                      const int nsplit, const int lane, floatx4 (&acc)[TM][2],
                                                      PixState<2> &px) {
    constexpr int kRing = 2;
    const int col = lane & 15, slot = lane >> 4;
    const int cbase = (mb0 / g.kg16) * g.Cg;
    const int PQ = g.P * g.Q;                             // H * W: stride 1, no padding
    const int n = nb0 * 16 + col * 2;
    const bool valid = n < g.npix;                        // npix is even: a pair is inside or outside as one
    const int nn = valid ? n : 0;
    const int img = g.N == 1 ? 0 : nn / PQ;
    const int pq = nn - img * PQ;
#pragma unroll
    for (int t = 0; t < 2; ++t) { px.img[t] = img; px.pq[t] = pq + t; px.valid[t] = valid; }
    const uint32_t voff = valid ? (uint32_t)((img * g.C + cbase + slot * 8) * PQ + pq) * 2u : kOobOffset;
    const int cblocks = g.cblocks;
    const int per = (cblocks + nsplit - 1) / nsplit;
    const int u_begin = min(cblocks, ks * per), u_end = min(cblocks, u_begin + per);
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, g.x_bytes);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, g.w_bytes);
    const __amdgpu_buffer_rsrc_t zres = make_rsrc(g.x, 0u);        // units past the range read zeros
    uint32_t a_voff[TM], a_base[TM];
#pragma unroll
    for (int m = 0; m < TM; ++m) {
        const bool ok = mb0 + m < g.K16;
        a_voff[m] = ok ? (uint32_t)lane * 16u : kOobOffset;
        a_base[m] = ok ? (uint32_t)(mb0 + m) * (uint32_t)cblocks : 0u;
    }
    half8 a[kRing][TM];
    uint32_t b[kRing][8];
    auto load_unit = [&](const int buf, const int u) __attribute__((always_inline)) {
        const bool ok = u < u_end;                                  // uniform
        const int cb = ok ? u : 0;
        const __amdgpu_buffer_rsrc_t wsel = ok ? wres : zres, xsel = ok ? xres : zres;
#pragma unroll
        for (int m = 0; m < TM; ++m) a[buf][m] = buf_load<half8>(wsel, a_voff[m], (a_base[m] + (uint32_t)cb) * 1024u);
        const bool part = g.c_rem != 0 && cb == cblocks - 1;        // uniform
        const int left = part ? g.c_rem - slot * 8 : 8;             // channels of this lane's eight that exist
#pragma unroll
        for (int i = 0; i < 8; ++i)
            b[buf][i] = __builtin_amdgcn_raw_buffer_load_b32(xsel, i < left ? voff : kOobOffset,
                                                             (uint32_t)cb * g.cb_stride + (uint32_t)i * g.plane_bytes, 0);
    };
    auto compute = [&](const int buf) __attribute__((always_inline)) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        u32x4 lo, hi;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            lo[i] = __builtin_amdgcn_perm(b[buf][2 * i + 1], b[buf][2 * i], 0x05040100u);
            hi[i] = __builtin_amdgcn_perm(b[buf][2 * i + 1], b[buf][2 * i], 0x07060302u);
        }
        const half8 b0 = __builtin_bit_cast(half8, lo), b1 = __builtin_bit_cast(half8, hi);
#pragma unroll
        for (int m = 0; m < TM; ++m) {
            acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[buf][m], b0, acc[m][0], 0, 0, 0);
            acc[m][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[buf][m], b1, acc[m][1], 0, 0, 0);
        }
    };
#pragma unroll
    for (int m = 0; m < TM; ++m) acc[m][0] = acc[m][1] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (u_begin >= u_end) return;
#pragma unroll
    for (int i = 0; i < kRing - 1; ++i) load_unit(i, u_begin + i);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    int u = u_begin;
    while (u + kRing - 1 < u_end) {
#pragma unroll
        for (int i = 0; i < kRing; ++i) {
            load_unit((i + kRing - 1) % kRing, u + i + kRing - 1);
            __builtin_amdgcn_sched_barrier(0);
            compute(i);
            __builtin_amdgcn_sched_barrier(0);
        }
        u += kRing;
    }
    if (u < u_end) {
#pragma unroll
        for (int i = 0; i < kRing - 1; ++i) compute(i);
    }
}

// Row state of a lane's outputs: for each of its 4 * TM rows the element offset of the row in y
// (k * P * Q, or out of range) and the bias value.
template <int TM> struct RowState {
    uint32_t off[TM][4];      // byte offset of (image 0, row k, pixel 0), kOobOffset for rows beyond K
    float bias[TM][4];
};

// Output channel of accumulator register (m, j) of a lane of `slot`, counted from the first panel of the tile;
// `mixed`: the blocks' rows are dealt out as in gemm_a_offset.
__device__ __forceinline__ int gemm_row(const bool mixed, const int tm, const int m, const int slot, const int j) {
    if (!mixed) return m * 16 + slot * 4 + j;
    const int qm = 16 / tm, i = slot * 4 + j;
    return i / qm * 16 + tm * (i % qm) + m;
}

template <int TM, bool MIXED = false>
__device__ __forceinline__ void gemm_rows(const GemmParams &g, const int mb0, const int slot, RowState<TM> &rs) {
    const int PQ = g.P * g.Q, Kg = g.Kg;
    const uint32_t esz = g.half_out ? 2u : 4u;
    const float *bias = g.bias;
    const int grp = mb0 / g.kg16, mbl = mb0 - grp * g.kg16;
    const __amdgpu_buffer_rsrc_t bres = make_rsrc(bias, bias ? (uint32_t)g.K * 4u : 0u);   // no bias: every load reads 0
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int kl = mbl * 16 + gemm_row(MIXED, TM, m, slot, j);         // row within the group
            const int k = grp * Kg + kl;
            const bool ok = kl < Kg;
            rs.off[m][j] = ok ? (uint32_t)(k * PQ) * esz : kOobOffset;
            rs.bias[m][j] = buf_load<float>(bres, ok ? (uint32_t)k * 4u : kOobOffset, 0u);
        }
}

// One finished output: bias, optional clamp at zero, one rounding to the storage type; the store is
// range-checked, so rows beyond K and pixels beyond the layer (offset out of range) write nothing.
__device__ __forceinline__ void gemm_store(const __amdgpu_buffer_rsrc_t yres, const bool relu, const bool half,
                                           const uint32_t off, const float bias, const float v) {
    float r = v + bias;
    if (relu) r = fmaxf(r, 0.f);
    if (half) {
        const _Float16 h = (_Float16)r;      // round to nearest even
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, h), yres, off, 0u, 0);
    } else {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, r), yres, off, 0u, 0);
    }
}

// Two neighbouring float16 outputs of a row.
__device__ __forceinline__ void gemm_store_pair(const __amdgpu_buffer_rsrc_t yres, const bool relu, const uint32_t off,
                                                const float bias, const float v0, const float v1) {
    typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
    float r0 = v0 + bias, r1 = v1 + bias;
    if (relu) { r0 = fmaxf(r0, 0.f); r1 = fmaxf(r1, 0.f); }
    const half2_t h = {(_Float16)r0, (_Float16)r1};      // round to nearest even
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, h), yres, off, 0u, 0);
}

// Byte offset of pixel (img, pq) within its row of y, or out of range.
__device__ __forceinline__ uint32_t gemm_pixel_offset(const GemmParams &g, const int img, const int pq, const bool valid) {
    const uint32_t esz = g.half_out ? 2u : 4u;
    return valid ? ((uint32_t)img * (uint32_t)(g.K * g.P * g.Q) + (uint32_t)pq) * esz : kOobOffset;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t gemm_y_rsrc(const GemmParams &g) {
    return make_rsrc(g.y, (uint32_t)g.N * (uint32_t)(g.K * g.P * g.Q) * (g.half_out ? 2u : 4u));
}

// ---- reductions cut into ranges: the partial sums of a tile meet in the workspace, and the wavefront or workgroup that stores the last of them adds
// them up, in the order of the ranges, and stores y.  A launch of its own for that took 4-6.5 us behind all items; here most tiles are added up while others
// are still multiplied.  What is left of it is latency, one trip to memory for the stores, one or two for the word of arrivals, one per few ranges.  us a call, launch / this:
// ResNet-18-shaped stack 39.2 / 36.5, MobileNetV2-shaped plan 33.6 / 30.0, ResNet-50 in float16 39.1 / 34.5.
// Nothing in the workspace has to be cleared: a tile's word of arrivals counts while its upper 48 bits are the launch's mark, any other content means that
// nobody has arrived, and the last one clears it.  Every launch has a mark of its own (a replayed one the same each time): what a launch leaves behind
// whose workspace another call overwrote while it ran, which spoils these two, means nothing to a later one.  The partial sums are stored through to memory and read past the caches that other
// XCDs do not share (sc1, the scope of one GPU); a wavefront waits for its stores before it, or the workgroup's first thread, arrives.
// More than kSplitMost ranges go in two steps, groups of them first: one wavefront takes 1.5 us for every three ranges of a 64 x 32 tile (ResNet-18-shaped stack at 130x111, whose
// 512-channel layers have 43, 42.2 -> 30.7 us a call; a launch behind the items took 34.3).
struct SplitTile {
    char *tile;         // [range][wavefront][block of 16 x 16][lane] floatx4, then the words of arrivals in 256 bytes: of the tile, of its groups
    int ks, n;          // which range; ranges in all (1: the item stores y itself)
    unsigned long long mark;
};
constexpr int kSplitScope = 16;                         // sc1
constexpr unsigned long long kSplitMark = 0x7fa5c3e996b1ull;    // of the first launch; 48 bits
constexpr size_t kSplitWord = 256;
constexpr int kSplitMost = 12, kSplitGroup = 6, kSplitGroups = 31;

__device__ __forceinline__ unsigned long long split_look(const char *word) {
    return __hip_atomic_load(reinterpret_cast<const unsigned long long *>(word), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One thread, which has looked at the word before (on its way beside the partial sums); true for the last of n.  (Every exchange that fails means that
// another arrival's went through since, and there are n of them.)
__device__ __forceinline__ bool split_arrive(char *word, const int n, unsigned long long seen, const unsigned long long mark) {
    unsigned long long *w = reinterpret_cast<unsigned long long *>(word);
    for (;;) {
        const int before = seen >> 16 == mark ? (int)(seen & 0xffff) : 0;
        const bool last = before + 1 >= n;
        if (__hip_atomic_compare_exchange_strong(w, &seen, last ? 0ull : mark << 16 | (unsigned long long)(before + 1), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return last;
    }
}

template <int TM, int TN>
__device__ __forceinline__ void split_put(const floatx4 (&acc)[TM][TN], const __amdgpu_buffer_rsrc_t res, const uint32_t off) {
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc[m][t]), res, off + (m * TN + t) * 1024u, 0u, kSplitScope);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// acc = the sum of n partial sums `stride` bytes apart, as many of them on their way as registers allow.
template <int TM, int TN>
__device__ __forceinline__ void split_sum(floatx4 (&acc)[TM][TN], const __amdgpu_buffer_rsrc_t res, const uint32_t off, const uint32_t first, const uint32_t stride, const int n) {
    constexpr int NB = TM * TN, G = NB >= 12 ? 2 : NB >= 7 ? 3 : 6;
    asm volatile("" ::: "memory");
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b / TN][b % TN] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int z = 0; z < n; z += G) {
        // (ranges past the last one load the last one again and are not added)
        floatx4 p[G][NB];
#pragma unroll
        for (int i = 0; i < G; ++i)
#pragma unroll
            for (int b = 0; b < NB; ++b)
                p[i][b] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(res, off + b * 1024u, first + (uint32_t)min(z + i, n - 1) * stride, kSplitScope));
#pragma unroll
        for (int i = 0; i < G; ++i)
            if (z + i < n) {
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b / TN][b % TN] += p[i][b];
            }
    }
}

// The sums of a tile whose reduction is cut, added by whichever of its wavefronts (WG: workgroups of four) is done last.  true: acc holds them.
// mine: the lane's place in a range; lds: WG, of the workgroup, no longer read by any of its wavefronts once they are here.
template <bool WG, int TM, int TN>
__device__ __forceinline__ bool split_fold(const SplitTile &sp, const uint32_t mine, char *lds, floatx4 (&acc)[TM][TN]) {
    constexpr uint32_t BYTES = (WG ? 4 : 1) * TM * TN * 1024;
    const __amdgpu_buffer_rsrc_t res = make_rsrc(sp.tile, (uint32_t)sp.n * BYTES);
    char *words = sp.tile + (size_t)sp.n * BYTES;
    const int size = sp.n <= kSplitMost ? sp.n : max(kSplitGroup, (sp.n + kSplitGroups - 1) / kSplitGroups);      // ranges of a group
    const int groups = (sp.n + size - 1) / size, grp = sp.ks / size;
    const bool one = WG ? threadIdx.x == 0 : (threadIdx.x & 63) == 0;
    // a group's ranges, unless there is one group only; then the groups' sums, each where its first range was
    int at = sp.ks, first = grp * size, step = 1, n = min(size, sp.n - first);
    char *word = words + (groups > 1 ? 8 + 8 * grp : 0);
#pragma unroll 1
    for (;;) {
        unsigned long long seen = 0;
        if (one) seen = split_look(word);
        split_put<TM, TN>(acc, res, (uint32_t)at * BYTES + mine);
        int last = 0;
        if constexpr (WG) {
            int *flag = reinterpret_cast<int *>(lds);
            __syncthreads();
            if (one) flag[0] = split_arrive(word, n, seen, sp.mark);
            __syncthreads();
            last = flag[0];
        } else if (one) last = split_arrive(word, n, seen, sp.mark);
        if (__builtin_amdgcn_readfirstlane(last) == 0) return false;
        split_sum<TM, TN>(acc, res, mine, (uint32_t)first * BYTES, (uint32_t)step * BYTES, n);
        if (word == words) return true;
        word = words;
        at = first;
        first = 0;
        step = size;
        n = groups;
    }
}

#include "tile_gemm.h"

// The KS partial tiles of a workgroup's tile nt meet in LDS: red[((nt * KS + ks) * NREG + reg) * 64 + lane].
template <int TM, int TN>
__device__ __forceinline__ void gemm_put_partial(const floatx4 (&acc)[TM][TN], float *red, const int KS, const int place, const int lane) {
    if (KS > 1) {
        constexpr int NREG = TM * TN * 4;
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) red[(place * NREG + (m * TN + t) * 4 + j) * 64 + lane] = acc[m][t][j];
    }
}

// ... and are added in fixed order; `share` of the tile's `sharers` wavefronts finishes the accumulator registers share,
// share + sharers, ..  Lane holds rows 4 * slot + j, column col of each block.  A barrier lies between, for the whole workgroup.
template <int TM, int TN, bool MIXED>
__device__ __forceinline__ void gemm_finish(const GemmParams &g, const int mb0, const int KS, const int share, const int sharers, const int nt, const int lane,
                                            const floatx4 (&acc)[TM][TN], const PixState<TN> &px, const float *red) {
    constexpr int NREG = TM * TN * 4;
    if (KS > 1) __syncthreads();
    RowState<TM> rs;
    gemm_rows<TM, MIXED>(g, mb0, lane >> 4, rs);
    const __amdgpu_buffer_rsrc_t yres = gemm_y_rsrc(g);
    const bool relu = g.relu, half_out = g.half_out;
    uint32_t pixoff[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) pixoff[t] = gemm_pixel_offset(g, px.img[t], px.pq[t], px.valid[t]);
#pragma unroll
    for (int m = 0; m < TM; ++m) {
#pragma unroll
        for (int t = 0; t < TN; ++t) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int reg = (m * TN + t) * 4 + j;
                if ((reg & (sharers - 1)) != share) continue;
                float v = acc[m][t][j];
                if (KS > 1) {
                    v = 0.f;
                    for (int z = 0; z < KS; ++z) v += red[((nt * KS + z) * NREG + reg) * 64 + lane];
                }
                // either offset may be the out-of-range constant 2^31; both at once would wrap to a small sum
                const uint32_t off = rs.off[m][j] == kOobOffset ? kOobOffset : rs.off[m][j] + pixoff[t];
                gemm_store(yres, relu, half_out, off, rs.bias[m][j], v);
            }
        }
    }
}

// One layer per launch: a workgroup of KS wavefronts owns one output tile, the wavefronts split
// the channel blocks and add their partial sums through LDS in fixed order.
// What bounds such a launch is the vector memory path of its CUs beside the latency of the first loads.  float32 3x3 tiles run the
// loop of the work items: one load carries the weights of both panels, and with a third of the registers the loads of a row do not queue
// behind three chunks of others.  us, whole chunks of nine taps in rings of 2 to 4 -> rows in a ring of 3: 128 channels at 28x28
// 8.1 -> 7.7, 512 at 7x7 14.7 -> 13.3, 512 -> 64 at 14x14 14.9 -> 12.5, 96 -> 100 at 20x30 8.9 -> 6.8.
// (the 32 x 32 tile is launched as one wavefront per workgroup only, and needs more than the 128
// registers a 16-wavefront workgroup leaves each lane)
template <bool HALF, int TM, int TN, int MODE, int NBUF>
__global__ __launch_bounds__(TM * TN == 8 ? 256 : TM * TN == 4 ? 64 : 1024) void im2col_gemm_kernel(const GemmParams g) {
    extern __shared__ __align__(16) float red[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar
    const int slot = lane >> 4;
    const int KS = 1 << g.ks_shift;
    const int ks = wave & (KS - 1), nt = wave >> g.ks_shift;             // k-split index, tile within the workgroup
    const int tiles_per_wg = (blockDim.x >> 6) >> g.ks_shift;
    const int ltile = xcd_logical_tile(g.grid_nx * g.grid_ny);
    if (ltile < 0) return;                                               // whole workgroup: grid padding
    const int bx = g.m_major ? ltile % g.grid_nx : ltile / g.grid_ny;
    const int by = g.m_major ? ltile / g.grid_nx : ltile % g.grid_ny;
    const int mb0 = by * TM;                              // panel index over all groups; TM panels stay in one group
    const int nb0 = (bx * tiles_per_wg + nt) * TN;
    floatx4 acc[TM][TN];
    PixState<TN> px;
    constexpr bool ROWS3 = !HALF && MODE == 3 && (TM == 4 || TN == 1), PATCH = MODE == kModePatch, MIXED = ROWS3 || PATCH;
    if constexpr (PATCH) {
        gemm_accumulate_patch(g, mb0, nb0, ks, KS, lane, red + wave * kPatchFloats, acc, px);
        if (KS > 1) __syncthreads();                                     // the partial sums take the place of the pixels
    } else if constexpr (ROWS3) gemm_accumulate_3x3<TM, TN, TM * TN <= 2 ? 2 : 1>(g, mb0, nb0, ks, KS, lane, acc, px);
    else if constexpr (MODE == kModeTaps) gemm_accumulate_taps<TM, TN>(g, mb0, nb0, ks, KS, lane, acc, px);
    else gemm_accumulate<HALF, TM, TN, MODE, NBUF>(g, mb0, nb0, ks, KS, lane, acc, px);

    gemm_put_partial<TM, TN>(acc, red, KS, nt * KS + ks, lane);
    gemm_finish<TM, TN, MIXED>(g, mb0, KS, ks, KS, nt, lane, acc, px, red);
}

// ---------------------------------------------------------------- many layers in one launch
// A batch-1 layer neither fills 256 CUs nor runs long enough to hide its launch, its first loads
// and its epilogue.  Independent layers (what the decision stage profiles, and what a model's
// parallel branches are) therefore go into ONE launch of single-wavefront workgroups, one per
// work item: an item is one output tile (TM x 2 blocks of 16 x 16) of one layer over one of the
// nsplit ranges its reduction is cut into, the ranges sized so that items of different layers
// take about the same time.  The chip's dispatcher balances the items over the CUs; two to four
// items are resident per SIMD, so one item's addressing and first loads run under another's
// MFMAs.  A split layer's items store partial tiles; the last of a tile's items adds them in fixed order.
struct GemmItemLayer {
    GemmParams g;
    char *part;         // partial tiles of a split layer (workspace)
    unsigned long long mark;    // of the launch, in the words of arrivals
    int ntn;            // tiles along the pixels
    int nsplit;         // ranges of the reduction (1: the item stores y itself)
    int mode, tm;       // chunking mode (ModeT); 16-row panels per tile (1, 2 or 4)
};
// A layer as the kernel argument carries it: 64 bytes, so that the layers of one call mostly fit one
// launch (56 of them; 20 with GemmItemLayer itself, which a wavefront derives from this in scalar registers).
// Three launches of a third of the layers each end with a nearly empty chip three times: the
// ResNet-50-shaped stack in float16 spent 40 + 29 + 24 us in them, the last with 368 workgroups.
struct GemmItemRec {
    const void *x, *wp;
    const float *bias;
    void *y;
    uint32_t part256;                    // offset of the partial tiles from the table's base, in 256 bytes
    int H, W;
    uint16_t N, C, K, nsplit, sh, sw, ph, pw;
    uint8_t R, S, groups;
    uint8_t mode : 3, tm : 3, relu : 1, tile : 1;
    // tile = 1: items of whole workgroups (tile_gemm.h), all of one group.  tm: panels per wavefront, + 4 if it holds seven blocks of 16 pixels, not
    // four.  mode: 3, 3x3 filters at equal strides (sh) and pads (ph), the fields that are free hold the tile: S, groups: its rows and columns; sw, pw: tiles
    // per row and per column of an image.  1, 1x1 filters.  kModeTaps, few channels, not split: the tile's rows and columns * 256 in part256.
    // 0, a depthwise layer (depthwise.h), R x R; groups: its filters are untransformed.
};
static_assert(sizeof(GemmItemRec) == 64, "sixteen scalar registers");
struct GemmItemTable {
    GemmItemRec layer[kMaxGemmLayers];
    // first item of each layer, INT_MAX beyond the last layer: a workgroup finds its layer by counting the entries it has reached (table_find)
    int item0[kMaxGemmLayers];
    char *part_base;
    unsigned long long mark;
    int nitems;
    int group;          // consecutive items handed to one XCD
};
static_assert(sizeof(GemmItemTable) <= 4096, "the table is passed by value as the kernel argument");

template <bool HALF, int TM, int MODE, int NBUF = 2>
__device__ __forceinline__ void gemm_item(const GemmItemLayer &L, const int local, const int lane) {
    constexpr int TN = 2;
    const int nb = local % L.ntn, rest = local / L.ntn;
    const int ks = rest % L.nsplit, mt = rest / L.nsplit;       // order: tile row, range, tile column (fastest)
    floatx4 acc[TM][TN];
    PixState<TN> px;
    if constexpr (!HALF && MODE == 3) gemm_accumulate_3x3<TM, TN, 1>(L.g, mt * TM, nb * TN, ks, L.nsplit, lane, acc, px);
    else if constexpr (MODE == kModeOctets) gemm_accumulate_octets<TM, TN>(L.g, mt * TM, nb * TN, ks, L.nsplit, lane, acc, px);
    else if constexpr (MODE == kModeTaps) gemm_accumulate_taps<TM, TN>(L.g, mt * TM, nb * TN, ks, L.nsplit, lane, acc, px);
    else if constexpr (MODE == kModePairs) gemm_accumulate_pairs<TM>(L.g, mt * TM, nb * TN, ks, L.nsplit, lane, acc, px);
    else if constexpr (!HALF && MODE == 1) gemm_accumulate_1x1<TM, TN>(L.g, mt * TM, nb * TN, ks, L.nsplit, lane, acc, px);
    else gemm_accumulate<HALF, TM, TN, MODE, NBUF>(L.g, mt * TM, nb * TN, ks, L.nsplit, lane, acc, px);
    __builtin_amdgcn_s_setprio(3);
    if (L.nsplit > 1) {
        const SplitTile sp{L.part + (size_t)(mt * L.ntn + nb) * ((size_t)L.nsplit * (TM * TN * 1024) + kSplitWord), ks, L.nsplit, L.mark};
        if (!split_fold<false, TM, TN>(sp, (uint32_t)lane * 16u, nullptr, acc)) return;
    }
    {
        RowState<TM> rs;
        gemm_rows<TM, !HALF && (MODE == 1 || MODE == 3)>(L.g, mt * TM, lane >> 4, rs);
        const __amdgpu_buffer_rsrc_t yres = gemm_y_rsrc(L.g);
        const bool relu = L.g.relu, half_out = L.g.half_out;
        uint32_t pixoff[TN];
#pragma unroll
        for (int t = 0; t < TN; ++t) pixoff[t] = gemm_pixel_offset(L.g, px.img[t], px.pq[t], px.valid[t]);
        __builtin_amdgcn_sched_barrier(0);      // parameters and bias values first, then nothing but stores
        if constexpr (MODE == kModePairs) {
            // the two blocks' values of a row are neighbouring pixels: one 4-byte store (even planes keep it aligned)
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t off = rs.off[m][j] == kOobOffset ? kOobOffset : rs.off[m][j] + pixoff[0];
                    gemm_store_pair(yres, relu, off, rs.bias[m][j], acc[m][0][j], acc[m][1][j]);
                }
            return;
        }
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t off = rs.off[m][j] == kOobOffset ? kOobOffset : rs.off[m][j] + pixoff[t];
                    gemm_store(yres, relu, half_out, off, rs.bias[m][j], acc[m][t][j]);
                }
    }
}

// The table is the kernel argument; the kernel reads it through the kernel-argument segment
// pointer (constant address space, scalar loads at computed offsets).  Indexing the by-value
// parameter itself with a run-time layer number makes the compiler copy all 4 KB of it to
// scratch memory first, in every wavefront.
typedef const __attribute__((address_space(4))) GemmItemTable *GemmItemTablePtr;

// All of it is uniform: scalar arithmetic on one 64-byte scalar load.
__device__ __forceinline__ void load_item_layer(GemmItemLayer &L, const GemmItemTablePtr tbl, const GemmItemRec &r, const bool half) {
    GemmParams &g = L.g;
    g.x = r.x; g.wp = r.wp; g.bias = r.bias; g.y = r.y;
    g.N = r.N; g.C = r.C; g.H = r.H; g.W = r.W; g.K = r.K; g.R = r.R; g.S = r.S;
    g.sh = r.sh; g.sw = r.sw; g.ph = r.ph; g.pw = r.pw;
    // (a division by a run-time value costs tens of instructions; strides are 1 or 2, groups 1, nearly always)
    auto out_size = [](int span, int stride) { return (stride == 1 ? span : stride == 2 ? span >> 1 : span / stride) + 1; };
    g.P = out_size(g.H + 2 * g.ph - g.R, g.sh);
    g.Q = out_size(g.W + 2 * g.pw - g.S, g.sw);
    g.npix = g.N * g.P * g.Q;
    g.Kg = r.groups == 1 ? g.K : g.K / r.groups;
    g.Cg = r.groups == 1 ? g.C : g.C / r.groups;
    g.kg16 = (g.Kg + 15) >> 4;
    g.K16 = r.groups * g.kg16;
    g.ks_shift = 0;
    g.grid_nx = g.grid_ny = g.m_major = 0;
    L.mode = r.mode;
    gemm_derived(g, half, r.mode);
    g.relu = r.relu;
    L.part = tbl->part_base + (size_t)r.part256 * 256;
    L.mark = tbl->mark;
    L.ntn = (g.npix + 31) >> 5;
    L.nsplit = r.nsplit;
    L.tm = r.tm;
}

constexpr int kItemWaves = 4;      // items per workgroup (one wavefront each)

// The tile of a record with tile = 1.
__device__ __forceinline__ void load_tile_layer(TileLayer &T, const GemmItemRec &r, const bool half) {
    T.x = r.x; T.wp = r.wp; T.bias = r.bias; T.y = r.y;
    T.N = r.N; T.C = r.C; T.H = r.H; T.W = r.W; T.K = r.K; T.pad = r.ph;
    T.K16 = (T.K + 15) >> 4;
    T.cblocks = half ? (T.C + 31) >> 5 : (T.C + 3) >> 2;
    T.relu = r.relu;
    if (!half || r.mode == 3) {
        T.st = half ? r.sh : 1;
        T.P = (half && T.st == 2 ? (r.H + 2 * T.pad - 3) >> 1 : r.H + 2 * T.pad - 3) + 1;
        T.Q = (half && T.st == 2 ? (r.W + 2 * T.pad - 3) >> 1 : r.W + 2 * T.pad - 3) + 1;
        T.th = r.S; T.tw = r.groups; T.ntw = r.sw; T.nth = r.pw;
        return;
    }
    T.R = r.R; T.S = r.S; T.sh = r.sh; T.sw = r.sw; T.padw = r.pw;
    T.P = (r.H + 2 * T.pad - T.R) / T.sh + 1;
    T.Q = (r.W + 2 * T.padw - T.S) / T.sw + 1;
    T.th = T.tw = T.nth = T.ntw = 1;
    if (r.mode == kModeTaps) {
        T.th = r.part256 & 255; T.tw = r.part256 >> 8;         // (not split)
        T.nth = (T.P + T.th - 1) / T.th;
        T.ntw = (T.Q + T.tw - 1) / T.tw;
    }
}
__device__ __forceinline__ int tile_regs(const GemmItemRec &r) { return (r.tm & 3) * (r.tm & 4 ? 28 : 16); }      // accumulator registers of a wavefront

__device__ __forceinline__ GemmItemRec load_item_rec(const GemmItemTablePtr tbl, const int li) {
    GemmItemRec r;
    const __attribute__((address_space(4))) uint32_t *src = (const __attribute__((address_space(4))) uint32_t *)&tbl->layer[li];
    uint32_t d[sizeof(GemmItemRec) / 4];
#pragma unroll
    for (int i = 0; i < (int)(sizeof(GemmItemRec) / 4); ++i) d[i] = src[i];
    __builtin_memcpy(&r, d, sizeof r);
    return r;
}

// Which whole-workgroup items a launch holds besides the others.  (A kernel with all of them is 25-30 KB longer than one without depthwise
// items, which costs launches that have none 2-4 %.)
constexpr int kNoTiles = 0, kTiles = 1, kLargeTiles = 2, kDepthwise = 3, kTilesDepthwise = 4;

__device__ __forceinline__ int one_tiles(const TileLayer &T, const GemmItemRec &r) {
    const int px = r.tm & 4 ? 112 : 64;
    return __builtin_amdgcn_readfirstlane((T.N * T.P * T.Q + px - 1) / px);
}

template <bool HALF>
__device__ __forceinline__ void run_depthwise_item(const GemmItemRec &r, const int blk) {
    DwParams d{r.N, r.C, r.H, r.W, r.sh, r.ph, r.pw, 0, 0, r.relu};
    d.P = (d.st == 2 ? (d.H + 2 * d.ph - r.R) >> 1 : d.H + 2 * d.ph - r.R) + 1;
    d.Q = (d.st == 2 ? (d.W + 2 * d.pw - r.R) >> 1 : d.W + 2 * d.pw - r.R) + 1;
    depthwise_workgroup<typename std::conditional<HALF, __half, float>::type>(r.x, r.wp, r.bias, r.y, d, r.R, r.groups != 0, blk);
}

template <bool HALF, int TILE, bool SPLIT>
__device__ __forceinline__ void run_tile_item(const GemmItemTablePtr tbl, const GemmItemRec &r, const int local, char *lds) {
    TileLayer T;
    load_tile_layer(T, r, HALF);
    // order: pixel tile fastest, then the range of channels, then the panels
    const int ntiles = HALF && r.mode == 1 ? one_tiles(T, r) : T.N * T.nth * T.ntw, nsplit = SPLIT ? r.nsplit : 1;
    const int rest = __builtin_amdgcn_readfirstlane(local / ntiles), nt = local - rest * ntiles;
    const int mt = __builtin_amdgcn_readfirstlane(rest / nsplit), ks = rest - mt * nsplit;
    const int chunks = (T.C + kTileChannels - 1) / kTileChannels;
    int per = chunks;
    if (nsplit > 1) per = __builtin_amdgcn_readfirstlane((chunks + nsplit - 1) / nsplit);
    const int c0 = ks * per, c1 = min(chunks, c0 + per);
    const SplitTile sp{tbl->part_base + (size_t)r.part256 * 256 + (size_t)(mt * ntiles + nt) * ((size_t)nsplit * (tile_regs(r) * 1024u) + kSplitWord), ks, SPLIT ? nsplit : 1, tbl->mark};
    if constexpr (HALF && TILE != kLargeTiles) {
        if (r.mode == kModeTaps) {
            if (r.tm == 5) few_item<7>(T, mt, nt, lds);
            else few_item<4>(T, mt, nt, lds);
            return;
        }
        if (r.mode == 3 && r.sh == 2) {
            tile_item<true, 1, 4, true, kTilePatch2 / 64>(T, mt, nt, c0, c1, sp, lds);
            return;
        }
        if (r.mode == 1) {
            switch (r.tm) {
                case 6: one_item<2, 7, true>(T, mt, nt, c0, c1, sp, lds); break;
                case 5: one_item<1, 7, true>(T, mt, nt, c0, c1, sp, lds); break;
                case 2: one_item<2, 4, false>(T, mt, nt, c0, c1, sp, lds); break;
                default: one_item<1, 4, false>(T, mt, nt, c0, c1, sp, lds); break;
            }
            return;
        }
    }
    if constexpr (TILE == kLargeTiles) tile_item<HALF, 2, 7, true>(T, mt, nt, c0, c1, sp, lds);
    else if (r.tm == 5) tile_item<HALF, 1, 7, false>(T, mt, nt, c0, c1, sp, lds);
    else tile_item<HALF, 1, 4, false>(T, mt, nt, c0, c1, sp, lds);
}

template <bool HALF, int TILE, bool SPLIT>
__global__ __launch_bounds__(64 * kItemWaves, TILE == kLargeTiles ? 2 : 3) void gemm_items_kernel(const GemmItemTable tbl_arg) {
    constexpr int NBUF = 2;
    const GemmItemTablePtr tbl = (GemmItemTablePtr)__builtin_amdgcn_kernarg_segment_ptr();
    // Workgroup i runs on XCD i % 8.  Groups of `group` consecutive items (neighbouring tiles of
    // one layer: they share a weight panel) are dealt to the XCDs in turn, so every XCD sees the
    // same mix of layers in the same order and a panel is fetched into one L2.
    // An item's addressing competes for issue slots with the MFMA loops of the other wavefronts on
    // its SIMD, which always have an instruction ready: without a higher priority it is served
    // last and takes several microseconds.  The k-loop drops back to the default priority.
    __builtin_amdgcn_s_setprio(3);
    // The wavefronts of a workgroup take consecutive items (neighbouring tiles along the pixels:
    // the same weight fragments at about the same time, so three of four reads of them hit in
    // the CU's L1); they share nothing else and never wait for one another.
    const int G = tbl->group;
    const int i = blockIdx.x, xcd = i & 7, j = i >> 3;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int item = (((j / G) * 8 + xcd) * G + j % G) * kItemWaves + wave;
    if (item >= tbl->nitems) return;
    int first;
    const int li = table_find<kMaxGemmLayers>(&tbl->item0[0], item, first);
    const GemmItemRec rec = load_item_rec(tbl, li);
    if constexpr (TILE == kDepthwise || TILE == kTilesDepthwise) {
        if (rec.tile && rec.mode == 0) {
            __builtin_amdgcn_s_setprio(0);
            run_depthwise_item<HALF>(rec, (item - first) / kItemWaves);
            return;
        }
    }
    if constexpr (TILE == kTiles || TILE == kTilesDepthwise || TILE == kLargeTiles) {
        __shared__ __align__(16) char tile_lds[HALF ? (TILE == kLargeTiles ? 8 * kTilePatch * 16 : 8 * kTilePatch2 * 16) : TILE == kLargeTiles ? 2 * kTileBuffer : kTileBuffer];
        // (every layer of such a launch starts with a workgroup of its own: all four wavefronts come here or none does)
        if (TILE == kLargeTiles || rec.tile) {
            run_tile_item<HALF, TILE, SPLIT>(tbl, rec, (item - first) / kItemWaves, tile_lds);
            return;
        }
    }
    GemmItemLayer L;
    load_item_layer(L, tbl, rec, HALF);
    if (!SPLIT) L.nsplit = 1;
    const int local = item - first;
    if (TILE != kNoTiles && local >= ((L.g.K16 + L.tm - 1) / L.tm) * L.ntn * L.nsplit) return;      // the layer's last workgroup is not full
    const int lane = threadIdx.x & 63;
    if (L.tm == 4) {
        if constexpr (!HALF) {
            if (L.mode == 3) gemm_item<false, 4, 3, NBUF>(L, local, lane);
            else if (L.mode == 7) gemm_item<false, 4, 7, NBUF>(L, local, lane);
            else gemm_item<false, 4, 1, NBUF>(L, local, lane);
        } else {
            if (L.mode == kModePairs) gemm_item<true, 4, kModePairs>(L, local, lane);
            else if (L.mode == kModeOctets) gemm_item<true, 4, kModeOctets>(L, local, lane);
            else gemm_item<true, 4, kModeTaps>(L, local, lane);
        }
    } else if (L.tm == 2) {
        switch (L.mode) {
            case 1: gemm_item<HALF, 2, 1, NBUF>(L, local, lane); break;
            case kModePairs: if constexpr (HALF) gemm_item<HALF, 2, kModePairs>(L, local, lane); break;
            case kModeTaps: if constexpr (HALF) gemm_item<HALF, 2, kModeTaps>(L, local, lane); break;
            case 3: gemm_item<HALF, 2, 3, NBUF>(L, local, lane); break;
            case 5: if constexpr (!HALF) gemm_item<HALF, 2, 5, NBUF>(L, local, lane); break;
            case 7: if constexpr (!HALF) gemm_item<HALF, 2, 7, NBUF>(L, local, lane); break;
            default: gemm_item<HALF, 2, 0, NBUF>(L, local, lane); break;
        }
    } else {
        switch (L.mode) {
            case 1: gemm_item<HALF, 1, 1, NBUF>(L, local, lane); break;
            case kModePairs: if constexpr (HALF) gemm_item<HALF, 1, kModePairs>(L, local, lane); break;
            case kModeTaps: if constexpr (HALF) gemm_item<HALF, 1, kModeTaps>(L, local, lane); break;
            case 3: gemm_item<HALF, 1, 3, NBUF>(L, local, lane); break;
            case 5: if constexpr (!HALF) gemm_item<HALF, 1, 5, NBUF>(L, local, lane); break;
            case 7: if constexpr (!HALF) gemm_item<HALF, 1, 7, NBUF>(L, local, lane); break;
            default: gemm_item<HALF, 1, 0, NBUF>(L, local, lane); break;
        }
    }
}

// ---------------------------------------------------------------- several layers, each as its own launch would run it
// Layers of a cold pass that do not depend on one another, in one launch: the tiles and the splits of the reduction are those of
// im2col_gemm_kernel, and so are the results, bit for bit (a caller may not see whether a layer shared a launch).  What it
// saves: a batch-1 layer leaves most of the chip idle for most of its 8-16 us.  Workgroups of eight wavefronts hold 8 / KS tiles, or one
// of KS = 16, whose wavefronts then take two ranges each.  Every layer's blocks are a multiple of eight, so that the XCD of a
// block does not depend on what else is in the launch.  Measured, us a cold pass of a stack (batch 1, 224 x 224), one launch a layer ->
// this: ResNet-18-shaped 206 -> 113, ResNet-50 463 -> 296, GoogLeNet 362 -> 89, SqueezeNet 151 -> 52, AlexNet 76 -> 51; MobileNetV2 (a chain)
// 224 -> 221.  Two workgroups per CU; with fewer registers, for a third one, it takes as long.
// What bounds a launch of such layers is the sum of their wavefronts, each of them mostly latency, over what the chip holds at once: a
// wavefront whose share of the products would be below the chip's average takes a tile of two panels, then two blocks of pixels as well (the sums stay the same).  us a cold pass, tiles as
// alone (two blocks of pixels in launches of more than 1024 workgroups) / this: ResNet-18 123 / 113, ResNet-50 318 / 296, AlexNet 57 / 51, GoogLeNet 94 / 89 (2x130x300 139 / 128).
constexpr int kLayerWaves = 8;      // 1 << 3
constexpr int kLayerResident = 256 * 2 * kLayerWaves;       // wavefronts
constexpr int kLayerRed = 16 * 8 * 64;      // partial tiles: KS = 16, two panels, or KS = 8, two and two blocks of pixels
struct GemmLayersTable {
    GemmParams g[kMaxMergedLayers];           // grid_nx, grid_ny: workgroups along the pixels, tiles along the panels
    int block0[kMaxMergedLayers];             // first workgroup of each layer, INT_MAX beyond the last one
    uint8_t variant[kMaxMergedLayers];        // mode + 16 if a tile has two panels, + 32 if two blocks of pixels
};
static_assert(sizeof(GemmLayersTable) <= 4096, "the table is passed by value as the kernel argument");
typedef const __attribute__((address_space(4))) GemmLayersTable *GemmLayersTablePtr;

template <int TM, int TN, int MODE>
__device__ __forceinline__ void gemm_layer_block(const GemmParams &g, const int blk, float *red) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int KS = 1 << g.ks_shift, pshift = min(g.ks_shift, 3), per_tile = 1 << pshift, ks = wave & (per_tile - 1);
    const int nt = wave >> pshift, tiles = kLayerWaves >> pshift;
    const int total = g.grid_nx * g.grid_ny, per = (total + 7) >> 3, ltile = (blk & 7) * per + (blk >> 3);
    if (ltile >= total) return;                            // whole workgroup: padding
    const int div = g.m_major ? g.grid_nx : g.grid_ny, hi = __builtin_amdgcn_readfirstlane(ltile / div), lo = ltile - hi * div;
    const int mb0 = (g.m_major ? hi : lo) * TM, nb0 = ((g.m_major ? lo : hi) * tiles + nt) * TN;
    floatx4 acc[TM][TN];
    PixState<TN> px;
#pragma nounroll
    for (int z = ks; z < KS; z += per_tile) {
        if constexpr (MODE == 3) gemm_accumulate_3x3<TM, TN, 2>(g, mb0, nb0, z, KS, lane, acc, px);
        else if constexpr (MODE == kModePatch) gemm_accumulate_patch(g, mb0, nb0, z, KS, lane, red + kLayerRed + wave * kPatchFloats, acc, px);
        else gemm_accumulate<false, TM, TN, MODE, 2>(g, mb0, nb0, z, KS, lane, acc, px);
        gemm_put_partial<TM, TN>(acc, red, KS, nt * KS + z, lane);
    }
    gemm_finish<TM, TN, MODE == 3 || MODE == kModePatch>(g, mb0, KS, ks, per_tile, nt, lane, acc, px, red);
}

__global__ __launch_bounds__(64 * kLayerWaves, 4) void gemm_layers_kernel(const GemmLayersTable tbl_arg) {
    __shared__ __align__(16) float red[kLayerRed + kLayerWaves * kPatchFloats];
    const GemmLayersTablePtr tbl = (GemmLayersTablePtr)__builtin_amdgcn_kernarg_segment_ptr();
    int first;
    const int li = table_find<kMaxMergedLayers>(&tbl->block0[0], (int)blockIdx.x, first);
    GemmParams g;
    {
        static_assert(sizeof(GemmParams) % 4 == 0, "copied word by word");
        const __attribute__((address_space(4))) uint32_t *src = (const __attribute__((address_space(4))) uint32_t *)&tbl->g[li];
        uint32_t d[sizeof(GemmParams) / 4];
#pragma unroll
        for (int i = 0; i < (int)(sizeof(GemmParams) / 4); ++i) d[i] = src[i];
        __builtin_memcpy(&g, d, sizeof g);
    }
    const int blk = (int)blockIdx.x - first;
#define NNV_LAYER_BLOCK(V, TM, TN)                                     \
    case V + 1: gemm_layer_block<TM, TN, 1>(g, blk, red); break;       \
    case V + 3: gemm_layer_block<TM, TN, 3>(g, blk, red); break;       \
    case V + 5: gemm_layer_block<TM, TN, 5>(g, blk, red); break;       \
    case V + 7: gemm_layer_block<TM, TN, 7>(g, blk, red); break;       \
    case V: gemm_layer_block<TM, TN, 0>(g, blk, red); break;
    switch (tbl->variant[li]) {
        NNV_LAYER_BLOCK(0, 1, 1)
        NNV_LAYER_BLOCK(16, 2, 1)
        NNV_LAYER_BLOCK(32, 1, 2)
        NNV_LAYER_BLOCK(48, 2, 2)
        case kModePatch: gemm_layer_block<1, 1, kModePatch>(g, blk, red); break;
    }
#undef NNV_LAYER_BLOCK
}

// half NCHW -> half [N][cpad / 8][H][W][8]: octets of channels, zero padded to a multiple of 32.
// Lanes 0..15 of a fragment load are 16 pixels of one octet: here they read 256 consecutive bytes.  (From
// [N][H][W][cpad], the first version, each of them read another cache line, and a load took 64 cycles of the
// CU's memory path instead of 16.  Measured, us a call: VGG-16-shaped stack 161 -> 85, ResNet-50 75 -> 62,
// ResNet-18 48 -> 39.)  A thread converts one pixel of an octet; both sides are coalesced.
__device__ __forceinline__ void to_octet(const __half *__restrict__ x, __half *__restrict__ xt, const int C, const int HW,
                                         const int octs, const int img, const int oct, const int pix) {
    __half v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int c = oct * 8 + j;
        v[j] = (c < C) ? x[((size_t)img * C + c) * HW + pix] : __float2half(0.f);
    }
    *reinterpret_cast<uint4 *>(xt + (((size_t)img * octs + oct) * HW + pix) * 8) = *reinterpret_cast<uint4 *>(v);
}

__global__ __launch_bounds__(256) void to_octets_kernel(const __half *__restrict__ x, __half *__restrict__ xt, int C, int HW) {
    const int pix = blockIdx.x * 256 + threadIdx.x;
    if (pix < HW) to_octet(x, xt, C, HW, gridDim.y, blockIdx.z, blockIdx.y, pix);
}

// The same conversion for several layers in one launch: a workgroup finds its layer by its index,
// as the item kernel does, then converts 256 pixels of 32 channels of one image.
struct OctetTable {
    const __half *x[kMaxGemmLayers];
    __half *xt[kMaxGemmLayers];
    int C[kMaxGemmLayers], HW[kMaxGemmLayers], octs[kMaxGemmLayers];
    int block0[kMaxGemmLayers];      // first workgroup of each layer, INT_MAX beyond the last one
    int nblocks;
};
static_assert(sizeof(OctetTable) <= 4096, "the table is passed by value as the kernel argument");
typedef const __attribute__((address_space(4))) OctetTable *OctetTablePtr;
constexpr int kOctetsPerBlock = 4;

__global__ __launch_bounds__(256) void to_octets_many_kernel(const OctetTable tbl_arg) {
    const OctetTablePtr tbl = (OctetTablePtr)__builtin_amdgcn_kernarg_segment_ptr();
    const int b = blockIdx.x;
    if (b >= tbl->nblocks) return;
    int first;
    const int li = table_find<kMaxGemmLayers>(&tbl->block0[0], b, first);
    const int C = tbl->C[li], HW = tbl->HW[li], octs = tbl->octs[li];
    const __half *x = tbl->x[li];
    __half *xt = tbl->xt[li];
    // (pixels, octets) of an image in one run: small planes fill their workgroups too
    const int per_img = HW * octs, npb = (per_img + 256 * kOctetsPerBlock - 1) / (256 * kOctetsPerBlock);
    const int local = b - first;
    const int img = local / npb, e0 = (local - img * npb) * (256 * kOctetsPerBlock) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < kOctetsPerBlock; ++i) {
        const int e = e0 + i * 256;
        if (e < per_img) to_octet(x, xt, C, HW, octs, img, e / HW, e % HW);
    }
}

// ---------------------------------------------------------------- host side

struct GemmPlan {
    int tm, tn, ks_shift, mode, nbuf;
    size_t xt_bytes;
};

// channels of the float16 copy of x
static int copy_channels(const Geo &g, int mode) { return mode == kModeTaps ? 8 : ceil_div(g.c, 32) * 32; }

static GemmPlan plan_im2col(const Geo &g) {
    GemmPlan pl{};
    const bool half = g.dtype == NNV_F16;
    const int kg16 = ceil_div(g.kg, 16);
    const int K16 = g.groups * kg16;
    const int npix16 = ceil_div(g.n * g.p * g.q, 16);
    const int cblocks = half ? ceil_div(g.cg, 32) : ceil_div(g.cg, 4);
    const bool partial = !half && (g.cg % 4) != 0;
    if (g.r == 1 && g.s == 1 && !partial) pl.mode = 1;
    else if (half && g.groups == 1 && g.c <= kTapsMaxChannels) pl.mode = kModeTaps;
    else if (g.r == 3 && g.s == 3) pl.mode = 3;
    else if (g.s == 7 && !half) pl.mode = 7;
    else if (g.s == 5 && !half) pl.mode = 5;
    else pl.mode = 0;
    const bool row = pl.mode == 5 || pl.mode == 7 || (pl.mode == 3 && half);
    const int nunits = pl.mode == kModeTaps ? ceil_div(g.r * g.s, 4) : pl.mode == 0 ? cblocks * g.r * g.s : row ? cblocks * g.r : cblocks;
    const int unit_steps = (pl.mode == 0 || pl.mode == kModeTaps) ? 1 : row ? pl.mode : g.r * g.s;
    auto tiles = [&](int tm, int tn) { return (long)ceil_div(K16, tm) * ceil_div(npix16, tn); };
    // Batch-1 layers are latency-bound.  What pays (measured on ResNet-18-shaped layers): the
    // 32x32 tile only with thousands of tiles; the 32x16 tile while it still leaves >= 160 tiles,
    // its units split over KS wavefronts up to ~2048 wavefronts (1536 for float32 3x3, whose wavefronts of two channel blocks are mostly start: 64 channels at 56x56
    // 7.8 -> 7.7 us, weights from HBM 7.4, 128 at 28x28 8.0 -> 7.6, 64 at 56x56 -> 128 at stride 2 7.9 -> 6.9; a wavefront's two chains of products keep the error where
    // twice the wavefronts had it, gemm_accumulate_3x3); else the 16x16 tile with a
    // moderate split (>= 768 wavefronts) and a deeper register ring, because its few workgroups
    // stream the weights from HBM and each CU keeps only so many misses in flight.
    auto split_for = [&](long t, long target) {
        int shift = 0;
        while (shift < 4 && (t << shift) < target && (nunits >> (shift + 1)) >= 1 &&
               (((long)nunits * unit_steps) >> (shift + 1)) >= 9)
            ++shift;
        return shift;
    };
    // Large float32 3x3 layers: 64 x 32 tiles, 9 loads per 24 MFMAs.  One such tile of 256 channels is 61 us of matrix
    // instructions, so a workgroup of two or four wavefronts shares it: as many as give every SIMD one
    // (1400), and more as long as each keeps 108 steps.  Below that number the smaller tiles are the better ones,
    // unless the reduction is long.  Measured, us (channels, maps, tiles): 256, 8x56x56, 3136: 283 -> 252;
    // 256, 1x56x56, 392: 49 -> 44; 512, 8x14x14, 392: 100 -> 81; 512, 16x7x7, 200: 59 -> 48; 200 to 400, 8x20x20, 700: 62 -> 51; 64, 1x224x224, 1568:
    // 46.5 -> 44.5; 64, 1x112x112, 392: 17.2 -> 17.0; 64, 1x56x56, 98: 7.7 against 12.2 (kept).  1x1 layers lose 20 %.
    if (!half && g.groups == 1 && pl.mode == 3 && (kg16 % 4 == 0 || kg16 >= 12)) {
        const long t = tiles(4, 2);
        const int steps = cblocks * 9;
        int shift = 0;
        while (shift < 2 && ((t << shift) < 1400 || (steps >> (shift + 1)) >= 108)) ++shift;
        if ((t << shift) >= 1400 || (t >= 180 && steps >= 576)) {
            pl.tm = 4; pl.tn = 2; pl.nbuf = 2;
            pl.ks_shift = shift;
            return pl;
        }
    }
    // (the float16 1x1 gather keeps eight loads per fragment in flight: no room for the 32x32 tile)
    if (tiles(2, 2) >= 4096 && !(half && pl.mode == 1)) { pl.tm = 2; pl.tn = 2; pl.ks_shift = 0; }
    else if (tiles(2, 1) >= 160) { pl.tm = 2; pl.tn = 1; pl.ks_shift = split_for(tiles(2, 1), !half && pl.mode == 3 ? 1536 : 2048); }
    else {
        pl.tm = 1; pl.tn = 1;
        pl.ks_shift = split_for(tiles(1, 1), 768);
        // float32 3x3, whose loop keeps fewer registers (two filter rows ahead): twice the wavefronts as long as each keeps 72 steps.
        // us without / with, [channels, maps -> outputs]: [256, 14x14 -> 256] 9.6 / 8.0, [999, 12x32 -> 148] 27.5 / 20.7, [1024, 7x7 -> 1024] 39 /
        // 26; below 72 steps [256, 2x7x7 -> 256] 8.4 / 8.9.
        if (!half && pl.mode == 3 && pl.ks_shift < 3 && (tiles(1, 1) << pl.ks_shift) < 1536 && (((long)nunits * unit_steps) >> (pl.ks_shift + 1)) >= 72) ++pl.ks_shift;
    }
    if (g.groups > 1 && kg16 % pl.tm != 0) {       // a wavefront's panels must belong to one group
        pl.tm = 1; pl.tn = 1;
        pl.ks_shift = split_for(tiles(1, 1), 2048);
    }
    // depth of the register ring: never more sets than the wavefront has chunks to load
    const int units_per_wave = ceil_div(nunits, 1 << pl.ks_shift);
    const int chunk_units = pl.mode == 1 ? (half ? 2 : 8) : 1;
    const int chunks = ceil_div(units_per_wave, chunk_units);
    pl.nbuf = 2;
    if (pl.tm == 1 && chunks >= 6) pl.nbuf = 4;
    else if (pl.tm * pl.tn <= 2 && chunks >= 3) pl.nbuf = 3;
    if (half || pl.tm * pl.tn == 4 || pl.mode == 3) pl.nbuf = 2;       // (float32 3x3: rings of three filter rows, gemm_accumulate_3x3)
    // float16 needs the copy of x in octets of channels, except for 1x1 filters (gathered from NCHW)
    pl.xt_bytes = (half && pl.mode != 1) ? align_up((size_t)g.n * g.h * g.w * copy_channels(g, pl.mode) * sizeof(__half), 256) : 0;
    return pl;
}

size_t im2col_workspace_bytes(const Geo &g) { return plan_im2col(g).xt_bytes; }

// Where the pixels of a tile go through LDS (gemm_accumulate_patch): tiles of 16 x 16 whose wavefronts have enough channels to make up for a longer start.  us a layer alone, gathered /
// through LDS, [channel blocks of a wavefront, channels, maps -> outputs], weights and pixels from HBM: [12, 200, 28x28 -> 64] 8.6 / 8.3, [12, 189, 6x21x9 -> 49] 9.8 / 10.3, [15, 248, 2x18x52 -> 26] 11.6 / 10.0,
// [16, 512, 7x7 -> 512] 14.2 / 12.5, [14, 462, 4x18x13 -> 48] 13.2 / 12.0, [22, 721, 2x9x8 -> 294] 18.5 / 16.4, [30, 973, 2x26x15 -> 81] 40.3 / 31.3; 72 layers, geometric mean 0.90 (0.74-1.05).  Read again and again,
// out of the caches, gathered pixels are close by and the longer start counts up to 15 blocks of four wavefronts: the same layers 6.6 / 8.3, 9.5 / 10.3, 7.6 / 9.6, 11.6 / 12.3, 12.8 / 11.8, 15.7 / 15.9, 39.3 /
// 31.0, geometric mean 0.97 (0.74-1.29).  A layer of a network finds its operands displaced by the others' (cold ResNet-18-shaped pass 118 / 113), which is what the line is drawn for.
// Tiles of two panels gain nothing (60 outputs of 318 channels at 73x75 27.6 / 30.3), nor does stride 2, whose rows are twice as long (256, 14x14 -> 512 8.4 / 9.6).
constexpr int kPatchMinBlocks = 12;
static bool patch_pays(const Geo &g, const GemmPlan &pl) {
    if (g.dtype != NNV_F32 || pl.mode != 3 || pl.tm * pl.tn != 1 || g.sh != 1 || g.sw != 1 || g.pw != 1) return false;
    return ceil_div(g.cg, 4) >> pl.ks_shift >= kPatchMinBlocks;
}

template <bool HALF, int TM, int TN, int NBUF>
static void launch_gemm_mode(int mode, const GemmParams &gp, dim3 grid, dim3 block, size_t lds, hipStream_t st) {
    switch (mode) {
        case 1: if constexpr (!HALF || TM * TN < 4) { hipLaunchKernelGGL((im2col_gemm_kernel<HALF, TM, TN, 1, NBUF>), grid, block, lds, st, gp); } break;
        case 3: if constexpr (NBUF == 2) { hipLaunchKernelGGL((im2col_gemm_kernel<HALF, TM, TN, 3, NBUF>), grid, block, lds, st, gp); } break;
        case kModeTaps: if constexpr (HALF) { hipLaunchKernelGGL((im2col_gemm_kernel<HALF, TM, TN, kModeTaps, NBUF>), grid, block, lds, st, gp); } break;
        case kModePatch: if constexpr (!HALF && NBUF == 2 && TM * TN == 1) { hipLaunchKernelGGL((im2col_gemm_kernel<HALF, TM, TN, kModePatch, NBUF>), grid, block, lds, st, gp); } break;
        case 5: if constexpr (!HALF) { hipLaunchKernelGGL((im2col_gemm_kernel<HALF, TM, TN, 5, NBUF>), grid, block, lds, st, gp); } break;
        case 7: if constexpr (!HALF) { hipLaunchKernelGGL((im2col_gemm_kernel<HALF, TM, TN, 7, NBUF>), grid, block, lds, st, gp); } break;
        default: hipLaunchKernelGGL((im2col_gemm_kernel<HALF, TM, TN, 0, NBUF>), grid, block, lds, st, gp); break;
    }
}

template <bool HALF>
static void launch_gemm_variant(const GemmPlan &pl, const GemmParams &gp, dim3 grid, dim3 block, size_t lds, hipStream_t st) {
    if (pl.tm == 4) {
        if constexpr (!HALF) hipLaunchKernelGGL((im2col_gemm_kernel<false, 4, 2, 3, 2>), grid, block, lds, st, gp);
    } else if (pl.tm == 2 && pl.tn == 2) launch_gemm_mode<HALF, 2, 2, 2>(pl.mode, gp, grid, block, lds, st);
    else if constexpr (HALF) {      // rings of two only
        if (pl.tm == 2) launch_gemm_mode<true, 2, 1, 2>(pl.mode, gp, grid, block, lds, st);
        else launch_gemm_mode<true, 1, 1, 2>(pl.mode, gp, grid, block, lds, st);
    } else if (pl.tm == 2) {
        if (pl.nbuf >= 3) launch_gemm_mode<false, 2, 1, 3>(pl.mode, gp, grid, block, lds, st);
        else launch_gemm_mode<false, 2, 1, 2>(pl.mode, gp, grid, block, lds, st);
    } else {
        if (pl.nbuf >= 4) launch_gemm_mode<false, 1, 1, 4>(pl.mode, gp, grid, block, lds, st);
        else if (pl.nbuf == 3) launch_gemm_mode<false, 1, 1, 3>(pl.mode, gp, grid, block, lds, st);
        else launch_gemm_mode<false, 1, 1, 2>(pl.mode, gp, grid, block, lds, st);
    }
}

// Kernel parameters of a layer apart from the tile plan.
static GemmParams gemm_params(const Geo &g, int mode, const void *x, const void *w, const float *bias, void *y) {
    const bool half = g.dtype == NNV_F16;
    GemmParams gp{};
    gp.x = x; gp.wp = w; gp.bias = bias; gp.y = y;
    gp.N = g.n; gp.C = g.c; gp.H = g.h; gp.W = g.w; gp.K = g.k; gp.R = g.r; gp.S = g.s;
    gp.sh = g.sh; gp.sw = g.sw; gp.ph = g.ph; gp.pw = g.pw; gp.P = g.p; gp.Q = g.q;
    gp.npix = g.n * g.p * g.q;
    gp.kg16 = ceil_div(g.kg, 16);
    gp.K16 = g.groups * gp.kg16;
    gp.Kg = g.kg; gp.Cg = g.cg;
    gp.relu = g.relu;
    gemm_derived(gp, half, mode);
    return gp;
}

// float16 layers with a filter larger than 1x1 read x from a copy in octets of channels in the workspace.
static void launch_octets(const Geo &g, const GemmParams &gp, const void *x, void *xt, hipStream_t st) {
    dim3 grid(ceil_div(g.h * g.w, 256), gp.cpad / 8, g.n);
    hipLaunchKernelGGL(to_octets_kernel, grid, dim3(256), 0, st, static_cast<const __half *>(x),
                       static_cast<__half *>(xt), g.c, g.h * g.w);
}

static hipError_t launch_im2col_plain(const Geo &g, const void *x, const void *w, const float *bias, void *y, void *ws, hipStream_t st) {
    GemmPlan pl = plan_im2col(g);
    const bool half = g.dtype == NNV_F16;
    GemmParams gp = gemm_params(g, pl.mode, x, w, bias, y);
    gp.ks_shift = pl.ks_shift;
    if (half && pl.mode != 1) {
        launch_octets(g, gp, x, ws, st);
        gp.x = ws;
    }
    const int KS = 1 << pl.ks_shift;
    const int waves = KS;
    const int tiles_per_wg = waves / KS;
    const int npix16 = ceil_div(gp.npix, 16);
    gp.grid_nx = ceil_div(ceil_div(npix16, pl.tn), tiles_per_wg);
    gp.grid_ny = ceil_div(gp.K16, pl.tm);
    gp.m_major = gp.w_bytes >= gp.x_bytes;
    dim3 grid(xcd_grid(gp.grid_nx * gp.grid_ny), 1, 1);
    size_t lds = KS > 1 ? (size_t)waves * pl.tm * pl.tn * 4 * 64 * sizeof(float) : 0;
    if (patch_pays(g, pl)) {
        pl.mode = kModePatch;
        lds = std::max(lds, (size_t)waves * kPatchFloats * sizeof(float));
    }
    if (half) launch_gemm_variant<true>(pl, gp, grid, dim3(64 * waves), lds, st);
    else launch_gemm_variant<false>(pl, gp, grid, dim3(64 * waves), lds, st);
    return hipGetLastError();
}

// ---- many layers in one launch: item plan of one layer
// Tile of a layer whose items are whole workgroups (tile_gemm.h).
struct TileShape {
    int th, tw, nth, ntw;   // outputs of a tile, tiles per column and row of an image
};

// The fewest tiles of at most bn outputs whose patch fits, then the smallest patch; false if none does.
static bool plan_tile_shape(const Geo &g, const int bn, const int patch, TileShape *out) {
    long best = LONG_MAX;
    const int n0 = ceil_div(g.q, bn);
    for (int n = n0; n < n0 + 4 && n <= g.q; ++n) {
        const int tw = ceil_div(g.q, n), ntw = ceil_div(g.q, tw);
        const long pw = (long)(tw - 1) * g.sw + g.s;
        int rows = std::min(g.p, bn / tw);
        while (rows > 0 && ((rows - 1L) * g.sh + g.r) * pw > patch) --rows;
        if (rows < 1) continue;
        const int nth = ceil_div(g.p, rows);
        if ((long)nth * ntw * 4096 >= best) continue;
        const int th = ceil_div(g.p, nth);
        const long key = (long)nth * ntw * 4096 + ((th - 1L) * g.sh + g.r) * pw;
        if (key < best && nth < 65536 && ntw < 65536) { best = key; *out = TileShape{th, tw, nth, ntw}; }
    }
    return best != LONG_MAX;
}

// Length of the items of a launch: k-steps of a single-wavefront item, chunks of 32 channels of a whole workgroup's (0: none of these); few: float16
// layers of few channels in items of workgroups; wide: float32 7x7 layers with four panels per tile.
struct ItemTarget { int steps, chunks; bool few, wide; };

struct ItemPlan {
    int mode, tm, nmt, ntn, nsplit;
    int tile, tn;           // tile: items of whole workgroups, 4 tm panels x tn blocks of 16 pixels
    TileShape shape;
    int steps;              // k-steps of the whole reduction
    size_t part_bytes;      // partial tiles (0 if the layer is not split)
    size_t xt_bytes;        // float16 copy of x in octets of channels (0 if not needed)
};

// k-steps (one MFMA per 16 x 16 block each) a work item aims at: long enough to amortise an
// item's addressing, first loads and store, short enough that the chip's last round of items
// stays small against the whole launch.
constexpr int kItemSteps = 144;

// Layers that may run in items of whole workgroups: 3x3, stride 1 (float16: or 2), and sizes that fill most of a tile: 48 input
// channels (a chunk is 32), 33 output channels (a workgroup takes 64), two thirds of its pixels.
// (SqueezeNet-shaped stack, the expand layers of 16 and 32 channels in tiles or not: 38.8 / 34.3 us.)
static bool plan_tile(const Geo &g, ItemPlan *ip) {
    if (g.groups != 1 || g.r != 3 || g.s != 3 || g.sh != g.sw || g.ph != g.pw || g.ph >= 65536) return false;
    if (g.sh != 1 && (g.sh != 2 || g.dtype != NNV_F16)) return false;
    if (g.c < 48 || g.k < 33) return false;
    TileShape wide{}, narrow{};
    const bool okw = g.sh == 1 && plan_tile_shape(g, 112, kTilePatch, &wide), okn = plan_tile_shape(g, 64, g.sh == 1 ? kTilePatch : kTilePatch2, &narrow);
    if (!okw && !okn) return false;
    const long nw = okw ? (long)wide.nth * wide.ntw * 7 : LONG_MAX, nn = okn ? (long)narrow.nth * narrow.ntw * 4 : LONG_MAX;
    if (std::min(nw, nn) * 32 > 3L * g.p * g.q + 64) return false;
    ip->tile = 1;
    ip->mode = 3;
    ip->tm = 1;
    const int K16 = ceil_div(g.k, 16);
    ip->tn = nw <= nn ? 7 : 4;
    ip->shape = nw <= nn ? wide : narrow;
    ip->nmt = ceil_div(K16, 4 * ip->tm);
    ip->ntn = g.n * ip->shape.nth * ip->shape.ntw;
    return true;
}

// ... and float16 layers of 1x1 filters, under the same rule (one_item).  128 channels per item unless 64 leave fewer empty.
static bool plan_one(const Geo &g, ItemPlan *ip) {
    if (g.dtype != NNV_F16 || g.groups != 1 || g.r != 1 || g.s != 1 || g.sh >= 65536 || g.sw >= 65536 || g.ph >= 65536 || g.pw >= 65536) return false;
    if (g.c < 48 || g.k < 33) return false;
    const bool pairs = g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0 && (g.h * g.w) % 2 == 0;
    const int bn = pairs ? 112 : 64, npix = g.n * g.p * g.q;
    if (2L * ceil_div(npix, bn) * bn > 3L * npix + 64) return false;
    const int K16 = ceil_div(g.k, 16);
    ip->tile = 1;
    ip->mode = 1;
    ip->tm = ceil_div(K16, 8) * 8 * 100 <= ceil_div(K16, 4) * 4 * 115 ? 2 : 1;
    ip->tn = pairs ? 7 : 4;
    ip->nmt = ceil_div(K16, 4 * ip->tm);
    ip->ntn = ceil_div(npix, bn);
    return true;
}

// ... and float16 layers of up to eight channels (few_item).
static bool plan_few(const Geo &g, ItemPlan *ip) {
    if (g.dtype != NNV_F16 || g.groups != 1 || g.c > kTapsMaxChannels || g.r * g.s < 2 || g.sh >= 65536 || g.sw >= 65536 || g.ph >= 65536 || g.pw >= 65536) return false;
    TileShape wide{}, narrow{};
    const bool okw = plan_tile_shape(g, 112, kFewPatch, &wide), okn = plan_tile_shape(g, 64, kFewPatch, &narrow);
    if (!okw && !okn) return false;
    const long nw = okw ? (long)wide.nth * wide.ntw * 7 : LONG_MAX, nn = okn ? (long)narrow.nth * narrow.ntw * 4 : LONG_MAX;
    if (std::min(nw, nn) * 32 > 3L * g.p * g.q + 64) return false;
    ip->tile = 1;
    ip->mode = kModeTaps;
    ip->tm = 1;
    ip->tn = nw <= nn ? 7 : 4;
    ip->shape = nw <= nn ? wide : narrow;
    ip->nmt = ceil_div(g.k, 64);
    ip->ntn = g.n * ip->shape.nth * ip->shape.ntw;
    ip->nsplit = 1;
    ip->steps = ceil_div(g.r * g.s, 4);
    return true;
}

// ... its channels cut into ranges of about `chunks` chunks of 32
static void split_tile(const Geo &g, const int chunks, ItemPlan *ip) {
    const int all = ceil_div(g.c, kTileChannels);
    const int most = std::min(all, chunks), n = g.dtype == NNV_F16 ? std::max(1, (all + most / 2) / most) : ceil_div(all, most);
    const int per = ceil_div(all, n);
    ip->nsplit = ceil_div(all, per);
    ip->steps = all * g.r * g.s;
    ip->part_bytes = ip->nsplit > 1 ? (size_t)ip->nmt * ip->ntn * (ip->nsplit * (size_t)(ip->tm * ip->tn * 4096) + kSplitWord) : 0;
}

// The layer in items of whole workgroups, before its channels are cut (tile = 0: it has none).
static ItemPlan plan_whole(const Geo &g) {
    ItemPlan ip{};
    if (!plan_tile(g, &ip) && !plan_one(g, &ip)) plan_few(g, &ip);
    return ip;
}

// What does not depend on the target, for callers that plan a layer several times.
struct LayerPlan {
    ItemPlan whole;
    GemmPlan gemm;
};

static ItemPlan plan_items(const Geo &g, const ItemTarget target_len, const LayerPlan *known = nullptr) {
    ItemPlan ip{};
    if (target_len.chunks > 0 || target_len.few) {
        ip = known ? known->whole : plan_whole(g);
        if (ip.tile && (ip.mode == kModeTaps ? target_len.few : target_len.chunks > 0)) {
            if (ip.mode != kModeTaps) split_tile(g, ip.mode == 1 ? 4 * target_len.chunks : target_len.chunks, &ip);
            return ip;
        }
        ip = ItemPlan{};
    }
    const GemmPlan pl = known ? known->gemm : plan_im2col(g);
    const bool half = g.dtype == NNV_F16;
    ip.mode = pl.mode;
    ip.xt_bytes = pl.xt_bytes;
    const int kg16 = ceil_div(g.kg, 16);
    const int K16 = g.groups * kg16;
    // two panels per tile unless that leaves a third or more of the tile rows empty
    // (a tile's panels must belong to one group)
    ip.tm = (kg16 % 2 == 0 || (g.groups == 1 && kg16 >= 5)) ? 2 : 1;
    // float32 3x3 and 1x1 layers with at least 64 output channels: four panels per tile
    if (!half && g.groups == 1 && (pl.mode == 3 || pl.mode == 1) && (kg16 % 4 == 0 || kg16 >= 12)) ip.tm = 4;
    // float16 1x1, stride 1, no padding, an even plane: pixels in pairs, and four panels under the same rule
    if (half && pl.mode == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0 && (g.h * g.w) % 2 == 0) {
        ip.mode = kModePairs;
        if (g.groups == 1 && (kg16 % 4 == 0 || kg16 >= 12)) ip.tm = 4;
    } else if (half && pl.mode == 1 && g.groups == 1 && ceil_div(g.c, 32) >= kOctetsMinBlocks && kg16 >= kOctetsMinPanels) {
        ip.mode = kModeOctets;
        ip.tm = 4;
        ip.xt_bytes = align_up((size_t)g.n * g.h * g.w * copy_channels(g, ip.mode) * sizeof(__half), 256);
    }
    if (pl.mode == kModeTaps && (kg16 % 4 == 0 || kg16 >= 12)) ip.tm = 4;
    // float32 7x7: four where the launch wants them (items_target)
    if (target_len.wide && !half && g.groups == 1 && pl.mode == 7 && kg16 % 4 == 0) ip.tm = 4;
    ip.nmt = ceil_div(K16, ip.tm);
    ip.ntn = ceil_div(ceil_div(g.n * g.p * g.q, 16), 2);
    const int cblocks = half ? ceil_div(g.cg, 32) : ceil_div(g.cg, 4);
    const bool row = pl.mode == 5 || pl.mode == 7 || (pl.mode == 3 && half);
    int nunits = pl.mode == kModeTaps ? ceil_div(g.r * g.s, 4) : pl.mode == 0 ? cblocks * g.r * g.s : row ? cblocks * g.r : cblocks;
    int unit_steps = (pl.mode == 0 || pl.mode == kModeTaps) ? 1 : row ? pl.mode : g.r * g.s;
    int chunk_units = pl.mode == 1 ? (half ? 2 : 8) : 1;
    int target = target_len.steps;
    if (ip.tm == 4) {
        // a wide item does twice the MFMAs per k-step: somewhat fewer steps per item
        target = std::max(9, target * 3 / 4);
    }
    if (!half && pl.mode == 1) { nunits = ceil_div(cblocks, 4); unit_steps = 4; chunk_units = 1; }   // float32 1x1: the kernel splits whole chunks of 4 blocks
    const long steps = (long)nunits * unit_steps;
    ip.steps = (int)steps;
    long nsplit = (steps + target / 2) / target;
    const long most = std::max(1, nunits / chunk_units);          // every range holds at least one chunk
    nsplit = std::max(1L, std::min(nsplit, most));
    // ranges are ceil(nunits / nsplit) units long: drop ranges that would come out empty
    const int per = ceil_div(nunits, (int)nsplit);
    ip.nsplit = ceil_div(nunits, per);
    ip.part_bytes = ip.nsplit > 1 ? (size_t)ip.nmt * ip.ntn * (ip.nsplit * (size_t)(ip.tm * 2048) + kSplitWord) : 0;
    return ip;
}

// Item length of a launch of these layers.
// float16 items of a call that fills the chip fewer than three times over are a third as long:
// such a launch ends with its longest items (a 512-channel 3x3 layer is one item of 144 steps per tile
// otherwise), and a float16 step moves eight times the channels of a float32 one.  Measured (us, one
// call, items of 36 / 48 / 144 steps): ResNet-18-shaped stack 48.2 / 48.3 / 62.7, AlexNet 26.6 / 27.2 / 36.5,
// GoogLeNet 60.2 / 55.8 / 56.0, SqueezeNet 43.7 / 43.5 / 43.8; above the line (10840 items of 144 steps or
// more) ResNet-50 78.7 / 77.7 / 77.0 and VGG-16 179 / 178 / 162 (all of them before 3x3 and 1x1 layers ran in items of workgroups).
// float32: a launch whose items all fit the chip at once (kItemsResident, less a sixteenth: a launch
// that fills every slot was measured slower than one that leaves a few free) takes the shortest
// item length, in steps of 12 down to kItemStepsMin, with which they still do: the launch lasts as
// long as an item, and the free slots would stay idle.  Measured (us, one call, 48 / 72 / 144 steps):
// AlexNet-shaped stack 35.8 / 42.8 / 63.3, SqueezeNet 42.2 / 37.6 / 38.3; launches above the line keep the long
// items: ResNet-18 65.7 / 62.9 / 52.1, ResNet-50 131 / 111 / 98, MobileNetV1 48 / 46 / 44 (all of them before 3x3 layers ran in items of workgroups,
// and before the share of a SIMD counted, below, by which the ResNet-18-shaped launch takes items of 60 steps).
constexpr int kItemStepsShortHalf = 48, kItemStepsMin = 48;
constexpr int kItemsResident = 256 * 3 * kItemWaves;

// Items of whole workgroups: with W of them if each took one chunk (weighted by their blocks of pixels), an item takes W / 450, at least two
// chunks: three workgroups fit a CU, and an item spends 5 us outside its products.  Launches of fewer than
// 220 keep to single-wavefront items.  Measured over 50 launches of five stacks at batch 1-4 and 96-320 pixels, us at 1 / 2 / 4 / 8
// chunks against none: W = 232 (AlexNet-shaped) 35 / 34 / 41 / 67 against 43, 803 (ResNet-18) 59 / 48 / 54 / 83 against 56, 995 (ResNet-50) 106 / 101 / 98 / 119
// against 106, 2146 (ResNet-18, 3x162x237) 126 / 112 / 103 / 105 against 116, 7488 (VGG-16) 285 / 233 / 211 / 203 (16: 198) against 296; below, W = 216 (GoogLeNet, 201 x 134)
// 53 / 59 / 86 / 100 against 60.  Taken together 4 % over the best of 0, 1, 2, 3, 4, 6, 8 and 16 for each launch; no other line, divisor or least range tried came below 3 %
// (three chunks at least: ResNet-18 48 -> 53).  The worst: W = 397 (AlexNet, 2x225x156), 60 where three chunks give 42 and fill the chip once.
// (Three to six chunks where that makes one round of one to one and a half take AlexNet-shaped stacks at 2x314x246 from 81 to 66 us, 3x224x200 75 / 61, 4x200x180 82 / 64, but a chain of sums two or three
// times as long is further from the exact ones: 1.3e-7 -> 1.6e-7 to 2.3e-7 of their 2-norm.)
// float16, W in chunks of 3x3 filters of 64 x 112 outputs, four chunks of 1x1 filters to one: below 600 single-wavefront items; else the channels stay whole
// if no layer has more than 12 chunks (48 of 1x1 filters), since partial tiles and their sums cost 3 us (6 when a launch added them), and otherwise a range is W / 330 chunks, at
// least four: an item of 512 channels takes 24 us.  us a call at 0 / 4 / 8 / 12 or more chunks, none longer than 12: W = 662 (AlexNet-shaped, 2x211x317) 25 / 29 / 29 / 23, 1273
// (GoogLeNet, 3x210x173) 64 / 66 / 58 / 58, 1380 (MobileNetV1, 3x273x258) 48 / 39 / 35 / 35; longer: 983 (ResNet-18) 38 / 23 / 31 / 31, 1381 (ResNet-18, 295x215) 38 / 27 / 30 / 37, 3374
// (ResNet-50, 301x227) 72 / 60 / 55 / 63, 5085 (ResNet-50, 2x217x257) 103 / 85 / 74 / 69, 7488 (VGG-16) 92 / 80 / 69 / 59; W = 197 (SqueezeNet, 2x132x119) 16 / 22 / 22 / 22.
// Layers of few channels are items of workgroups where that saves the launch that copies x, not beside other copies (MobileNetV2-shaped plan 50 / 44;
// ResNet-18 at 4x108x114, whose last layers keep their copy, 30 / 36).
// known: filled in for n layers.
static ItemTarget items_target(int n, const Geo *geos, LayerPlan *known) {
    ItemTarget target{kItemSteps, 0, false, false};
    long w = 0;                      // in chunks of 1x1 filters of 64 x 16 outputs
    int longest_whole = 0;           // reduction, in chunks of 1x1 filters
    for (int i = 0; i < n; ++i) {
        known[i] = LayerPlan{plan_whole(geos[i]), plan_im2col(geos[i])};
        const ItemPlan &whole = known[i].whole;
        if (!whole.tile || whole.mode == kModeTaps) continue;
        const int chunks = ceil_div(geos[i].c, kTileChannels) * (whole.mode == 3 ? 4 : 1);
        w += (long)whole.nmt * whole.ntn * whole.tn * chunks;
        longest_whole = std::max(longest_whole, chunks);
    }
    w /= 28;
    if (geos[0].dtype == NNV_F16) {
        if (w >= 600) target.chunks = longest_whole <= 48 ? 12 : (int)std::min(std::max(4L, w / 330), 65536L);
        // (decided last: plans without `few` first)
        bool copies = false;
        for (int i = 0; i < n && !copies; ++i) copies = known[i].whole.mode != kModeTaps && plan_items(geos[i], target, &known[i]).xt_bytes > 0;
        target.few = !copies;
    } else if (w >= 220) target.chunks = std::max(2, (int)std::min((w + 449) / 450, 65536L));
    auto total_at = [&](int t) {
        long tot = 0;
        for (int i = 0; i < n; ++i) {
            const ItemPlan p = plan_items(geos[i], ItemTarget{t, target.chunks, target.few, target.wide}, &known[i]);
            tot += (long)p.nmt * p.ntn * p.nsplit * (p.tile ? kItemWaves : 1);
        }
        return tot;
    };
    const long total = total_at(kItemSteps);
    if (geos[0].dtype == NNV_F16) {
        if (total < 3L * kItemsResident) target.steps = kItemStepsShortHalf;
        return target;
    }
    constexpr long fit = (long)kItemsResident * 15 / 16;
    long items = total;                 // at target.steps
    if (total <= fit)
        for (int t = kItemSteps - 12; t >= kItemStepsMin; t -= 12) {
            const long at = total_at(t);
            if (at > fit) break;
            target.steps = t;
            items = at;
        }
    const int fitting = target.steps;
    // float32, whatever their number: no item longer than a SIMD's share of the launch's matrix instructions, or the launch ends with
    // a few long items (the deep layers of a mobile network: 20 us each, and all others are done after 12).  us a call, items of 144 steps
    // or what the rule above chose / this: MobileNetV2-shaped plan 47 / 40, MobileNetV1 44 / 42, ResNet-18 at batch 2, 150 x 187 74 / 63;
    // shares longer than the items change nothing (ResNet-50, SqueezeNet, where items of 72 cost 9 %).
    double share = 0;                   // in steps of a panel
    int longest[5] = {0, 0, 0, 0, 0};   // steps of the longest reduction among the layers of 1, 2 and 4 panels per tile
    for (int i = 0; i < n; ++i) {
        const ItemPlan p = plan_items(geos[i], ItemTarget{kItemSteps, target.chunks, false, target.wide}, &known[i]);
        if (p.tile) continue;
        share += (double)p.nmt * p.ntn * p.steps * p.tm / 1024;
        longest[p.tm] = std::max(longest[p.tm], p.steps);
    }
    for (int tm : {1, 2, 4})
        if ((double)longest[tm] * tm > share)
            while (target.steps > kItemStepsMin && target.steps * (tm == 4 ? 0.75 : 1.0) * tm > share) target.steps -= 12;
    // Launches of between one and one and a half times the items that are resident at once end with a round that fills the chip in part: there the
    // 7x7 layers, whose items are many and bound by their gathers of pixels, take four panels per tile (half the items and gathers).  54 launches of three stacks at
    // batch 1-3 and 96-320 pixels, times without / with (geometric means, in brackets the smallest and largest), by items over those resident: 0.66-0.9 0.98 (0.92-1.03), 1.0-1.5 1.02
    // (0.95-1.08; ResNet-18-shaped stack at 192x253 55.0 / 51.0 us, at 318x182 62.4 / 65.3), 1.5-1.9 0.97 (0.93-1.02), 2.0-2.5 1.00 (0.98-1.01), more 1.01 (0.98-1.03):
    // a partly filled round counts while it is the second.
    if (target.steps != fitting) items = total_at(target.steps);
    target.wide = items > kItemsResident && items <= kItemsResident * 3L / 2;
    return target;
}

long depthwise_items(const Geo &g) {
    if (g.ph >= 65536 || g.pw >= 65536) return LONG_MAX / kMaxGemmLayers;
    return dw_workgroups(DwParams{g.n, g.c, g.h, g.w, g.sh, g.ph, g.pw, g.p, g.q, 0});
}

// The launch's 64-byte layer records hold filter sizes and groups in 8 bits, strides, pads and the
// number of ranges in 16 (channels and images are below 2^16 everywhere).  Only a stride or a pad of 2^16
// and more does not fit: such a layer is launched by itself.
bool im2col_items_supported(const Geo &g) {
    return g.sh < 65536 && g.sw < 65536 && g.ph < 65536 && g.pw < 65536 && plan_items(g, ItemTarget{kItemStepsMin / 2, 0, false, false}).nsplit < 65536;
}

void im2col_items_workspace_bytes(int n, const Geo *geos, size_t *bytes) {
    if (n <= 0 || n > kMaxGemmLayers) return;
    LayerPlan known[kMaxGemmLayers];
    const ItemTarget target = items_target(n, geos, known);
    for (int i = 0; i < n; ++i) {
        const ItemPlan ip = plan_items(geos[i], target, &known[i]);
        bytes[i] = align_up(ip.part_bytes, 256) + align_up(ip.xt_bytes, 256);
    }
}

// One item launch of n planned layers of one storage type, with the copies of x in front of it that they need; ws[i]: layer i's partial tiles and copy.
// Behind them ndw depthwise layers (geos, x, w, bias, y [n ..]; raw: their filters are untransformed).
static hipError_t launch_planned(int n, const Geo *geos, const ItemPlan *plans, const void *const *x, const void *const *w,
                                 const float *const *bias, void *const *y, void *const *ws, hipStream_t st, int ndw = 0, const char *raw = nullptr) {
    const bool half = geos[0].dtype == NNV_F16;
    // Order: layers with the longest items first, so that the chip's last round of items is made
    // of the short ones.
    // (items of whole workgroups before the others: these fill what they leave)
    int order[kMaxGemmLayers];
    bool tiles = false;
    for (int i = 0; i < n; ++i) {
        order[i] = i;
        tiles = tiles || plans[i].tile;
    }
    // 128 x 112 outputs per workgroup: planned for single layers only, and that kernel runs no other items
    const bool large = n == 1 && plans[0].tile && plans[0].mode == 3 && plans[0].tm == 2;
    auto item_len = [&](int i) {
        const ItemPlan &p = plans[i];
        // float16: a step that gathers pixels from NCHW takes about four times as long as one that reads octets, one that reads pairs half as
        // long again (ResNet-50-shaped stack without items of workgroups, in that order or by steps alone: 54 / 59 us)
        const long cost = !half ? 1 : p.mode == 1 ? 16 : p.mode == kModePairs ? 6 : 4;
        const long len = (long)ceil_div(p.steps, p.nsplit) * p.tm * cost;
        if (p.tile && half) return (long)ceil_div(p.steps, p.nsplit) * (p.mode == 1 ? 2 : 1) << 20;
        return p.tile ? (len * p.tn) << 20 : len;
    };
    std::stable_sort(order, order + n, [&](int a, int b) { return item_len(a) > item_len(b); });
    GemmItemTable tbl{};
    OctetTable cl{};
    int items = 0, ncl = 0, clblocks = 0;
    char *base = static_cast<char *>(ws[0]);
    for (int i = 1; i < n; ++i) base = std::min(base, static_cast<char *>(ws[i]));
    for (int o = 0; o < n; ++o) {
        const int i = order[o];
        const Geo &g = geos[i];
        const ItemPlan &ip = plans[i];
        GemmItemRec &L = tbl.layer[o];
        L.x = x[i]; L.wp = w[i]; L.bias = bias ? bias[i] : nullptr; L.y = y[i];
        L.H = g.h; L.W = g.w;
        L.N = (uint16_t)g.n; L.C = (uint16_t)g.c; L.K = (uint16_t)g.k;
        L.sh = (uint16_t)g.sh; L.sw = (uint16_t)g.sw; L.ph = (uint16_t)g.ph; L.pw = (uint16_t)g.pw;
        L.R = (uint8_t)g.r; L.S = (uint8_t)g.s; L.groups = (uint8_t)g.groups;
        L.relu = g.relu ? 1 : 0;
        char *region = static_cast<char *>(ws[i]);
        if (ip.xt_bytes) {
            // all copies of the call are made by one launch in front of the item launch
            void *xt = region + align_up(ip.part_bytes, 256);
            cl.x[ncl] = static_cast<const __half *>(x[i]);
            cl.xt[ncl] = static_cast<__half *>(xt);
            cl.C[ncl] = g.c;
            cl.HW[ncl] = g.h * g.w;
            cl.octs[ncl] = copy_channels(g, ip.mode) / 8;
            cl.block0[ncl] = clblocks;
            clblocks += ceil_div(g.h * g.w * cl.octs[ncl], 256 * kOctetsPerBlock) * g.n;
            ++ncl;
            L.x = xt;
        }
        L.part256 = (uint32_t)((region - base) / 256);
        tbl.item0[o] = items;
        L.nsplit = (uint16_t)ip.nsplit;
        L.mode = ip.mode;
        L.tm = ip.tm;
        const int count = ip.nmt * ip.ntn * ip.nsplit;
        if (ip.tile) {
            L.tile = 1;
            L.tm = ip.tm + (ip.tn == 7 ? 4 : 0);
            if (ip.mode == kModeTaps) L.part256 = (uint32_t)(ip.shape.th + ip.shape.tw * 256);
            else if (ip.mode == 3) {
                L.S = (uint8_t)ip.shape.th; L.groups = (uint8_t)ip.shape.tw;
                L.sw = (uint16_t)ip.shape.ntw; L.pw = (uint16_t)ip.shape.nth;
            }
            items += count * kItemWaves;
        } else {
            items += tiles || ndw > 0 ? ceil_div(count, kItemWaves) * kItemWaves : count;
        }
    }
    for (int i = n; i < n + ndw; ++i) {
        const Geo &g = geos[i];
        GemmItemRec &L = tbl.layer[i];
        L.x = x[i]; L.wp = w[i]; L.bias = bias ? bias[i] : nullptr; L.y = y[i];
        L.H = g.h; L.W = g.w;
        L.N = (uint16_t)g.n; L.C = (uint16_t)g.c;
        L.sh = (uint16_t)g.sh; L.ph = (uint16_t)g.ph; L.pw = (uint16_t)g.pw;
        L.R = (uint8_t)g.r; L.groups = raw[i - n] ? 1 : 0;
        L.relu = g.relu ? 1 : 0;
        L.tile = 1;
        tbl.item0[i] = items;
        items += (int)dw_workgroups(DwParams{g.n, g.c, g.h, g.w, g.sh, g.ph, g.pw, g.p, g.q, 0}) * kItemWaves;
    }
    for (int i = n + ndw; i < kMaxGemmLayers; ++i) tbl.item0[i] = INT_MAX;
    tbl.nitems = items;
    tbl.group = 2;       // workgroups (of kItemWaves items) handed to one XCD in a row
    tbl.part_base = base;
    static std::atomic<unsigned long long> launches{0};
    tbl.mark = (kSplitMark + launches.fetch_add(1, std::memory_order_relaxed)) & 0xffffffffffffull;
    if (ncl > 0) {
        for (int i = ncl; i < kMaxGemmLayers; ++i) cl.block0[i] = INT_MAX;
        cl.nblocks = clblocks;
        hipLaunchKernelGGL(to_octets_many_kernel, dim3(clblocks), dim3(256), 0, st, cl);
    }
    const int wgs = ceil_div(items, kItemWaves);
    const int per_xcd = ceil_div(ceil_div(wgs, tbl.group), 8) * tbl.group;
    const bool split = std::any_of(plans, plans + n, [](const ItemPlan &ip) { return ip.nsplit > 1; });
#define NNV_ITEMS(HALF, TILE, SPLIT) hipLaunchKernelGGL((gemm_items_kernel<HALF, TILE, SPLIT>), dim3(per_xcd * 8), dim3(64 * kItemWaves), 0, st, tbl)
#define NNV_ITEMS_OF(HALF)                                           \
    if (large) NNV_ITEMS(HALF, kLargeTiles, HALF);                   \
    else if (tiles && ndw > 0) NNV_ITEMS(HALF, kTilesDepthwise, true); \
    else if (ndw > 0) NNV_ITEMS(HALF, kDepthwise, true);             \
    else if (tiles && split) NNV_ITEMS(HALF, kTiles, true);          \
    else if (tiles) NNV_ITEMS(HALF, kTiles, false);                  \
    else if (split) NNV_ITEMS(HALF, kNoTiles, true);                 \
    else NNV_ITEMS(HALF, kNoTiles, false);
    if (half) { NNV_ITEMS_OF(true) } else { NNV_ITEMS_OF(false) }
#undef NNV_ITEMS_OF
#undef NNV_ITEMS
    return hipGetLastError();
}

// Launches layers [0, n) (all of one storage type, n <= kMaxGemmLayers) as one item launch, with a
// launch of copies in front if a float16 layer reads one.  ws[i] is layer i's own workspace region of
// im2col_items_workspace_bytes of these layers.
hipError_t launch_im2col_items(int n, const Geo *geos, const void *const *x, const void *const *w, const float *const *bias,
                               void *const *y, void *const *ws, hipStream_t st, int ndw, const char *raw) {
    if (n <= 0) return hipSuccess;
    if (n + ndw > kMaxGemmLayers) return hipErrorInvalidValue;
    for (int i = 0; i < n + ndw; ++i)
        if (geos[i].dtype != geos[0].dtype) return hipErrorInvalidValue;
    LayerPlan known[kMaxGemmLayers];
    const ItemTarget target = items_target(n, geos, known);
    ItemPlan plans[kMaxGemmLayers];
    for (int i = 0; i < n; ++i) plans[i] = plan_items(geos[i], target, &known[i]);
    return launch_planned(n, geos, plans, x, w, bias, y, ws, st, ndw, raw);
}

// A single layer in items of whole workgroups, its channels not split: an item takes the whole channel loop, so that there have to be enough of
// them.  The lines stand where a sweep of 590 layers changes sides (48-2048 channels, planes of 7x7 to 224x224, batches of 1-16, half of the sizes those of networks,
// half random; weights and pixels from HBM; geometric means of the time without / with such items, in brackets the smallest and largest):
//   float32, by items of 64 channels x 16 pixels (an item holds 7 or 4 of them): 7 x 140-179 items 0.92 (0.74-1.06), 180-199 1.06 (0.98-1.20), 200-229 1.22 (0.95-1.35), 280-399
//     1.15 (0.90-1.28), above 1.33 (0.97-1.72); 4 x 250-299 0.80 (0.64-1.01), 300-349 0.88 (0.72-1.15), 350-399 1.00 (0.85-1.19), 400-499 1.10 (0.89-1.29), above 1.14 (0.83-1.47).
//   float16 3x3, items: 1-59 0.81 (0.48-1.03), 80-99 1.07 (0.87-1.58), 100-119 1.17 (0.94-1.46), 120-199 1.40 (1.13-2.21), above 1.43 (1.10-2.27); stride 2:
//     100-130 0.89 (0.76-1.11), 168 1.14, 200-299 1.24 (1.00-1.36), above 1.28 (1.09-1.58).
//   float16 1x1: 150-199 0.84 (0.73-0.96), 200-249 0.97 (0.83-1.51), 250-299 1.13 (0.97-1.47), 300-339 1.23 (1.07-1.70), above 1.52 (0.95-2.50); at stride 2 200-249 1.22 (0.95-1.60).
//   float16 few channels, if one row of tiles holds all 33 to 64 panels' channels: below 70 1.00 (0.94-1.06), 100-199 1.09 (1.07-1.12), above 1.14 (0.99-1.29);
//     fewer channels 1.03 (0.80-1.20), more 1.02 (0.84-1.26).
// 128 x 112 outputs (times of 64 x 112 / 128 x 112): float32, with two buffers, two workgroups per CU and not three: where they all fit the chip and
// those of 64 need a second round, 1.03 (1.00-1.07, 29 layers; 256 channels at 8x56x56 189 / 177 us); fewer 0.87, more 0.82-1.00.  float16 3x3, whose LDS reads
// they halve: where those of 64 would share CUs, 257-449 items 1.11 (1.04-1.25), 450-999 1.17 (1.02-1.30), more 1.08 (0.99-1.16; 256 channels at 8x56x56
// 51 / 41 us); one to a CU 0.86 (0.78-0.92, 52 layers; 512 at 4x28x28 27 / 31 us).
static bool plan_tile_single(const Geo &g, ItemPlan *ip) {
    const bool half = g.dtype == NNV_F16;
    const int K16 = ceil_div(g.k, 16), nmt = ceil_div(K16, 8);
    const bool fits = nmt * 8 * 100 <= ceil_div(K16, 4) * 4 * 115;       // 128 channels per item leave no more empty than 64
    if (plan_few(g, ip)) return g.k > 32 && g.k <= 64 && ip->ntn >= 100;
    if (!plan_tile(g, ip) && !plan_one(g, ip)) return false;
    const long items = (long)ip->nmt * ip->ntn * ip->tm;
    if (half ? items < (ip->mode == 1 ? 250 : g.sh == 1 ? 80 : 160) : items * ip->tn < 200 * 7) return false;
    constexpr int kChipSmall = 256 * 3, kChipLarge = 256 * 2;            // workgroups resident at once
    if (fits && ip->mode == 3 && ip->tn == 7 && (half ? items > 256 : items > kChipSmall && (long)nmt * ip->ntn <= kChipLarge)) {
        ip->tm = 2;
        ip->nmt = nmt;
    }
    split_tile(g, INT_MAX, ip);
    return true;
}

// Layers that gemm_layers_kernel may run: float32 with the small tiles of im2col_gemm_kernel.
bool im2col_layer_mergeable(const Geo &g) {
    ItemPlan tile{};
    if (g.dtype != NNV_F32 || plan_tile_single(g, &tile)) return false;
    const GemmPlan pl = plan_im2col(g);
    return pl.tn == 1 && pl.tm <= 2 && pl.ks_shift <= 4;
}

// n <= kMaxMergedLayers mergeable layers, none of which reads or writes what another one writes: one launch, results as by launch_im2col.
hipError_t launch_im2col_layers(int n, const Geo *geos, const void *const *x, const void *const *w, void *const *y, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (n > kMaxMergedLayers) return hipErrorInvalidValue;
    GemmPlan plans[kMaxMergedLayers];
    int order[kMaxMergedLayers], tn[kMaxMergedLayers];
    long work[kMaxMergedLayers];         // about the products of a wavefront
    long all = 0;
    auto products = [&](int i) { return (long)ceil_div(geos[i].cg, 4) * geos[i].r * geos[i].s; };
    for (int i = 0; i < n; ++i) {
        plans[i] = plan_im2col(geos[i]);
        order[i] = i;
        all += products(i) * ceil_div(geos[i].n * geos[i].p * geos[i].q, 16) * geos[i].groups * ceil_div(geos[i].kg, 16);
    }
    for (int i = 0; i < n; ++i) {
        GemmPlan &pl = plans[i];
        tn[i] = 1;
        work[i] = products(i) * pl.tm >> std::min(pl.ks_shift, 3);
        if (work[i] < all / kLayerResident && pl.tm == 1 && ceil_div(geos[i].kg, 16) % 2 == 0) { pl.tm = 2; work[i] *= 2; }
        if (work[i] < all / kLayerResident && pl.ks_shift <= 3) { tn[i] = 2; work[i] *= 2; }       // (KS = 16: the partial tiles would not fit)
    }
    std::stable_sort(order, order + n, [&](int a, int b) { return work[a] > work[b]; });
    GemmLayersTable tbl{};
    long blocks = 0;
    for (int o = 0; o < n; ++o) {
        const int i = order[o];
        const GemmPlan &pl = plans[i];
        GemmParams &gp = tbl.g[o];
        gp = gemm_params(geos[i], pl.mode, x[i], w[i], nullptr, y[i]);
        gp.ks_shift = pl.ks_shift;
        gp.grid_nx = ceil_div(ceil_div(gp.npix, 16 * tn[i]), kLayerWaves >> std::min(pl.ks_shift, 3));
        gp.grid_ny = ceil_div(gp.K16, pl.tm);
        gp.m_major = gp.w_bytes >= gp.x_bytes;
        const int mode = tn[i] == 1 && patch_pays(geos[i], pl) ? kModePatch : pl.mode;
        tbl.variant[o] = (uint8_t)(mode + (pl.tm == 2 ? 16 : 0) + (tn[i] == 2 ? 32 : 0));
        tbl.block0[o] = (int)blocks;
        blocks += xcd_grid(gp.grid_nx * gp.grid_ny);
        if (blocks >= (1L << 30)) return hipErrorInvalidValue;
    }
    for (int o = n; o < kMaxMergedLayers; ++o) tbl.block0[o] = INT_MAX;
    hipLaunchKernelGGL(gemm_layers_kernel, dim3((unsigned)blocks), dim3(64 * kLayerWaves), 0, st, tbl);
    return hipGetLastError();
}

hipError_t launch_im2col(const Geo &g, const void *x, const void *w, const float *bias, void *y, void *ws, hipStream_t st) {
    ItemPlan tile{};
    if (plan_tile_single(g, &tile)) return launch_planned(1, &g, &tile, &x, &w, bias ? &bias : nullptr, &y, &ws, st);
    return launch_im2col_plain(g, x, w, bias, y, ws, st);
}

}  // namespace nnv
