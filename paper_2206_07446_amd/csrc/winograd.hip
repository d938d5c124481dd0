// Winograd F(2x2,3x3) / F(4x4,3x3) / F(6x6,3x3) convolution from transformed weights (the fastest
// executing, most expensive to prepare kernel family of Table 2).  Three kernels:
//   1. input transform   V[xi][tile block][c][tiles] = (B^T d B)[xi]      (vector ALU)
//   2. batched tile GEMM M[xi] = U[xi] (K x C) * V[xi] (C x T), alpha^2 independent
//      products on the matrix cores; U and V are stored as ready-made 16-row operand
//      fragments, so both are read with one coalesced load per fragment and no LDS;
//      deep layers with few tiles split the channels over the wavefronts of a workgroup
//      and add the partial sums through LDS in fixed order
//   3. output transform  Y = A^T M A, clipped to P x Q, plus bias        (vector ALU)
// V and M live in the caller's workspace.  float16 storage keeps U, V and y in half
// precision; the transforms and the accumulation are float32.
// float32 F(2x2) / F(4x4) layers with many tiles for their channels run instead as ONE kernel
// (wino_fused_kernel below) that keeps V in LDS and M in registers, or, with one step of channels, both in registers (wino_wave_kernel).
#include <algorithm>
#include <climits>
#include <type_traits>
#include <vector>
#include "nnv_internal.h"
#include "buf.h"
#include "wino_consts.h"

namespace nnv {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef half8_t half8;

struct WinoParams {
    const void *x;
    const void *U;
    void *V;
    float *M;
    const float *bias;
    void *y;
    int N, C, H, W, K, ph, pw, P, Q;
    int th, tw, T;          // tiles per image (rows, cols), total tiles
    int tn, nblk, Tpad;     // tiles come in nblk blocks of 16 tn (tn: 1 or 2), of which the last may hold 16 only; Tpad: T padded to 16
    int K16, cpad, csteps;  // cpad: channels padded to 4 (float32) / 32 (float16); csteps = cpad / that
    int ks_shift;           // wavefronts sharing one output tile (splitting the channels) = 1 << ks_shift
    uint32_t u_bytes, v_bytes;   // sizes of U and V (range-checked loads)
    uint32_t x_bytes;            // size of x
    int relu;                    // outputs clamped at zero before the store
    int gemm_wgs_per_xi;         // workgroups per frequency in the tile GEMM
    int alpha2;                  // number of frequencies
};

// out[i][j] = sum_k L[i][k] * in[k][j] with a compile-time matrix L (zeros skipped).
#define NNV_MATMUL_LEFT(L, ROWS, INNER, COLS, in, out)                                  \
    _Pragma("unroll") for (int i_ = 0; i_ < ROWS; ++i_) _Pragma("unroll") for (int j_ = 0; j_ < COLS; ++j_) { \
        float acc_ = 0.f;                                                               \
        _Pragma("unroll") for (int k_ = 0; k_ < INNER; ++k_) if (L[i_][k_] != 0.f) acc_ += L[i_][k_] * in[k_][j_]; \
        out[i_][j_] = acc_;                                                             \
    }
// out[i][j] = sum_k in[i][k] * Rm[j][k]   (right-multiply by Rm^T)
#define NNV_MATMUL_RIGHT_T(Rm, ROWS, INNER, COLS, in, out)                              \
    _Pragma("unroll") for (int i_ = 0; i_ < ROWS; ++i_) _Pragma("unroll") for (int j_ = 0; j_ < COLS; ++j_) { \
        float acc_ = 0.f;                                                               \
        _Pragma("unroll") for (int k_ = 0; k_ < INNER; ++k_) if (Rm[j_][k_] != 0.f) acc_ += in[i_][k_] * Rm[j_][k_]; \
        out[i_][j_] = acc_;                                                             \
    }

// ---- patches.  float32, one column of padding, the 16 lanes of a row over neighbouring tiles: element by element a patch takes A^2
// gathers with M floats from lane to lane, and a gather of 64 lanes holds the CU's vector memory path for up to 64 cycles.  A lane therefore
// loads the M columns that only it begins with (4-byte aligned loads of two or four floats; floats past the end of x read as zero one by one), and takes the
// two outer columns from the lanes beside it; the first and the last lane of a row load theirs.  Columns outside the image are zero.
// Input transforms of a VGG-16-shaped F(4x4) stack 38.1 -> 26.5 us, ResNet-18 F(2x2) 11.0 -> 9.8.  (Other paddings: element by element.)
// row(u): byte offset of row u of the lane's channel, or out of range.
template <int M, typename Row>
__device__ __forceinline__ void patch_load(float (&d)[M + 2][M + 2], const __amdgpu_buffer_rsrc_t xres, const int tj, const int tw, const int lane, Row row, const uint32_t soff) {
    const int edge = (lane & 15) == 0 ? tj * M - 1 : tj * M + M;
    const bool has_edge = (lane & 15) == 0 ? tj > 0 : (lane & 15) == 15 && tj + 1 < tw;
#pragma unroll
    for (int u = 0; u < M + 2; ++u) {
        const uint32_t o = row(u);
        const uint32_t c = o + (uint32_t)tj * (4u * M);
        if constexpr (M >= 4) {
            const auto v = buf_load_floats<4>(xres, c, soff);
#pragma unroll
            for (int i = 0; i < 4; ++i) d[u][1 + i] = v[i];
        }
        if constexpr (M % 4 == 2) {
            const auto v = buf_load_floats<2>(xres, c + (M / 4) * 16u, soff);
#pragma unroll
            for (int i = 0; i < 2; ++i) d[u][1 + M / 4 * 4 + i] = v[i];
        }
        d[u][0] = buf_load<float>(xres, has_edge ? o + (uint32_t)edge * 4u : kOobOffset, soff);
    }
}
template <int M>
__device__ __forceinline__ void patch_finish(float (&d)[M + 2][M + 2], const int tj, const int tw, const int W) {
    auto beside = [](const float edge, const float v, auto right) __attribute__((always_inline)) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, edge), __builtin_bit_cast(int, v), decltype(right)::value ? 0x101 : 0x111, 0xf, 0xf, false));
    };
#pragma unroll
    for (int u = 0; u < M + 2; ++u) {
        const float left = beside(d[u][0], d[u][M], std::false_type{}), right = beside(d[u][0], d[u][1], std::true_type{});
        d[u][0] = tj > 0 ? left : 0.f;
        d[u][M + 1] = tj + 1 < tw ? right : 0.f;
    }
    if (W % M != 0) {           // (uniform)
#pragma unroll
        for (int i = 1; i < M; ++i)
#pragma unroll
            for (int u = 0; u < M + 2; ++u) d[u][1 + i] = tj * M + i < W ? d[u][1 + i] : 0.f;
    }
}

// ---- 1. input transform.  Workgroup = a block of 16 tn tiles x as many channels as its threads cover.
// (tb, by): tile block and channel group of the workgroup; bdim: its threads
// V, float32: [xi][block][c][16 tn tiles], so that lane n of the tile GEMM reads its tn tiles tn n ..
// with one load.  float16: [xi][block][t][operand fragments of 16 tiles x 32 channels], tile tn n + t of
// the block being row n of its t-th fragment (the GEMM then stores neighbouring tiles together).
// tn = 2 with an odd number of 16-tile blocks: the last block has 16 tiles in the first 8 of these lanes, [c][16 tiles],
// or one row of fragments with tile 2 n + t in row n + 8 t, so that V and M are no larger than the tiles need.
__device__ __forceinline__ bool wino_short_block(const WinoParams &w, const int tb) { return (tb + 1) * 16 * w.tn > w.Tpad; }
template <int SET, bool HALF>
__device__ __forceinline__ void wino_input_block(const WinoParams &w, const int tb, const int by, const int bdim) {
    using Wm = WinoMat<SET>;
    constexpr int A = Wm::A, M = Wm::M;
    typedef typename std::conditional<HALF, __half, float>::type T;
    int tl, c;      // tile within the block, channel
    if (HALF) {   // lanes: 8 channels fastest, then tiles -> 128 B contiguous half stores; 16 tiles x 16 channels per workgroup
        tl = ((threadIdx.x >> 3) & 15) * w.tn + by % w.tn;
        c = (by / w.tn) * 16 + (threadIdx.x >> 7) * 8 + (threadIdx.x & 7);
    } else {      // lanes: the tiles of the block fastest, then channels -> 256 B contiguous stores
        const int sh = w.tn == 2 ? 5 : 4;
        tl = threadIdx.x & ((1 << sh) - 1);
        c = (by * bdim + threadIdx.x) >> sh;
    }
    const int t = tb * 16 * w.tn + tl;
    if (c >= w.cpad || t >= w.Tpad) return;
    const bool narrow = wino_short_block(w, tb);
    // The alpha x alpha patch, all loads in flight at once: elements in the zero padding, of
    // tiles past the end and of padding channels get an out-of-range offset and read as zero.
    float d[A][A];
    {
        const bool live = t < w.T && c < w.C;
        const int tt = live ? t : 0, cc = live ? c : 0;
        const int per = w.th * w.tw;
        const int img = tt / per, rem = tt - img * per;
        const int ti = rem / w.tw, tj = rem - ti * w.tw;
        const int ih0 = ti * M - w.ph, iw0 = tj * M - w.pw;
        const int base = (img * w.C + cc) * w.H * w.W;
        const __amdgpu_buffer_rsrc_t xres = make_rsrc(w.x, w.x_bytes);
        if (!HALF && w.pw == 1) {                 // (uniform)
            if constexpr (!HALF) {
                const int lane = threadIdx.x & 63;
                patch_load<M>(d, xres, tj, w.tw, lane, [&](int u) __attribute__((always_inline)) {
                    return live && (unsigned)(ih0 + u) < (unsigned)w.H ? (uint32_t)(base + (ih0 + u) * w.W) * 4u : kOobOffset;
                }, 0u);
                patch_finish<M>(d, tj, w.tw, w.W);
            }
        } else {
#pragma unroll
            for (int u = 0; u < A; ++u) {
                const int ih = ih0 + u;
                const bool rok = live && (unsigned)ih < (unsigned)w.H;
#pragma unroll
                for (int v = 0; v < A; ++v) {
                    const int iw = iw0 + v;
                    const bool ok = rok && (unsigned)iw < (unsigned)w.W;
                    d[u][v] = buf_load_x<T>(xres, ok ? (uint32_t)(base + ih * w.W + iw) * (uint32_t)sizeof(T) : kOobOffset, 0u);
                }
            }
        }
    }
    float tmp[A][A], V[A][A];
    NNV_MATMUL_LEFT(Wm::BT, A, A, A, d, tmp)
    NNV_MATMUL_RIGHT_T(Wm::BT, A, A, A, tmp, V)
    if (HALF) {
        const int frag = narrow ? 0 : tl % w.tn, row = narrow ? (tl >> 1) + 8 * (tl & 1) : tl / w.tn;
        __half *o = static_cast<__half *>(w.V) + ((size_t)(tb * w.tn + frag) * w.csteps + c / 32) * 512 + ((c % 32) / 8) * 128 + row * 8 + (c & 7);
        const size_t xs = (size_t)w.Tpad * w.cpad;
#pragma unroll
        for (int u = 0; u < A; ++u)
#pragma unroll
            for (int v = 0; v < A; ++v) o[(u * A + v) * xs] = __float2half_rn(V[u][v]);
    } else {
        float *o = static_cast<float *>(w.V) + (size_t)tb * w.cpad * (16 * w.tn) + c * (narrow ? 16 : 16 * w.tn) + tl;
        const size_t xs = (size_t)w.Tpad * w.cpad;
#pragma unroll
        for (int u = 0; u < A; ++u)
#pragma unroll
            for (int v = 0; v < A; ++v) o[(u * A + v) * xs] = V[u][v];
    }
}

template <int SET, bool HALF>
__global__ __launch_bounds__(256) void wino_input_kernel(const WinoParams w) {
    wino_input_block<SET, HALF>(w, blockIdx.x, blockIdx.y, blockDim.x);
}

// ---- 2. batched tile GEMM: per frequency xi, M[xi] (K x T) = U[xi] (K x C) V[xi] (C x T) on the matrix cores.
//
// float32: what bounds a 16x16x4 GEMM fed by one load per operand fragment is the CU's vector memory path (a
// 256-byte wave load takes it 5-9 cycles, four SIMDs want one fragment each per 32-cycle MFMA), so here a
// load carries the fragments of several blocks: which row of a block is which output channel is free, as
// long as the store agrees.  With TM panels (16 output channels x 4 channels, [c][k] in memory) per tile, lane
// (i, slot) takes TM consecutive floats, rows TM (i % (16/TM)) .. of panel i / (16/TM), channel slot: element
// m is its operand of the m-th row block.  One 16-byte load replaces four, and V is stored so that the TN tile
// blocks of a lane are neighbours too: 2 loads per 8 MFMAs instead of 6 (64 x 32 tile).
// What bounds a launch now is U, V and M through the fabric: the tile GEMMs of all layers of a VGG-16-shaped F(4x4) stack move
// 497 MB (U is 235) in 110 us, 0.88 of the rate of a plain copy; a pass of three launches 207 -> 176 us.  64 x 64 tiles
// (TN = 4) move less through L1 and took the same time there, 10 % more on a ResNet-18-shaped stack.
// float16: fragments are 16 bytes per lane to begin with.
typedef uint32_t uint32x2 __attribute__((ext_vector_type(2)));
template <int N> __device__ static inline void buf_store_floats(const typename FloatVec<N>::type &v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    if constexpr (N == 1) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, voff, soff, 0);
    else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint32x2, v), r, voff, soff, 0);
}
// One step (4 or 32 channels) of a tile's operands.
template <bool HALF, int TM, int TN> struct WinoStep;
template <int TM, int TN> struct WinoStep<false, TM, TN> {
    typename FloatVec<TM>::type a;
    typename FloatVec<TN>::type b;
};
template <int TM, int TN> struct WinoStep<true, TM, TN> {
    half8 a[TM], b[TN];
};

// The k-loop is kept to loads and MFMAs: a lone wavefront on a SIMD issues one instruction
// every four cycles, so every select or address computation in the loop costs as much as a
// quarter of a float32 MFMA.  Offsets are a per-lane constant (or an out-of-range constant
// for panels outside the problem) plus a scalar that advances by one fragment per step.
// One wavefront's work on one frequency: `run` tiles, TM panels x the TN = w.tn 16-tile blocks of the tile blocks
// tb, tb + 1, ..., summed over the ks-th of KS ranges of the channel steps (KS > 1: run = 1); `red` is the
// workgroup's LDS (used if KS > 1), nt the wavefront's tile slot in it.  The first loads of a tile are
// in flight while the one before it is finished and stored: with 64 channels a tile is 2 us of matrix
// instructions, as much as it takes to look the layer up and get the first operands, and a launch of
// such tiles ran at a third of the rate of its long ones.  kb0 >= K16: nothing is loaded, nothing stored.
template <bool HALF, int TM, int TN, int D>
__device__ __forceinline__ void wino_gemm_tile(const WinoParams &w, const int xi, const int kb0, const int tb, const int run,
                                               const int ks, const int KS, const int ks_shift, const int nt,
                                               const int lane, float *red) {
    const __amdgpu_buffer_rsrc_t ures = make_rsrc(w.U, w.u_bytes);
    const __amdgpu_buffer_rsrc_t vres = make_rsrc(w.V, w.v_bytes);
    const int col = lane & 15, slot = lane >> 4;
    constexpr int QM = 16 / TM;          // float32: lanes per panel
    constexpr uint32_t FRAG = HALF ? 1024 : 256;
    const bool any = kb0 < w.K16;
    uint32_t a_voff[HALF ? TM : 1], b_voff;
    // the last block may be short (then KS = 1 runs end with it): its tiles are those of the lanes col < 8
    auto is_short = [&](int r) __attribute__((always_inline)) { return TN == 2 && (tb + r + 1) * (16 * TN) > w.Tpad; };
    const uint32_t b_step = !HALF && is_short(0) ? FRAG : FRAG * TN;      // float32: bytes of V per step
    const uint32_t panel = (uint32_t)w.csteps * FRAG;        // bytes of a panel of U
    if constexpr (HALF) {
#pragma unroll
        for (int m = 0; m < TM; ++m) a_voff[m] = kb0 + m < w.K16 ? (uint32_t)m * panel + lane * 16u : kOobOffset;
        b_voff = lane * 16u;
    } else {
        a_voff[0] = kb0 + col / QM < w.K16 ? (uint32_t)(col / QM) * panel + (uint32_t)slot * 64u + (uint32_t)(col % QM) * (4u * TM) : kOobOffset;
        b_voff = (uint32_t)slot * (b_step / 4u) + (uint32_t)col * (4u * TN);
        if (is_short(0) && col >= 8) b_voff = kOobOffset;
    }
    if (!any) b_voff = kOobOffset;
    const uint32_t a_base = any ? ((uint32_t)xi * w.K16 + kb0) * panel : 0u;
    const uint32_t b_base = any ? ((uint32_t)xi * (w.Tpad >> 4) + (uint32_t)tb * TN) * panel : 0u;
    const int per_wave = (w.csteps + KS - 1) >> ks_shift;
    const int s_begin = min(w.csteps, ks * per_wave);
    const int s_end = min(w.csteps, s_begin + per_wave);

    WinoStep<HALF, TM, TN> st[2][D];
    // chunk of D steps of tile r starting at step s0; steps past the end read as zero (their products are
    // added like any others: one path through the loop keeps one set of accumulator registers)
    auto load_chunk = [&](int buf, int r, int s0) __attribute__((always_inline)) {
        const uint32_t b_tile = b_base + (uint32_t)r * (TN * panel);
        const bool narrow = HALF && is_short(r);     // uniform; float16: fragment 1 of a short block is the rows 8.. of fragment 0
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const bool in = s0 + d < s_end;          // uniform
            const uint32_t s = in ? (uint32_t)(s0 + d) : 0u;
            const uint32_t bo = in ? b_voff : kOobOffset;
            if constexpr (HALF) {
#pragma unroll
                for (int m = 0; m < TM; ++m) st[buf][d].a[m] = buf_load<half8>(ures, in ? a_voff[m] : kOobOffset, a_base + s * FRAG);
#pragma unroll
                for (int t = 0; t < TN; ++t) {
                    const uint32_t bt = t > 0 && narrow ? (col < 8 ? bo + t * 128u : kOobOffset) : bo;
                    st[buf][d].b[t] = buf_load<half8>(vres, bt, b_tile + (narrow ? 0u : (uint32_t)t * panel) + s * FRAG);
                }
            } else {
                st[buf][d].a = buf_load_floats<TM>(ures, in ? a_voff[0] : kOobOffset, a_base + s * FRAG);
                st[buf][d].b = buf_load_floats<TN>(vres, bo, b_tile + s * b_step);
            }
        }
    };
    floatx4 acc[TM][TN];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t) acc[m][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    };
    auto mfma_step = [&](int buf, int d) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                if constexpr (HALF)
                    acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(st[buf][d].a[m], st[buf][d].b[t], acc[m][t], 0, 0, 0);
                else
                    acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(float_of<TM>(st[buf][d].a, m), float_of<TN>(st[buf][d].b, t), acc[m][t], 0, 0, 0);
            }
    };
    // M[xi][k][Tpad tiles]: register (m, t, j) of lane (col, slot) is block row i = 4 slot + j of row block m, tile
    // TN col + t.  float32: row TM (i % QM) + m of panel i / QM, a lane's part and a part that depends on
    // (m, j) alone.
    const uint32_t m_row = (uint32_t)w.Tpad * 4u;
    const __amdgpu_buffer_rsrc_t mres = make_rsrc(w.M, (uint32_t)w.alpha2 * (uint32_t)w.K16 * 16u * m_row);
    const int lane_panel = HALF ? 0 : slot * 4 / QM, lane_row = HALF ? slot * 4 : TM * (slot * 4 % QM);
    const uint32_t m_voff = kb0 + lane_panel < w.K16 && !(!HALF && is_short(0) && col >= 8) ? (uint32_t)(lane_panel * 16 + lane_row) * m_row + (uint32_t)col * (4u * TN) : kOobOffset;
    const uint32_t m_base = any ? ((uint32_t)xi * w.K16 + kb0) * 16u * m_row + (uint32_t)tb * (64u * TN) : 0u;
    auto store_row = [&](const int r, const int m, const typename FloatVec<TN>::type &v, const uint32_t off) __attribute__((always_inline)) {
        if (!HALF || kb0 + m < w.K16) buf_store_floats<TN>(v, mres, HALF && is_short(r) && col >= 8 ? kOobOffset : m_voff, off);
    };
    auto finish = [&](int r) __attribute__((always_inline)) {
        uint32_t off = m_base + (uint32_t)r * (64u * TN);
#pragma unroll
        for (int q = 0; q < TM * 4; ++q) {          // rows in the order of their uniform part
            const int m = HALF ? q / 4 : q % TM, j = HALF ? q % 4 : q / TM;
            typename FloatVec<TN>::type v;
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                if constexpr (TN == 1) v = acc[m][t][j];
                else v[t] = acc[m][t][j];
            }
            store_row(r, m, v, off);
            off += HALF && j == 3 ? 13u * m_row : m_row;
        }
        clear();
    };
    // (scheduling barriers: the loads of the next chunk stay in front of this chunk's MFMAs)
    int r = 0, s = s_begin;
    clear();
    load_chunk(0, 0, s);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    for (bool more = true; more;) {
#pragma unroll
        for (int buf = 0; buf < 2; ++buf) {
            if (buf == 1 && !more) break;
            const bool last = s + D >= s_end;
            const int rn = last ? r + 1 : r, sn = last ? s_begin : s + D;
            load_chunk(buf ^ 1, min(rn, run - 1), sn);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int d = 0; d < D; ++d) mfma_step(buf, d);
            __builtin_amdgcn_sched_barrier(0);
            if (last && KS == 1) finish(r);
            more = rn < run;
            r = rn;
            s = sn;
        }
    }
    if (KS > 1) {
        constexpr int NREG = TM * TN * 4;
        float *mine = red + (nt * KS + ks) * NREG * 64 + lane;
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) mine[((m * 4 + j) * TN + t) * 64] = acc[m][t][j];
        __syncthreads();
        for (int q = ks; q < TM * 4; q += KS) {
            const int m = HALF ? q / 4 : q % TM, j = HALF ? q % 4 : q / TM;
            const float *p = red + (nt * KS * NREG + (m * 4 + j) * TN) * 64 + lane;
            typename FloatVec<TN>::type v;
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                float e = 0.f;
                for (int z = 0; z < KS; ++z) e += p[(z * NREG + t) * 64];
                if constexpr (TN == 1) v = e;
                else v[t] = e;
            }
            store_row(0, m, v, m_base + (uint32_t)(HALF ? m * 16 + j : q) * m_row);
        }
    }
}

template <bool HALF, int TM, int TN, int D>
__global__ __launch_bounds__(1024) void wino_gemm_kernel(const WinoParams w) {
    extern __shared__ __align__(16) float red[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar
    const int KS = 1 << w.ks_shift;
    const int ks = wave & (KS - 1), nt = wave >> w.ks_shift;
    const int tiles_per_wg = (blockDim.x >> 6) >> w.ks_shift;
    // logical workgroup order: frequency slowest, so an XCD works on a few frequencies and keeps
    // their U and V panels in its own L2
    const int lwg = xcd_logical_tile(w.gemm_wgs_per_xi * w.alpha2);
    if (lwg < 0) return;
    const int xi = lwg / w.gemm_wgs_per_xi;
    const int tile = (lwg - xi * w.gemm_wgs_per_xi) * tiles_per_wg + nt;   // flattened (panel group, tile block)
    const int kbt = tile / w.nblk, tb = tile - kbt * w.nblk;
    wino_gemm_tile<HALF, TM, TN, D>(w, xi, kbt * TM, tb, 1, ks, KS, w.ks_shift, nt, lane, red);   // kb0 >= K16 for surplus wavefronts
}

// Bias, optional clamp at zero and store of the M x M outputs of tile t, channel k, clipped to P x Q.
template <int M, bool HALF>
__device__ __forceinline__ void wino_store_tile(const WinoParams &w, float (&Y)[M][M], int t, int k) {
    const float bv = w.bias ? w.bias[k] : 0.f;
#pragma unroll
    for (int a = 0; a < M; ++a)
#pragma unroll
        for (int b = 0; b < M; ++b) {
            Y[a][b] += bv;
            if (w.relu) Y[a][b] = fmaxf(Y[a][b], 0.f);
        }
    const int per = w.th * w.tw;
    const int img = t / per, rem = t - img * per;
    const int ti = rem / w.tw, tj = rem - ti * w.tw;
    const size_t base = ((size_t)img * w.K + k) * w.P * w.Q;
    // Rows of a tile are stored VW elements at a time where Q is a multiple of VW (every group
    // of VW columns is then entirely inside the image and aligned): adjacent lanes hold
    // adjacent tiles, so a wavefront writes contiguous runs instead of 4-byte pieces.
    constexpr int VW = M % 4 == 0 ? 4 : 2;
    const bool vec = w.Q % VW == 0;
#pragma unroll
    for (int a = 0; a < M; ++a) {
        const int p = ti * M + a;
        if (p >= w.P) continue;
        if (vec) {
#pragma unroll
            for (int b = 0; b < M; b += VW) {
                const int q = tj * M + b;
                if (q >= w.Q) continue;
                const size_t o = base + (size_t)p * w.Q + q;
                if constexpr (HALF) {
                    uint32_t pk[VW / 2];
#pragma unroll
                    for (int i = 0; i < VW / 2; ++i) {
                        __half2 h = __floats2half2_rn(Y[a][b + 2 * i], Y[a][b + 2 * i + 1]);
                        pk[i] = *reinterpret_cast<uint32_t *>(&h);
                    }
                    if constexpr (VW == 4) *reinterpret_cast<uint2 *>(static_cast<__half *>(w.y) + o) = make_uint2(pk[0], pk[1]);
                    else *reinterpret_cast<uint32_t *>(static_cast<__half *>(w.y) + o) = pk[0];
                } else {
                    if constexpr (VW == 4)
                        *reinterpret_cast<float4 *>(static_cast<float *>(w.y) + o) =
                            make_float4(Y[a][b], Y[a][b + 1], Y[a][b + 2], Y[a][b + 3]);
                    else
                        *reinterpret_cast<float2 *>(static_cast<float *>(w.y) + o) = make_float2(Y[a][b], Y[a][b + 1]);
                }
            }
        } else {
#pragma unroll
            for (int b = 0; b < M; ++b) {
                const int q = tj * M + b;
                if (q >= w.Q) continue;
                const float v = Y[a][b];
                if (HALF) static_cast<__half *>(w.y)[base + (size_t)p * w.Q + q] = __float2half_rn(v);
                else static_cast<float *>(w.y)[base + (size_t)p * w.Q + q] = v;
            }
        }
    }
}

// ---- 3. output transform.  A thread owns one tile of one output channel; a frequency of M is a contiguous
// [k][Tpad] array, so the threads take its elements in order and every load of a wavefront is one piece.
template <int SET, bool HALF>
__device__ __forceinline__ void wino_output_block(const WinoParams &w, const int blk, const int bdim) {
    using Wm = WinoMat<SET>;
    constexpr int A = Wm::A, M = Wm::M;
    const int e = blk * bdim + threadIdx.x;
    const int k = e / w.Tpad, t = e - k * w.Tpad;
    if (t >= w.T || k >= w.K) return;
    const float *mp = w.M + e;
    const size_t xs = (size_t)w.K16 * 16 * w.Tpad;
    float m[A][A];
#pragma unroll
    for (int u = 0; u < A; ++u)
#pragma unroll
        for (int v = 0; v < A; ++v) m[u][v] = mp[(u * A + v) * xs];
    float tmp[M][A], Y[M][M];
    NNV_MATMUL_LEFT(Wm::AT, M, A, A, m, tmp)
    NNV_MATMUL_RIGHT_T(Wm::AT, M, A, M, tmp, Y)
    wino_store_tile<M, HALF>(w, Y, t, k);
}

template <int SET, bool HALF>
__global__ __launch_bounds__(256) void wino_output_kernel(const WinoParams w) {
    wino_output_block<SET, HALF>(w, blockIdx.x, blockDim.x);
}

// ---- many layers of one Winograd variant and storage type in three launches (input transforms,
// tile GEMMs, output transforms of all of them), for the same reason as the implicit GEMM's
// work-item launch: a batch-1 layer fills neither the chip nor the time its launch takes.
// A workgroup finds its layer by counting the entries of a prefix array it has reached.
constexpr int kWinoItemWaves = 4;
constexpr int kWinoGroup = 8;      // consecutive tile-GEMM workgroups handed to one XCD
struct WinoTable {
    WinoParams layer[kMaxWinoLayers];
    int in0[kMaxWinoLayers];      // first workgroup of each layer: input transform,
    int gemm0[kMaxWinoLayers];    //   tile GEMM (workgroups of work items: frequency x tile),
    int out0[kMaxWinoLayers];     //   output transform; INT_MAX beyond the last layer
    int in_by[kMaxWinoLayers];    // channel groups per tile block (the "y" extent of the single launch)
    int tm[kMaxWinoLayers];       // panels per tile of the GEMM items
    int run[kMaxWinoLayers];      // tile blocks per item
    int n_in, n_gemm, n_out;
};
static_assert(sizeof(WinoTable) <= 4096, "the table is passed by value as the kernel argument");
typedef const __attribute__((address_space(4))) WinoTable *WinoTablePtr;

__device__ __forceinline__ void load_wino_layer(WinoParams &dst, const WinoTablePtr tbl, const int li) {
    static_assert(sizeof(WinoParams) % 4 == 0, "copied word by word");
    const __attribute__((address_space(4))) uint32_t *src = (const __attribute__((address_space(4))) uint32_t *)&tbl->layer[li];
    uint32_t *d = reinterpret_cast<uint32_t *>(&dst);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(WinoParams) / 4); ++i) d[i] = src[i];
}

#define NNV_FIND_LAYER(prefix, b, li, first) \
    int first;                               \
    const int li = table_find<kMaxWinoLayers>(&tbl->prefix[0], (b), first);

template <int SET, bool HALF>
__global__ __launch_bounds__(256) void wino_input_many_kernel(const WinoTable tbl_arg) {
    const WinoTablePtr tbl = (WinoTablePtr)__builtin_amdgcn_kernarg_segment_ptr();
    const int b = blockIdx.x;
    NNV_FIND_LAYER(in0, b, li, first)
    WinoParams w;
    load_wino_layer(w, tbl, li);
    const int local = b - first, by_n = tbl->in_by[li];
    wino_input_block<SET, HALF>(w, local / by_n, local % by_n, 256);
}

template <int SET, bool HALF>
__global__ __launch_bounds__(256) void wino_output_many_kernel(const WinoTable tbl_arg) {
    const WinoTablePtr tbl = (WinoTablePtr)__builtin_amdgcn_kernarg_segment_ptr();
    const int b = blockIdx.x;
    NNV_FIND_LAYER(out0, b, li, first)
    WinoParams w;
    load_wino_layer(w, tbl, li);
    wino_output_block<SET, HALF>(w, b - first, 256);
}

// Tile GEMM work items (frequency x tile) in workgroups of kWinoItemWaves wavefronts, which take
// consecutive items (the same panels of U, neighbouring tile blocks: three of four reads of U hit the CU's
// L1).  The items of a layer with many channel steps are given to 2 or 4 of them that split the steps
// (summed through LDS in a fixed order).  Items of a layer are ordered frequency slowest; groups of 8
// consecutive workgroups go to one XCD.
template <bool HALF>
__global__ __launch_bounds__(64 * kWinoItemWaves, 5) void wino_gemm_many_kernel(const WinoTable tbl_arg) {
    extern __shared__ __align__(16) float red[];      // kWinoItemWaves x 32 accumulator registers x 64 lanes
    const WinoTablePtr tbl = (WinoTablePtr)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int G = kWinoGroup;
    const int i = blockIdx.x, xcd = i & 7, j = i >> 3;
    const int wg = ((j / G) * 8 + xcd) * G + j % G;
    if (wg >= tbl->n_gemm) return;
    __builtin_amdgcn_s_setprio(3);       // the look-up competes for issue slots with the k-loops of the resident wavefronts
    NNV_FIND_LAYER(gemm0, wg, li, first)
    WinoParams w;
    load_wino_layer(w, tbl, li);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int KS = 1 << w.ks_shift, ks = wave & (KS - 1), nt = wave >> w.ks_shift;
    const int local = (wg - first) * (kWinoItemWaves >> w.ks_shift) + nt;
    const int tm = tbl->tm[li], run = tbl->run[li];
    const int per_row = (w.nblk + run - 1) / run;         // items per frequency and panel group: runs of tile blocks
    const int per_xi = w.gemm_wgs_per_xi;                 // items per frequency
    const bool surplus = local >= per_xi * w.alpha2;      // the last workgroup of a layer may hold fewer items
    const int xi = surplus ? 0 : local / per_xi, tile = local - xi * per_xi;
    const int kbt = surplus ? w.K16 : tile / per_row, tb = surplus ? 0 : (tile - kbt * per_row) * run;   // kb0 >= K16: nothing loaded, nothing stored
#define NNV_WINO_ITEM(TM, TN, D) wino_gemm_tile<HALF, TM, TN, D>(w, xi, kbt * TM, tb, HALF ? min(run, w.nblk - tb) : 1, ks, KS, w.ks_shift, nt, lane, red)
    if constexpr (HALF) {
        if (w.tn == 2) { if (tm == 2) NNV_WINO_ITEM(2, 2, 2); else NNV_WINO_ITEM(1, 2, 2); }
        else { if (tm == 2) NNV_WINO_ITEM(2, 1, 2); else NNV_WINO_ITEM(1, 1, 2); }
    } else {
        if (w.tn == 2) { if (tm == 4) NNV_WINO_ITEM(4, 2, 4); else if (tm == 2) NNV_WINO_ITEM(2, 2, 4); else NNV_WINO_ITEM(1, 2, 4); }
        else { if (tm == 4) NNV_WINO_ITEM(4, 1, 4); else if (tm == 2) NNV_WINO_ITEM(2, 1, 4); else NNV_WINO_ITEM(1, 1, 4); }
    }
#undef NNV_WINO_ITEM
}

// ---- fused variant (float32, F(2x2) and F(4x4)): all three steps in one kernel, V and M never in memory.
// A workgroup owns 16 TN tiles x 16 TM output channels at all frequencies, FW of them per wavefront.  A chunk is 4 / TN steps of four input channels:
// while the products of a chunk run, four wavefronts transform the patches of the next one, each those of one step and one block of 16 tiles, lane (tile
// l % 16, channel l / 16), and lay them down in LDS as ready-made operand fragments.  U comes from L2 in the layout of the tile GEMM, a load per TM TN
// products, requested a chunk ahead.  At the end the frequencies meet in LDS, a row block at a time, and a thread transforms and stores one tile.
// What bounds it is the matrix cores, at three quarters of the rate of a large product while a workgroup per CU is resident: a chunk of F(4x4) (16 channels) takes 3.0 us,
// 1.9 of them products at 2.4 GHz; 2.7 without the transforms, as long without the loads of U.  Patches in single elements held the vector memory path
// instead (4.4 us).  Over a whole launch the matrix pipe is busy 54 % of the cycles in F(2x2) (eight layers of a VGG-16-shaped stack, 116 us) and 30 % in F(4x4) (five, of up to 8 chunks,
// 61 us): the rest is a workgroup's start and end.  F(4x4) has twelve wavefronts for the products and four of their own for the transforms: one wavefront that did both would wait for
// patches whenever it waits for U, since loads come back in order (5.0 us).  F(2x2), with four times fewer elements in a patch, has eight that do both; twelve,
// one workgroup per CU instead of two, take a VGG-16-shaped stack from 166 to 200 us.  32 x 32 tiles (TM = TN = 2) for F(4x4), half the loads of U and twice the transforms: 3.9 us a chunk.
constexpr int kWinoFusedFreqs[2] = {2, 3};        // frequencies of a wavefront
constexpr int kWinoFusedOwn[2] = {0, 4};          // wavefronts that only transform (0: the first four do both)
constexpr int wino_fused_threads(int set) { return ((set == 0 ? 16 : 36) / kWinoFusedFreqs[set] + kWinoFusedOwn[set]) * 64; }
template <int SET, int TM, int TN, bool WIDE>
__device__ __forceinline__ void wino_fused_block(const WinoParams &w, const int blk, float *lds) {
    using Wm = WinoMat<SET>;
    constexpr int A = Wm::A, M = Wm::M, AA = A * A, FW = kWinoFusedFreqs[SET], WAVES = AA / FW, OWN = kWinoFusedOwn[SET], STEPS = 4 / TN, QM = 16 / TM;
    static_assert(AA % FW == 0 && WAVES >= 8 && STEPS % 2 == 0, "the first four wavefronts transform, eight store");
    constexpr int kBuffer = AA * 256;                     // floats: a chunk of V, or a row block of M of 16 tiles
    const int lane = threadIdx.x & 63, col = lane & 15, slot = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nt = ((w.Tpad >> 4) + TN - 1) / TN;
    const int kbt = blk / nt, tb = blk - kbt * nt, kb0 = kbt * TM;       // tile blocks fastest: neighbours share U
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(w.x, w.x_bytes);
    const __amdgpu_buffer_rsrc_t ures = make_rsrc(w.U, w.u_bytes);
    const int jt = wave % TN, js = (wave & 3) / TN;             // the block of tiles and the step of a chunk that this wavefront transforms
    // Byte offsets of the patch's rows and columns in channel `slot`.  Those in the zero padding, of tiles past the end and of
    // missing channels carry 2^30 each, beyond the end of x (smaller than 2^30 bytes on this route): their elements read as zero.
    constexpr uint32_t kOut = 0x40000000u;
    const uint32_t plane4 = (uint32_t)(w.H * w.W) * 16u;  // bytes of 4 channel planes
    uint32_t rowoff[A];
    int tj;
    {
        const int t = (tb * TN + jt) * 16 + col;
        const bool live = t < w.T;
        const int tt = live ? t : 0, per = w.th * w.tw;
        const int img = tt / per, rem = tt - img * per;
        const int ti = rem / w.tw, ih0 = ti * M - w.ph;
        tj = rem - ti * w.tw;
        const int base = (img * w.C + slot) * w.H * w.W;
#pragma unroll
        for (int u = 0; u < A; ++u) {
            const int ih = ih0 + u;
            rowoff[u] = live && (unsigned)ih < (unsigned)w.H ? (uint32_t)(base + ih * w.W) * 4u : kOut;
        }
    }
    const uint32_t panel = (uint32_t)w.csteps * 256u;
    const uint32_t a_voff = kb0 + col / QM < w.K16 ? (uint32_t)(col / QM) * panel + (uint32_t)slot * 64u + (uint32_t)(col % QM) * (4u * TM) : kOobOffset;
    const uint32_t a_xi = (uint32_t)w.K16 * panel, a_base = (uint32_t)(wave * FW) * a_xi + (uint32_t)kb0 * panel;
    typename FloatVec<TM>::type a[STEPS][FW];   // of the steps s, s + 1, ...
    float d[A][A];
    // (steps past the last one read as zero, both operands: one path through the loop keeps one set of accumulators)
    auto load_a = [&](const int p, const int f, const int s) __attribute__((always_inline)) {
        a[p][f] = buf_load_floats<TM>(ures, s < w.csteps ? a_voff : kOobOffset, a_base + (uint32_t)f * a_xi + (s < w.csteps ? (uint32_t)s * 256u : 0u));
    };
    auto load_patch = [&](const int ch) __attribute__((always_inline)) {
        const int s = ch * STEPS + js;                    // (past the last step: nothing)
        const uint32_t miss = s * 4 + slot < w.C ? 0u : kOut, soff = s < w.csteps ? (uint32_t)s * plane4 : 0u;
        if constexpr (WIDE) patch_load<M>(d, xres, tj, w.tw, lane, [&](int u) __attribute__((always_inline)) { return rowoff[u] + miss; }, soff);
        else {
#pragma unroll
            for (int v = 0; v < A; ++v) {
                const int iw = tj * M - w.pw + v;
                const uint32_t coloff = (unsigned)iw < (unsigned)w.W ? (uint32_t)iw * 4u : kOut;
#pragma unroll
                for (int u = 0; u < A; ++u) d[u][v] = buf_load<float>(xres, rowoff[u] + miss + coloff, soff);
            }
        }
    };
    auto put_patch = [&](const int ch) __attribute__((always_inline)) {
        float *o = lds + (ch & 1) * kBuffer + (js * AA * 64 + lane) * TN + jt;
        if constexpr (WIDE) patch_finish<M>(d, tj, w.tw, w.W);
        // column by column in place, then row by row: few registers beside the patch itself
#pragma unroll
        for (int v = 0; v < A; ++v) {
            float in[A][1], out[A][1];
#pragma unroll
            for (int u = 0; u < A; ++u) in[u][0] = d[u][v];
            NNV_MATMUL_LEFT(Wm::BT, A, A, 1, in, out)
#pragma unroll
            for (int u = 0; u < A; ++u) d[u][v] = out[u][0];
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int u = 0; u < A; ++u) {
            float in[1][A], out[1][A];
#pragma unroll
            for (int v = 0; v < A; ++v) in[0][v] = d[u][v];
            NNV_MATMUL_RIGHT_T(Wm::BT, 1, A, A, in, out)
#pragma unroll
            for (int v = 0; v < A; ++v) o[(u * A + v) * 64 * TN] = out[0][v];
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    floatx4 acc[FW][TM][TN];
#pragma unroll
    for (int f = 0; f < FW; ++f)
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t) acc[f][m][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int chunks = (w.csteps + STEPS - 1) / STEPS;
    auto chunk_loop = [&](auto transforms, auto multiplies) __attribute__((always_inline)) {
        constexpr bool T = decltype(transforms)::value, P = decltype(multiplies)::value;
        if constexpr (T) {
            load_patch(0);
            __builtin_amdgcn_sched_barrier(0);
            put_patch(0);
            load_patch(1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (P) {
#pragma unroll
            for (int f = 0; f < STEPS * FW; ++f) load_a(f / FW, f % FW, f / FW);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        for (int ch = 0; ch < chunks; ++ch) {
            if constexpr (T) {
                put_patch(ch + 1);
                __builtin_amdgcn_sched_barrier(0);
                    load_patch(ch + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            const float *vb = lds + (ch & 1) * kBuffer + (wave * FW * 64 + lane) * TN;
            if constexpr (P) {
#pragma unroll
                for (int i = 0; i < STEPS; ++i) {
                    typename FloatVec<TN>::type b[FW];
#pragma unroll
                    for (int f = 0; f < FW; ++f) b[f] = *reinterpret_cast<const typename FloatVec<TN>::type *>(vb + (i * AA + f) * 64 * TN);
#pragma unroll
                    for (int f = 0; f < FW; ++f) {
#pragma unroll
                        for (int m = 0; m < TM; ++m)
#pragma unroll
                            for (int t = 0; t < TN; ++t)
                                acc[f][m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(float_of<TM>(a[i][f], m), float_of<TN>(b[f], t), acc[f][m][t], 0, 0, 0);
                        load_a(i, f, (ch + 1) * STEPS + i);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            __syncthreads();
        }
    };
    // A loop for each role, so that no wavefront waits for what it does not use; all pass 1 + chunks barriers.
    if (wave >= WAVES) __builtin_amdgcn_s_setprio(3);
    if (wave >= WAVES) chunk_loop(std::true_type{}, std::false_type{});
    else if (OWN == 0 && wave < 4) chunk_loop(std::true_type{}, std::true_type{});
    else chunk_loop(std::false_type{}, std::true_type{});
    // Row i = 4 slot + j of row block m is row TM (i % QM) + m of panel i / QM.  Two row blocks at a time, four wavefronts each.
    constexpr int Q = TM * TN;
#pragma unroll
    for (int q0 = 0; q0 < Q; q0 += 2) {
        if (q0 > 0) __syncthreads();
#pragma unroll
        for (int q = q0; q < q0 + 2 && q < Q; ++q)
#pragma unroll
            for (int f = 0; f < FW && wave < WAVES; ++f)
#pragma unroll
                for (int j = 0; j < 4; ++j) lds[(q & 1) * kBuffer + (wave * FW + f) * 256 + j * 64 + lane] = acc[f][q / TN][q % TN][j];
        __syncthreads();
        const int q = q0 + (wave >> 2), row = slot * 4 + (wave & 3);
        const int k = (kb0 + row / QM) * 16 + TM * (row % QM) + q / TN, tile = (tb * TN + q % TN) * 16 + col;
        if (wave < 8 && q < Q && k < w.K && tile < w.T) {
            const float *in_lds = lds + (wave >> 2) * kBuffer + (wave & 3) * 64 + lane;
            float in[A][A], tmp[M][A], Y[M][M];
#pragma unroll
            for (int u = 0; u < A; ++u)
#pragma unroll
                for (int v = 0; v < A; ++v) in[u][v] = in_lds[(u * A + v) * 256];
            NNV_MATMUL_LEFT(Wm::AT, M, A, A, in, tmp)
            NNV_MATMUL_RIGHT_T(Wm::AT, M, A, M, tmp, Y)
            wino_store_tile<M, false>(w, Y, tile, k);
        }
    }
}

struct WinoFusedTable {
    WinoParams layer[kMaxWinoLayers];
    int block0[kMaxWinoLayers];
    int tm[kMaxWinoLayers];
    int n;
};
static_assert(sizeof(WinoFusedTable) <= 4096, "the table is passed by value as the kernel argument");
typedef const __attribute__((address_space(4))) WinoFusedTable *WinoFusedTablePtr;
// WIDE: layers whose patches are read in wide loads (one column of padding): 0 none, 1 all, 2 some
template <int SET, int TN, int WIDE>
__global__ __launch_bounds__(wino_fused_threads(SET)) void wino_fused_kernel(const WinoFusedTable tbl_arg) {
    constexpr int A = WinoMat<SET>::A;
    __shared__ __align__(16) float lds[2 * A * A * 256];
    const WinoFusedTablePtr tbl = (WinoFusedTablePtr)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int G = kWinoGroup;
    const int i = blockIdx.x, xcd = i & 7, j = i >> 3;
    const int wg = ((j / G) * 8 + xcd) * G + j % G;
    if (wg >= tbl->n) return;
    int first;
    const int li = table_find<kMaxWinoLayers>(&tbl->block0[0], wg, first);
    WinoParams w;
    {
        const __attribute__((address_space(4))) uint32_t *src = (const __attribute__((address_space(4))) uint32_t *)&tbl->layer[li];
        uint32_t *dst = reinterpret_cast<uint32_t *>(&w);
#pragma unroll
        for (int k = 0; k < (int)(sizeof(WinoParams) / 4); ++k) dst[k] = src[k];
    }
    const int tm = tbl->tm[li];
    auto block = [&](auto wide) __attribute__((always_inline)) {
        constexpr bool W = decltype(wide)::value;
        if (tm == 4) wino_fused_block<SET, 4, TN, W>(w, wg - first, lds);
        else if (tm == 2) wino_fused_block<SET, 2, TN, W>(w, wg - first, lds);
        else wino_fused_block<SET, 1, TN, W>(w, wg - first, lds);
    };
    if (WIDE == 1 || (WIDE == 2 && w.pw == 1)) block(std::true_type{});
    if (WIDE == 0 || (WIDE == 2 && w.pw != 1)) block(std::false_type{});
}

// ---- layers of one step of channels (four of them: the first layer of a network) by themselves.  A workgroup of the kernel above is all start and end there: its wavefronts wait
// for four that transform, then M goes through LDS once more.  Here a wavefront owns 16 tiles x 16 output channels and every lane transforms the patch of one (tile, channel) pair in
// registers: lane (tile l%16, channel l/16) then holds, for every frequency, exactly its element
// of the B operand of the 16x16x4 MFMA.  The alpha^2 accumulators stay in registers and the
// output transform is applied to them in place (accumulator register j of lane l is output
// channel 4*(l/16)+j of tile l%16).  The input transform is repeated by every 16-channel block
// of K, and a wavefront has nobody beside it to wait for its patches: no longer worth it from two steps on (wino_waves).
// The sums are those of the kernel above, bit for bit.
template <int SET>
__global__ __launch_bounds__(256) void wino_wave_kernel(const WinoParams w) {
    using Wm = WinoMat<SET>;
    constexpr int A = Wm::A, M = Wm::M, AA = A * A;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // logical order: tile blocks fastest, so neighbouring workgroups share U; the four
    // wavefronts of a workgroup share the patches (same tiles, four blocks of output channels)
    const int lwg = xcd_logical_tile(w.gemm_wgs_per_xi);
    if (lwg < 0) return;
    const int T16 = (w.T + 15) >> 4;
    const int kbg = lwg / T16, tb = lwg - kbg * T16;
    const int kb = kbg * 4 + wave;
    if (kb >= w.K16) return;
    const int col = lane & 15, slot = lane >> 4;
    const int t = tb * 16 + col;
    const bool live = t < w.T;
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(w.x, w.x_bytes);
    const __amdgpu_buffer_rsrc_t ures = make_rsrc(w.U, w.u_bytes);
    const uint32_t plane4 = (uint32_t)(w.H * w.W) * 16u;     // bytes of 4 channel planes
    // per-lane byte offsets of the patch rows and columns in channel `slot`; a step adds its
    // channel base as the scalar offset.  Rows and columns in the zero padding (and every row of
    // a surplus tile) carry 2^30 instead, which puts the sum beyond the end of x (x is smaller
    // than 2^30 bytes on this route), so those elements read as zero.
    constexpr uint32_t kOut = 0x40000000u;
    uint32_t rowoff[A], coloff[A];
    {
        const int tt = live ? t : 0;
        const int per = w.th * w.tw;
        const int img = tt / per, rem = tt - img * per;
        const int ti = rem / w.tw, tj = rem - ti * w.tw;
        const int ih0 = ti * M - w.ph, iw0 = tj * M - w.pw;
        const int base = (img * w.C + slot) * w.H * w.W;
#pragma unroll
        for (int u = 0; u < A; ++u) {
            const int ih = ih0 + u;
            rowoff[u] = (live && (unsigned)ih < (unsigned)w.H) ? (uint32_t)(base + ih * w.W) * 4u : kOut;
        }
#pragma unroll
        for (int v = 0; v < A; ++v) {
            const int iw = iw0 + v;
            coloff[v] = (unsigned)iw < (unsigned)w.W ? (uint32_t)iw * 4u : kOut;
        }
    }
    const uint32_t a_voff = lane * 4u;
    const uint32_t a_base = (uint32_t)kb * w.csteps;          // fragment index at frequency 0, step 0
    const uint32_t a_xi = (uint32_t)w.K16 * w.csteps;         // fragments per frequency
    floatx4 acc[AA];
#pragma unroll
    for (int i = 0; i < AA; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    // Everything a step needs is requested one step earlier.  Patches alternate between two
    // register sets; the U fragment of frequency i is re-requested for the next step right
    // after the MFMA that consumed it, into the same register.  Loads complete in order, and
    // the order of issue is patch(s), U(s), patch(s+1), U(s+1), ..., so waiting for one of
    // them never waits for anything requested later.  The scheduling barriers keep that order.
    float d[2][A][A], a[AA];
    const int full = w.C >> 2;                                // steps whose 4 channels all exist
    const int last = w.csteps - 1;
    auto load_patch = [&](int buf, int s) __attribute__((always_inline)) {
        const uint32_t soff = (uint32_t)s * plane4;
#pragma unroll
        for (int u = 0; u < A; ++u)
#pragma unroll
            for (int v = 0; v < A; ++v) d[buf][u][v] = buf_load<float>(xres, rowoff[u] + coloff[v], soff);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto load_a = [&](int i, int s) __attribute__((always_inline)) {
        a[i] = buf_load<float>(ures, a_voff, (a_base + (uint32_t)i * a_xi + s) * 256u);
    };
    auto step = [&](int buf, int s) __attribute__((always_inline)) {
        float tmp[A][A], V[A][A];
        NNV_MATMUL_LEFT(Wm::BT, A, A, A, d[buf], tmp)
        NNV_MATMUL_RIGHT_T(Wm::BT, A, A, A, tmp, V)
        const int sn = min(s + 1, last);
#pragma unroll
        for (int i = 0; i < AA; ++i) {
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], V[i / A][i % A], acc[i], 0, 0, 0);
            load_a(i, sn);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    if (full > 0) load_patch(0, 0);
#pragma unroll
    for (int i = 0; i < AA; ++i) load_a(i, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (full > 0) {
        int s = 0;
        for (; s + 2 <= full; s += 2) {
            load_patch(1, s + 1);
            step(0, s);
            load_patch(0, min(s + 2, full - 1));
            step(1, s + 1);
        }
        if (s < full) step(0, s);
    }
    if (w.C & 3) {
        // last step of a channel count that is not a multiple of 4: lanes of missing channels read zero
        const bool cok = full * 4 + slot < w.C;
        const uint32_t soff = (uint32_t)full * plane4;
#pragma unroll
        for (int u = 0; u < A; ++u)
#pragma unroll
            for (int v = 0; v < A; ++v) d[0][u][v] = buf_load<float>(xres, cok ? rowoff[u] + coloff[v] : kOobOffset, soff);
        __builtin_amdgcn_sched_barrier(0);
        step(0, full);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = kb * 16 + slot * 4 + j;
        if (!live || k >= w.K) continue;
        float m[A][A], tmp[M][A], Y[M][M];
#pragma unroll
        for (int u = 0; u < A; ++u)
#pragma unroll
            for (int v = 0; v < A; ++v) m[u][v] = acc[u * A + v][j];
        NNV_MATMUL_LEFT(Wm::AT, M, A, A, m, tmp)
        NNV_MATMUL_RIGHT_T(Wm::AT, M, A, M, tmp, Y)
        wino_store_tile<M, false>(w, Y, t, k);
    }
}

// ---------------------------------------------------------------- host side

struct WinoPlan {
    int m, alpha, th, tw, T, T16, tn, nblk, Tpad, K16, cpad, csteps;
    size_t v_bytes, m_bytes;
};

static WinoPlan plan_wino(const Geo &g, int kind) {
    WinoPlan p{};
    const bool half = g.dtype == NNV_F16;
    p.m = wino_m(kind);
    p.alpha = p.m + 2;
    p.th = ceil_div(g.p, p.m);
    p.tw = ceil_div(g.q, p.m);
    p.T = g.n * p.th * p.tw;
    p.T16 = ceil_div(p.T, 16);
    p.tn = p.T > 16 ? 2 : 1;
    p.nblk = ceil_div(p.T, 16 * p.tn);
    p.Tpad = 16 * p.T16;
    p.K16 = ceil_div(g.k, 16);
    const int cb = half ? 32 : 4;
    p.csteps = ceil_div(g.c, cb);
    p.cpad = p.csteps * cb;
    const size_t aa = (size_t)p.alpha * p.alpha;
    p.v_bytes = align_up(aa * p.Tpad * p.cpad * (half ? 2 : 4), 256);
    p.m_bytes = align_up(aa * p.K16 * 16 * p.Tpad * sizeof(float), 256);
    return p;
}

// Panels per tile of a tile GEMM: two, or four (float32) where that leaves at most a seventh more rows empty than two would (three
// panels: as many).
static int wino_tm(const WinoPlan &p, bool half, int most = 4) {
    if (half || most < 4) return std::min(most, p.K16 >= 2 ? 2 : 1);
    if (p.K16 >= 3 && ceil_div(p.K16, 4) * 4 * 100 <= ceil_div(p.K16, 2) * 2 * 115) return 4;
    return p.K16 >= 2 ? 2 : 1;
}

// Which layers run as the fused kernel.  The three launches are bound by V and M, written and read in between, and by U; the fused kernel reads U once per block
// of tiles, from L2, and has no parallelism along the channels: a layer of many channels on few tiles is one long chain.  Both are estimated,
// in us, and a launch of several layers takes those of at most so many channel steps that the sum is least, if that is 3 % less than none (wino_fused_layers).  A layer whose
// channel steps the three launches would split keeps them: added up in one chain, 512 channels are 1.4 to 2 times further from the exact sums.
//   three = base + (V + M) / in_out + max((V + M + U) / gemm, operations / rate)                                (sums over the layers)
//   fused = start + max(ceil(workgroups / 256) x mean of (chunks x chunk + each), longest (chunks x chunk x lone) + first)
// MB and MFLOP over us; chunk and each: those of 64 outputs (less: their part for fewer).  Patches that are read element by element (padding other than one column) make a chunk
// `single` times as long, and three launches by `narrow` per MB of V.  Fitted to 716 layers and launches of five stacks with every line drawn (3-512 channels,
// 8-512 outputs, 7-320 pixels, batch 1-8), which it meets within 8 %; what it chooses is 0.1 to 0.4 % over the best line for each on average, and the slowest 1.05 times none fused.  us a call, three launches / all
// layers fused / chosen: VGG-16-shaped stack F(2x2) at 3x115x114 172 / 156 / 156, F(4x4) 1x263x191 168 / 161 / 160, 2x166x278 302 / 265 / 264; ResNet-18 F(2x2) 3x222x177 80 / 85 / 73, F(4x4)
// 1x224x224 51 / 75 / 51; SqueezeNet F(2x2) at 224x224 25.6 / 13.6 / 13.5, F(4x4) 4x157x241 39 / 31 / 31.  One layer, three / fused: F(4x4), 64 channels at 224x224 35.7 / 23.1, 256 at 112x112 68 / 58, at 56x56 24.8 / 56; F(2x2),
// 128 at 112x112 44 / 30.
struct WinoRates {
    double base, in_out, gemm, rate, start, chunk, each, lone, less, first, single, narrow;
};
constexpr WinoRates kWinoRates[2] = {{9.15, 4.29, 5.58, 86.3, 2.55, 1.22, 2.94, 1.43, 0.473, 1.74, 1.32, 0.026}, {9.82, 3.23, 5.47, 91.3, 3.18, 2.93, 8.15, 1.27, 0.477, 3.51, 1.81, 0.048}};

// (of one kernel or three: launch_wino takes no more blocks of tiles)
constexpr int kWinoMostT16 = 65535 * 16;

static bool wino_fused_able(const Geo &g, int kind) {
    return g.dtype == NNV_F32 && (kind == NNV_WINO_F2 || kind == NNV_WINO_F4) && (size_t)g.n * g.c * g.h * g.w * 4 < ((size_t)1 << 30);
}

// Layers with many tiles and few channels and outputs, which have no workspace and so no other route (the lines are those of an
// estimate of their own: what a program is told to allocate stays the same).
static bool wino_no_workspace(const Geo &g, int kind, const WinoPlan &p) {
    if (!wino_fused_able(g, kind) || p.T16 < 32 || p.K16 > 8 || p.csteps > 16) return false;
    const double wgs = (double)p.T16 * ceil_div(p.K16, 4);
    const double rounds = wgs > 256.0 ? wgs / 256.0 : 1.0;
    const int waves = p.K16 < 4 ? p.K16 : 4;
    const double step_us = kind == NNV_WINO_F2 ? 0.47 + 0.16 * (waves - 1) : 1.9 + 0.5 * (waves - 1);
    const double y_mb = (double)g.n * g.k * g.p * g.q * 4e-6;
    const double fused_us = 4.0 + y_mb / 2.3 + p.csteps * step_us * rounds;
    const double three_us = 8.0 + 2.0 * (double)(p.v_bytes + p.m_bytes) * 1e-6 / 3.0;
    return fused_us < three_us;
}

// Panels per workgroup of the fused kernel.
static int wino_fused_panels(const WinoPlan &p, const int most) { return p.K16 >= 3 ? most : std::min(p.K16, most); }

// Blocks of tiles and, at most, panels of its workgroups.
struct WinoForm { int tn, most; };
constexpr int kWinoForms = 4;
constexpr WinoForm kWinoForm[2][kWinoForms] = {{{2, 4}, {1, 4}, {1, 2}, {1, 1}}, {{1, 4}, {1, 4}, {1, 2}, {1, 1}}};
static long wino_form_blocks(const WinoPlan &p, const WinoForm &f) { return (long)ceil_div(p.T16, f.tn) * ceil_div(p.K16, wino_fused_panels(p, f.most)); }

// Which of them a launch takes; all: its workgroups in each.
// F(2x2) in fewer workgroups than the chip has CUs: one block of tiles each, twice as many and half as many chunks.  us a layer, two blocks / one: 10 channels at 5x73x22 -> 36 10.8 / 7.9,
// 20 at 4x46x31 -> 126 11.6 / 9.4.
// Fewer panels per workgroup, so more of them, while each still has a CU of its own (a workgroup of F(4x4) fills one).
// us a layer, four panels / two / one [workgroups]: F(4x4), 7 channels at 3x23x70 -> 122 [42 / 84 / 168] 14.3 / 10.4 / 8.7, 64 at 2x125x77 -> 59 [80 / 160 / 320] 23.0 / 17.2 / 25.1, 12 at
// 3x110x31 -> 206 [168 / 294 / 546] 14.2 / 18.2 / 21.1; F(2x2), 13 at 5x106x7 -> 33 [67 / 134 / 201] 6.7 / 5.4 / 4.9, 26 at 3x21x77 -> 153 [249 / 415 / 830] 9.6 / 10.9 / 12.0.
static int wino_form(const long (&all)[kWinoForms]) {
    if (all[0] >= 256) return 0;
    int f = 1;
    while (f + 1 < kWinoForms && all[f + 1] <= 256) ++f;
    return f;
}

// Layers that do better as wavefronts of their own (wino_wave_kernel) than as workgroups, where a launch of workgroups of four panels fills the chip.
// us a layer, workgroups / wavefronts: F(4x4), 3 channels at 224x224 -> 64 12.7 / 11.3, at 4x224x224 40.8 / 35.2, 4 at 4x224x224 40.6 / 39.5, 8 40.8 / 52.1, 3 -> 32 30.5 / 32.0 (-> 16 25.5 /
// 29.5); F(2x2), 3 at 112x112 -> 64 7.1 / 6.1, -> 128 9.7 / 7.2, at 224x224 -> 64 12.6 / 11.9, -> 32 8.8 / 10.3, -> 16 6.5 / 5.9, 4x224x224 -> 16 17.5 / 14.5, 8 at 4x56x56 -> 64 7.1 / 7.6,
// 7 at 8x31x74 -> 38 9.1 / 8.0 (three panels of four), 4 at 4x224x224 -> 96 57.9 / 62.5, at
// 112x112 21.0 / 20.6.
static bool wino_waves(int kind, const WinoPlan &p) {
    if (p.K16 > 8) return false;                // (more repeat the input transform too often)
    if (kind == NNV_WINO_F4) return p.csteps == 1 && p.K16 >= 3;
    return p.csteps == 1 ? p.K16 != 2 && (p.K16 < 5 || p.T16 <= 1024) : p.csteps == 2 && p.K16 == 3;
}

// Panels per tile of a layer's own tile GEMM, and over how many (1 << shift) wavefronts its channel steps are split.
// Latency-bound at batch 1 (measured on ResNet-18-shaped layers): the largest wavefront tile that still leaves >= 768 wavefronts; then
// the channel steps are split over the wavefronts of a workgroup towards ~4 per SIMD, keeping >= 16 steps each.
struct WinoSplit { int tm, shift; };
static WinoSplit wino_split(const WinoPlan &p, bool half) {
    const long aa = (long)p.alpha * p.alpha;
    int tm = wino_tm(p, half);
    while (tm > 1 && aa * ceil_div(p.K16, tm) * p.nblk < 768) tm = tm == 4 ? wino_tm(p, half, 2) : 1;
    int shift = 0;
    const long tiles = (long)ceil_div(p.K16, tm) * p.nblk;
    while (shift < 4 && ((aa * tiles) << shift) < 4096 && (p.csteps >> (shift + 1)) >= (half ? 4 : 16)) ++shift;
    return {tm, shift};
}

// The channel steps of the layers of one launch: split over 1 << shifts[i] wavefronts; runs[i]: tile blocks per item; mfmas[i]: matrix instructions of an
// item.  Returns those of the launch per SIMD.
// An item's wavefront should not outlast its share of the launch: matrix instructions of an item against
// those of the launch per SIMD; the channel steps of longer items are split over 2 or 4 wavefronts, and the
// layers with the longest wavefronts go first (but see below).  float16 F(2x2) items much shorter than a wavefront slot's
// share (four per SIMD) take several tile blocks one after the other (VGG-16-shaped stack 163 -> 157 us; the same on
// F(4x4) 106 -> 108, float32 F(4x4) 175 -> 177, F(6x6) 196 -> 208).
static long wino_many_split(int n, const WinoPlan *plans, int kind, bool half, long *mfmas, int *shifts, int *runs) {
    long total = 0, items = 0;
    for (int i = 0; i < n; ++i) {
        const WinoPlan &p = plans[i];
        const int tm = wino_tm(p, half);
        total += (long)p.csteps * p.tn * p.alpha * p.alpha * p.K16 * p.nblk;
        items += (long)p.alpha * p.alpha * ceil_div(p.K16, tm) * p.nblk;
        // a step's panels come from HBM once per frequency, whatever the number of tile blocks that share them: at
        // four wavefronts per SIMD 256 bytes of them take as long as three matrix instructions (half: a quarter of that per KB)
        mfmas[i] = (long)p.csteps * std::max(tm * p.tn, (half ? 6 : 13) * tm / 4 / p.nblk);
    }
    const long per_simd = total / 1024;      // matrix instructions of the launch per SIMD
    // The shortest wavefront worth a split, in matrix instructions.  float32: 128 while the launch has fewer items than the
    // chip has SIMDs (a split puts idle ones to work), else 512: wavefronts that have to queue gain nothing from being
    // shorter.  Measured over 110 launches of six stacks at batch 1-6 and 80-320 pixels, weights from HBM, geometric means of
    // 256 / 512 / 1024 against 128: up to 1008 items 1.02 / 1.06 / 1.12, 1472 to 4000 items 0.99 / 0.97 / 0.98, to 8000
    // 0.99 / 0.98 / 0.99, beyond (per_simd / 6 rules) 1.00 / 1.00 / 1.01.  float16: 64 to 384 take the same time within
    // 1-2 %, 32 costs a launch of few items 5 %.
    const long shortest = half ? 96 : items < 1024 ? 128 : 512;
    const long most = std::max(shortest, per_simd / 6), least = per_simd / 4 / 4;
    for (int i = 0; i < n; ++i) {
        shifts[i] = 0;
        while (shifts[i] < 2 && (mfmas[i] >> shifts[i]) > most && (plans[i].csteps >> (shifts[i] + 1)) >= (half ? 2 : 8)) ++shifts[i];
        runs[i] = 1;
        if (half && kind == NNV_WINO_F2 && shifts[i] == 0 && mfmas[i] < least) {
            const int r = (int)std::min<long>(least / mfmas[i], plans[i].nblk);
            runs[i] = ceil_div(plans[i].nblk, ceil_div(plans[i].nblk, r));      // equal runs
            mfmas[i] *= runs[i];
        }
    }
    return per_simd;
}

void wino_fused_layers(int n, const Geo *geos, int kind, char *fused) {
    std::fill(fused, fused + n, 0);
    if (n > kMaxWinoLayers || (kind != NNV_WINO_F2 && kind != NNV_WINO_F4) || geos[0].dtype == NNV_F16) return;
    const WinoRates &r = kWinoRates[kind == NNV_WINO_F2 ? 0 : 1];
    const int set = kind == NNV_WINO_F2 ? 0 : 1;
    struct Cost { int steps; double three; double blocks[kWinoForms], work[kWinoForms], chain[kWinoForms]; };
    Cost cost[kMaxWinoLayers];
    WinoPlan plans[kMaxWinoLayers], many[kMaxWinoLayers];
    bool only[kMaxWinoLayers];          // no other route
    int m = 0;
    for (int i = 0; i < n; ++i) {
        plans[i] = plan_wino(geos[i], kind);
        only[i] = wino_no_workspace(geos[i], kind, plans[i]);
        if (!only[i]) many[m++] = plans[i];
    }
    long mfmas[kMaxWinoLayers];
    int shifts[kMaxWinoLayers], runs[kMaxWinoLayers];       // of the others, in three launches
    if (m > 1) wino_many_split(m, many, kind, false, mfmas, shifts, runs);
    else if (m == 1) shifts[0] = wino_split(many[0], false).shift;
    int order[kMaxWinoLayers];
    double three = 0;
    for (int i = 0, j = 0; i < n; ++i) {
        const WinoPlan &p = plans[i];
        const double aa = (double)p.alpha * p.alpha, v = (double)p.v_bytes * 1e-6, vm = v + (double)p.m_bytes * 1e-6, u = aa * p.K16 * p.csteps * 256e-6;
        const double ops = 2.0 * aa * p.csteps * 4 * p.K16 * 16 * p.Tpad * 1e-6;
        Cost &c = cost[i];
        order[i] = i;
        c.steps = !wino_fused_able(geos[i], kind) || p.T16 > kWinoMostT16 ? INT_MAX : only[i] ? 0 : shifts[j] == 0 ? p.csteps : INT_MAX;
        j += only[i] ? 0 : 1;
        c.three = vm / r.in_out + (geos[i].pw != 1 ? v * r.narrow : 0.0) + std::max((vm + u) / r.gemm, ops / r.rate);
        three += c.three;
        for (int f = 0; f < kWinoForms; ++f) {
            const WinoForm &form = kWinoForm[set][f];
            const double part = wino_fused_panels(p, form.most) == 4 ? 1.0 : r.less;
            const double chunks = ceil_div(p.csteps, 4 / form.tn) * r.chunk * part * (geos[i].pw != 1 ? r.single : 1.0);
            c.blocks[f] = (double)wino_form_blocks(p, form);
            c.work[f] = c.blocks[f] * (chunks + r.each * part);
            c.chain[f] = chunks * r.lone;
        }
    }
    std::sort(order, order + n, [&](int a, int b) { return cost[a].steps < cost[b].steps; });
    // the layers in this order move to the fused launch one after the other
    int best = 0;
    double none = 0, best_us = 0, work[kWinoForms] = {}, chain[kWinoForms] = {};
    long all[kWinoForms] = {};
    for (int o = 0; o <= n; ++o) {
        const int next = o < n ? cost[order[o]].steps : INT_MAX;
        if (next > 0 && (o == 0 || next != cost[order[o - 1]].steps)) {
            double us = o < n ? r.base + three : 0.0;
            if (o > 0) {
                const int f = wino_form(all);
                us += r.start + std::max((double)((all[f] + 255) / 256) * work[f] / (double)all[f], chain[f] + r.first);
            }
            const int line = o > 0 ? cost[order[o - 1]].steps : 0;
            if (none == 0) none = best_us = us;
            else if (us < best_us && us < 0.97 * none) { best = line; best_us = us; }
        }
        if (o == n || next == INT_MAX) break;
        const Cost &c = cost[order[o]];
        three -= c.three;
        for (int f = 0; f < kWinoForms; ++f) {
            all[f] += (long)c.blocks[f];
            work[f] += c.work[f];
            chain[f] = std::max(chain[f], c.chain[f]);
        }
    }
    for (int i = 0; i < n; ++i) fused[i] = cost[i].steps <= best;
}

size_t wino_workspace_bytes(const Geo &g, int kind) {
    const WinoPlan p = plan_wino(g, kind);
    if (wino_no_workspace(g, kind, p)) return 0;
    return p.v_bytes + p.m_bytes;
}

template <bool HALF>
static void launch_wino_gemm(int tm, int tn, const WinoParams &w, dim3 grid, dim3 block, size_t lds, hipStream_t st) {
#define NNV_WINO_GEMM(TM, TN, D) hipLaunchKernelGGL((wino_gemm_kernel<HALF, TM, TN, D>), grid, block, lds, st, w)
    constexpr int D = HALF ? 2 : 4;
    if (tn == 2) {
        if (tm == 4) { if constexpr (!HALF) NNV_WINO_GEMM(4, 2, D); }
        else if (tm == 2) NNV_WINO_GEMM(2, 2, D);
        else NNV_WINO_GEMM(1, 2, D);
    } else {
        if (tm == 4) { if constexpr (!HALF) NNV_WINO_GEMM(4, 1, D); }
        else if (tm == 2) NNV_WINO_GEMM(2, 1, D);
        else NNV_WINO_GEMM(1, 1, D);
    }
#undef NNV_WINO_GEMM
}

template <int SET, bool HALF>
static hipError_t launch_wino_t(const Geo &g, const WinoPlan &p, WinoParams &w, hipStream_t st) {
    {
        // one wavefront per workgroup while that keeps the launch small: a batch-1 layer then occupies four times as many CUs
        const int bt = (!HALF && (long)p.T16 * ceil_div(p.cpad, 16) < 4096) ? 64 : 256;
        dim3 grid(p.nblk, HALF ? p.tn * ceil_div(p.cpad, 16) : ceil_div(p.cpad * 16 * p.tn, bt), 1);
        hipLaunchKernelGGL((wino_input_kernel<SET, HALF>), grid, dim3(bt), 0, st, w);
    }
    {
        const long aa = (long)p.alpha * p.alpha;
        const WinoSplit sp = wino_split(p, HALF);
        const int tm = sp.tm, shift = sp.shift;
        const long tiles = (long)ceil_div(p.K16, tm) * p.nblk;
        w.ks_shift = shift;
        w.gemm_wgs_per_xi = (int)tiles;
        const int waves = 1 << shift;
        const size_t lds = waves > 1 ? (size_t)waves * tm * p.tn * 4 * 64 * sizeof(float) : 0;
        launch_wino_gemm<HALF>(tm, p.tn, w, dim3(xcd_grid(w.gemm_wgs_per_xi * (int)aa)), dim3(64 * waves), lds, st);
    }
    {
        const int bt = (long)p.T16 * p.K16 < 4096 ? 64 : 256;
        hipLaunchKernelGGL((wino_output_kernel<SET, HALF>), dim3((unsigned)(((long)g.k * p.Tpad + bt - 1) / bt)), dim3(bt), 0, st, w);
    }
    return hipGetLastError();
}

static WinoParams wino_params(const Geo &g, const WinoPlan &p, const void *x, const void *U, const float *bias, void *y,
                              void *ws) {
    const bool half = g.dtype == NNV_F16;
    WinoParams w{};
    w.x = x; w.U = U; w.bias = bias; w.y = y;
    w.V = ws;
    w.M = reinterpret_cast<float *>(static_cast<char *>(ws) + p.v_bytes);
    w.N = g.n; w.C = g.c; w.H = g.h; w.W = g.w; w.K = g.k; w.ph = g.ph; w.pw = g.pw; w.P = g.p; w.Q = g.q;
    w.x_bytes = (uint32_t)((size_t)g.n * g.c * g.h * g.w * (half ? 2 : 4));
    w.relu = g.relu;
    w.th = p.th; w.tw = p.tw; w.T = p.T; w.tn = p.tn; w.nblk = p.nblk; w.Tpad = p.Tpad;
    w.K16 = p.K16; w.cpad = p.cpad; w.csteps = p.csteps;
    const size_t aa = (size_t)p.alpha * p.alpha;
    w.u_bytes = (uint32_t)(aa * p.K16 * p.csteps * 64 * (half ? 16 : 4));
    w.v_bytes = (uint32_t)(aa * p.Tpad * p.cpad * (half ? 2 : 4));
    w.alpha2 = (int)aa;
    return w;
}

bool wino_many_supported(const Geo &g, int kind) {
    const WinoPlan p = plan_wino(g, kind);
    return !wino_no_workspace(g, kind, p) && p.T16 <= (1 << 20) && p.K16 <= 65535;
}

template <int SET, bool HALF>
static void launch_wino_many_t(const WinoTable &tbl, hipStream_t st) {
    hipLaunchKernelGGL((wino_input_many_kernel<SET, HALF>), dim3(tbl.n_in), dim3(256), 0, st, tbl);
    hipLaunchKernelGGL((wino_gemm_many_kernel<HALF>), dim3(ceil_div(tbl.n_gemm, 8 * kWinoGroup) * 8 * kWinoGroup), dim3(64 * kWinoItemWaves),
                       (size_t)kWinoItemWaves * 32 * 64 * sizeof(float), st, tbl);
    hipLaunchKernelGGL((wino_output_many_kernel<SET, HALF>), dim3(tbl.n_out), dim3(256), 0, st, tbl);
}

// Layers [0, n) of one Winograd kind and storage type (n <= kMaxWinoLayers, all of them with a
// workspace) in three launches; ws[i] is layer i's own region of wino_workspace_bytes.
hipError_t launch_wino_many(int n, const Geo *geos, int kind, const void *const *x, const void *const *U,
                            const float *const *bias, void *const *y, void *const *ws, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (n > kMaxWinoLayers) return hipErrorInvalidValue;
    const bool half = geos[0].dtype == NNV_F16;
    WinoTable tbl{};
    long n_in = 0, n_gemm = 0, n_out = 0;
    WinoPlan plans[kMaxWinoLayers];
    int order[kMaxWinoLayers];
    long mfmas[kMaxWinoLayers];
    for (int i = 0; i < n; ++i) {
        if ((geos[i].dtype == NNV_F16) != half || !wino_many_supported(geos[i], kind)) return hipErrorInvalidValue;
        plans[i] = plan_wino(geos[i], kind);
        order[i] = i;
    }
    int shifts[kMaxWinoLayers], runs[kMaxWinoLayers];
    const long per_simd = wino_many_split(n, plans, kind, half, mfmas, shifts, runs);
    // Longest first, except in float32 F(4x4) and F(6x6) launches of fewer than 2000 instructions per SIMD: they are bound by
    // U, and deep layers first put all of it in front of the arithmetic.  Same 110 launches, sorted against not, geometric means: F(2x2)
    // 0.99 (0.94-1.05), F(4x4) and F(6x6) below the line 1.01 (0.93-1.07), beyond it 0.98 (0.96-1.03).  float16: 0.98 (0.91-1.03).
    if (half || kind == NNV_WINO_F2 || per_simd >= 2000)
        std::stable_sort(order, order + n, [&](int a, int b) { return (mfmas[a] >> shifts[a]) > (mfmas[b] >> shifts[b]); });
    for (int o = 0; o < n; ++o) {
        const int i = order[o];
        const WinoPlan &p = plans[i];
        WinoParams &w = tbl.layer[o];
        w = wino_params(geos[i], p, x[i], U[i], bias ? bias[i] : nullptr, y[i], ws[i]);
        const int tm = wino_tm(p, half);
        w.ks_shift = shifts[i];
        w.gemm_wgs_per_xi = ceil_div(p.K16, tm) * ceil_div(p.nblk, runs[i]);
        tbl.tm[o] = tm;
        tbl.run[o] = runs[i];
        tbl.in_by[o] = half ? p.tn * (p.cpad / 16) : ceil_div(p.cpad * 16 * p.tn, 256);
        tbl.in0[o] = (int)n_in; tbl.gemm0[o] = (int)n_gemm; tbl.out0[o] = (int)n_out;
        n_in += (long)p.nblk * tbl.in_by[o];
        n_gemm += ceil_div(w.alpha2 * w.gemm_wgs_per_xi, kWinoItemWaves >> w.ks_shift);
        n_out += ((long)geos[i].k * p.Tpad + 255) / 256;
        if (n_in >= (1L << 30) || n_gemm >= (1L << 30) || n_out >= (1L << 30)) return hipErrorInvalidValue;
    }
    for (int i = n; i < kMaxWinoLayers; ++i) tbl.in0[i] = tbl.gemm0[i] = tbl.out0[i] = INT_MAX;
    tbl.n_in = (int)n_in; tbl.n_gemm = (int)n_gemm; tbl.n_out = (int)n_out;
    const int set = wino_set(kind, geos[0].dtype);
    if (set == WS_F2) { if (half) launch_wino_many_t<0, true>(tbl, st); else launch_wino_many_t<0, false>(tbl, st); }
    else if (set == WS_F4) launch_wino_many_t<1, false>(tbl, st);
    else if (set == WS_F6) launch_wino_many_t<3, false>(tbl, st);
    else launch_wino_many_t<2, true>(tbl, st);
    return hipGetLastError();
}

// Layers [0, n) on the fused route, of one kind (n <= kMaxWinoLayers), in one launch; the layers of the longest workgroups first.
hipError_t launch_wino_fused(int n, const Geo *geos, int kind, const void *const *x, const void *const *U, const float *const *bias, void *const *y, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (n > kMaxWinoLayers) return hipErrorInvalidValue;
    WinoFusedTable tbl{};
    int order[kMaxWinoLayers];
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order, order + n, [&](int a, int b) { return geos[a].c > geos[b].c; });
    const int set = kind == NNV_WINO_F2 ? 0 : 1;
    WinoPlan plans[kMaxWinoLayers];
    long all[kWinoForms] = {};
    for (int i = 0; i < n; ++i) {
        plans[i] = plan_wino(geos[i], kind);
        for (int f = 0; f < kWinoForms; ++f) all[f] += wino_form_blocks(plans[i], kWinoForm[set][f]);
    }
    const WinoForm form = kWinoForm[set][wino_form(all)];
    const int tn = form.tn;
    if (n == 1 && form.most == 4 && wino_waves(kind, plans[0])) {
        WinoParams w = wino_params(geos[0], plans[0], x[0], U[0], bias ? bias[0] : nullptr, y[0], nullptr);
        w.gemm_wgs_per_xi = plans[0].T16 * ceil_div(plans[0].K16, 4);
        const dim3 grid(xcd_grid(w.gemm_wgs_per_xi));
        if (kind == NNV_WINO_F2) hipLaunchKernelGGL((wino_wave_kernel<0>), grid, dim3(256), 0, st, w);
        else hipLaunchKernelGGL((wino_wave_kernel<1>), grid, dim3(256), 0, st, w);
        return hipGetLastError();
    }
    long blocks = 0;
    for (int o = 0; o < n; ++o) {
        const int i = order[o];
        if (!wino_fused_able(geos[i], kind)) return hipErrorInvalidValue;
        tbl.layer[o] = wino_params(geos[i], plans[i], x[i], U[i], bias ? bias[i] : nullptr, y[i], nullptr);
        tbl.tm[o] = wino_fused_panels(plans[i], form.most);
        tbl.block0[o] = (int)blocks;
        blocks += wino_form_blocks(plans[i], form);
        if (blocks >= (1L << 30)) return hipErrorInvalidValue;
    }
    for (int i = n; i < kMaxWinoLayers; ++i) tbl.block0[i] = INT_MAX;
    tbl.n = (int)blocks;
    const dim3 grid((unsigned)(((blocks + 8 * kWinoGroup - 1) / (8 * kWinoGroup)) * 8 * kWinoGroup));
    const auto is_wide = [](const Geo &g) { return g.pw == 1; };
    const bool all_wide = std::all_of(geos, geos + n, is_wide), some_wide = std::any_of(geos, geos + n, is_wide);
#define NNV_WINO_FUSED(SET, TN, WIDE) hipLaunchKernelGGL((wino_fused_kernel<SET, TN, WIDE>), grid, dim3(wino_fused_threads(SET)), 0, st, tbl)
#define NNV_WINO_FUSED_OF(SET, TN) { if (all_wide) NNV_WINO_FUSED(SET, TN, 1); else if (some_wide) NNV_WINO_FUSED(SET, TN, 2); else NNV_WINO_FUSED(SET, TN, 0); }
    if (kind == NNV_WINO_F4) NNV_WINO_FUSED_OF(1, 1)
    else if (tn == 2) NNV_WINO_FUSED_OF(0, 2)
    else NNV_WINO_FUSED_OF(0, 1)
#undef NNV_WINO_FUSED_OF
#undef NNV_WINO_FUSED
    return hipGetLastError();
}

hipError_t launch_wino(const Geo &g, int kind, const void *x, const void *U, const float *bias, void *y, void *ws,
                       hipStream_t st) {
    const WinoPlan p = plan_wino(g, kind);
    char fused = 0;
    wino_fused_layers(1, &g, kind, &fused);
    if (fused) return launch_wino_fused(1, &g, kind, &x, &U, &bias, &y, st);
    if (p.T16 > kWinoMostT16 || p.K16 > 65535) return hipErrorInvalidValue;
    WinoParams w = wino_params(g, p, x, U, bias, y, ws);
    const int set = wino_set(kind, g.dtype);
    if (set == WS_F2) {
        if (g.dtype == NNV_F16) return launch_wino_t<0, true>(g, p, w, st);
        return launch_wino_t<0, false>(g, p, w, st);
    }
    if (set == WS_F4) return launch_wino_t<1, false>(g, p, w, st);
    if (set == WS_F6) return launch_wino_t<3, false>(g, p, w, st);
    return launch_wino_t<2, true>(g, p, w, st);
}

}  // namespace nnv
