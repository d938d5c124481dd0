// Work items of whole workgroups (included by gemm.hip): float32 3x3 layers at stride 1 on the bfloat16 matrix cores; float16 3x3, 1x1 and few-channel
// layers (further down).
//
// float32.  What bounds the single-wavefront items of gemm.hip on such layers is the float32 matrix pipe (a 16x16x4 product runs 32
// cycles for 1024 FMAs, a bfloat16 16x16x32 one 16 cycles for 8192) and the vector memory path of a CU, which every operand
// fragment passes once per wavefront and filter tap.  Here
//   * a float32 is the exact sum of three bfloat16 (8 + 8 + 8 significant bits, each rounded to nearest), x = h + m + l,
//     and a product of two of them eight bfloat16 products: h h' + (h m' + m h') + (m m' + h l' + l h') + (m l' + l m'); l l', what is left
//     out, is at most 2^-34 of the product, a thousandth of what rounding the product to float32 takes.  h h' and the small terms have an accumulator each,
//     so a long sum rounds its large part once per 32 channels and tap instead of once per channel.  Sums of one product, 115 million of them: at
//     most 5.99e-8 of it away from it, a float32 product 5.96e-8 (with six products, m l' and l m' left out, 1.09e-7).  Relative 2-norm of the error against float64, random
//     data, this / one chain of float32 products: 3.7e-8 / 1.0e-7 over 32 terms, 1.3e-7 / 4.4e-7 over 576, 4.1e-7 / 1.2e-6
//     over 4608.  The matrix unit takes bfloat16 below 2^-126 for zero, so both operands are taken times 2^23 and the sums times 2^-46:
//     a part of any float32, being a multiple of 2^-149, is then zero or at least 2^-126, and what products lose is below 2^-172 each, no sum of
//     which a float32 shows.  Operands that bfloat16 cannot hold (infinite, NaN, from 2^105 on) and sums from 2^82 on leave a scaled sum that
//     is not finite: a workgroup that finds one computes its tile once more with float32 products (tile_accumulate_float; us a call with
//     ordinary values / one infinite pixel / every sum not finite: 256 channels at 8x56x56 165 / 285 / 405, 512 at 4x28x28 112 / 270 / 270, 64 at 224x224
//     38 / 45 / 93; each wavefront for itself, its operands straight from memory, took 480 / 605, 1290 / 1290 and 75 / 140).
//   * the four wavefronts of a workgroup share the pixels of a tile: 32 channels of the patch of x are split once, laid
//     down in LDS and read by all wavefronts and all filter taps; each wavefront reads and splits the weights of its own
//     output channels only.
// What bounds it now: large layers the power limit (256 channels at 8x56x56 take 20 % less time when the pixels are zeros),
// small launches the issue of vector instructions beside the products (a 16x16x32 product leaves room for one, splitting
// takes one for each) and 5 us of an item before its first and after its last product.  Measured, us a call with weights and pixels from HBM,
// single-wavefront kernels -> this: 256 channels at 8x56x56 253 -> 177 (165 in a row of calls, 179 TFLOP/s), 512 at 4x28x28 156 -> 125, 128 at 112x112
// 44.7 -> 33.2, 64 at 224x224 44.7 -> 40.7; VGG-16-shaped stack 296 -> 197, ResNet-50 106 -> 98, ResNet-18 56 -> 48.5, AlexNet 43 -> 34.  (32x32x16 products
// leave room for four vector instructions, but blocks of 32 pixels fill a row of 28 or 56 worse: 256 channels at 8x56x56 with six products 156 against 134.
// 1x1 layers lose: a chunk of theirs is one tap, over before the next chunk has arrived.)
//
// Patch in LDS: [part h, m, l][channel slot c % 4][pixel][8 channels], 16 bytes per pixel and slot, so that the 16
// pixels of a fragment are 256 consecutive bytes.  The eight channels of slot s are s, s + 4, .., s + 28: what a lane of
// that slot finds in eight consecutive fragments of the packed weights.  DOUBLE: two
// buffers, the next 32 channels are fetched, split and written beside the products of these (two workgroups per CU); else one
// buffer, and the two other workgroups of the CU work meanwhile.
// A wavefront: TM panels of 16 output channels x TN blocks of 16 pixels.  The pixels of a tile are th x tw outputs of one image.

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kTilePatch = 192;                                // pixels of a patch, at most: 64 per filter row
constexpr int kTileBuffer = 12 * kTilePatch * 16;              // bytes of its 3 parts x 4 slots
constexpr int kTilePatch2 = 320;                               // pixels of a float16 patch at stride 2
constexpr int kTileChannels = 32;                              // channels of a chunk

struct TileLayer {
    const void *x, *wp;
    const float *bias;
    void *y;
    int N, C, H, W, K, P, Q, pad;
    int st;                               // 3x3 filters: stride (float32: 1)
    int R, S, sh, sw, padw;               // the other filters
    int K16, cblocks;
    int th, tw, nth, ntw;                 // outputs of a tile, tiles per image
    int relu;
};

// Both operands are taken times 2^23, the sums times 2^-46: whatever part of a float32 is not zero is then at least 2^-126.
constexpr float kTileScale = 0x1p23f, kTileUnscale = 0x1p-46f;

__device__ __forceinline__ void bf3_split(const float x, const float y, uint32_t &h, uint32_t &m, uint32_t &l) {
    const float a = x * kTileScale, b = y * kTileScale;
    // (the empty statements keep the compiler from converting a second time for the value it shifts out)
    const bf16x2 hp = {(__bf16)a, (__bf16)b};
    h = __builtin_bit_cast(uint32_t, hp);
    asm("" : "+v"(h));
    const float ra = a - __builtin_bit_cast(float, h << 16), rb = b - __builtin_bit_cast(float, h & 0xffff0000u);
    const bf16x2 mp = {(__bf16)ra, (__bf16)rb};
    m = __builtin_bit_cast(uint32_t, mp);
    asm("" : "+v"(m));
    const float sa = ra - __builtin_bit_cast(float, m << 16), sb = rb - __builtin_bit_cast(float, m & 0xffff0000u);
    const bf16x2 lp = {(__bf16)sa, (__bf16)sb};
    l = __builtin_bit_cast(uint32_t, lp);
}

// n / d for 0 <= n <= 256 and 1 <= d <= 256 (n d < 2^16): exact.
struct SmallDiv {
    uint32_t magic;
    __device__ __forceinline__ explicit SmallDiv(int d) : magic(65536u / (uint32_t)d + 1u) {}
    __device__ __forceinline__ int operator()(int n) const { return (int)(((uint32_t)n * magic) >> 16); }
};

// Position of a tile: image, first output row and column, first panel of the wavefront.
struct TilePos { int img, p0, q0, mb0; };

// Offset of output pixel n of the tile in a plane of y, or -1.
__device__ __forceinline__ int tile_out_pixel(const TileLayer &g, const TilePos &at, const SmallDiv &by_tw, const int n) {
    const int r = by_tw(n), c = n - r * g.tw, p = at.p0 + r, q = at.q0 + c;
    return r < g.th && p < g.P && q < g.Q ? p * g.Q + q : -1;
}

// acc + acs = the tile's sums over the channel chunks [c0, c1).  All four wavefronts call it with the same tile and range.
template <int TM, int TN, bool DOUBLE>
__device__ __forceinline__ void tile_accumulate(const TileLayer &g, const TilePos &at, const int c0, const int c1, char *lds,
                                                floatx4 (&acc)[TM][TN], floatx4 (&acs)[TM][TN]) {
    constexpr int NT = kTilePatch / 64;                         // staging tasks of a wavefront: 64 pixels x 8 channels
    static_assert(NT == 3, "a task per filter row");
    constexpr uint32_t SUB = kTilePatch * 16, PART = 4 * SUB;
    const int lane = threadIdx.x & 63, col = lane & 15, slot = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pw = g.tw + 2, npatch = pw * (g.th + 2);
    const SmallDiv by_pw(pw), by_tw(g.tw);
    const int HW = g.H * g.W;

    // ---- staging: wavefront w fetches the channels w, w + 4, .. of pixel 64 j + lane
    uint32_t sv[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int f = j * 64 + lane, r = by_pw(f), c = f - r * pw;
        const int ih = at.p0 - g.pad + r, iw = at.q0 - g.pad + c;
        const bool ok = f < npatch && (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
        sv[j] = ok ? (uint32_t)((at.img * g.C + wave) * HW + ih * g.W + iw) * 4u : kOobOffset;
    }
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, (uint32_t)(g.N * g.C) * (uint32_t)HW * 4u);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, (uint32_t)g.K16 * (uint32_t)g.cblocks * (9 * 256u));
    const uint32_t cb_stride = (uint32_t)HW * 16u;
    auto fetch = [&](float (&v)[8], const uint32_t pix, const int chunk) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int cb = chunk * 8 + i;
            const bool ok = cb * 4 + wave < g.C;                 // uniform
            v[i] = buf_load<float>(xres, ok ? pix : kOobOffset, ok ? (uint32_t)cb * cb_stride : 0u);
        }
    };
    auto put = [&](const float (&v)[8], const int j, const uint32_t buf) __attribute__((always_inline)) {
        u32x4_t h, m, l;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t a, b, c;
            bf3_split(v[2 * i], v[2 * i + 1], a, b, c);
            h[i] = a; m[i] = b; l[i] = c;
        }
        char *o = lds + buf + wave * SUB + (j * 64 + lane) * 16;
        *reinterpret_cast<u32x4_t *>(o) = h;
        *reinterpret_cast<u32x4_t *>(o + PART) = m;
        *reinterpret_cast<u32x4_t *>(o + 2 * PART) = l;
    };
    // ---- pixels of the lane's columns (columns past the tile read pixel 0 and are not stored)
    uint32_t baddr[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int n = t * 16 + col, r = by_tw(n), c = n - r * g.tw;
        baddr[t] = (uint32_t)slot * SUB + (r < g.th ? (uint32_t)(r * pw + c) * 16u : 0u);
    }
    // ---- weights: TM consecutive floats per lane, rows dealt out as in gemm_a_offset
    constexpr int QM = 16 / TM;
    const uint32_t a_voff = at.mb0 + col / QM < g.K16
        ? (uint32_t)(col / QM) * (uint32_t)g.cblocks * (9 * 256u) + (uint32_t)slot * 64u + (uint32_t)(col % QM) * (4u * TM) : kOobOffset;
    const uint32_t a_base = (uint32_t)at.mb0 * (uint32_t)g.cblocks * 9u;
    typename FloatVec<TM>::type araw[8];
    // the weights of tap (row, s) of a chunk (channel blocks past the last read the last one again: the pixels of those
    // channels are zeros)
    auto load_a = [&](const int chunk, const int row, const int s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int cb = min(chunk * 8 + i, g.cblocks - 1);
            araw[i] = buf_load_floats<TM>(wres, a_voff + s * 256u, (a_base + (uint32_t)(cb * 9 + row * 3)) * 256u);
        }
    };
    struct Parts { u32x4_t h, m, l; };
    Parts af[2][TM], bf[2];
    auto split_a = [&](const int set, const int q) __attribute__((always_inline)) {
        const int m = q >> 2, i = q & 3;
        uint32_t h, mm, l;
        bf3_split(float_of<TM>(araw[2 * i], m), float_of<TM>(araw[2 * i + 1], m), h, mm, l);
        af[set][m].h[i] = h; af[set][m].m[i] = mm; af[set][m].l[i] = l;
    };
    auto read_b = [&](const int set, const int t, const uint32_t off, const int s) __attribute__((always_inline)) {
        const char *b = lds + (baddr[t] + off) + s * 16;
        bf[set].h = *reinterpret_cast<const u32x4_t *>(b);
        bf[set].m = *reinterpret_cast<const u32x4_t *>(b + PART);
        bf[set].l = *reinterpret_cast<const u32x4_t *>(b + 2 * PART);
    };
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[m][t] = acs[m][t] = floatx4{0.f, 0.f, 0.f, 0.f};

    // ---- first chunk, first two taps of the weights
    {
        float v[NT][8];
        load_a(c0, 0, 0);
#pragma unroll
        for (int j = 0; j < NT; ++j) fetch(v[j], sv[j], c0);
#pragma unroll
        for (int q = 0; q < 4 * TM; ++q) split_a(0, q);
        load_a(c0, 0, 1);
#pragma unroll
        for (int j = 0; j < NT; ++j) put(v[j], j, 0);
    }
    __syncthreads();

    __builtin_amdgcn_s_setprio(0);
    float st[8];
    uint32_t cur = 0;
    int ch = c0, row = 0;
    bool turned = true;
    for (int it = (c1 - c0) * 3; it > 0; --it) {
        // one filter row of a chunk: three taps of TN blocks
        const bool turn = row == 2;
        const int nx = min(ch + 1, c1 - 1), nch = turn ? nx : ch, nrow = turn ? 0 : row + 1;
        const uint32_t off = cur + (uint32_t)(row * pw) * 16u, noff = turn ? off : off + (uint32_t)pw * 16u;
        if (turned) read_b(0, 0, off, 0);
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const int sa = s & 1;
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                const int e = s * TN + t, sb = e & 1;
                __builtin_amdgcn_sched_barrier(0);
                if (e + 1 < 3 * TN) read_b(sb ^ 1, (e + 1) % TN, off, (e + 1) / TN);
                else read_b(sb ^ 1, 0, noff, 0);        // the next row's first block (after the last row: not used)
                __builtin_amdgcn_sched_barrier(0);
                // the next tap's weights are split beside this tap's first products, then those of the tap after it requested
#pragma unroll
                for (int q = t * TM; q < (t + 1) * TM && q < 4 * TM; ++q) split_a(sa ^ 1, q);
                if (t == (TN > 4 ? 4 : 3)) {
                    if (s == 0) load_a(ch, row, 2);
                    else load_a(nch, nrow, s - 1);
                }
                // the next chunk's patch: a task per filter row (after the last chunk the last one again, unread)
                if constexpr (DOUBLE) {
                    if (s == 0 && t == TN - 1) {
                        uint32_t pix = sv[0];
#pragma unroll
                        for (int r = 1; r < NT; ++r) pix = row == r ? sv[r] : pix;
                        fetch(st, pix, nx);
                    }
                    if (s == 2 && t == TN - 2) put(st, row, cur ^ (uint32_t)kTileBuffer);
                }
#define NNV_BF(X) __builtin_bit_cast(bf16x8, X)
#define NNV_TILE_MFMA(X, Y, Z) \
    _Pragma("unroll") for (int m = 0; m < TM; ++m) Z[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(NNV_BF(af[sa][m].X), NNV_BF(bf[sb].Y), Z[m][t], 0, 0, 0);
                NNV_TILE_MFMA(l, m, acs) NNV_TILE_MFMA(m, l, acs) NNV_TILE_MFMA(l, h, acs) NNV_TILE_MFMA(h, h, acc)
                NNV_TILE_MFMA(m, h, acs) NNV_TILE_MFMA(m, m, acs) NNV_TILE_MFMA(h, m, acs) NNV_TILE_MFMA(h, l, acs)
#undef NNV_TILE_MFMA
#undef NNV_BF
                // (vector instructions dealt out over the products)
#pragma unroll
                for (int i = 0; i < 8 * TM; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // (three taps: the next row starts with the first of the two sets again)
#pragma unroll
        for (int m = 0; m < TM; ++m) af[0][m] = af[1][m];
        if (TN & 1) bf[0] = bf[1];
        if (turn) {
            if constexpr (DOUBLE) cur ^= (uint32_t)kTileBuffer;
            else if (ch + 1 < c1) {
                float v[NT][8];
#pragma unroll
                for (int j = 0; j < NT; ++j) fetch(v[j], sv[j], ch + 1);
                __syncthreads();        // all have read this chunk
#pragma unroll
                for (int j = 0; j < NT; ++j) put(v[j], j, 0);
            }
            __syncthreads();
        }
        turned = turn;
        ch = turn ? ch + 1 : ch;
        row = nrow;
    }
}

// The same sums with float32 products, for tiles whose sums are not finite.  All four wavefronts call it with the same tile and range,
// and none reads lds any more.  The patch of a chunk is laid down as it is, [slot][pixel][8 channels].
template <int TM, int TN>
__device__ __forceinline__ void tile_accumulate_float(const TileLayer &g, const TilePos &at, const int c0, const int c1, char *lds, floatx4 (&acc)[TM][TN]) {
    constexpr int NT = kTilePatch / 64, QM = 16 / TM;
    constexpr uint32_t SUB = kTilePatch * 32;
    static_assert(4 * SUB <= kTileBuffer, "the patch fits");
    const int lane = threadIdx.x & 63, col = lane & 15, slot = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pw = g.tw + 2, npatch = pw * (g.th + 2), HW = g.H * g.W;
    const SmallDiv by_pw(pw), by_tw(g.tw);
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, (uint32_t)(g.N * g.C) * (uint32_t)HW * 4u);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, (uint32_t)g.K16 * (uint32_t)g.cblocks * (9 * 256u));
    const uint32_t a_voff = at.mb0 + col / QM < g.K16
        ? (uint32_t)(col / QM) * (uint32_t)g.cblocks * (9 * 256u) + (uint32_t)slot * 64u + (uint32_t)(col % QM) * (4u * TM) : kOobOffset;
    const uint32_t a_base = (uint32_t)at.mb0 * (uint32_t)g.cblocks * 9u;
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[m][t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int ch = c0; ch < c1; ++ch) {
        __syncthreads();            // all have read the chunk before
#pragma unroll 1
        for (int j = 0; j < NT; ++j) {
            const int f = j * 64 + lane, r = by_pw(f), c = f - r * pw;
            const int ih = at.p0 - g.pad + r, iw = at.q0 - g.pad + c;
            const bool in = f < npatch && (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
            floatx4 v[2];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int cc = (ch * 8 + i) * 4 + wave;
                v[i >> 2][i & 3] = buf_load<float>(xres, in && cc < g.C ? (uint32_t)((at.img * g.C + cc) * HW + ih * g.W + iw) * 4u : kOobOffset, 0u);
            }
            floatx4 *o = reinterpret_cast<floatx4 *>(lds + wave * SUB + f * 32);
            o[0] = v[0];
            o[1] = v[1];
        }
        __syncthreads();
#pragma unroll 1
        for (int row = 0; row < 3; ++row) {
            typename FloatVec<TM>::type a[3][8];
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int cb = ch * 8 + i;          // past the last channel block: zeros, as its pixels are
                    a[s][i] = buf_load_floats<TM>(wres, cb < g.cblocks ? a_voff : kOobOffset, (a_base + (uint32_t)(min(cb, g.cblocks - 1) * 9 + row * 3 + s)) * 256u);
                }
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                const int n = t * 16 + col, r = by_tw(n), c = n - r * g.tw;
                const char *pix = lds + slot * SUB + (r < g.th ? ((r + row) * pw + c) * 32 : 0);
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    const floatx4 b[2] = {reinterpret_cast<const floatx4 *>(pix + s * 32)[0], reinterpret_cast<const floatx4 *>(pix + s * 32)[1]};
#pragma unroll
                    for (int i = 0; i < 8; ++i)
#pragma unroll
                        for (int m = 0; m < TM; ++m)
                            acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(float_of<TM>(a[s][i], m), b[i >> 2][i & 3], acc[m][t], 0, 0, 0);
                }
            }
        }
    }
}

// ---- float16 3x3 filters: the same tiles.  What bounds the single-wavefront items is the vector memory path of a CU: every wavefront fetches its
// pixels once per tap (2 fragments of weights and 2 of pixels for 4 products) from a copy of x in octets of channels that a launch in front
// has to make.  Here the patch of 32 channels is read once per workgroup, straight from NCHW, the weights' fragments as they are packed (16 bytes
// per lane: channels 8 slot .. + 7), nine taps of them on their way at a time.  Beside the products: LDS (a fragment of pixels takes 8 cycles, TM products 16 TM of
// four SIMDs; with TM = 1 both take as long), 8 NT + 9 TM requests and, at the end of a chunk, NT writes of a patch that has two buffers.
// Measured, us a call, single-wavefront items -> this: 256 channels at 8x56x56 76 -> 39 (1.5 PFLOP/s), 512 at 4x28x28 66 -> 27, 64 at 224x224 22 -> 16, VGG-16-shaped
// stack 92 -> 59; with the other two kinds of items below ResNet-50 54 -> 42, ResNet-18 38 -> 23.
// NT tasks of 64 pixels: 3 at stride 1, 5 at stride 2.
template <int TM, int TN, int NT>
__device__ __forceinline__ void tile_accumulate_half(const TileLayer &g, const TilePos &at, const int c0, const int c1, char *lds, floatx4 (&acc)[TM][TN]) {
    constexpr uint32_t SUB = NT * 64 * 16, BUFFER = 4 * SUB;
    const int lane = threadIdx.x & 63, col = lane & 15, slot = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pw = (g.tw - 1) * g.st + 3, npatch = pw * ((g.th - 1) * g.st + 3);
    const SmallDiv by_pw(pw), by_tw(g.tw);
    const int HW = g.H * g.W;
    // staging: wavefront w fetches the channels 8 w .. + 7 of pixel 64 j + lane
    uint32_t sv[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int f = j * 64 + lane, r = NT == 3 ? by_pw(f) : f / pw, c = f - r * pw;
        const int ih = at.p0 * g.st - g.pad + r, iw = at.q0 * g.st - g.pad + c;
        const bool ok = f < npatch && (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
        sv[j] = ok ? (uint32_t)((at.img * g.C + wave * 8) * HW + ih * g.W + iw) * 2u : kOobOffset;
    }
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, (uint32_t)(g.N * g.C) * (uint32_t)HW * 2u);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, (uint32_t)g.K16 * (uint32_t)g.cblocks * (9 * 1024u));
    const uint32_t plane = (uint32_t)HW * 2u;
    uint32_t st[NT][8];
    auto fetch = [&](const int j, const int i, const int chunk) __attribute__((always_inline)) {
        const bool ok = chunk * 32 + wave * 8 + i < g.C;         // uniform
        st[j][i] = __builtin_amdgcn_raw_buffer_load_b16(xres, ok ? sv[j] : kOobOffset, ok ? (uint32_t)(chunk * 32 + i) * plane : 0u, 0);
    };
    auto put = [&](uint32_t (&v)[8], const int j, const uint32_t buf) __attribute__((always_inline)) {
        u32x4_t o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // (the empty statement keeps the compiler from packing, and so waiting for, the values where they are requested)
            asm volatile("" : "+v"(v[2 * i]), "+v"(v[2 * i + 1]));
            o[i] = __builtin_amdgcn_perm(v[2 * i + 1], v[2 * i], 0x05040100u);
        }
        *reinterpret_cast<u32x4_t *>(lds + buf + wave * SUB + (j * 64 + lane) * 16) = o;
    };
    uint32_t baddr[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int n = t * 16 + col, r = by_tw(n), c = n - r * g.tw;
        baddr[t] = (uint32_t)slot * SUB + (r < g.th ? (uint32_t)(r * g.st * pw + c * g.st) * 16u : 0u);
    }
    uint32_t a_voff[TM], a_base[TM];
#pragma unroll
    for (int m = 0; m < TM; ++m) {
        const bool ok = at.mb0 + m < g.K16;
        a_voff[m] = ok ? (uint32_t)lane * 16u : kOobOffset;
        a_base[m] = ok ? (uint32_t)(at.mb0 + m) * (uint32_t)g.cblocks * 9u : 0u;
    }
    constexpr int NB = TM == 1 ? 8 : 6;                        // blocks of pixels on their way from LDS
    half8 a[9][TM], b[NB];
    auto load_a = [&](const int rs, const int chunk) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < TM; ++m) a[rs][m] = buf_load<half8>(wres, a_voff[m] + rs % 3 * 1024u, (a_base[m] + (uint32_t)(chunk * 9 + rs / 3 * 3)) * 1024u);
    };
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[m][t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < 8; ++i) fetch(j, i, c0);
#pragma unroll
    for (int rs = 0; rs < 9; ++rs) load_a(rs, c0);
#pragma unroll
    for (int j = 0; j < NT; ++j) put(st[j], j, 0);
    __syncthreads();
    __builtin_amdgcn_s_setprio(0);
    uint32_t cur = 0;
    // a chunk; MORE: the next one's patch is requested at its start and laid down at its end, its weights tap by tap as these are done
    auto chunk_of = [&](auto more, const int ch) __attribute__((always_inline)) {
        constexpr bool MORE = decltype(more)::value;
        uint32_t off[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) off[r] = cur + (uint32_t)(r * pw) * 16u;
        auto read_b = [&](const int e) __attribute__((always_inline)) {
            const int rs = e / TN, t = e % TN;
            if (e < 9 * TN) b[e % NB] = *reinterpret_cast<const half8 *>(lds + (baddr[t] + off[rs / 3]) + rs % 3 * 16);
        };
#pragma unroll
        for (int e = 0; e + 1 < NB; ++e) read_b(e);
#pragma unroll
        for (int e = 0; e < 9 * TN; ++e) {
            read_b(e + NB - 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < TM; ++m) acc[m][e % TN] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[e / TN][m], b[e % NB], acc[m][e % TN], 0, 0, 0);
            if (MORE) {
                // (one or two requests at a time, beside the products: 24 in a row held these up by 0.7 us)
                constexpr int STEPS = NT == 3 ? 6 * TN : 9 * TN;        // over the first two filter rows, or all
#pragma unroll
                for (int f = e * 8 * NT / STEPS; f < (e + 1) * 8 * NT / STEPS && f < 8 * NT; ++f) fetch(f / 8, f % 8, ch + 1);
                if (e % TN == TN - 1) load_a(e / TN, ch + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (MORE) {
            cur ^= BUFFER;
#pragma unroll
            for (int j = 0; j < NT; ++j) put(st[j], j, cur);
            __syncthreads();
        }
    };
#pragma unroll 1
    for (int ch = c0; ch + 1 < c1; ++ch) chunk_of(std::true_type{}, ch);
    chunk_of(std::false_type{}, c1 - 1);
}

// Bias, clamp and store; off: offsets of the lane's pixels in channel 0 of their image, or out of range.  PAIRS: blocks 2 i and 2 i + 1
// hold neighbouring pixels of an even number (one_pixel).
template <bool HALF, int TM, int TN, bool PAIRS = false>
__device__ __forceinline__ void tile_store(const TileLayer &g, const int mb0, const int slot, const uint32_t (&off)[TN], const floatx4 (&acc)[TM][TN]) {
    constexpr uint32_t ESZ = HALF ? 2u : 4u;
    const int PQ = g.P * g.Q;
    const __amdgpu_buffer_rsrc_t yres = make_rsrc(g.y, (uint32_t)(g.N * g.K) * (uint32_t)PQ * ESZ);
    const __amdgpu_buffer_rsrc_t bres = make_rsrc(g.bias, g.bias ? (uint32_t)g.K * 4u : 0u);
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = mb0 * 16 + gemm_row(!HALF, TM, m, slot, j);
            const bool ok = k < g.K;
            const float bv = buf_load<float>(bres, ok ? (uint32_t)k * 4u : kOobOffset, 0u);
            const uint32_t base = (uint32_t)(k * PQ) * ESZ;
            if constexpr (PAIRS) {
#pragma unroll
                for (int t = 0; t + 1 < TN; t += 2)
                    gemm_store_pair(yres, g.relu, ok && off[t] != kOobOffset ? base + off[t] : kOobOffset, bv, acc[m][t][j], acc[m][t + 1][j]);
            }
#pragma unroll
            for (int t = PAIRS ? TN & ~1 : 0; t < TN; ++t)
                gemm_store(yres, g.relu, HALF, ok && off[t] != kOobOffset ? base + off[t] : kOobOffset, bv, acc[m][t][j]);
        }
}

// Pixel of a 1x1 item's tile that column col of block t holds: with pairs, those of two blocks alternate, and so do the halves of a last one.
__device__ __forceinline__ int one_pixel(const bool pairs, const int tn, const int t, const int col) {
    if (!pairs) return t * 16 + col;
    return t == tn - 1 && (tn & 1) ? t * 16 + (col & 7) * 2 + (col >> 3) : (t >> 1) * 32 + col * 2 + (t & 1);
}

// Offset of pixel n of a float16 layer in channel 0 of its image, or out of range.
__device__ __forceinline__ uint32_t one_out_offset(const TileLayer &g, const int n) {
    const int PQ = g.P * g.Q;
    if (n >= g.N * PQ) return kOobOffset;
    const int img = n / PQ;
    return (uint32_t)(img * g.K * PQ + n - img * PQ) * 2u;
}

// One work item: tile (mt, nt) over the chunks [c0, c1).
template <bool HALF, int TM, int TN, bool DOUBLE, int NT = 3>
__device__ __forceinline__ void tile_item(const TileLayer &g, const int mt, const int nt, const int c0, const int c1, const SplitTile sp, char *lds) {
    const int lane = threadIdx.x & 63, col = lane & 15, slot = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rest = nt / g.ntw, img = rest / g.nth;
    const TilePos at{__builtin_amdgcn_readfirstlane(img), __builtin_amdgcn_readfirstlane((rest - img * g.nth) * g.th),
                     __builtin_amdgcn_readfirstlane((nt - rest * g.ntw) * g.tw), (mt * 4 + wave) * TM};
    floatx4 acc[TM][TN];
    if constexpr (HALF) tile_accumulate_half<TM, TN, NT>(g, at, c0, c1, lds, acc);
    else {
        floatx4 acs[TM][TN];
        tile_accumulate<TM, TN, DOUBLE>(g, at, c0, c1, lds, acc, acs);
        float z = 0.f;                    // NaN if any sum is not finite
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                acc[m][t] += acs[m][t];
#pragma unroll
                for (int j = 0; j < 4; ++j) z = fmaf(acc[m][t][j], 0.f, z);
                acc[m][t] *= kTileUnscale;
            }
        // (a workgroup's wavefronts decide together: the float32 products share the patch as well.  The products end with a barrier, so that
        // lds may be written.)
        int *bad = reinterpret_cast<int *>(lds);
        const bool mine = __ballot(z != 0.f) != 0;
        if (lane == 0) bad[wave] = mine;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(bad[0] | bad[1] | bad[2] | bad[3]) != 0) tile_accumulate_float<TM, TN>(g, at, c0, c1, lds, acc);
    }
    __builtin_amdgcn_s_setprio(3);
    // (tiles of 128 channels are not split; the float16 one's compiler spills 672 bytes per lane if no branch stands between its loop and its stores)
    if constexpr (HALF || TM == 1) {
        if (sp.n > 1 && !split_fold<true, TM, TN>(sp, (uint32_t)wave * (TM * TN * 1024) + (uint32_t)lane * 16u, lds, acc)) return;
    }
    const SmallDiv by_tw(g.tw);
    uint32_t off[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int pix = tile_out_pixel(g, at, by_tw, t * 16 + col);
        off[t] = pix >= 0 ? (uint32_t)(at.img * g.K * (g.P * g.Q) + pix) * (HALF ? 2u : 4u) : kOobOffset;
    }
    tile_store<HALF, TM, TN>(g, at.mb0, slot, off, acc);
}

// ---- float16 1x1 filters, any stride: the wavefronts share the pixels, whose x is gathered from NCHW once per workgroup instead of once per
// wavefront (in pairs, a step of single-wavefront items is 4 fragments of weights and 8 loads of pixels for 8 products; here 2 and 8 for 14).  In the
// ResNet-50-shaped stack they take it from 51 to 42 us, its vector loads from 860 to 640 thousand.  PAIRS: stride 1, no padding and an even plane: two neighbouring pixels per load.  kOneChunks chunks of 32 channels
// are in LDS, the next ones on their way to registers; a chunk is TM TN products only, so that less in flight would wait for memory.
constexpr int kOneChunks = 4;
template <int TM, int TN, bool PAIRS>
__device__ __forceinline__ void one_item(const TileLayer &g, const int mt, const int nt, const int c0, const int c1, const SplitTile sp, char *lds) {
    static_assert(PAIRS ? TN <= 8 : TN <= 4, "a wavefront's 64 lanes cover the pixels");
    constexpr uint32_t SUB = TN * 256, CHUNK = 4 * SUB;
    const int lane = threadIdx.x & 63, col = lane & 15, slot = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = nt * (TN * 16), PQ = g.P * g.Q, npix = g.N * PQ, HW = g.H * g.W, mb0 = (mt * 4 + wave) * TM;
    // wavefront w fetches the channels 8 w .. + 7 of pixel `lane`, or of the pixels 2 lane and 2 lane + 1
    uint32_t sv = kOobOffset;
    {
        const int f = PAIRS ? 2 * lane : lane, n = n0 + f;
        if (f < TN * 16 && n < npix) {
            const int img = n / PQ, pq = n - img * PQ;
            int pix = pq;
            bool ok = true;
            if (!PAIRS) {
                const int p = pq / g.Q, ih = p * g.sh - g.pad, iw = (pq - p * g.Q) * g.sw - g.padw;
                ok = (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
                pix = ih * g.W + iw;
            }
            if (ok) sv = (uint32_t)((img * g.C + wave * 8) * HW + pix) * 2u;
        }
    }
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, (uint32_t)(g.N * g.C) * (uint32_t)HW * 2u);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, (uint32_t)g.K16 * (uint32_t)g.cblocks * 1024u);
    const uint32_t plane = (uint32_t)HW * 2u;
    uint32_t st[kOneChunks][8];
    auto fetch = [&](const int f, const int chunk) __attribute__((always_inline)) {
        const int u = f / 8, i = f % 8, c = (chunk + u) * 32 + i;
        const bool ok = chunk + u < c1 && c + wave * 8 < g.C;     // uniform
        const uint32_t v = ok ? sv : kOobOffset, s = ok ? (uint32_t)c * plane : 0u;
        if constexpr (PAIRS) st[u][i] = __builtin_amdgcn_raw_buffer_load_b32(xres, v, s, 0);
        else st[u][i] = __builtin_amdgcn_raw_buffer_load_b16(xres, v, s, 0);
    };
    auto put = [&]() __attribute__((always_inline)) {
        constexpr int HALF_BLOCK = TN / 2 * 16;         // (first lane of a last block without a partner)
        if (PAIRS && lane >= TN * 8) return;
        char *o = lds + wave * SUB + (PAIRS ? lane + (lane & ~15) : lane) * 16;
        const uint32_t odd = lane < HALF_BLOCK ? 256 : 128;
#pragma unroll
        for (int u = 0; u < kOneChunks; ++u) {
            u32x4_t lo, hi;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                asm volatile("" : "+v"(st[u][2 * i]), "+v"(st[u][2 * i + 1]));
                lo[i] = __builtin_amdgcn_perm(st[u][2 * i + 1], st[u][2 * i], 0x05040100u);
                if (PAIRS) hi[i] = __builtin_amdgcn_perm(st[u][2 * i + 1], st[u][2 * i], 0x07060302u);
            }
            *reinterpret_cast<u32x4_t *>(o + u * CHUNK) = lo;
            if (PAIRS) *reinterpret_cast<u32x4_t *>(o + u * CHUNK + odd) = hi;
        }
    };
    uint32_t a_voff[TM], a_base[TM];
#pragma unroll
    for (int m = 0; m < TM; ++m) {
        const bool ok = mb0 + m < g.K16;
        a_voff[m] = ok ? (uint32_t)lane * 16u : kOobOffset;
        a_base[m] = ok ? (uint32_t)(mb0 + m) * (uint32_t)g.cblocks : 0u;
    }
    half8 a[kOneChunks][TM];
    auto load_a = [&](const int u, const int chunk) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < TM; ++m) a[u][m] = buf_load<half8>(wres, a_voff[m], (a_base[m] + (uint32_t)min(chunk + u, c1 - 1)) * 1024u);
    };
    floatx4 acc[TM][TN];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[m][t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int f = 0; f < 8 * kOneChunks; ++f) fetch(f, c0);
#pragma unroll
    for (int u = 0; u < kOneChunks; ++u) load_a(u, c0);
    const char *bptr = lds + slot * SUB + col * 16;
    auto chunks_of = [&](auto more, const int ch) __attribute__((always_inline)) {
        constexpr bool MORE = decltype(more)::value;
        put();
        __syncthreads();
        if constexpr (MORE) {
#pragma unroll
            for (int f = 0; f < 8 * kOneChunks; ++f) fetch(f, ch + kOneChunks);
        }
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int NB = TM == 1 ? 8 : 4;
        half8 b[NB];
        auto read_b = [&](const int e) __attribute__((always_inline)) {
            if (e < kOneChunks * TN) b[e % NB] = *reinterpret_cast<const half8 *>(bptr + e / TN * CHUNK + e % TN * 256);
        };
#pragma unroll
        for (int e = 0; e + 1 < NB; ++e) read_b(e);
#pragma unroll
        for (int u = 0; u < kOneChunks; ++u) {
            if (!MORE && ch + u >= c1) break;          // uniform
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                read_b(u * TN + t + NB - 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int m = 0; m < TM; ++m) acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[u][m], b[(u * TN + t) % NB], acc[m][t], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (MORE) load_a(u, ch + kOneChunks);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int ch = c0;
#pragma unroll 1
    for (; ch + kOneChunks < c1; ch += kOneChunks) {
        chunks_of(std::true_type{}, ch);
        __syncthreads();        // all have read these
    }
    chunks_of(std::false_type{}, ch);
    __builtin_amdgcn_s_setprio(3);
    if (sp.n > 1 && !split_fold<true, TM, TN>(sp, (uint32_t)wave * (TM * TN * 1024) + (uint32_t)lane * 16u, lds, acc)) return;
    uint32_t off[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) off[t] = one_out_offset(g, n0 + one_pixel(PAIRS, TN, t, col));
    tile_store<true, TM, TN, PAIRS>(g, mb0, slot, off, acc);
}

// ---- float16 layers of up to eight channels (the first of a network): a reduction step is four taps of eight channels.  The patch of a
// tile is laid down once, a pixel's eight channels in 16 bytes, straight from NCHW; the copy in octets of channels was a launch
// of 5 us in front (ResNet-50-shaped stack 48 -> 42 us).  A wavefront: one panel; tap 4 u + slot of a step lies in that slot's lanes.
constexpr int kFewPatch = 2400;                               // pixels, at most; a pixel of zeros behind them
template <int TN>
__device__ __forceinline__ void few_item(const TileLayer &g, const int mt, const int nt, char *lds) {
    constexpr int kRing = 4;
    const int lane = threadIdx.x & 63, col = lane & 15, slot = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rest = __builtin_amdgcn_readfirstlane(nt / g.ntw), img = __builtin_amdgcn_readfirstlane(rest / g.nth);
    const int p0 = (rest - img * g.nth) * g.th, q0 = (nt - rest * g.ntw) * g.tw, mb0 = mt * 4 + wave;
    const int pw = (g.tw - 1) * g.sw + g.S, npatch = pw * ((g.th - 1) * g.sh + g.R), HW = g.H * g.W, RS = g.R * g.S;
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, (uint32_t)(g.N * g.C) * (uint32_t)HW * 2u);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, (uint32_t)g.K16 * (uint32_t)RS * 1024u);
    const bool panel = mb0 < g.K16;                            // uniform
    const uint32_t abase = panel ? (uint32_t)mb0 * (uint32_t)RS * 1024u : 0u;
    half8 a[kRing];
    auto load_a = [&](const int i, const int u) __attribute__((always_inline)) {
        const int tap = u * 4 + slot;
        a[i] = buf_load<half8>(wres, panel && tap < RS ? (uint32_t)(tap * 64 + col) * 16u : kOobOffset, abase);
    };
#pragma unroll
    for (int i = 0; i < kRing; ++i) load_a(i, i);
    for (int f0 = 0; f0 < npatch; f0 += 512) {                 // two pixels of a thread at a time
        uint32_t v[2][8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int f = f0 + h * 256 + (int)threadIdx.x, r = f / pw, c = f - r * pw;
            const int ih = p0 * g.sh - g.pad + r, iw = q0 * g.sw - g.padw + c;
            const bool ok = f < npatch && (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
            const uint32_t vo = ok ? (uint32_t)(img * g.C * HW + ih * g.W + iw) * 2u : kOobOffset;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[h][i] = 0;
                if (i < g.C) v[h][i] = __builtin_amdgcn_raw_buffer_load_b16(xres, vo, (uint32_t)(i * HW) * 2u, 0);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4_t o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_perm(v[h][2 * i + 1], v[h][2 * i], 0x05040100u);
            const int f = f0 + h * 256 + (int)threadIdx.x;
            if (f < npatch) *reinterpret_cast<u32x4_t *>(lds + f * 16) = o;
        }
    }
    if (threadIdx.x == 0) *reinterpret_cast<u32x4_t *>(lds + kFewPatch * 16) = u32x4_t{0u, 0u, 0u, 0u};
    __syncthreads();
    if (!panel) return;                                        // uniform
    __builtin_amdgcn_s_setprio(0);
    const SmallDiv by_tw(g.tw);
    uint32_t baddr[TN], off[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int n = t * 16 + col, r = by_tw(n), c = n - r * g.tw, p = p0 + r, q = q0 + c;
        baddr[t] = r < g.th ? (uint32_t)(r * g.sh * pw + c * g.sw) * 16u : 0u;
        off[t] = r < g.th && p < g.P && q < g.Q ? (uint32_t)(img * g.K * (g.P * g.Q) + p * g.Q + q) * 2u : kOobOffset;
    }
    floatx4 acc[1][TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) acc[0][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    const uint32_t magic = 65536u / (uint32_t)g.S + 1u;        // (tap * magic) >> 16 == tap / S, as in gemm_accumulate_taps
    const int steps = (RS + 3) >> 2;
#pragma unroll 1
    for (int u = 0; u < steps; u += kRing) {
#pragma unroll
        for (int i = 0; i < kRing; ++i) {
            if (u + i >= steps) break;                         // uniform
            const int tap = (u + i) * 4 + slot, r = (int)(((uint32_t)tap * magic) >> 16), s = tap - r * g.S;
            const uint32_t to = (uint32_t)(r * pw + s) * 16u;
            half8 b[TN];
#pragma unroll
            for (int t = 0; t < TN; ++t) b[t] = *reinterpret_cast<const half8 *>(lds + (tap < RS ? baddr[t] + to : kFewPatch * 16u));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < TN; ++t) acc[0][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[i], b[t], acc[0][t], 0, 0, 0);
            load_a(i, u + i + kRing);                          // (past the last tap: nothing)
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __builtin_amdgcn_s_setprio(3);
    tile_store<true, 1, TN>(g, mb0, slot, off, acc);
}
