// Work items of whole workgroups for float32 3x3 layers at stride 1: implicit GEMM on the bfloat16 matrix cores (included by gemm.hip).
//
// What bounds the single-wavefront items of gemm.hip on such layers is the float32 matrix pipe (a 16x16x4 product runs 32
// cycles for 1024 FMAs, a bfloat16 16x16x32 one 16 cycles for 8192) and the vector memory path of a CU, which every operand
// fragment passes once per wavefront and filter tap.  Here
//   * a float32 is the exact sum of three bfloat16 (8 + 8 + 8 significant bits, each rounded to nearest), x = h + m + l,
//     and a product of two of them six bfloat16 products: h h' + (h m' + m h') + (m m' + h l' + l h'); what is left out is
//     at most 2^-23 of the product and of either sign.  h h' and the small terms have an accumulator each, so a long sum rounds its large part
//     once per 32 channels and tap instead of once per channel.  Relative 2-norm of the error against float64, random
//     data, this / one chain of float32 products: 3.7e-8 / 1.0e-7 over 32 terms, 1.3e-7 / 4.4e-7 over 576, 4.1e-7 / 1.2e-6
//     over 4608.  Values that bfloat16 cannot hold (infinite, NaN, rounded up to infinity) leave a sum that is not finite, and
//     parts below 2^-126, which the matrix unit takes for zero, matter only in sums of tiny values: a wavefront that finds a sum
//     not finite, or not zero and below 2^-60, computes its tile once more with float32 products (tile_exact).
//   * the four wavefronts of a workgroup share the pixels of a tile: 32 channels of the patch of x are split once, laid
//     down in LDS and read by all wavefronts and all filter taps; each wavefront reads and splits the weights of its own
//     output channels only.
// What bounds it now: large layers the power limit (256 channels at 8x56x56 take 20 % less time when the pixels are zeros),
// small launches the issue of vector instructions beside the products (a 16x16x32 product leaves room for one, splitting
// takes one for each) and 5 us of an item before its first and after its last product.  Measured, us a call,
// single-wavefront kernels -> this: 256 channels at 8x56x56 252 -> 134 (221 TFLOP/s), 512 at 4x28x28 156 -> 101, 64 at 224x224
// 44.5 -> 35, VGG-16-shaped stack 278 -> 166, ResNet-50 100 -> 85, ResNet-18 50.4 -> 41.6, AlexNet 45 -> 33.  (32x32x16 products
// leave room for four vector instructions, but blocks of 32 pixels fill a row of 28 or 56 worse: 256 channels at 8x56x56 156.
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
constexpr int kTileChannels = 32;                              // channels of a chunk

struct TileLayer {
    const float *x, *wp, *bias;
    float *y;
    int N, C, H, W, K, P, Q, pad;
    int K16, cblocks;
    int th, tw, nth, ntw;                 // outputs of a tile, tiles per image
    int relu;
};

__device__ __forceinline__ void bf3_split(const float a, const float b, uint32_t &h, uint32_t &m, uint32_t &l) {
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
                NNV_TILE_MFMA(l, h, acs) NNV_TILE_MFMA(h, h, acc) NNV_TILE_MFMA(m, h, acs)
                NNV_TILE_MFMA(m, m, acs) NNV_TILE_MFMA(h, m, acs) NNV_TILE_MFMA(h, l, acs)
#undef NNV_TILE_MFMA
#undef NNV_BF
                // (vector instructions dealt out over the products)
#pragma unroll
                for (int i = 0; i < 6 * TM; ++i) {
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

// The same sums with float32 products, every operand straight from memory: for tiles whose result is not finite.
template <int TM, int TN>
__device__ __forceinline__ void tile_exact(const TileLayer &g, const TilePos &at, const int c0, const int c1, floatx4 (&acc)[TM][TN]) {
    constexpr int QM = 16 / TM;
    const int lane = threadIdx.x & 63, col = lane & 15, slot = lane >> 4;
    const SmallDiv by_tw(g.tw);
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(g.x, (uint32_t)(g.N * g.C) * (uint32_t)(g.H * g.W) * 4u);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(g.wp, (uint32_t)g.K16 * (uint32_t)g.cblocks * (9 * 256u));
    const uint32_t a_voff = at.mb0 + col / QM < g.K16
        ? (uint32_t)(col / QM) * (uint32_t)g.cblocks * (9 * 256u) + (uint32_t)slot * 64u + (uint32_t)(col % QM) * (4u * TM) : kOobOffset;
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[m][t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int cb = c0 * 8; cb < min(c1 * 8, g.cblocks); ++cb) {
        const int c = cb * 4 + slot;
#pragma unroll 1
        for (int rs = 0; rs < 9; ++rs) {
            const auto a = buf_load_floats<TM>(wres, a_voff, ((uint32_t)at.mb0 * (uint32_t)g.cblocks * 9u + (uint32_t)(cb * 9 + rs)) * 256u);
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                const int n = t * 16 + col, r = by_tw(n), q = n - r * g.tw;
                const int ih = at.p0 + r - g.pad + rs / 3, iw = at.q0 + q - g.pad + rs % 3;
                const bool ok = r < g.th && c < g.C && (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
                const float b = buf_load<float>(xres, ok ? (uint32_t)(((at.img * g.C + c) * g.H + ih) * g.W + iw) * 4u : kOobOffset, 0u);
#pragma unroll
                for (int m = 0; m < TM; ++m) acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(float_of<TM>(a, m), b, acc[m][t], 0, 0, 0);
            }
        }
    }
}

// One work item: tile (mt, nt) over the chunks [c0, c1); part: where its sums go if the layer's channels are split, else null.
template <int TM, int TN, bool DOUBLE>
__device__ __forceinline__ void tile_item(const TileLayer &g, const int mt, const int nt, const int c0, const int c1, float *part, char *lds) {
    const int lane = threadIdx.x & 63, col = lane & 15, slot = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rest = nt / g.ntw, img = rest / g.nth;
    const TilePos at{__builtin_amdgcn_readfirstlane(img), __builtin_amdgcn_readfirstlane((rest - img * g.nth) * g.th),
                     __builtin_amdgcn_readfirstlane((nt - rest * g.ntw) * g.tw), (mt * 4 + wave) * TM};
    floatx4 acc[TM][TN];
    {
        floatx4 acs[TM][TN];
        tile_accumulate<TM, TN, DOUBLE>(g, at, c0, c1, lds, acc, acs);
        float z = 0.f;                    // NaN if any sum is not finite
        uint32_t least = 0xffffffffu;     // twice the bits of the smallest one that is not zero, less one
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                acc[m][t] += acs[m][t];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    z = fmaf(acc[m][t][j], 0.f, z);
                    least = min(least, (__builtin_bit_cast(uint32_t, acc[m][t][j]) << 1) - 1u);
                }
            }
        constexpr uint32_t kTiny = (127u - 60u) << 24;      // 2^-60
        if (__ballot(z != 0.f || least < kTiny) != 0) tile_exact<TM, TN>(g, at, c0, c1, acc);
    }
    __builtin_amdgcn_s_setprio(3);
    if (part) {
        float *o = part + (size_t)wave * (TM * TN * 256) + lane;
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) o[((m * TN + t) * 4 + j) * 64] = acc[m][t][j];
        return;
    }
    const int PQ = g.P * g.Q;
    const SmallDiv by_tw(g.tw);
    int pix[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) pix[t] = tile_out_pixel(g, at, by_tw, t * 16 + col);
    const __amdgpu_buffer_rsrc_t yres = make_rsrc(g.y, (uint32_t)(g.N * g.K) * (uint32_t)PQ * 4u);
    const __amdgpu_buffer_rsrc_t bres = make_rsrc(g.bias, g.bias ? (uint32_t)g.K * 4u : 0u);
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = at.mb0 * 16 + gemm_row(true, TM, m, slot, j);
            const bool ok = k < g.K;
            const float bv = buf_load<float>(bres, ok ? (uint32_t)k * 4u : kOobOffset, 0u);
            const uint32_t base = (uint32_t)((at.img * g.K + k) * PQ);
#pragma unroll
            for (int t = 0; t < TN; ++t)
                gemm_store(yres, g.relu, false, ok && pix[t] >= 0 ? (base + (uint32_t)pix[t]) * 4u : kOobOffset, bv, acc[m][t][j]);
        }
}
