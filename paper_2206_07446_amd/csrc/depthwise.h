// Depthwise 3x3 and 5x5 filters at stride 1 or 2: the outputs of a layer dealt out to the threads of workgroups of 256, for launches of many layers.
#pragma once
#include <type_traits>
#include "buf.h"

namespace nnv {

struct DwParams {
    int N, C, H, W, st, ph, pw, P, Q, relu;
};

// Outputs of a thread: that many rows of one column.  What bounds the launch is the latency of a wavefront (look-up of its layer, divisions, loads) and the
// loads per output, 18 of them with an output per thread (taps and pixels), 6.75 with four in a column, whose windows share their rows.
// us a call, two outputs per thread, each with loads of its own (5x5: one), / two rows / four / seven (5x5: four): the 17 layers of a MobileNetV2-shaped stack
// 12.5 / 12.1 / 11.3 / 11.8, at 4x120x300 31.2 / 28.0 / 22.0 / 23.3, at batch 3 in float16 49.0 / 29.0 / 22.0 / 20.2; EfficientNet-B0, with 5x5
// filters, 16.2 / 17.2 (two) / 14.9 (four).
constexpr int kDwRows = 4;
static inline long dw_workgroups(const DwParams &d) {
    return ((long)d.N * d.C * ((d.P + kDwRows - 1) / kDwRows) * d.Q + 255) / 256;
}

__device__ __forceinline__ void dw_store(const __amdgpu_buffer_rsrc_t r, const uint32_t off, const float v, float) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0u, 0);
}
__device__ __forceinline__ void dw_store(const __amdgpu_buffer_rsrc_t r, const uint32_t off, const float v, __half) {
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, (_Float16)v), r, off, 0u, 0);
}

// RAW: wv holds the untransformed float32 filters [c][FS * FS].
template <typename T, int FS, int ST, bool RAW>
__device__ __forceinline__ void depthwise_column(const void *x, const void *wv, const float *bias, void *y, const DwParams &d, const int blk) {
    constexpr int R = kDwRows, NR = (R - 1) * ST + FS;
    constexpr uint32_t ESZ = sizeof(T);
    typedef typename std::conditional<RAW, float, T>::type W;
    const int groups = (d.P + R - 1) / R, per_plane = groups * d.Q, planes = d.N * d.C;
    const int e = blk * 256 + (int)threadIdx.x;
    const int plane = e / per_plane, rest = e - plane * per_plane, pg = rest / d.Q, q = rest - pg * d.Q;
    const bool live = plane < planes;
    const int c = d.N == 1 ? plane : plane % d.C, p0 = pg * R;
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(x, (uint32_t)planes * (uint32_t)(d.H * d.W) * ESZ);
    const __amdgpu_buffer_rsrc_t yres = make_rsrc(y, (uint32_t)planes * (uint32_t)(d.P * d.Q) * ESZ);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(wv, RAW ? (uint32_t)(d.C * FS * FS) * 4u : (uint32_t)((d.C + 31) / 32 * 32 * FS * FS) * ESZ);
    const __amdgpu_buffer_rsrc_t bres = make_rsrc(bias, bias ? (uint32_t)d.C * 4u : 0u);       // no bias: zero
    const int ih0 = p0 * ST - d.ph, iw0 = q * ST - d.pw;
    const uint32_t base = (uint32_t)(plane * d.H * d.W) * ESZ;
    uint32_t col[FS];
#pragma unroll
    for (int s = 0; s < FS; ++s) col[s] = live && (unsigned)(iw0 + s) < (unsigned)d.W ? base + (uint32_t)(iw0 + s) * ESZ : kOobOffset;
    float xv[NR][FS], w[FS][FS];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const bool ok = (unsigned)(ih0 + r) < (unsigned)d.H;
        const uint32_t row = (uint32_t)((ih0 + r) * d.W) * ESZ;
#pragma unroll
        for (int s = 0; s < FS; ++s) xv[r][s] = buf_load_x<T>(xres, ok && col[s] != kOobOffset ? col[s] + row : kOobOffset, 0u);
    }
    const uint32_t wo = !live ? kOobOffset : RAW ? (uint32_t)(c * FS * FS) * 4u : (uint32_t)((c >> 5) * (FS * FS * 32) + (c & 31)) * ESZ;
#pragma unroll
    for (int r = 0; r < FS; ++r)
#pragma unroll
        for (int s = 0; s < FS; ++s) w[r][s] = buf_load_x<W>(wres, wo + (uint32_t)((r * FS + s) * (RAW ? 4 : 32 * ESZ)), 0u);
    const float bv = buf_load<float>(bres, live ? (uint32_t)c * 4u : kOobOffset, 0u);
    const uint32_t yo = (uint32_t)(plane * d.P * d.Q + p0 * d.Q + q) * ESZ;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        float acc = bv;
#pragma unroll
        for (int r = 0; r < FS; ++r)
#pragma unroll
            for (int s = 0; s < FS; ++s) acc = fmaf(xv[i * ST + r][s], w[r][s], acc);
        if (d.relu) acc = fmaxf(acc, 0.f);
        dw_store(yres, live && p0 + i < d.P ? yo + (uint32_t)(i * d.Q) * ESZ : kOobOffset, acc, T());
    }
}

// Workgroup blk of a layer; all of it is uniform but the thread.
template <typename T>
__device__ __forceinline__ void depthwise_workgroup(const void *x, const void *w, const float *bias, void *y, const DwParams &d, const int fs, const bool raw, const int blk) {
#define NNV_DW(FS, ST) (raw ? depthwise_column<T, FS, ST, true>(x, w, bias, y, d, blk) : depthwise_column<T, FS, ST, false>(x, w, bias, y, d, blk))
    if (fs == 3) { if (d.st == 1) NNV_DW(3, 1); else NNV_DW(3, 2); }
    else { if (d.st == 1) NNV_DW(5, 1); else NNV_DW(5, 2); }
#undef NNV_DW
}

}  // namespace nnv
