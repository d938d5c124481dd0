// Internal declarations shared by the host dispatch and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>
#include <stddef.h>
#include "nnv.h"

namespace nnv {

// Validated geometry of one conv layer (host side).
struct Geo {
    int n, c, h, w, k, r, s, sh, sw, ph, pw, groups, dtype;
    int p, q;      // output height / width
    int cg, kg;    // channels per group (input / output)
    int relu;      // clamp the outputs at zero before the store (not part of the descriptor)
};

static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
static inline bool is_wino(int kind) { return kind == NNV_WINO_F2 || kind == NNV_WINO_F4 || kind == NNV_WINO_F6; }
static inline int wino_m(int kind) { return kind == NNV_WINO_F2 ? 2 : kind == NNV_WINO_F4 ? 4 : 6; }
static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Fewest input channels for which Winograd runs with float16 storage (see nnv_kind_supported).
constexpr int kWinoHalfMinChannels = 16;

// Winograd matrix sets (see wino_consts.h)
enum WinoSet { WS_F2 = 0, WS_F4 = 1, WS_F4H = 2, WS_F6 = 3 };
static inline int wino_set(int kind, int dtype) {
    if (kind == NNV_WINO_F2) return WS_F2;
    if (kind == NNV_WINO_F6) return WS_F6;
    return dtype == NNV_F16 ? WS_F4H : WS_F4;
}

// One weight-transformation job of a grouped launch.
enum JobType { JOB_WINO = 0, JOB_GEMM = 1, JOB_DW = 2 };
struct TransformJob {
    const float *src;
    void *dst;
    uint16_t K, C, RS;      // rows, channels per row, taps
    uint16_t cchunk;        // channels handled by one block
    uint16_t nchunks;       // blocks per 16-row group
    uint8_t type;           // JobType
    uint8_t wset;           // WinoSet (JOB_WINO)
    uint8_t half;           // output float16
    uint8_t unused[3];
};
// 112 jobs of 32 bytes + 112 block offsets fit the 4 KB of kernel arguments: the candidates of every
// stack here but two go out in one launch (a second one for the last few jobs ran 15 us by itself).
constexpr int kMaxJobs = 112;
struct JobTable {
    TransformJob job[kMaxJobs];
    int first_block[kMaxJobs];   // first block of each job in the launch, INT_MAX beyond the last job: a block
                                 // finds its job by counting the entries it has reached (no chain of dependent loads)
};
static_assert(sizeof(JobTable) <= 4096, "the job table is passed by value as the kernel argument");
constexpr int kMaxGemmGroups = 64;   // groups of an IM2COL_GEMM layer: a transformation job each

// Records the text of a failed HIP call for nnv_last_hip_error and returns NNV_E_HIP.
int record_hip_error(hipError_t e);

int fill_transform_job(const Geo &g, int kind, const float *src, void *dst, TransformJob *job, int *nblocks);
size_t transform_job_lds_bytes(const TransformJob &job);
// jobs [0, njobs) of tbl with their first_block entries set; the entries beyond are filled in here
hipError_t launch_transform_jobs(JobTable &tbl, int njobs, int total_blocks, size_t lds, hipStream_t st);
hipError_t launch_copy_f32(const float *src, float *dst, size_t n, hipStream_t st);
hipError_t launch_fill_u32(uint32_t *dst, size_t n, uint32_t v, hipStream_t st);

hipError_t launch_direct(const Geo &g, const void *x, const float *w, const float *bias, void *y, hipStream_t st);
hipError_t launch_depthwise(const Geo &g, const void *x, const void *w, const float *bias, void *y, hipStream_t st);

// Many layers in one launch: direct convolution (layers for which direct_many_supported holds) and
// depthwise convolution; one storage type per call.
constexpr int kMaxDirectLayers = 32;
constexpr int kMaxDwLayers = 40;
bool direct_many_supported(const Geo &g);
hipError_t launch_direct_many(int n, const Geo *geos, const void *const *x, const void *const *w, const float *const *bias,
                              void *const *y, hipStream_t st);
// raw: w[i] are the untransformed float32 filters (depthwise layers run by the direct kind), else the
// channel-blocked tap-major ones of the depthwise kind.
hipError_t launch_depthwise_many(int n, const Geo *geos, const void *const *x, const void *const *w,
                                 const float *const *bias, void *const *y, bool raw, hipStream_t st);

size_t im2col_workspace_bytes(const Geo &g);
hipError_t launch_im2col(const Geo &g, const void *x, const void *w, const float *bias, void *y, void *ws, hipStream_t st);

// Many independent IM2COL_GEMM layers (one storage type, at most kMaxGemmLayers) in one launch of
// work items, of single wavefronts or whole workgroups (tile_gemm.h), plus one launch in front if a float16 layer reads a copy of x; ws[i] is layer i's own region of im2col_items_workspace_bytes.
constexpr int kMaxGemmLayers = 56;
bool im2col_items_supported(const Geo &g);
void im2col_items_workspace_bytes(int n, const Geo *geos, size_t *bytes);      // of each of the layers of a launch
hipError_t launch_im2col_items(int n, const Geo *geos, const void *const *x, const void *const *w,
                               const float *const *bias, void *const *y, void *const *ws, hipStream_t st, int ndw = 0, const char *raw = nullptr);
// Behind the n layers, ndw depthwise ones of the same storage type may ride along (n + ndw <= kMaxGemmLayers, n > 0): geos, x, w, bias and y go on
// with them, ws does not; raw[j]: filters of the j-th untransformed.
// depthwise_items: workgroups of a layer (more than any launch should take where a layer record cannot hold it).
long depthwise_items(const Geo &g);

// Several IM2COL_GEMM layers without bias that do not depend on one another, in one launch whose results are those of
// launch_im2col on each of them, bit for bit (at most kMaxMergedLayers, each mergeable).
constexpr int kMaxMergedLayers = 24;
bool im2col_layer_mergeable(const Geo &g);
hipError_t launch_im2col_layers(int n, const Geo *geos, const void *const *x, const void *const *w, void *const *y, hipStream_t st);

size_t wino_workspace_bytes(const Geo &g, int kind);
// Many layers of one Winograd kind and storage type in three launches (see winograd.hip).
constexpr int kMaxWinoLayers = 20;
bool wino_many_supported(const Geo &g, int kind);
hipError_t launch_wino_many(int n, const Geo *geos, int kind, const void *const *x, const void *const *U,
                            const float *const *bias, void *const *y, void *const *ws, hipStream_t st);
// Several layers of one kind that run as one fused kernel (see winograd.hip), without a workspace.
// wino_fused_layers: which of n layers of one kind and storage type (n <= kMaxWinoLayers) run so in one call.
void wino_fused_layers(int n, const Geo *geos, int kind, char *fused);
hipError_t launch_wino_fused(int n, const Geo *geos, int kind, const void *const *x, const void *const *U,
                             const float *const *bias, void *const *y, hipStream_t st);
hipError_t launch_wino(const Geo &g, int kind, const void *x, const void *w, const float *bias, void *y, void *ws, hipStream_t st);

}  // namespace nnv
