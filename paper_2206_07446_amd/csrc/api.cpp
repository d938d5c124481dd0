// Host side of the C ABI declared in nnv.h: descriptor validation, size queries,
// dispatch by kernel kind and the per-operation timing.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>
#include "nnv_internal.h"

using namespace nnv;

// Scratch of nnv_conv_forward_static: one array per GPU, part of the loaded code object, so no
// call ever allocates it.  In host code this name is only a handle for hipGetSymbolAddress; the
// device address it yields (per device) is what kernels and copies get.
static __device__ __align__(256) unsigned char nnv_static_scratch[NNV_STATIC_SCRATCH_BYTES];

namespace {

thread_local std::string g_hip_error;

int hip_fail(hipError_t e) {
    g_hip_error = hipGetErrorString(e);
    return NNV_E_HIP;
}
}  // namespace

int nnv::record_hip_error(hipError_t e) { return hip_fail(e); }

namespace {

int make_geo(const nnv_conv_desc *d, Geo *g) {
    if (!d) return NNV_E_NULL;
    if (d->n <= 0 || d->c <= 0 || d->h <= 0 || d->w <= 0 || d->k <= 0 || d->r <= 0 || d->s <= 0) return NNV_E_BAD_DESC;
    if (d->stride_h <= 0 || d->stride_w <= 0 || d->pad_h < 0 || d->pad_w < 0 || d->groups <= 0) return NNV_E_BAD_DESC;
    if (d->c % d->groups || d->k % d->groups) return NNV_E_BAD_DESC;
    if (d->dtype != NNV_F32 && d->dtype != NNV_F16) return NNV_E_BAD_DESC;
    // padded extents and output sizes in 64 bits: a huge pad must not wrap around
    const int64_t hp = (int64_t)d->h + 2 * (int64_t)d->pad_h, wp = (int64_t)d->w + 2 * (int64_t)d->pad_w;
    if (hp < d->r || wp < d->s) return NNV_E_BAD_DESC;
    const int64_t p64 = (hp - d->r) / d->stride_h + 1, q64 = (wp - d->s) / d->stride_w + 1;
    if (p64 >= ((int64_t)1 << 30) || q64 >= ((int64_t)1 << 30)) return NNV_E_BAD_DESC;
    if (d->n > 65535 || d->c > 65535 || d->k > 65535) return NNV_E_BAD_DESC;
    g->n = d->n; g->c = d->c; g->h = d->h; g->w = d->w; g->k = d->k; g->r = d->r; g->s = d->s;
    g->sh = d->stride_h; g->sw = d->stride_w; g->ph = d->pad_h; g->pw = d->pad_w;
    g->groups = d->groups; g->dtype = d->dtype;
    g->p = (int)p64;
    g->q = (int)q64;
    g->cg = d->c / d->groups;
    g->kg = d->k / d->groups;
    g->relu = 0;
    const int64_t lim = (int64_t)1 << 30;   // element counts are indexed with 32-bit ints
    if ((int64_t)g->n * g->c * g->h * g->w >= lim || (int64_t)g->n * g->k * g->p * g->q >= lim) return NNV_E_BAD_DESC;
    if ((int64_t)g->n * g->h * g->w * (ceil_div(g->c, 32) * 32) >= lim) return NNV_E_BAD_DESC;
    if ((int64_t)g->k * g->cg * g->r * g->s >= lim) return NNV_E_BAD_DESC;
    return NNV_OK;
}

size_t tx_bytes(const Geo &g, int kind);
size_t ws_bytes(const Geo &g, int kind);

bool kind_rules(const Geo &g, int kind);

// A kind runs a layer if its shape rules hold and every buffer it touches stays below 2 GiB
// (the kernels address them with 32-bit byte offsets).
bool supported(const Geo &g, int kind) {
    if (!kind_rules(g, kind)) return false;
    const size_t lim = (size_t)1 << 31;
    const size_t esz = g.dtype == NNV_F16 ? 2 : 4;
    if ((size_t)g.n * g.c * g.h * g.w * esz >= lim || (size_t)g.n * g.k * g.p * g.q * esz >= lim) return false;
    return tx_bytes(g, kind) < lim && ws_bytes(g, kind) < lim;
}

bool kind_rules(const Geo &g, int kind) {
    switch (kind) {
        case NNV_DIRECT: return true;
        case NNV_IM2COL_GEMM: {
            // the pack stages 16 rows x one fragment column of taps in LDS
            if (g.r > 32 || g.s > 32 || g.r * g.s > (g.dtype == NNV_F16 ? 64 : 128)) return false;
            if (g.groups == 1) return true;
            // groups: one panel block and one transformation job per group; the float16
            // copy in octets of channels needs each group's channels on a fragment boundary
            if (g.groups > kMaxGemmGroups) return false;
            return g.dtype == NNV_F32 || (g.r == 1 && g.s == 1) || g.cg % 32 == 0;
        }
        case NNV_WINO_F2:
        case NNV_WINO_F4:
            // float16 storage of U and V: with fewer than 16 input channels the error relative to
            // max|y| has a heavy tail that crosses the float16 bound of this library (5e-3), so
            // that pairing is refused like F(6x6) in float16
            if (g.dtype == NNV_F16 && g.c < kWinoHalfMinChannels) return false;
            return g.groups == 1 && g.r == 3 && g.s == 3 && g.sh == 1 && g.sw == 1;
        case NNV_WINO_F6: return g.groups == 1 && g.r == 3 && g.s == 3 && g.sh == 1 && g.sw == 1 && g.dtype == NNV_F32;
        case NNV_DEPTHWISE:
            return g.groups == g.c && g.c == g.k && g.r == g.s && (g.r == 3 || g.r == 5) && g.sh == g.sw && (g.sh == 1 || g.sh == 2);
        default: return false;
    }
}

size_t tx_bytes(const Geo &g, int kind) {
    const bool half = g.dtype == NNV_F16;
    const size_t frag = half ? (size_t)ceil_div(g.cg, 32) * 512 * 2 : (size_t)ceil_div(g.cg, 4) * 64 * 4;
    const size_t k16 = ceil_div(g.k, 16);
    switch (kind) {
        case NNV_DIRECT: return (size_t)g.k * g.cg * g.r * g.s * sizeof(float);
        case NNV_IM2COL_GEMM: return (size_t)g.groups * ceil_div(g.kg, 16) * frag * g.r * g.s;
        case NNV_WINO_F2: return 16 * k16 * frag;
        case NNV_WINO_F4: return 36 * k16 * frag;
        case NNV_WINO_F6: return 64 * k16 * frag;
        case NNV_DEPTHWISE: return (size_t)ceil_div(g.c, 32) * g.r * g.s * 32 * (half ? 2 : 4);
        default: return 0;
    }
}

size_t ws_bytes(const Geo &g, int kind) {
    switch (kind) {
        case NNV_IM2COL_GEMM: return im2col_workspace_bytes(g);
        case NNV_WINO_F2:
        case NNV_WINO_F4:
        case NNV_WINO_F6: return wino_workspace_bytes(g, kind);
        default: return 0;
    }
}

inline bool misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) != 0; }

int transform_many(int n, const nnv_conv_desc *descs, const nnv_kind *kinds, const float *const *w_raw,
                   void *const *w_tx, hipStream_t st) {
    if (n < 0) return NNV_E_ARG;
    if (n == 0) return NNV_OK;
    if (!descs || !kinds || !w_raw || !w_tx) return NNV_E_NULL;
    std::vector<Geo> geos(n);
    for (int i = 0; i < n; ++i) {
        int rc = make_geo(&descs[i], &geos[i]);
        if (rc) return rc;
        if (kinds[i] < 0 || kinds[i] >= NNV_KIND_COUNT) return NNV_E_ARG;
        if (!supported(geos[i], kinds[i])) return NNV_E_UNSUPPORTED;
        if (!w_raw[i] || !w_tx[i]) return NNV_E_NULL;
        if (misaligned(w_raw[i]) || misaligned(w_tx[i])) return NNV_E_ALIGN;
    }
    JobTable tbl;
    int njobs = 0, blocks = 0;
    size_t lds = 0;
    auto flush = [&]() -> hipError_t {
        if (njobs == 0) return hipSuccess;
        hipError_t e = launch_transform_jobs(tbl, njobs, blocks, lds, st);
        njobs = 0; blocks = 0; lds = 0;
        return e;
    };
    for (int i = 0; i < n; ++i) {
        if (kinds[i] == NNV_DIRECT) {
            if (static_cast<const void *>(w_raw[i]) != w_tx[i]) {
                hipError_t e = launch_copy_f32(w_raw[i], static_cast<float *>(w_tx[i]),
                                               (size_t)geos[i].k * geos[i].cg * geos[i].r * geos[i].s, st);
                if (e != hipSuccess) return hip_fail(e);
            }
            continue;
        }
        // a grouped GEMM layer is one pack job per group: rows [g * Kg, (g + 1) * Kg) of the raw
        // tensor into the g-th panel block
        const bool grouped = kinds[i] == NNV_IM2COL_GEMM && geos[i].groups > 1;
        Geo one = geos[i];
        if (grouped) { one.k = one.kg; one.c = one.cg; one.groups = 1; }
        const size_t src_step = (size_t)one.k * one.cg * one.r * one.s;
        const size_t dst_step = grouped ? tx_bytes(one, NNV_IM2COL_GEMM) : 0;
        for (int gi = 0; gi < (grouped ? geos[i].groups : 1); ++gi) {
            TransformJob &job = tbl.job[njobs];
            int nblocks;
            if (fill_transform_job(one, kinds[i], w_raw[i] + gi * src_step, static_cast<char *>(w_tx[i]) + gi * dst_step, &job, &nblocks))
                return NNV_E_UNSUPPORTED;
            tbl.first_block[njobs] = blocks;
            blocks += nblocks;
            lds = std::max(lds, transform_job_lds_bytes(job));
            if (++njobs == kMaxJobs) {
                hipError_t e = flush();
                if (e != hipSuccess) return hip_fail(e);
            }
        }
    }
    hipError_t e = flush();
    if (e != hipSuccess) return hip_fail(e);
    return NNV_OK;
}

int forward_checked(const Geo &g, int kind, const void *x, const void *w_tx, const float *bias, void *y, void *ws,
                    hipStream_t st) {
    hipError_t e = hipSuccess;
    switch (kind) {
        case NNV_DIRECT: e = launch_direct(g, x, static_cast<const float *>(w_tx), bias, y, st); break;
        case NNV_IM2COL_GEMM: e = launch_im2col(g, x, w_tx, bias, y, ws, st); break;
        case NNV_WINO_F2:
        case NNV_WINO_F4:
        case NNV_WINO_F6: e = launch_wino(g, kind, x, w_tx, bias, y, ws, st); break;
        case NNV_DEPTHWISE: e = launch_depthwise(g, x, w_tx, bias, y, st); break;
        default: return NNV_E_ARG;
    }
    if (e != hipSuccess) return hip_fail(e);
    return NNV_OK;
}

int forward_args(const nnv_conv_desc *desc, nnv_kind kind, const void *x, const void *w_tx, const float *bias,
                 void *y, void *ws, size_t ws_size, Geo *g) {
    int rc = make_geo(desc, g);
    if (rc) return rc;
    if (kind < 0 || kind >= NNV_KIND_COUNT) return NNV_E_ARG;
    if (!supported(*g, kind)) return NNV_E_UNSUPPORTED;
    if (!x || !w_tx || !y) return NNV_E_NULL;
    const size_t need = ws_bytes(*g, kind);
    if (need > 0 && !ws) return NNV_E_NULL;
    if (ws_size < need) return NNV_E_WORKSPACE;
    if (misaligned(x) || misaligned(w_tx) || misaligned(y) || (need && misaligned(ws)) || (bias && (reinterpret_cast<uintptr_t>(bias) & 3)))
        return NNV_E_ALIGN;
    return NNV_OK;
}

// ---- the convolutions of a stage of a cold pass: layers that do not depend on one another share a launch where they can
struct Span {
    uintptr_t begin, end;
    Span(const void *p, size_t n) : begin(reinterpret_cast<uintptr_t>(p)), end(begin + n) {}
    bool meets(const Span &o) const { return begin < o.end && o.begin < end; }
};

// Executes layers [0, n) as one after the other would.  A layer's level is one above the highest of the earlier layers whose
// output it reads or writes over, or whose input or weights it writes over; the mergeable layers of a level go out
// in one launch.  Buffers that lie in the workspace follow no rule here: then one layer after the other.
constexpr int kMergeWindow = 64;      // layers looked at together: at most 2016 pairs
int forward_levels(int n, const Geo *geos, const nnv_kind *kinds, const void *const *x, void *const *w_tx, void *const *y, void *ws,
                   size_t ws_size, hipStream_t st) {
    int level[kMergeWindow], last = 0, mergeable = 0;
    bool merge[kMergeWindow], plain = false;
    for (int i = 0; i < n; ++i) {
        level[i] = i;
        merge[i] = kinds[i] == NNV_IM2COL_GEMM && im2col_layer_mergeable(geos[i]);
        mergeable += merge[i] ? 1 : 0;
    }
    last = n - 1;
    if (mergeable > 1) {
        std::vector<Span> xs, wt, ys;
        const Span scratch(ws, ws ? ws_size : 0);
        for (int i = 0; i < n; ++i) {
            const Geo &g = geos[i];
            const size_t esz = g.dtype == NNV_F16 ? 2 : 4;
            xs.emplace_back(x[i], (size_t)g.n * g.c * g.h * g.w * esz);
            wt.emplace_back(w_tx[i], tx_bytes(g, kinds[i]));
            ys.emplace_back(y[i], (size_t)g.n * g.k * g.p * g.q * esz);
            plain = plain || scratch.meets(xs[i]) || scratch.meets(wt[i]) || scratch.meets(ys[i]);
        }
        last = 0;
        for (int j = 0; j < n && !plain; ++j) {
            level[j] = 0;
            for (int i = 0; i < j; ++i)
                if (level[i] >= level[j] && (ys[i].meets(xs[j]) || ys[i].meets(ys[j]) || ys[i].meets(wt[j]) || ys[j].meets(xs[i]) || ys[j].meets(wt[i])))
                    level[j] = level[i] + 1;
            last = std::max(last, level[j]);
        }
        if (plain) last = n - 1;
    }
    for (int v = 0; v <= last; ++v) {
        std::vector<Geo> bg;
        std::vector<const void *> bx, bw;
        std::vector<void *> by;
        int one = -1;
        for (int i = 0; i < n; ++i) {
            if (level[i] != v) continue;
            if (merge[i]) {
                bg.push_back(geos[i]); bx.push_back(x[i]); bw.push_back(w_tx[i]); by.push_back(y[i]);
                one = i;
                continue;
            }
            const int rc = forward_checked(geos[i], kinds[i], x[i], w_tx[i], nullptr, y[i], ws, st);
            if (rc) return rc;
        }
        if (bg.size() == 1) {
            const int rc = forward_checked(geos[one], kinds[one], x[one], w_tx[one], nullptr, y[one], ws, st);
            if (rc) return rc;
        }
        for (size_t b = 0; bg.size() > 1 && b < bg.size(); b += kMaxMergedLayers) {
            const int m = (int)std::min<size_t>(kMaxMergedLayers, bg.size() - b);
            const hipError_t e = launch_im2col_layers(m, &bg[b], &bx[b], &bw[b], &by[b], st);
            if (e != hipSuccess) return hip_fail(e);
        }
    }
    return NNV_OK;
}

// Device address of nnv_static_scratch on the current device, looked up once per device.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void *g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev < 0 || dev >= kMaxDevices) return NNV_E_ARG;
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(nnv_static_scratch));
        if (e != hipSuccess) return hip_fail(e);
        if (!p || misaligned(p)) return NNV_E_ALIGN;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return NNV_OK;
}

// ---- nnv_conv_forward_grouped: which layers share a launch, and where their scratch lies.
// Layers of one launch run concurrently, so each needs a workspace region of its own; launches
// follow one another on the stream, so the regions of different launches overlap.
struct GroupedPlan {
    enum Class { SINGLE = 0, GEMM_ITEMS = 1, WINO_MANY = 2, DIRECT_MANY = 3, DW_MANY = 4, DW_RAW_MANY = 5, WINO_FUSED = 6 };
    struct Batch {
        int cls;
        int kind;                   // WINO_MANY: the Winograd kind of the batch
        std::vector<int> layers;
        std::vector<size_t> offset; // workspace offset of each layer's region
        std::vector<int> depthwise; // GEMM_ITEMS: depthwise layers that ride along
    };
    std::vector<Batch> batches;
    size_t bytes = 0;
};

GroupedPlan plan_grouped(int n, const Geo *geos, const nnv_kind *kinds) {
    GroupedPlan gp;
    std::vector<char> taken(n, 0);
    // collect the layers that satisfy `pick` into batches of at most `cap`, each layer with a
    // workspace region of its own
    // A batch below `least` layers is given back (its layers then run by themselves): the many-layer
    // kernels are laid out for launches that fill the chip - work items of 144 k-steps, tiles resident
    // all at once - and one or two layers through them take 2-5 times as long as their own launches
    // (measured: a 512-channel 7x7 layer 30 against 15 us through the item GEMM).
    auto collect = [&](int cls, int kind, int cap, int least, auto pick, auto region_bytes) {
        GroupedPlan::Batch cur{cls, kind, {}, {}, {}};
        size_t off = 0;
        auto close = [&]() {
            if ((int)cur.layers.size() >= least) { gp.bytes = std::max(gp.bytes, off); gp.batches.push_back(cur); }
            else for (int i : cur.layers) taken[i] = 0;
            cur.layers.clear(); cur.offset.clear(); off = 0;
        };
        for (int i = 0; i < n; ++i) {
            if (taken[i] || !pick(i)) continue;
            taken[i] = 1;
            cur.layers.push_back(i);
            cur.offset.push_back(off);
            off += align_up(region_bytes(i), 256);
            if ((int)cur.layers.size() == cap) close();
        }
        close();
    };
    for (int half = 0; half < 2; ++half) {
        auto same_type = [&](int i) { return (geos[i].dtype == NNV_F16) == (half == 1); };
        // (the regions of an item launch depend on the item length, which depends on the whole batch: laid out below)
        // (more layers than one launch carries are dealt out evenly: a last launch of a few layers leaves most of the chip idle)
        auto gemm_item = [&](int i) { return kinds[i] == NNV_IM2COL_GEMM && same_type(i) && im2col_items_supported(geos[i]); };
        int gemm_layers = 0;
        for (int i = 0; i < n; ++i) gemm_layers += gemm_item(i) ? 1 : 0;
        const int gemm_launches = std::max(1, ceil_div(gemm_layers, kMaxGemmLayers));
        collect(GroupedPlan::GEMM_ITEMS, NNV_IM2COL_GEMM, std::max(1, ceil_div(gemm_layers, gemm_launches)), 4,
                gemm_item, [&](int) { return (size_t)0; });
        collect(GroupedPlan::DIRECT_MANY, NNV_DIRECT, kMaxDirectLayers, 3,
                [&](int i) { return kinds[i] == NNV_DIRECT && same_type(i) && direct_many_supported(geos[i]); },
                [&](int) { return (size_t)0; });
        collect(GroupedPlan::DW_MANY, NNV_DEPTHWISE, kMaxDwLayers, 2,
                [&](int i) { return kinds[i] == NNV_DEPTHWISE && same_type(i); }, [&](int) { return (size_t)0; });
        // depthwise layers given to the direct kind: the depthwise launch, reading the untransformed filters
        collect(GroupedPlan::DW_RAW_MANY, NNV_DIRECT, kMaxDwLayers, 2,
                [&](int i) { return kinds[i] == NNV_DIRECT && same_type(i) && supported(geos[i], NNV_DEPTHWISE); },
                [&](int) { return (size_t)0; });
        // float32 F(2x2) and F(4x4).  The workspace holds the region of every layer that has one, also of those that run fused: which ones do depends on all layers of the
        // call, and a workspace for many layers has to be enough for some of them.
        for (int kind : {NNV_WINO_F2, NNV_WINO_F4}) {
            std::vector<int> of_kind;
            for (int i = 0; i < n && !half; ++i)
                if (kinds[i] == kind && same_type(i)) of_kind.push_back(i);
            if (of_kind.size() < 2) continue;          // (one layer: runs by itself)
            std::vector<char> fused(n, 0);
            size_t off = 0;
            int regions = 0;
            for (int i : of_kind) {
                if (!wino_many_supported(geos[i], kind)) continue;
                off = (regions++ % kMaxWinoLayers ? off : 0) + align_up(ws_bytes(geos[i], kind), 256);
                gp.bytes = std::max(gp.bytes, off);
            }
            for (size_t at = 0; at < of_kind.size(); at += kMaxWinoLayers) {
                Geo part[kMaxWinoLayers];
                char yes[kMaxWinoLayers];
                const size_t m = std::min<size_t>(of_kind.size() - at, kMaxWinoLayers);
                for (size_t j = 0; j < m; ++j) part[j] = geos[of_kind[at + j]];
                wino_fused_layers((int)m, part, kind, yes);
                for (size_t j = 0; j < m; ++j) fused[of_kind[at + j]] = yes[j];
            }
            collect(GroupedPlan::WINO_FUSED, kind, kMaxWinoLayers, 1, [&](int i) { return fused[i] != 0; }, [&](int) { return (size_t)0; });
        }
        for (int kind : {NNV_WINO_F2, NNV_WINO_F4, NNV_WINO_F6})
            collect(GroupedPlan::WINO_MANY, kind, kMaxWinoLayers, 2,
                    [&](int i) { return kinds[i] == kind && same_type(i) && wino_many_supported(geos[i], kind); },
                    [&](int i) { return ws_bytes(geos[i], kind); });
    }
    // Depthwise layers ride along with an item launch of their storage type: the items leave half of the memory path idle and end one by one, and a launch
    // less is 4 us.  Up to kMostDepthwise workgroups of them, ten rounds of what the item kernel's registers let the chip hold; more do better in a launch of
    // their own, four wavefronts per SIMD instead of three and a fourth of the code.  us a call, apart / together, [workgroups]: ShuffleNet-shaped [460] 23.5 / 19.8, MobileNetV1 [1970] 38.1 / 29.0,
    // MobileNetV2 [2350] 32.3 / 27.4, float16 28.1 / 20.9, EfficientNet-B0 [2370] 49.9 / 45.0, MobileNetV2 in float16 at batch 2 [4700] 38.0 / 33.4 and 3 [7050] 49.8 / 48.2,
    // EfficientNet-B0 at batch 3 [7120] 105 / 100; beyond the line MobileNetV2 at batch 4 [9400] 98 / 98, float16 69 / 70.6, at 4x320x320 [18600] 176 / 182, float16 125 / 133.
    constexpr long kMostDepthwise = 7680;
    for (GroupedPlan::Batch &d : gp.batches) {
        if (d.cls != GroupedPlan::DW_MANY && d.cls != GroupedPlan::DW_RAW_MANY) continue;
        for (GroupedPlan::Batch &b : gp.batches) {
            if (b.cls != GroupedPlan::GEMM_ITEMS || geos[b.layers[0]].dtype != geos[d.layers[0]].dtype) continue;
            if ((int)(b.layers.size() + b.depthwise.size() + d.layers.size()) > kMaxGemmLayers) continue;
            long items = 0;
            for (int i : b.depthwise) items += depthwise_items(geos[i]);
            for (int i : d.layers) items += depthwise_items(geos[i]);
            if (items > kMostDepthwise) continue;
            b.depthwise.insert(b.depthwise.end(), d.layers.begin(), d.layers.end());
            d.layers.clear();
            break;
        }
    }
    gp.batches.erase(std::remove_if(gp.batches.begin(), gp.batches.end(), [](const GroupedPlan::Batch &b) { return b.layers.empty(); }), gp.batches.end());
    for (GroupedPlan::Batch &b : gp.batches) {
        if (b.cls != GroupedPlan::GEMM_ITEMS) continue;
        std::vector<Geo> bg;
        for (int i : b.layers) bg.push_back(geos[i]);
        std::vector<size_t> bytes(bg.size());
        im2col_items_workspace_bytes((int)bg.size(), bg.data(), bytes.data());
        size_t off = 0;
        for (size_t j = 0; j < b.layers.size(); ++j) {
            b.offset[j] = off;
            off += align_up(bytes[j], 256);
        }
        gp.bytes = std::max(gp.bytes, off);
    }
    for (int i = 0; i < n; ++i) {
        if (taken[i]) continue;
        gp.batches.push_back(GroupedPlan::Batch{GroupedPlan::SINGLE, kinds[i], {i}, {0}, {}});
        gp.bytes = std::max(gp.bytes, ws_bytes(geos[i], kinds[i]));
    }
    return gp;
}

int grouped_geos(int n, const nnv_conv_desc *descs, const nnv_kind *kinds, std::vector<Geo> *geos) {
    if (!descs || !kinds) return NNV_E_NULL;
    geos->resize(n);
    for (int i = 0; i < n; ++i) {
        int rc = make_geo(&descs[i], &(*geos)[i]);
        if (rc) return rc;
        if (kinds[i] < 0 || kinds[i] >= NNV_KIND_COUNT) return NNV_E_ARG;
        if (!supported((*geos)[i], kinds[i])) return NNV_E_UNSUPPORTED;
    }
    return NNV_OK;
}

double median(std::vector<float> v) {
    std::sort(v.begin(), v.end());
    const size_t n = v.size();
    return n % 2 ? v[n / 2] : 0.5 * (v[n / 2 - 1] + v[n / 2]);
}

}  // namespace

extern "C" {

int nnv_layout_version(void) { return 1; }

const char *nnv_status_string(int status) {
    switch (status) {
        case NNV_OK: return "ok";
        case NNV_E_NULL: return "a required pointer is NULL";
        case NNV_E_BAD_DESC: return "invalid convolution descriptor";
        case NNV_E_UNSUPPORTED: return "kernel kind does not support this layer";
        case NNV_E_WORKSPACE: return "workspace too small";
        case NNV_E_ALIGN: return "device pointer not 16-byte aligned";
        case NNV_E_HIP: return "HIP runtime error";
        case NNV_E_ARG: return "invalid argument";
        case NNV_E_IO: return "cache file could not be opened, read or written";
        case NNV_E_CACHE: return "cache file does not match the requested layer, kind or layout version";
        default: return "unknown status";
    }
}

const char *nnv_last_hip_error(void) { return g_hip_error.c_str(); }

int nnv_kind_supported(const nnv_conv_desc *desc, nnv_kind kind) {
    Geo g;
    int rc = make_geo(desc, &g);
    if (rc) return rc;
    if (kind < 0 || kind >= NNV_KIND_COUNT) return NNV_E_ARG;
    return supported(g, kind) ? 1 : 0;
}

size_t nnv_transformed_bytes(const nnv_conv_desc *desc, nnv_kind kind) {
    Geo g;
    if (make_geo(desc, &g) || kind < 0 || kind >= NNV_KIND_COUNT || !supported(g, kind)) return 0;
    return tx_bytes(g, kind);
}

size_t nnv_workspace_bytes(const nnv_conv_desc *desc, nnv_kind kind) {
    Geo g;
    if (make_geo(desc, &g) || kind < 0 || kind >= NNV_KIND_COUNT || !supported(g, kind)) return 0;
    return ws_bytes(g, kind);
}

int nnv_transform_weights(const nnv_conv_desc *desc, nnv_kind kind, const float *w_raw, void *w_tx, void *hip_stream) {
    if (!desc) return NNV_E_NULL;
    const float *src[1] = {w_raw};
    void *dst[1] = {w_tx};
    return transform_many(1, desc, &kind, src, dst, static_cast<hipStream_t>(hip_stream));
}

int nnv_transform_weights_grouped(int n_layers, const nnv_conv_desc *descs, const nnv_kind *kinds,
                                  const float *const *w_raw, void *const *w_tx, void *hip_stream) {
    return transform_many(n_layers, descs, kinds, w_raw, w_tx, static_cast<hipStream_t>(hip_stream));
}

int nnv_conv_forward(const nnv_conv_desc *desc, nnv_kind kind, const void *x, const void *w_tx, const float *bias,
                     void *y, void *workspace, size_t workspace_bytes, void *hip_stream) {
    Geo g;
    int rc = forward_args(desc, kind, x, w_tx, bias, y, workspace, workspace_bytes, &g);
    if (rc) return rc;
    return forward_checked(g, kind, x, w_tx, bias, y, workspace, static_cast<hipStream_t>(hip_stream));
}

int nnv_conv_forward_relu(const nnv_conv_desc *desc, nnv_kind kind, const void *x, const void *w_tx, const float *bias,
                          void *y, void *workspace, size_t workspace_bytes, void *hip_stream) {
    Geo g;
    int rc = forward_args(desc, kind, x, w_tx, bias, y, workspace, workspace_bytes, &g);
    if (rc) return rc;
    g.relu = 1;
    return forward_checked(g, kind, x, w_tx, bias, y, workspace, static_cast<hipStream_t>(hip_stream));
}

size_t nnv_conv_forward_grouped_workspace_bytes(int n_layers, const nnv_conv_desc *descs, const nnv_kind *kinds) {
    if (n_layers <= 0) return 0;
    std::vector<Geo> geos;
    if (grouped_geos(n_layers, descs, kinds, &geos)) return 0;
    return plan_grouped(n_layers, geos.data(), kinds).bytes;
}

int nnv_conv_forward_grouped(int n_layers, const nnv_conv_desc *descs, const nnv_kind *kinds, const void *const *x,
                             const void *const *w_tx, const float *const *bias, void *const *y, void *workspace,
                             size_t workspace_bytes, unsigned flags, void *hip_stream) {
    if (n_layers < 0 || (flags & ~(unsigned)NNV_FORWARD_RELU)) return NNV_E_ARG;
    if (n_layers == 0) return NNV_OK;
    if (!x || !w_tx || !y) return NNV_E_NULL;
    std::vector<Geo> geos;
    int rc = grouped_geos(n_layers, descs, kinds, &geos);
    if (rc) return rc;
    for (int i = 0; i < n_layers; ++i) {
        if (!x[i] || !w_tx[i] || !y[i]) return NNV_E_NULL;
        if (misaligned(x[i]) || misaligned(w_tx[i]) || misaligned(y[i]) ||
            (bias && bias[i] && (reinterpret_cast<uintptr_t>(bias[i]) & 3)))
            return NNV_E_ALIGN;
        geos[i].relu = (flags & NNV_FORWARD_RELU) ? 1 : 0;
    }
    const GroupedPlan gp = plan_grouped(n_layers, geos.data(), kinds);
    if (gp.bytes > 0 && !workspace) return NNV_E_NULL;
    if (workspace_bytes < gp.bytes) return NNV_E_WORKSPACE;
    if (gp.bytes > 0 && misaligned(workspace)) return NNV_E_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    for (const GroupedPlan::Batch &b : gp.batches) {
        if (b.cls == GroupedPlan::SINGLE) {
            const int i = b.layers[0];
            rc = forward_checked(geos[i], kinds[i], x[i], w_tx[i], bias ? bias[i] : nullptr, y[i], workspace, st);
            if (rc) return rc;
            continue;
        }
        const int m = (int)b.layers.size(), ndw = (int)b.depthwise.size();
        std::vector<Geo> bg(m + ndw);
        std::vector<const void *> bx(m + ndw), bw(m + ndw);
        std::vector<const float *> bb(m + ndw);
        std::vector<void *> by(m + ndw), bws(m);
        std::vector<char> raw(ndw);
        for (int j = 0; j < m + ndw; ++j) {
            const int i = j < m ? b.layers[j] : b.depthwise[j - m];
            bg[j] = geos[i]; bx[j] = x[i]; bw[j] = w_tx[i]; bb[j] = bias ? bias[i] : nullptr; by[j] = y[i];
            if (j < m) bws[j] = static_cast<char *>(workspace) + b.offset[j];
            else raw[j - m] = kinds[i] == NNV_DIRECT;
        }
        hipError_t e = hipSuccess;
        switch (b.cls) {
            case GroupedPlan::GEMM_ITEMS:
                e = launch_im2col_items(m, bg.data(), bx.data(), bw.data(), bb.data(), by.data(), bws.data(), st, ndw, raw.data());
                break;
            case GroupedPlan::WINO_FUSED:
                e = launch_wino_fused(m, bg.data(), b.kind, bx.data(), bw.data(), bb.data(), by.data(), st);
                break;
            case GroupedPlan::WINO_MANY:
                e = launch_wino_many(m, bg.data(), b.kind, bx.data(), bw.data(), bb.data(), by.data(), bws.data(), st);
                break;
            case GroupedPlan::DIRECT_MANY:
                e = launch_direct_many(m, bg.data(), bx.data(), bw.data(), bb.data(), by.data(), st);
                break;
            default:
                e = launch_depthwise_many(m, bg.data(), bx.data(), bw.data(), bb.data(), by.data(),
                                          b.cls == GroupedPlan::DW_RAW_MANY, st);
                break;
        }
        if (e != hipSuccess) return hip_fail(e);
    }
    return NNV_OK;
}

int nnv_conv_forward_static(const nnv_conv_desc *desc, nnv_kind kind, const void *x, const void *w_tx,
                            const float *bias, void *y, void *hip_stream) {
    Geo g;
    // argument checks as in nnv_conv_forward, against a workspace of the static size; the
    // address only has to be non-NULL and aligned here
    void *probe = reinterpret_cast<void *>(static_cast<uintptr_t>(256));
    int rc = forward_args(desc, kind, x, w_tx, bias, y, probe, NNV_STATIC_SCRATCH_BYTES, &g);
    if (rc) return rc;
    void *ws = nullptr;
    rc = static_scratch(&ws);
    if (rc) return rc;
    return forward_checked(g, kind, x, w_tx, bias, y, ws, static_cast<hipStream_t>(hip_stream));
}

int nnv_cold_stack(int n_layers, const nnv_conv_desc *descs, const nnv_kind *kinds, const float *const *w_raw,
                   void *const *w_tx, const void *const *x, void *const *y, void *workspace, size_t workspace_bytes,
                   int stage_layers, void *stream_exec, void *stream_tx) {
    if (n_layers < 0) return NNV_E_ARG;
    if (n_layers == 0) return NNV_OK;
    if (!descs || !kinds || !w_raw || !w_tx || !x || !y) return NNV_E_NULL;
    // validate everything before the first launch
    std::vector<Geo> geos(n_layers);
    for (int i = 0; i < n_layers; ++i) {
        int rc = forward_args(&descs[i], kinds[i], x[i], w_tx[i], nullptr, y[i], workspace, workspace_bytes, &geos[i]);
        if (rc) return rc;
        if (!w_raw[i]) return NNV_E_NULL;
        if (misaligned(w_raw[i])) return NNV_E_ALIGN;
    }
    hipStream_t se = static_cast<hipStream_t>(stream_exec), stx = static_cast<hipStream_t>(stream_tx);
    const bool two = se != stx;
    const int per = stage_layers <= 0 ? n_layers : stage_layers;
    const int stages = (n_layers + per - 1) / per;
    std::vector<hipEvent_t> ev;     // [0]: fork, [1 + s]: stage s transformed
    auto cleanup = [&]() { for (hipEvent_t e : ev) (void)hipEventDestroy(e); };
    auto fail = [&](hipError_t e) { cleanup(); return hip_fail(e); };
    hipError_t e;
    if (two) {
        ev.reserve(stages + 1);
        for (int i = 0; i < stages + 1; ++i) {
            hipEvent_t h;
            e = hipEventCreateWithFlags(&h, hipEventDisableTiming);
            if (e != hipSuccess) return fail(e);
            ev.push_back(h);
        }
        e = hipEventRecord(ev[0], se);
        if (e == hipSuccess) e = hipStreamWaitEvent(stx, ev[0], 0);
        if (e != hipSuccess) return fail(e);
    }
    // Stage s + 1 is handed to stream_tx before the convolutions of stage s are handed to
    // stream_exec, so the host never holds the transformation stream back.
    auto issue_tx = [&](int s) -> int {
        const int b = s * per, n = std::min(per, n_layers - b);
        int rc = transform_many(n, descs + b, kinds + b, w_raw + b, w_tx + b, stx);
        if (rc) return rc;
        if (two) {
            hipError_t er = hipEventRecord(ev[1 + s], stx);
            if (er != hipSuccess) return hip_fail(er);
        }
        return NNV_OK;
    };
    int rc = issue_tx(0);
    for (int s = 0; s < stages && rc == NNV_OK; ++s) {
        if (s + 1 < stages) rc = issue_tx(s + 1);
        if (rc) break;
        if (two) {
            e = hipStreamWaitEvent(se, ev[1 + s], 0);
            if (e != hipSuccess) { rc = hip_fail(e); break; }
        }
        const int b = s * per, n = std::min(per, n_layers - b);
        for (int i = b; i < b + n && rc == NNV_OK; i += kMergeWindow)
            rc = forward_levels(std::min(kMergeWindow, b + n - i), &geos[i], kinds + i, x + i, w_tx + i, y + i, workspace, workspace_bytes, se);
    }
    if (two && rc != NNV_OK) {
        // an error cut the pass short: still join stream_tx back into stream_exec, so that a
        // capture that is under way stays well-formed
        if (hipEventRecord(ev[0], stx) == hipSuccess) (void)hipStreamWaitEvent(se, ev[0], 0);
    }
    cleanup();
    return rc;
}

int nnv_time_layer(const nnv_conv_desc *desc, nnv_kind kind, const float *w_raw, void *w_tx, const void *x, void *y,
                   void *workspace, size_t workspace_bytes, void *flush, size_t flush_bytes, int warmup, int reps,
                   void *hip_stream, nnv_timing *out) {
    if (!out || !w_raw) return NNV_E_NULL;
    if (reps <= 0 || warmup < 0) return NNV_E_ARG;
    Geo g;
    int rc = forward_args(desc, kind, x, w_tx, nullptr, y, workspace, workspace_bytes, &g);
    if (rc) return rc;
    if (misaligned(w_raw) || (flush && misaligned(flush))) return NNV_E_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    hipEvent_t e0, e1;
    hipError_t e = hipEventCreate(&e0);
    if (e != hipSuccess) return hip_fail(e);
    e = hipEventCreate(&e1);
    if (e != hipSuccess) { (void)hipEventDestroy(e0); return hip_fail(e); }
    std::vector<float> t_tx, t_fw;
    const bool tx_is_noop = kind == NNV_DIRECT && static_cast<const void *>(w_raw) == w_tx;
    rc = NNV_OK;
    // Warm repetitions time a short queue of back-to-back launches: a batch-1 layer runs for a
    // few microseconds, less than a pair of events costs.  A cold repetition is one launch.
    const bool cold = flush && flush_bytes >= 16;
    const int inner = cold ? 1 : 8;
    for (int it = 0; it < warmup + reps && rc == NNV_OK; ++it) {
        for (int phase = 0; phase < 2 && rc == NNV_OK; ++phase) {
            if (cold) {
                e = launch_fill_u32(static_cast<uint32_t *>(flush), flush_bytes / 4, (uint32_t)it, st);
                if (e != hipSuccess) { rc = hip_fail(e); break; }
            }
            float ms = 0.f;
            if (phase == 0 && tx_is_noop) {
                // nothing to run: the raw layout is the execution layout
            } else {
                if ((e = hipEventRecord(e0, st)) != hipSuccess) { rc = hip_fail(e); break; }
                for (int k = 0; k < inner && rc == NNV_OK; ++k) {
                    if (phase == 0) rc = nnv_transform_weights(desc, kind, w_raw, w_tx, hip_stream);
                    else rc = forward_checked(g, kind, x, w_tx, nullptr, y, workspace, st);
                }
                if (rc) break;
                if ((e = hipEventRecord(e1, st)) != hipSuccess) { rc = hip_fail(e); break; }
                if ((e = hipEventSynchronize(e1)) != hipSuccess) { rc = hip_fail(e); break; }
                if ((e = hipEventElapsedTime(&ms, e0, e1)) != hipSuccess) { rc = hip_fail(e); break; }
                ms /= (float)inner;
            }
            if (it >= warmup) (phase == 0 ? t_tx : t_fw).push_back(ms);
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e);
    const double esz = g.dtype == NNV_F16 ? 2.0 : 4.0;
    const double raw_b = (double)g.k * g.cg * g.r * g.s * 4.0;
    const double tx_b = (double)tx_bytes(g, kind);
    out->transform_ms = median(t_tx);
    out->forward_ms = median(t_fw);
    out->transform_bytes = tx_is_noop ? 0.0 : raw_b + tx_b;
    out->forward_bytes = esz * ((double)g.n * g.c * g.h * g.w + (double)g.n * g.k * g.p * g.q) + tx_b;
    const double macs = (double)g.n * g.k * g.p * g.q * g.cg * g.r * g.s;
    out->direct_equiv_flops = 2.0 * macs;
    if (is_wino(kind)) {
        const int m = wino_m(kind);
        const double tiles = (double)g.n * ceil_div(g.p, m) * ceil_div(g.q, m);
        out->forward_flops = 2.0 * (m + 2) * (m + 2) * g.k * g.c * tiles;
    } else {
        out->forward_flops = 2.0 * macs;
    }
    return NNV_OK;
}

}  // extern "C"
