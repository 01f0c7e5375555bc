// nyx_runtime.hip -- host runtime and C ABI (include/nyx.h).
//
// Planning discovers the ROIs once, chooses the LDS accumulation mode and the
// split of large ROIs, sizes the work queue and scratch, and captures the
// whole step (discovery, binning, accumulation, features) in a HIP graph
// replayed by nyx_plan_execute.  nyx_plan_execute_per_roi runs the same step
// with one accumulation launch per ROI instead of the persistent queue.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <numeric>
#include <string>
#include <vector>

#include "../../include/nyx.h"
#include "nyx_launch.h"
#include "nyx_types.h"

using namespace nyx;

namespace {

const char *const kFeatureNames[kNumFeat] = {
    "ASM", "ACOR", "CLUPROM", "CLUSHADE", "CLUTEND", "CONTRAST", "CORR", "DIFAVE", "DIFENTRO", "DIFVAR",
    "DIS", "ENERGY", "ENTROPY", "HOM1", "HOM2", "IDM", "INFOMEAS1", "INFOMEAS2", "IDMN", "ID",
    "IDN", "IV", "JAVE", "JE", "JMAX", "SUMAVE", "SUMENT", "JVAR", "SUMVAR", "VARIANCE"};

const char *const kIntensityNames[kNumIntensityFeat] = {
    "MEAN", "MIN", "MAX", "RANGE", "INTEGRATED_INTENSITY", "ENERGY", "RMS", "VARIANCE", "STDDEV",
    "STANDARD_ERROR", "SKEWNESS", "KURTOSIS", "HYPERSKEWNESS", "HYPERFLATNESS", "MEAN_ABSOLUTE_DEVIATION",
    "MEDIAN", "MEDIAN_ABSOLUTE_DEVIATION", "P01", "P10", "P25", "P75", "P90", "P99", "INTERQUARTILE_RANGE",
    "ROBUST_MEAN_ABSOLUTE_DEVIATION", "MODE", "ENTROPY", "UNIFORMITY", "UNIFORMITY_PIU", "WEIGHTED_CENTROID_X",
    "WEIGHTED_CENTROID_Y", "WEIGHTED_CENTROID_Z", "EDGE_INTEGRATED_INTENSITY", "EDGE_MIN", "EDGE_MAX",
    "EDGE_MEAN", "EDGE_STDDEV"};

const char *const kNeighbourNames[kNumNeighbourFeat] = {
    "NGLDM_DCENRG", "NGLDM_DCENT", "NGLDM_DCNU", "NGLDM_DCNUN", "NGLDM_DCM", "NGLDM_DCV", "NGLDM_GLNU",
    "NGLDM_GLNUN", "NGLDM_GLM", "NGLDM_GLV", "NGLDM_HDE", "NGLDM_HDHGLE", "NGLDM_HDLGLE", "NGLDM_HGLCE",
    "NGLDM_LDE", "NGLDM_LDHGLE", "NGLDM_LDLGLE", "NGLDM_LGLCE", "NGTDM_BUSYNESS", "NGTDM_COARSENESS",
    "NGTDM_COMPLEXITY", "NGTDM_CONTRAST", "NGTDM_STRENGTH", "GLDM_SDE", "GLDM_LDE", "GLDM_GLN", "GLDM_DN",
    "GLDM_DNN", "GLDM_GLV", "GLDM_DV", "GLDM_DE", "GLDM_LGLE", "GLDM_HGLE", "GLDM_SDLGLE", "GLDM_SDHGLE",
    "GLDM_LDLGLE", "GLDM_LDHGLE"};

constexpr uint32_t kLdsBudget = 160u * 1024u;   // LDS per CU on gfx950
constexpr uint32_t kRingMin = 2048u, kRingMax = 32768u;   // staged-accumulation level ring (bytes)
constexpr uint32_t kMaxGroupsPerCu = 5u;                  // k_batch, single precision: 5 waves per SIMD
constexpr uint32_t kMaxNgFused = 8191u;         // hash keys carry 13-bit levels
constexpr uint64_t kMaxLabelEntries = 1ull << 26;
// A context's block for the one-shot calls: what the largest call so far
// asked for, between these bounds (what exceeds it is allocated and freed by
// the call).
constexpr size_t kPoolMin = 32u << 20, kPoolMax = 512u << 20;
// Pinned staging memory: image descriptors up, counters and ROI descriptors down.
constexpr size_t kPinBytes = 512u << 10, kPinUp = 128u << 10, kPinDown = kPinBytes - kPinUp;
// Discovery fills the ROI descriptors (and the tile queue) in one go, sized by
// the label table, up to this many entries; above, the ROIs are counted first.
constexpr uint32_t kOnePassLabels = 1u << 17;
// Replays with the same outputs after which a plan's step is captured anew in
// two branches: that costs about 210 us more than one branch does, what some
// five replays give back (a caller that alternates two tables paid it on every
// call: 359 us a step before there was a branch, 441 with it, 243 so).
constexpr uint32_t kForkAfter = 4u;
// Banded accumulation (hash mode, symmetric matrices): ROIs above
// kBandMinVox voxels (and above the split size), LDS band of at most
// kBandLds bytes, work items of at least about kBandTile bbox voxels, bands
// of at least kBandWide levels per direction when several share a pass.
constexpr uint32_t kBandMinVox = 32768u, kBandLds = 128u * 1024u, kBandTile = 64u * 1024u, kBandMinW = 8u, kBandWide = 32u;

// Most device memory the packed hash may take beyond the configuration it
// takes the place of.
constexpr uint64_t kPackedExtra = 1ull << 30;

int log_level() {
    static int lvl = -1;
    if (lvl < 0) {
        const char *s = getenv("NYX_LOG");
        lvl = s ? atoi(s) : 0;
    }
    return lvl;
}

// A bump allocator over a device region, reused from its start by the next
// call: the fixed scratch of the no-allocation entry point, or a context's
// own block for the one-shot calls (spill: requests that do not fit come from
// hipMalloc, and the block grows to the call's demand before the next one).
struct Arena {
    uint8_t *base = nullptr;
    size_t cap = 0, used = 0;
    size_t wanted = 0;   // bytes the failed request would have needed in total
    size_t demand = 0;   // bytes asked for since the arena was last started
    bool spill = false;
    static size_t up(size_t n) { return (n + 255u) & ~(size_t)255u; }
    void *carve(size_t n) {
        const size_t at = up(used);
        demand += up(n);
        if (at + n > cap) {
            wanted = at + n;
            return nullptr;
        }
        used = at + n;
        return base + at;
    }
    bool fits(size_t n) const { return up(used) + n <= cap; }
    // gives back the tail of the latest request
    void trim(const void *p, size_t from, size_t to) {
        if (base && static_cast<const uint8_t *>(p) + from == base + used) used -= from - to;
    }
};

// Device buffer: owned (hipMalloc / hipFree), or carved from an Arena when
// one is given (never freed by the buffer).
struct DevBuf {
    void *p = nullptr;
    size_t bytes = 0;
    bool owned = false;
    Arena *arena = nullptr;
    DevBuf() = default;
    DevBuf(const DevBuf &) = delete;
    DevBuf &operator=(const DevBuf &) = delete;
    ~DevBuf() { release(); }
    void release() {
        if (p && owned) (void)hipFree(p);
        p = nullptr;
        bytes = 0;
        owned = false;
    }
    hipError_t alloc(size_t n) {
        release();
        if (n == 0) n = 16;
        if (arena) {
            p = arena->carve(n);
            if (p) {
                bytes = n;
                return hipSuccess;
            }
            if (!arena->spill) return hipErrorOutOfMemory;
        }
        hipError_t e = hipMalloc(&p, n);
        if (e == hipSuccess) {
            bytes = n;
            owned = true;
        } else {
            p = nullptr;
            (void)hipGetLastError();   // reported here: not to be found by the check of a later launch
        }
        return e;
    }
    // keeps the first n bytes
    void shrink(size_t n) {
        if (n == 0) n = 16;
        if (!p || n >= bytes) return;
        if (arena && !owned) arena->trim(p, bytes, n);
        bytes = n;
    }
    template <class T> T *as() const { return reinterpret_cast<T *>(p); }
};


uint32_t next_pow2(uint32_t v) {
    uint32_t p = 1;
    while (p < v) p <<= 1;
    return p;
}

}  // namespace

// Device memory of the no-allocation entry point: one array per GPU for the
// life of the process, shared by every call on that GPU.  Host code never
// uses the symbol itself (on the host it only names a stand-in): the device
// address is taken once per device with hipGetSymbolAddress and kept below.
constexpr size_t kScratchBytes = NYX_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint8_t *g_scratch_ptr[kMaxDevices] = {};

// The device address of `scratch` on `device` (current); nullptr on failure.
uint8_t *scratch_address(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[device] = static_cast<uint8_t *>(ptr);
    }
    return g_scratch_ptr[device];
}
}  // namespace

struct nyx_ctx {
    int device = 0;
    int n_cu = 0;
    std::string err;
    hipStream_t capture_stream = nullptr;
    hipStream_t side_stream = nullptr;    // a captured step's second branch, forked and joined by these events
    hipEvent_t fork_event = nullptr, join_event = nullptr;
    uint8_t *scratch = nullptr;   // this device's no-allocation scratch (device address)
    Arena pool;                   // device block of the one-shot calls
    uint8_t *pin = nullptr;       // kPinBytes of pinned host memory for the calls' small copies
};

// The sizes of a batch's ROIs by size class (size_class of their voxels), with
// each class's sums: what the planner asks of the ROIs up to a number of voxels
// comes from the sums of the classes below, and only larger ones are looked at
// one by one.  (Over the descriptors, each of its dozen questions walked all of
// them: a plan of 150000 regions took 17 ms on the host.)
struct RoiSizes {
    struct Box {
        uint32_t n, rows, width;
    };
    struct Sum {
        uint64_t count = 0, vox = 0;
        uint32_t most = 0;   // voxels of the largest
        void add(uint32_t n) {
            ++count;
            vox += n;
            most = std::max(most, n);
        }
        void add(const Sum &o) {
            count += o.count;
            vox += o.vox;
            most = std::max(most, o.most);
        }
    };
    std::vector<Box> box;                  // by class, ascending
    size_t first[kClasses + 1] = {};
    Sum of_class[kClasses], all;

    void fill(const std::vector<RoiDesc> &rois) {
        *this = RoiSizes{};
        for (const RoiDesc &r : rois) of_class[size_class(r.n)].add(r.n);
        for (int cl = 0; cl < kClasses; ++cl) {
            first[cl + 1] = first[cl] + of_class[cl].count;
            all.add(of_class[cl]);
        }
        box.resize(rois.size());
        size_t at[kClasses];
        std::copy(first, first + kClasses, at);
        for (const RoiDesc &r : rois)
            box[at[size_class(r.n)]++] = Box{r.n, r.rows, (uint32_t)(r.x1 - r.x0 + 1)};
    }
    // the ROIs of at most v voxels
    Sum up_to(uint32_t v) const {
        Sum s;
        const uint32_t c = size_class(v);
        for (uint32_t cl = 0; cl < c; ++cl) s.add(of_class[cl]);
        for (size_t i = first[c]; i < first[c + 1]; ++i)
            if (box[i].n <= v) s.add(box[i].n);
        return s;
    }
    // every ROI of more than v voxels
    template <class Fn> void above(uint32_t v, Fn &&fn) const {
        for (size_t i = first[size_class(v)]; i < box.size(); ++i)
            if (box[i].n > v) fn(box[i]);
    }
};

// All device state of one discovery/step over a batch of images.
struct Work {
    std::vector<ImgDesc> h_imgs;
    DevBuf imgs, tab[10], counters, rois, buckets, G, dsums, dsums_y, split_roi, band_roi, smarg, stot, splp, dict;
    uint64_t *vox_base = nullptr;      // first voxel of each image (device, behind the image descriptors)
    uint32_t n_split = 0, n_aux = 0;   // split ROIs and their extra storage (tile queue)
    uint32_t tab_total = 0, n_blocks = 0, n_counters = 0, total_chunks = 0;
    uint32_t n_rois = 0;
    uint64_t total_vox = 0;
    std::vector<RoiDesc> h_rois;
    RoiSizes sizes;                    // of h_rois
    StepArgs args{};
    bool have_rois = false;            // h_rois holds the descriptors
    // Carve every buffer from `ar` (nullptr: hipMalloc).
    void use_arena(Arena *ar) {
        for (DevBuf *b : {&imgs, &counters, &rois, &buckets, &G, &dsums, &dsums_y, &split_roi, &band_roi, &smarg, &stot,
                          &splp, &dict})
            b->arena = ar;
        for (DevBuf &b : tab) b.arena = ar;
    }
};

struct nyx_plan {
    nyx_ctx *ctx = nullptr;
    Work w;
    std::vector<nyx_image> imgs;
    int K = 0, ng = 0;
    nyx_precision prec = NYX_FP32;
    uint32_t grid = 0, block = 256;
    // second launch of the batch kernel (packed hash): the size classes below small_cls
    uint32_t small_cls = 0, small_kp = 0, small_grid = 0;
    LdsLayout small_lds{};
    bool banded = false, fork = false; // a planned ROI is banded; a step that is repeated forks
    // The step as a graph writing graph_table and graph_rois: of one branch,
    // and of two once it has been replayed `replays` times.
    struct Graph {
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
    } plain, forked;
    uint32_t replays = 0;
    void *graph_table = nullptr;
    nyx_roi_table graph_rois{};
    std::string desc;
    int64_t workspace_bytes = 0;
    float tuned_ms = 0.f;
    struct Cfg { int mode; uint32_t kp, block, split_vox, tile_vox, list_cap, hash_cap; int force_split; };
    Cfg cfg{};
};

namespace {

nyx_status fail(nyx_ctx *c, nyx_status s, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (c) c->err = buf;
    if (log_level() > 0) fprintf(stderr, "[nyx] error: %s\n", buf);
    return s;
}

#define HIPC(ctx, x)                                                                              \
    do {                                                                                          \
        hipError_t e_ = (x);                                                                      \
        if (e_ != hipSuccess)                                                                     \
            return fail(ctx, e_ == hipErrorOutOfMemory ? NYX_ERR_OOM : NYX_ERR_DEVICE, "%s: %s", #x, \
                        hipGetErrorString(e_));                                                   \
    } while (0)

nyx_status validate_images(nyx_ctx *ctx, const nyx_image *imgs, int32_t n) {
    if (!imgs || n <= 0) return fail(ctx, NYX_ERR_INVALID, "no images");
    for (int i = 0; i < n; ++i) {
        const nyx_image &m = imgs[i];
        if (!m.intensity || !m.labels) return fail(ctx, NYX_ERR_INVALID, "image %d: NULL array", i);
        if (m.nz <= 0 || m.ny <= 0 || m.nx <= 0) return fail(ctx, NYX_ERR_INVALID, "image %d: dimension <= 0", i);
        if (m.nz > 65535 || m.ny > 65535 || m.nx > 65535)
            return fail(ctx, NYX_ERR_INVALID, "image %d: dimension above 65535", i);
        if (m.nz * m.ny * m.nx >= (1ll << 31)) return fail(ctx, NYX_ERR_INVALID, "image %d: 2^31 voxels or more", i);
    }
    return NYX_OK;
}

nyx_status validate_offsets(nyx_ctx *ctx, const nyx_image *imgs, int32_t n_images, const nyx_offset *off,
                            int32_t K) {
    if (!off) return fail(ctx, NYX_ERR_INVALID, "offsets are NULL");
    if (K < 1 || K > kMaxOffsets) return fail(ctx, NYX_ERR_INVALID, "n_offsets must be in [1, 64]");
    bool any3d = false;
    for (int i = 0; i < n_images; ++i) any3d |= imgs[i].nz > 1;
    for (int k = 0; k < K; ++k) {
        if (off[k].dz == 0 && off[k].dy == 0 && off[k].dx == 0)
            return fail(ctx, NYX_ERR_INVALID, "offset %d is (0,0,0)", k);
        if (!any3d && off[k].dz != 0) return fail(ctx, NYX_ERR_INVALID, "offset %d has dz != 0 on 2D images", k);
        if (abs(off[k].dz) > 65535 || abs(off[k].dy) > 65535 || abs(off[k].dx) > 65535)
            return fail(ctx, NYX_ERR_INVALID, "offset %d out of range", k);
    }
    return NYX_OK;
}

nyx_status validate_bins(nyx_ctx *ctx, int32_t ng) {
    if (ng < 2 || ng > 65535) return fail(ctx, NYX_ERR_INVALID, "n_bins must be in [2, 65535]");
    if ((uint32_t)ng > kMaxNgFused)
        return fail(ctx, NYX_ERR_UNSUPPORTED, "n_bins above %u is not supported", kMaxNgFused);
    return NYX_OK;
}

// Distinct nonzero labels of every image, ascending, uploaded to w.dict;
// sets dict, dict_n and max_label (= dict_n) of w.h_imgs.  Labels present in
// a later execution but absent here have no table entry (E_LABEL_RANGE).
nyx_status build_label_dict(nyx_ctx *ctx, Work &w, int32_t n, hipStream_t st) {
    uint64_t max_vox = 0;
    for (int i = 0; i < n; ++i) max_vox = std::max<uint64_t>(max_vox, w.h_imgs[i].nvox);
    DevBuf list, cnt;
    list.arena = cnt.arena = w.imgs.arena;
    HIPC(ctx, cnt.alloc(sizeof(uint32_t)));
    uint32_t cap = 1u << 16, got = 0;
    for (int attempt = 0; attempt < 2; ++attempt) {
        HIPC(ctx, list.alloc(sizeof(uint64_t) * cap));
        const uint32_t zero = 0u;
        HIPC(ctx, hipMemcpyAsync(cnt.p, &zero, sizeof zero, hipMemcpyHostToDevice, st));
        HIPC(ctx, launch_label_collect(w.imgs.as<ImgDesc>(), n, max_vox, list.as<uint64_t>(), cap, cnt.as<uint32_t>(),
                                       st));
        HIPC(ctx, hipMemcpyAsync(&got, cnt.p, sizeof got, hipMemcpyDeviceToHost, st));
        HIPC(ctx, hipStreamSynchronize(st));
        if (got <= cap) break;
        cap = got;   // every entry fits the second time (same images)
    }
    if (got > cap) return fail(ctx, NYX_ERR_INTERNAL, "label collection did not converge");
    std::vector<uint64_t> h(got);
    if (got) HIPC(ctx, hipMemcpyAsync(h.data(), list.p, sizeof(uint64_t) * got, hipMemcpyDeviceToHost, st));
    HIPC(ctx, hipStreamSynchronize(st));
    std::sort(h.begin(), h.end());
    h.erase(std::unique(h.begin(), h.end()), h.end());
    std::vector<uint32_t> labels(h.size());
    std::vector<uint64_t> first(n + 1, 0);
    for (size_t k = 0; k < h.size(); ++k) {
        labels[k] = (uint32_t)h[k];
        first[(size_t)(h[k] >> 32) + 1u]++;
    }
    for (int i = 0; i < n; ++i) first[i + 1] += first[i];
    HIPC(ctx, w.dict.alloc(sizeof(uint32_t) * std::max<size_t>(labels.size(), 1)));
    if (!labels.empty())
        HIPC(ctx, hipMemcpyAsync(w.dict.p, labels.data(), sizeof(uint32_t) * labels.size(), hipMemcpyHostToDevice, st));
    HIPC(ctx, hipStreamSynchronize(st));
    for (int i = 0; i < n; ++i) {
        w.h_imgs[i].dict = w.dict.as<uint32_t>() + first[i];
        w.h_imgs[i].dict_n = (uint32_t)(first[i + 1] - first[i]);
        w.h_imgs[i].max_label = w.h_imgs[i].dict_n;
    }
    return NYX_OK;
}

// Waits for a call's stream where the call fails on the way: copies from the
// pinned memory and kernels on scratch that the next call uses, perhaps on
// another stream, may be under way.
struct CallGuard {
    hipStream_t st;
    bool done = false;
    explicit CallGuard(hipStream_t s) : st(s) {}
    ~CallGuard() {
        if (!done) (void)hipStreamSynchronize(st);
    }
    // the call's result; on success it has waited itself
    nyx_status end(nyx_status s) {
        done = s == NYX_OK;
        return s;
    }
};

// A one-shot call: its buffers come from the context's block, which earlier
// calls have finished with (each waits for its stream before it returns).
// Made once the arguments are found good and the context's device is the
// current one.
struct OneShot : CallGuard {
    OneShot(nyx_ctx *ctx, hipStream_t s) : CallGuard(s) {
        Arena &p = ctx->pool;
        const size_t want = std::min(std::max(p.demand + p.demand / 4u, kPoolMin), kPoolMax);
        if (!p.base || (p.demand > p.cap && want > p.cap)) {
            if (p.base) (void)hipFree(p.base);
            p.base = nullptr;
            p.cap = 0;
            void *q = nullptr;
            if (hipMalloc(&q, want) == hipSuccess) {
                p.base = static_cast<uint8_t *>(q);
                p.cap = want;
            } else {
                (void)hipGetLastError();   // every request spills
            }
        }
        p.spill = true;
        p.used = p.demand = p.wanted = 0;
    }
};

// Host to device through the pinned staging memory (at offset `at` of its
// upward part) where it fits there; the copy is then asynchronous and the
// staged bytes stay until the next synchronisation of the stream.
hipError_t copy_up(nyx_ctx *ctx, void *dst, const void *src, size_t n, size_t at, hipStream_t st) {
    if (at + n > kPinUp) return hipMemcpyAsync(dst, src, n, hipMemcpyHostToDevice, st);
    memcpy(ctx->pin + at, src, n);
    return hipMemcpyAsync(dst, ctx->pin + at, n, hipMemcpyHostToDevice, st);
}

// Tile queue asked of discovery: ROIs above tile_vox voxels are split.
struct TileQueue {
    uint32_t tile_vox = 0;
    uint32_t aux_values = 0;   // StepArgs::aux_values
};

// Work queue of a family whose items are tiles of about tile_vox voxels: the
// compaction cuts every ROI above tile_vox into fewer than 2 ceil(n / tile_vox)
// tiles (tiles_for), so the image's voxels bound the entries and the split
// ROIs.
nyx_status setup_tiles(nyx_ctx *ctx, Work &w, uint32_t roi_cap, const TileQueue &q) {
    StepArgs &a = w.args;
    const uint64_t n_split = std::min<uint64_t>(roi_cap, w.total_vox / q.tile_vox);
    const uint64_t n_items = roi_cap + 4u * (w.total_vox / q.tile_vox);
    if (n_items >= (1ull << 31)) return fail(ctx, NYX_ERR_UNSUPPORTED, "too many work items");
    HIPC(ctx, w.buckets.alloc((size_t)kClasses * std::max<uint64_t>(n_items, 1u) * sizeof(uint2)));
    HIPC(ctx, w.split_roi.alloc(std::max<uint64_t>(n_split, 1u) * 4u));
    a.buckets = w.buckets.as<uint2>();
    a.bucket_cap = (uint32_t)std::max<uint64_t>(n_items, 1u);
    a.split_roi = w.split_roi.as<uint32_t>();
    a.g_cap = (uint32_t)n_split;
    a.split_vox = a.tile_vox = q.tile_vox;
    a.aux_values = q.aux_values;
    a.enqueue = 1;
    return NYX_OK;
}

// Label tables, ROI discovery and the ROI descriptors (device), with the tile
// queue if one is asked for.  want_rois: the descriptors are wanted on the
// host too (fetch_rois).
nyx_status discover(nyx_ctx *ctx, const nyx_image *imgs, int32_t n, Work &w, hipStream_t st, bool want_rois,
                    const TileQueue *tiles = nullptr) {
    w.h_imgs.resize(n);
    uint32_t chunk = 0;
    uint64_t tv = 0, most_vox = 0;
    // one upload: image descriptors, first voxels, and the cleared label maxima
    std::vector<uint64_t> up((sizeof(ImgDesc) * n + 12u * n + 7u) / 8u, 0u);
    uint64_t *vbase = up.data() + sizeof(ImgDesc) / 8u * n;
    static_assert(sizeof(ImgDesc) % 8u == 0, "ImgDesc is followed by 64-bit words");
    for (int i = 0; i < n; ++i) {
        ImgDesc &d = w.h_imgs[i];
        memset(&d, 0, sizeof d);
        d.I = imgs[i].intensity;
        d.L = imgs[i].labels;
        d.B = nullptr;
        d.nz = (int32_t)imgs[i].nz;
        d.ny = (int32_t)imgs[i].ny;
        d.nx = (int32_t)imgs[i].nx;
        d.nvox = (uint32_t)(imgs[i].nz * imgs[i].ny * imgs[i].nx);
        d.chunk_base = chunk;
        {
            // discovery tiles: kScanTileRows rows (all planes flattened) by kScanTileCols columns
            uint64_t rows = (uint64_t)d.nz * (uint64_t)d.ny;
            chunk += (uint32_t)(((rows + kScanTileRows - 1u) / kScanTileRows) *
                                (((uint64_t)d.nx + kScanTileCols - 1u) / kScanTileCols));
        }
        vbase[i] = tv;
        tv += d.nvox;
        most_vox = std::max<uint64_t>(most_vox, d.nvox);
    }
    w.total_chunks = chunk;
    w.total_vox = tv;
    memcpy(up.data(), w.h_imgs.data(), sizeof(ImgDesc) * n);
    HIPC(ctx, w.imgs.alloc(up.size() * 8u));
    HIPC(ctx, copy_up(ctx, w.imgs.p, up.data(), up.size() * 8u, 0, st));
    w.vox_base = reinterpret_cast<uint64_t *>(w.imgs.as<ImgDesc>() + n);
    uint32_t *const dmax = reinterpret_cast<uint32_t *>(w.vox_base + n);
    // largest label per image sizes the label tables
    std::vector<uint32_t> big;
    uint32_t *hmax = reinterpret_cast<uint32_t *>(ctx->pin + kPinUp);
    if (sizeof(uint32_t) * n > kPinDown) {
        big.resize(n);
        hmax = big.data();
    }
    HIPC(ctx, launch_max_label(w.imgs.as<ImgDesc>(), n, most_vox, dmax, st));
    HIPC(ctx, hipMemcpyAsync(hmax, dmax, sizeof(uint32_t) * n, hipMemcpyDeviceToHost, st));
    HIPC(ctx, hipStreamSynchronize(st));
    uint64_t total = 0;
    for (int i = 0; i < n; ++i) total += (uint64_t)hmax[i] + 1u;
    if (total > kMaxLabelEntries || total > tv + (uint64_t)n) {
        // Label values too large (or too sparse) to index the table: the
        // table gets one entry per distinct label of each image instead.
        nyx_status s = build_label_dict(ctx, w, n, st);
        if (s != NYX_OK) return s;
        total = 0;
        for (int i = 0; i < n; ++i) total += (uint64_t)w.h_imgs[i].dict_n + 1u;
        if (total > kMaxLabelEntries)
            return fail(ctx, NYX_ERR_UNSUPPORTED, "%llu distinct labels (limit %llu)", (unsigned long long)total,
                        (unsigned long long)kMaxLabelEntries);
    } else {
        for (int i = 0; i < n; ++i) {
            w.h_imgs[i].dict = nullptr;
            w.h_imgs[i].dict_n = 0u;
            w.h_imgs[i].max_label = hmax[i];
        }
    }
    total = 0;
    for (int i = 0; i < n; ++i) {
        w.h_imgs[i].tab_base = (uint32_t)total;
        total += (uint64_t)w.h_imgs[i].max_label + 1u;
    }
    w.tab_total = (uint32_t)total;
    HIPC(ctx, copy_up(ctx, w.imgs.p, w.h_imgs.data(), sizeof(ImgDesc) * n, 0, st));
    for (auto &b : w.tab) HIPC(ctx, b.alloc(sizeof(uint32_t) * (size_t)total));
    w.n_blocks = (w.tab_total + 1023u) / 1024u;
    w.n_counters = C_BLOCKS + w.n_blocks;
    HIPC(ctx, w.counters.alloc(sizeof(uint32_t) * w.n_counters));

    StepArgs &a = w.args;
    memset(&a, 0, sizeof a);
    a.imgs = w.imgs.as<ImgDesc>();
    a.n_images = n;
    a.total_chunks = w.total_chunks;
    a.tab.cnt = w.tab[0].as<uint32_t>();
    a.tab.mn = w.tab[1].as<uint32_t>();
    a.tab.mx = w.tab[2].as<uint32_t>();
    a.tab.x0 = w.tab[3].as<int32_t>();
    a.tab.y0 = w.tab[4].as<int32_t>();
    a.tab.z0 = w.tab[5].as<int32_t>();
    a.tab.x1 = w.tab[6].as<int32_t>();
    a.tab.y1 = w.tab[7].as<int32_t>();
    a.tab.z1 = w.tab[8].as<int32_t>();
    a.tab.row = w.tab[9].as<uint32_t>();
    a.tab.total = w.tab_total;
    a.counters = w.counters.as<uint32_t>();
    HIPC(ctx, launch_reset(a, w.n_counters, st));
    HIPC(ctx, launch_scan(a, st));
    // The descriptors, in room for every label where that is little; else
    // the ROIs are counted first (a compaction with no ROI capacity writes
    // nothing) and the compaction repeated with room for them.
    const size_t roi_room = sizeof(RoiDesc) * (size_t)w.tab_total;
    const bool one_pass = w.tab_total <= kOnePassLabels && (!w.rois.arena || w.rois.arena->spill || w.rois.arena->fits(roi_room));
    const uint32_t *hc = reinterpret_cast<const uint32_t *>(ctx->pin + kPinUp);
    constexpr size_t kHead = 16u * sizeof(uint32_t);
    const uint32_t spec = want_rois && one_pass ? (uint32_t)std::min<size_t>(w.tab_total, (kPinDown - kHead) / sizeof(RoiDesc)) : 0u;
    nyx_status s = NYX_OK;
    for (int pass = one_pass ? 1 : 0; pass < 2; ++pass) {
        const uint32_t cap = pass == 0 ? 0u : (one_pass ? w.tab_total : w.n_rois);
        if (pass == 1) {
            if (tiles && (s = setup_tiles(ctx, w, cap, *tiles)) != NYX_OK) return s;
            HIPC(ctx, w.rois.alloc(sizeof(RoiDesc) * std::max<uint32_t>(cap, 1u)));
            a.rois = w.rois.as<RoiDesc>();
        }
        a.roi_cap = cap;
        if (pass == 1 && !one_pass) HIPC(ctx, launch_reset_counters(a, w.n_counters, st));
        HIPC(ctx, launch_compact(a, 0u, 0xFFFFFFFFu, st));
        HIPC(ctx, hipMemcpyAsync(ctx->pin + kPinUp, w.counters.p, kHead, hipMemcpyDeviceToHost, st));
        if (spec && pass == 1)
            HIPC(ctx, hipMemcpyAsync(ctx->pin + kPinUp + kHead, w.rois.p, sizeof(RoiDesc) * spec, hipMemcpyDeviceToHost, st));
        HIPC(ctx, hipStreamSynchronize(st));
        if (hc[C_ERR] & E_LABEL_RANGE) return fail(ctx, NYX_ERR_INTERNAL, "label range check failed during discovery");
        w.n_rois = hc[C_NROIS];
    }
    if (hc[C_ERR]) return fail(ctx, NYX_ERR_INTERNAL, "discovery failed (error bits %u)", hc[C_ERR]);
    if (w.n_rois <= spec) {
        const RoiDesc *h = reinterpret_cast<const RoiDesc *>(ctx->pin + kPinUp + kHead);
        w.h_rois.assign(h, h + w.n_rois);
        w.sizes.fill(w.h_rois);
        w.have_rois = true;
    }
    w.rois.shrink(sizeof(RoiDesc) * std::max<uint32_t>(w.n_rois, 1u));
    a.roi_cap = w.n_rois;
    w.n_split = std::min(hc[C_NSPLIT], a.g_cap);
    w.n_aux = hc[C_AUX];
    if (tiles) a.g_cap = w.n_split;
    return NYX_OK;
}

// The ROI descriptors on the host.
nyx_status fetch_rois(nyx_ctx *ctx, Work &w, hipStream_t st) {
    if (w.have_rois) return NYX_OK;
    w.h_rois.resize(w.n_rois);
    if (w.n_rois) {
        HIPC(ctx, hipMemcpyAsync(w.h_rois.data(), w.rois.p, sizeof(RoiDesc) * w.n_rois, hipMemcpyDeviceToHost, st));
        HIPC(ctx, hipStreamSynchronize(st));
    }
    w.sizes.fill(w.h_rois);
    w.have_rois = true;
    return NYX_OK;
}

struct Config {
    int mode = 0;            // 0 dense + list, 1 hash, 2 dense + scan, 3 packed dense + scan, 4 packed hash
    uint32_t kp = 1;
    uint32_t block = 256;
    uint32_t split_vox = 0, tile_vox = 0;
    uint32_t list_cap = 0, hash_cap = 0;
    int force_split = 0;
    int merged = 0;          // one matrix per ROI: the sum of the K offsets' matrices
    uint32_t copies = 1;     // privatised copies of each dense triangle (scan modes)
    float tile_scale = 1.f;  // split ROIs above tile_scale x the load-balance share
    int nonsym = 0;          // ordered counts: full squares (dense modes 2 and 3, or the hash)
    uint32_t small_cls = 0;  // packed hash: items of size classes below this take a launch of their own
    uint32_t small_kp = 0, small_cap = 0;   // with this many directions per pass and slots per direction
    uint32_t band_vox = 0;   // ROIs above this go to the banded kernel (0: none)
    uint32_t band_w = 0;     // band width (power of two)
    uint32_t band_dirs = 1;  // directions counted in one pass
};

// The banded kernel takes the large ROIs of hash-mode plans with symmetric
// matrices: band width = the largest power of two whose ng x width 32-bit
// cells fit kBandLds, for the most directions at once (each pass reads the
// region again) that leave a band of kBandWide levels: a narrower one sends
// too many pairs to global memory (60 M voxels at 1024 levels: the step took
// 1002 us with one direction of 32 levels, 3212 with two of 16; at 512 levels
// two of 32 took 690, one of 64 took 833).
void set_band(Config &c, uint32_t ng, int K) {
    c.band_vox = 0u;
    c.band_w = 0u;
    if ((c.mode != 1 && c.mode != 4) || c.nonsym) return;
    for (int dirs : {4, 2, 1}) {
        if (dirs > 1 && dirs > K) continue;
        uint32_t w = 1u;
        while (w * 2u <= ng && (uint64_t)ng * (w * 2u) * (uint32_t)dirs * 4u <= kBandLds) w *= 2u;
        c.band_dirs = (uint32_t)dirs;
        c.band_w = w;
        if (w >= kBandWide) break;
    }
    if (c.band_w < kBandMinW) c.band_w = 0u;
    else c.band_vox = std::max(c.split_vox, kBandMinVox);
}

// Voxels of a banded ROI's box per work item: as many as give every CU one
// item, as a block ends in a merge of its nonzero cells into global memory
// (one region of 60 M voxels, 1024 levels: 921 items of 2^18 voxels 535 us,
// 256 items 435), at least kBandTile (one of 4 M voxels: the step took 312 us
// at 2^18 voxels, 249 at 2^16).  Where regions smaller than a CU's share make
// that uneven, half a share, so that the tickets balance the work (a region of
// 64 M voxels beside 20 of 40000, 600 levels, k_band: 643 us with 256 items in
// all, 497 with half shares, 535 with 2^18 voxels; beside 300 at 1024 levels
// the whole step took 29.0 ms with the large region in one item, 4.8 so).
uint32_t band_tile(const Work &w, const Config &c, uint32_t n_cu, int K) {
    if (c.band_vox == 0u) return kBandTile;
    const uint32_t sets = ((uint32_t)K + c.band_dirs - 1u) / c.band_dirs;
    std::vector<RoiSizes::Box> box;   // the banded ROIs
    uint64_t total = 0;
    w.sizes.above(c.band_vox, [&](const RoiSizes::Box &r) {
        box.push_back(r);
        total += (uint64_t)r.rows * r.width;
    });
    const uint64_t share = std::min<uint64_t>(std::max<uint64_t>(kBandTile, total * sets / n_cu), 0x20000000u);
    for (uint64_t tile = share; tile <= share + share / 8u && box.size() * sets <= n_cu; tile += tile / 16u) {
        uint64_t items = 0;
        for (const RoiSizes::Box &b : box) items += band_blocks(b.rows, b.width, (uint32_t)tile) * (uint64_t)sets;
        if (items <= n_cu) return (uint32_t)tile;
    }
    return (uint32_t)std::max<uint64_t>(kBandTile, share / 2u);
}

const char *mode_name(int m) {
    switch (m) {
        case 0: return "dense-list";
        case 1:
        case 4: return "hash";
        case 2: return "dense-scan";
        default: return "dense16-scan";
    }
}

// Compaction entries (u32 cell indices) per lane of a scan chunk: one
// 16-byte read holds 8 packed 16-bit or 4 32-bit counters.
uint32_t scan_cells(int mode) { return mode == 3 ? (uint32_t)kScanCells : (uint32_t)kScanCells / 2u; }

// Cells of one dense matrix: the upper triangle, or the full square of
// ordered counts.
uint32_t mat_cells(uint32_t ng, bool nonsym) { return nonsym ? ng * ng : ng * (ng + 1u) / 2u; }

uint32_t u_words(int mode, uint32_t ng, bool nonsym = false) {
    uint32_t tri = mat_cells(ng, nonsym);
    uint32_t w = mode == 3 ? (tri + 1u) / 2u : tri;
    return (w + 3u) & ~3u;
}

// Marginal words per reducing wave: row, sum and difference marginals, plus
// the column marginal of an ordered matrix.
// (16-bit counters in the packed hash mode, whose items are small).
// (pair: row and difference marginals share words).
uint32_t marg_words(uint32_t ng, bool nonsym, int mode = 0, bool pair = false) {
    const uint32_t n = (nonsym ? 5u : (pair ? 3u : 4u)) * ng;
    return mode == 4 ? (n + 1u) / 2u : n;
}

// Bits of a 0-based level.
uint32_t level_bits(uint32_t ng) {
    uint32_t b = 1u;
    while ((1u << b) < ng) ++b;
    return b;
}

// Most voxels of a packed-hash item: the counts left in a slot's word, and
// marginals (at most four times the pairs of a direction) of 16 bits.
uint32_t packed_item_max(uint32_t ng) {
    const uint32_t lb = level_bits(ng);
    return lb > 12u ? 0u : std::min((1u << (32u - 2u * lb)) - 1u, 16383u);
}

// ring: reserve an LDS level ring for the staged accumulation, sized to the
// LDS the work-group can take without lowering its occupancy.
LdsLayout lay_out(const Config &c, uint32_t ng, int K, bool ring, bool pair) {
    LdsLayout L;
    memset(&L, 0, sizeof L);
    L.mode = (uint32_t)c.mode;
    L.kp = c.kp;
    L.nwaves = c.block / kWave;
    L.tri_pad = u_words(c.mode, ng, c.nonsym != 0);
    L.copies = (c.mode == 2 || c.mode == 3) ? c.copies : 1u;
    L.list_cap = c.list_cap;
    L.hash_cap = c.hash_cap;
    uint32_t off = 0;
    auto take = [&](uint32_t bytes) {
        uint32_t o = off;
        off += (bytes + 15u) & ~15u;
        return o;
    };
    if (c.mode == 4) {
        L.n_tri = c.kp;
        L.lvl_bits = level_bits(ng);
        L.cnt_bits = 32u - 2u * L.lvl_bits;
        L.item_max = std::min(packed_item_max(ng), packed_voxels(c.hash_cap));
        L.u_off = take(L.n_tri * c.hash_cap * 4u);
    } else if (c.mode != 1) {
        L.n_tri = c.merged ? 1u : c.kp;   // merged: one triangle for all offsets
        L.u_off = take(L.n_tri * L.copies * L.tri_pad * 4u);
    } else {
        L.hkey_off = take(c.hash_cap * 4u);
        L.hcnt_off = take(c.hash_cap * 4u);
    }
    L.list_off = take(c.kp * c.list_cap * 4u);
    L.lcnt_off = take(c.kp * 4u);
    L.buf_off = take((c.mode == 2 || c.mode == 3) ? L.nwaves * scan_buf_entries(scan_cells(c.mode)) * 2u : 0u);
    L.marg_sets = std::min(L.nwaves, c.merged ? 1u : c.kp);   // one set per wave that reduces a matrix
    L.marg_off = take(L.marg_sets * marg_words(ng, c.nonsym != 0, c.mode, pair) * 4u);
    L.marg_pair = pair ? 1u : 0u;
    L.misc_off = take(128u * 4u);
    if ((c.mode == 2 || c.mode == 3) && !c.nonsym) L.ro_off = take((ng + 1u) * 4u);
    L.item_off = take((uint32_t)kTicketChunk * kItemBytes);
    if (ring && ng <= 255u && c.mode != 1 && !c.nonsym) {
        // work-groups per CU: LDS-bound, and at most kMaxGroupsPerCu (the
        // single-precision kernel's register bound)
        const uint32_t per_group = kLdsBudget / std::max(1u, std::min(kMaxGroupsPerCu, kLdsBudget / off));
        const uint32_t bytes = off < per_group ? std::min(kRingMax, (per_group - off) & ~15u) : 0u;
        if (bytes >= kRingMin) {
            L.ring_off = take(bytes);
            L.ring_bytes = bytes;
        }
    }
    L.bytes = off;
    return L;
}

// Work-groups of the persistent kernel per CU for a given LDS footprint.
uint32_t groups_per_cu(uint64_t lds_bytes) {
    return (uint32_t)std::min<uint64_t>(kMaxGroupsPerCu, kLdsBudget / std::max<uint64_t>(lds_bytes, 1u));
}

// The row and difference marginals of a symmetric matrix share words where
// that lets a second work-group onto a CU (or one of 512 threads in the place
// of 256: widen_block) and an unsplit item's marginals (at most twice its
// voxels) stay below 2^16; what fits at all is found without it.  At 128
// levels: 4 directions two groups instead of one (2000 cells, batch kernel 104
// us with the best other split, 88 so), 8 directions 512 threads instead of
// 256 (4400 cells, distances 1 and 2: 696, 454).  From two groups to three it
// lost at 100 levels (320, 363).
LdsLayout make_layout(const Config &c, uint32_t ng, int K, bool ring) {
    const LdsLayout L = lay_out(c, ng, K, ring, false);
    if (c.mode != 3 || c.nonsym || c.merged || c.split_vox > 32767u || groups_per_cu(L.bytes) > 1u)
        return L;
    const LdsLayout P = lay_out(c, ng, K, ring, true);
    return groups_per_cu(P.bytes) > groups_per_cu(L.bytes) ? P : L;
}

// Work items of a ROI; banded ROIs (above band_vox voxels, 0: none) have none.
uint32_t tile_count(uint32_t n, uint32_t rows, uint32_t width, uint32_t split_vox, uint32_t tile_vox, uint32_t band_vox) {
    if (band_vox && n > band_vox) return 0u;
    const Tiling t = tiles_for(n, rows, width, split_vox, tile_vox);
    return t.row_blocks * t.col_blocks;
}

// Largest voxel count any work item can hold under a split rule.
uint64_t max_item_vox(const RoiSizes &rois, uint32_t split_vox, uint32_t tile_vox) {
    uint64_t m = rois.up_to(split_vox).most;
    rois.above(split_vox, [&](const RoiSizes::Box &r) {
        m = std::max<uint64_t>(m, item_bound(r.n, r.rows, r.width, tiles_for(r.n, r.rows, r.width, split_vox, tile_vox)));
    });
    return m;
}

// Packed hash tables, one per direction of a pass, for items much smaller
// than their triangle.  The main launch takes any item up to the split size;
// items of the smaller size classes take a second one whose tables (and so
// whose LDS) are sized for them, with every work-group slot that frees: the
// class boundary is the one with the least work per slot, counting an item
// as its voxels plus the fixed part of its reductions (about 500 voxels'
// worth at 256 levels).  mode 0 (not 4) when nothing fits.
Config packed_config(const nyx_ctx *ctx, const Work &w, uint32_t ng, int K, int force_split, uint32_t block,
                     uint32_t lb, bool nonsym, float tile_scale) {
    Config best;
    const uint32_t n_max = packed_item_max(ng);
    // The largest split that fits (a split ROI costs a merge in global
    // memory), then the most directions per pass: every pass repeats the
    // sweep and the fixed part of the reductions (2000 cells at 256 levels:
    // four directions in one 512-thread group per CU beat one in five groups).
    for (uint32_t kp = (uint32_t)K; kp >= 1u; kp = kp == 1u ? 0u : (kp + 1u) / 2u) {
        for (uint32_t split = std::min(lb, n_max);; split /= 2u) {
            const uint64_t mi = max_item_vox(w.sizes, split, split);
            if (mi <= n_max) {
                Config c;
                c.mode = 4; c.kp = kp; c.block = block; c.split_vox = c.tile_vox = split;
                // (room for a whole item of the split size, whatever the planned images hold)
                c.hash_cap = packed_slots((uint32_t)std::max<uint64_t>(mi, split), ~0u);
                c.force_split = force_split; c.nonsym = nonsym ? 1 : 0; c.tile_scale = tile_scale;
                if (make_layout(c, ng, K, false).bytes <= kLdsBudget) {
                    if (best.mode != 4 || split > best.split_vox) best = c;
                    break;
                }
            }
            if (split < 1024u) break;
        }
    }
    if (best.mode != 4) return best;
    set_band(best, ng, K);
    if (!force_split) {
        // voxels and items by size class, as the device will bucket them
        double vox[kClasses] = {}, num[kClasses] = {};
        const uint32_t sc = size_class(best.split_vox);
        for (uint32_t cl = 0; cl < sc; ++cl) {
            vox[cl] = (double)w.sizes.of_class[cl].vox;
            num[cl] = (double)w.sizes.of_class[cl].count;
        }
        w.sizes.above((1u << sc) - 1u, [&](const RoiSizes::Box &r) {
            if (best.band_vox && r.n > best.band_vox) return;   // (no batch items)
            const Tiling t = tiles_for(r.n, r.rows, r.width, best.split_vox, best.tile_vox);
            const uint32_t cl = size_class(item_bound(r.n, r.rows, r.width, t));
            vox[cl] += r.n;
            num[cl] += (double)t.row_blocks * t.col_blocks;
        });
        const double fixed = 500.0 * (1.0 + ng / 256.0);
        const auto work = [&](uint32_t lo, uint32_t hi) {
            double s = 0.0;
            for (uint32_t cl = lo; cl < hi; ++cl) s += vox[cl] + fixed * num[cl];
            return s;
        };
        const double g_main = groups_per_cu(make_layout(best, ng, K, false).bytes);
        double score = work(0u, kClasses) / g_main * 0.8;   // (a second launch has to be worth its cost)
        for (uint32_t cls = 6u; cls <= 11u; ++cls) {
            for (uint32_t kp = (uint32_t)K; kp >= 1u; kp = kp == 1u ? 0u : (kp + 1u) / 2u) {
                Config s = best;
                s.kp = kp;
                s.hash_cap = packed_slots((1u << cls) - 1u, ~0u);
                const uint32_t bytes = make_layout(s, ng, K, false).bytes;
                if (bytes > kLdsBudget || s.hash_cap >= best.hash_cap) continue;
                const double passes = ((double)K + kp - 1) / kp / (((double)K + best.kp - 1) / best.kp);
                const double t = work(0u, cls) * passes / groups_per_cu(bytes) + work(cls, kClasses) / g_main;
                if (t < score) {
                    score = t;
                    best.small_cls = cls;
                    best.small_kp = kp;
                    best.small_cap = s.hash_cap;
                }
            }
        }
    }
    return best;
}

// Item and split-slot counts implied by a configuration.
void count_items(const RoiSizes &rois, const Config &c, uint64_t *items, uint32_t *n_split) {
    const uint64_t whole = rois.up_to(c.split_vox).count;
    uint64_t it = whole, ns = c.force_split ? whole : 0u;
    rois.above(c.split_vox, [&](const RoiSizes::Box &r) {
        const uint32_t nt = tile_count(r.n, r.rows, r.width, c.split_vox, c.tile_vox, c.band_vox);
        it += nt;
        if (nt != 1u || c.force_split) ++ns;
    });
    *items = it;
    *n_split = (uint32_t)ns;
}

// Device memory of a step's queue, matrices and records.
uint64_t step_bytes(const Work &w, int K_out, uint32_t ng, bool nonsym, uint64_t items, uint32_t n_split) {
    const uint64_t mats = (uint64_t)n_split * K_out, mats1 = (uint64_t)std::max<uint32_t>(n_split, 1u) * K_out;
    const uint64_t records = (uint64_t)std::max<uint32_t>(w.n_rois, 1u) * K_out;
    return (uint64_t)kClasses * std::max<uint64_t>(items, 1u) * 8u + mats * ng * ng * 8u + records * sizeof(DirSums) +
           (nonsym ? records * sizeof(DirSumsY) : 16u) + n_split * 8u +
           mats1 * (16u * ng + 32u + 8u * std::max(1u, ng / 8u));
}

// Whether the packed hash `c` may take the place of `d`, what else the levels
// and regions fit.  Its tables hold fewer voxels, so it may split regions that
// `d` takes whole, and each of them then costs its matrices in global memory,
// cleared, merged into and reduced every pass at about 0.5 us a MB.  Measured
// savings are 1.3e-6 us a triangle cell of every item and direction against
// dense triangles, and 0.004 us an item and direction, or more, against 64-bit
// slots; so the extra bytes may be about those cells, or 7 KB each.  (400
// regions of 1100 voxels, one direction: 1100 levels 214 us in 64-bit slots and
// 1952 split in packed tables, 2048 levels 259 and 5780; 400 regions of 20000
// voxels among 30000 of 400 at 256 levels: 7039 us as triangles, 1441 packed
// with the 400 split.)  limit: bytes that the step may take (0: no limit).
bool packed_worth(const Work &w, const Config &c, const Config &d, uint32_t ng, int K, uint64_t limit) {
    uint64_t items_c, items_d;
    uint32_t split_c, split_d;
    count_items(w.sizes, c, &items_c, &split_c);
    count_items(w.sizes, d, &items_d, &split_d);
    const uint64_t need_c = step_bytes(w, K, ng, c.nonsym != 0, items_c, split_c),
                   need_d = step_bytes(w, K, ng, d.nonsym != 0, items_d, split_d);
    if (need_c <= need_d) return true;
    const uint64_t each = d.mode == 1 ? 7168u : mat_cells(ng, c.nonsym != 0);
    return need_c - need_d <= std::min<uint64_t>(items_d * (uint64_t)K * each, kPackedExtra) &&
           (limit == 0u || need_c <= limit);
}

Config default_config(const std::vector<Config> &cands, const Work &w, uint32_t ng, int K);

// Feasible LDS configurations for this workload, one per accumulation mode,
// each with as many directions per pass as fit.  Dense triangles first, then
// the packed hash where it is worth its splits (packed_worth); where no
// triangle fits, the hash of 64-bit slots in its place.
// merged: every offset counts into one LDS triangle in one pass, so only the
// dense scan modes qualify, and packed 16-bit counters need K x (voxels of an
// item) < 65536 (offered only when that bound leaves the load-balance tile
// size alone; 32-bit counters otherwise).  copies: privatised copies of each
// dense scan triangle (list and hash modes keep one); tile_scale scales the
// load-balance share above which ROIs are split; limit: see packed_worth.
std::vector<Config> candidate_configs(const nyx_ctx *ctx, const Work &w, uint32_t ng, int K, int force_split,
                                      uint32_t block, bool merged = false, uint32_t copies = 1u,
                                      float tile_scale = 1.f, bool nonsym = false, uint64_t limit = 0) {
    std::vector<Config> out;
    const uint32_t nw = block / kWave;
    const uint32_t tri = mat_cells(ng, nonsym);
    // LDS besides triangles / hash / lists: marginals for up to nw directions
    // at a time, misc, alignment slack
    auto fixed_for = [&](uint32_t kp) {
        // (marginal sets, misc words, staged item descriptors, row-offset table, alignment slack)
        return (std::min(nw, kp) * marg_words(ng, nonsym) * 4u + 15u) / 16u * 16u + 128u * 4u +
               (uint32_t)kTicketChunk * kItemBytes + ((ng + 1u) * 4u + 15u) / 16u * 16u + 64u * 4u + 64;
    };
    const uint32_t fixed = fixed_for(1u);
    const uint64_t total_vox = w.sizes.all.vox;
    // load balance: split ROIs that would take more than ~1/4 of one
    // work-group's share of the voxels
    uint64_t share = (uint64_t)((double)(total_vox / ((uint64_t)std::max(ctx->n_cu, 1) * 4u) + 1u) * tile_scale);
    const uint32_t lb = (uint32_t)std::min<uint64_t>(std::max<uint64_t>(share, 4096u), 1u << 20);
    std::vector<Config> later;
    for (int mode : {3, 2, 0}) {
        if ((merged || nonsym) && mode == 0) continue;   // the returning-atomic list keeps triangles only
        if (copies > 1u && mode == 0) continue;   // the returning-atomic list keeps one triangle
        const uint32_t cell_max = merged ? 65535u / (uint32_t)K : 65535u;   // 16-bit counters
        uint32_t split = mode == 3 ? std::min<uint32_t>(lb, cell_max) : lb;
        uint64_t mi = max_item_vox(w.sizes, split, split);
        while (mode == 3 && mi > cell_max && split > 64u) {
            split /= 2u;
            mi = max_item_vox(w.sizes, split, split);
        }
        if (mode == 3 && mi > cell_max) continue;
        if (merged && mode == 3 && split < std::min<uint32_t>(lb, 65535u)) continue;
        const bool scan = mode == 2 || mode == 3;
        const uint32_t list_cap = scan ? 0u : (uint32_t)std::min<uint64_t>(tri, std::max<uint64_t>(mi, 1u));
        const uint64_t scan_buf = scan ? (uint64_t)nw * scan_buf_entries(scan_cells(mode)) * 2u : 0u;
        const uint32_t cp = scan ? copies : 1u;
        for (uint32_t kp = (uint32_t)K; kp >= (merged ? (uint32_t)K : 1u); --kp) {
            const uint32_t n_tri = merged ? 1u : kp;
            uint64_t bytes = (uint64_t)n_tri * cp * u_words(mode, ng, nonsym) * 4u + (uint64_t)kp * list_cap * 4u + kp * 4u +
                             fixed_for(n_tri) + scan_buf;
            if (bytes <= kLdsBudget) {
                Config c;
                c.mode = mode; c.kp = kp; c.block = block; c.split_vox = split; c.tile_vox = split;
                c.list_cap = list_cap; c.force_split = force_split; c.merged = merged ? 1 : 0;
                c.copies = cp; c.tile_scale = tile_scale; c.nonsym = nonsym ? 1 : 0;
                out.push_back(c);
                if (merged) break;
                // many offsets: fewer directions per pass cost another pass
                // over the voxels but leave LDS for more work-groups per CU
                // (timed by the autotuner, never the default)
                if (mode == 3 && (K > 4 || groups_per_cu(bytes) < 3u))
                    for (uint32_t parts : {2u, 3u, 4u}) {
                        Config f = c;
                        f.kp = ((uint32_t)K + parts - 1u) / parts;
                        if (f.kp < kp && (later.empty() || later.back().kp != f.kp)) later.push_back(f);
                    }
                break;
            }
        }
    }
    out.insert(out.end(), later.begin(), later.end());
    if (merged || copies > 1u) return out;
    Config packed;
    if (packed_item_max(ng) > 0u) packed = packed_config(ctx, w, ng, K, force_split, block, lb, nonsym, tile_scale);
    if (!out.empty()) {
        if (packed.mode == 4 && packed_worth(w, packed, default_config(out, w, ng, K), ng, K, limit)) out.push_back(packed);
        return out;
    }
    // hash of 64-bit slots: items small enough that kp directions of pairs fill
    // at most half the table
    for (uint32_t kp = (uint32_t)K; kp >= 1u && fixed < kLdsBudget; --kp) {
        for (uint32_t hc = 1u << 14; hc >= 512u; hc >>= 1) {
            uint32_t per_dir = hc / (2u * kp);
            if (per_dir < 64u) continue;
            uint32_t split = std::min<uint32_t>(per_dir, lb);
            uint64_t mi = max_item_vox(w.sizes, split, split);
            while (mi > per_dir && split > 16u) {
                split /= 2u;
                mi = max_item_vox(w.sizes, split, split);
            }
            if (mi > per_dir) continue;
            uint32_t list_cap = (uint32_t)std::max<uint64_t>(mi, 1u);
            uint64_t bytes = (uint64_t)hc * 8u + (uint64_t)kp * list_cap * 4u + kp * 4u + fixed_for(kp);
            if (bytes <= kLdsBudget) {
                Config c;
                c.mode = 1; c.kp = kp; c.block = block; c.hash_cap = hc; c.split_vox = split; c.tile_vox = split;
                c.list_cap = list_cap; c.force_split = force_split; c.tile_scale = tile_scale;
                c.nonsym = nonsym ? 1 : 0;
                set_band(c, ng, K);
                out.push_back(packed.mode == 4 && packed_worth(w, packed, c, ng, K, limit) ? packed : c);
                return out;
            }
        }
    }
    if (packed.mode == 4) out.push_back(packed);
    return out;
}

// Default choice without timing.  An ordered scan of the triangle costs
// O(Ng^2) per direction and item and its LDS holds few work-groups, but its
// atomics return nothing; the packed hash costs O(pairs) and LDS in
// proportion to the item, with two LDS round trips a pair.  The line lies at
// a triangle of 16 times the average item.  Batch kernel, scan and hash, in
// us, on one 2048 x 2048 image: 2000 cells of 100-5000 voxels (1250 on
// average) 41 and 155 at 64 levels, 144 and 192 at 128 (6.6 times), 448 and
// 212 at 256 (26 times); 8000 of 30-600 (190) 90 and 138 at 64 levels (11
// times), 188 and 146 at 100 (27 times), 1384 and 188 at 256.  (The list of
// the returning-atomic mode lost to one of them everywhere: 81, 181, 332 on
// the first and 118, 269, 774 us on the second; it stays for callers that ask
// for it and where neither fits.)
Config default_config(const std::vector<Config> &cands, const Work &w, uint32_t ng, int K) {
    const RoiSizes::Sum &all = w.sizes.all;
    const uint64_t avg = all.count ? std::max<uint64_t>(1u, all.vox / all.count) : 1u;
    const uint64_t tri = (uint64_t)ng * (ng + 1u) / 2u;
    bool any_scan = false, any_hash = false;
    for (const Config &c : cands) {
        any_scan |= c.mode == 2 || c.mode == 3;
        any_hash |= c.mode == 4;
    }
    for (const Config &c : cands) {
        if (c.mode != 4) continue;
        // (the average of the regions that the banded kernel would leave it)
        const RoiSizes::Sum left = c.band_vox ? w.sizes.up_to(c.band_vox) : all;
        if (!any_scan || tri > 16u * (left.count ? std::max<uint64_t>(1u, left.vox / left.count) : avg)) return c;
    }
    const bool prefer_scan = any_scan && (any_hash || tri <= 8u * avg);
    // among the candidates of the preferred kind: fewest passes over the
    // voxels per work-group slot (passes / work-groups per CU); ties keep the
    // earlier candidate (more directions per pass)
    const Config *best = nullptr;
    double best_score = 0.0;
    for (const Config &c : cands) {
        const bool scan = c.mode == 2 || c.mode == 3;
        if (!(prefer_scan == scan || c.mode == 1)) continue;
        const uint32_t passes = ((uint32_t)K + c.kp - 1u) / c.kp;
        const double score = (double)passes / (double)std::max(1u, groups_per_cu(make_layout(c, ng, K, false).bytes));
        if (!best || score < best_score) { best = &c; best_score = score; }
    }
    return best ? *best : cands.front();
}

nyx_status choose_config(nyx_ctx *ctx, const Work &w, uint32_t ng, int K, int force_split, uint32_t block,
                         Config &cfg, bool nonsym = false) {
    std::vector<Config> c = candidate_configs(ctx, w, ng, K, force_split, block, false, 1u, 1.f, nonsym);
    if (c.empty()) return fail(ctx, NYX_ERR_UNSUPPORTED, "no LDS configuration fits n_bins=%u with %d offsets", ng, K);
    cfg = default_config(c, w, ng, K);
    return NYX_OK;
}

// Whether a candidate is what a forced accumulation mode names: the dense
// modes 0, 2 and 3 by number; the hash table, packed or not, where no dense
// triangle fits.
bool is_mode(const Config &c, int mode, const std::vector<Config> &cands) {
    if (mode != 1) return c.mode == mode && mode != 4;
    return (c.mode == 1 || c.mode == 4) && (cands.front().mode == 1 || cands.front().mode == 4);
}

// Row-sweep eligibility: all images 2D and every offset of each pass one of
// the four distance-1 in-plane classes, each class at most once per pass.
bool sweep_table(const std::vector<ImgDesc> &imgs, const nyx_offset *off, int K, uint32_t kp,
                 int8_t (*sweep)[4], uint32_t *flip, int max_passes) {
    memset(sweep, -1, sizeof(int8_t[4]) * max_passes);
    memset(flip, 0, sizeof(uint32_t) * max_passes);
    for (const ImgDesc &d : imgs)
        if (d.nz != 1) return false;
    int pass = 0;
    for (int d0 = 0; d0 < K; d0 += (int)kp, ++pass) {
        if (pass >= max_passes) return false;
        for (int d = d0; d < std::min(K, d0 + (int)kp); ++d) {
            const nyx_offset &o = off[d];
            if (o.dz != 0 || abs(o.dy) > 1 || abs(o.dx) > 1) return false;
            int cls;
            if (o.dy == 0) cls = 0;
            else if (o.dx == 0) cls = 1;
            else if (o.dy * o.dx < 0) cls = 2;   // (-1, +1) or (+1, -1)
            else cls = 3;                        // (-1, -1) or (+1, +1)
            if (sweep[pass][cls] >= 0) return false; // the same class twice in a pass
            sweep[pass][cls] = (int8_t)(d - d0);
            // the sweep's own directions: (0, 1), (-1, 0), (-1, 1) and (1, 1)
            const bool own = cls == 0 ? o.dx > 0 : (cls == 3 ? o.dy > 0 : o.dy < 0);
            if (!own) flip[pass] |= 1u << (d - d0);
        }
    }
    return true;
}

// 3D row-sweep eligibility: every offset of each pass a distance-1 offset,
// each of the 13 neighbour classes at most once per pass.
bool sweep3_table(const nyx_offset *off, int K, uint32_t kp, uint64_t *sweep, int max_passes) {
    memset(sweep, 0, sizeof(uint64_t) * max_passes);
    int pass = 0;
    for (int d0 = 0; d0 < K; d0 += (int)kp, ++pass) {
        if (pass >= max_passes) return false;
        for (int d = d0; d < std::min(K, d0 + (int)kp); ++d) {
            const nyx_offset &o = off[d];
            if (abs(o.dz) > 1 || abs(o.dy) > 1 || abs(o.dx) > 1) return false;
            const int at = 4 * class3d(o.dz, o.dy, o.dx);
            if (sweep[pass] >> at & 15u) return false;   // the same class twice in a pass
            sweep[pass] |= (uint64_t)(d - d0 + 1) << at;
        }
    }
    return true;
}

void set_sweep(StepArgs &a, const std::vector<ImgDesc> &imgs, const nyx_offset *off, int K, uint32_t kp) {
    a.sweep_ok = sweep_table(imgs, off, K, kp, a.sweep, a.sweep_flip, kMaxSweepPasses) ? 1 : 0;
    a.sweep3_ok = !a.sweep_ok && sweep3_table(off, K, kp, a.sweep3, kMaxSweepPasses) ? 1 : 0;
}

// A configuration whose LDS leaves room for one 256-thread work-group per CU
// runs with 512 threads instead when its layout (a scan buffer and a set of
// marginals per reducing wave) still fits: eight waves then share the CU's
// latency instead of four.  The 3D row sweep (vol) has no barrier inside its
// accumulation, so it takes 512 threads wherever they leave the number of
// work-groups on a CU alone, up to the two its registers allow (500 ellipsoids
// at 64 levels and 13 offsets: batch kernel 669 us with 256, 413 with 512).
Config widen_block(const Config &c, uint32_t ng, int K, bool vol) {
    if (c.block != 256u) return c;
    const uint32_t groups = groups_per_cu(make_layout(c, ng, K, false).bytes);
    if (groups > (vol ? 2u : 1u)) return c;
    Config w = c;
    w.block = 512u;
    const uint32_t bytes = make_layout(w, ng, K, false).bytes;
    return bytes <= kLdsBudget && groups_per_cu(bytes) == groups ? w : c;
}

// Whether the 3D row sweep accumulates a configuration's passes.
bool takes_sweep3(const Work &w, const Config &c, const nyx_offset *off, int K) {
    StepArgs t;
    set_sweep(t, w.h_imgs, off, K, c.kp);
    return !c.nonsym && t.sweep3_ok;
}

// Allocates queue, split matrices and fills the step arguments.
nyx_status setup_step(nyx_ctx *ctx, Work &w, const Config &cfg, const nyx_offset *off, int K, uint32_t ng,
                      int fp64, uint32_t g_cap_override, int64_t cap_bytes, int64_t *ws_bytes) {
    StepArgs &a = w.args;
    uint64_t items;
    uint32_t n_split;
    count_items(w.sizes, cfg, &items, &n_split);
    if (g_cap_override) n_split = g_cap_override;
    if (items >= (1ull << 31)) return fail(ctx, NYX_ERR_UNSUPPORTED, "too many work items");
    uint32_t bucket_cap = (uint32_t)std::max<uint64_t>(items, 1u);
    const int K_out = cfg.merged ? 1 : K;
    uint64_t g_bytes = (uint64_t)n_split * K_out * (uint64_t)ng * ng * 8u;
    const uint64_t sums_bytes = (uint64_t)std::max<uint32_t>(w.n_rois, 1u) * K_out * sizeof(DirSums);
    const uint64_t sums_y_bytes =
        cfg.nonsym ? (uint64_t)std::max<uint32_t>(w.n_rois, 1u) * K_out * sizeof(DirSumsY) : 16u;
    uint64_t need = step_bytes(w, K_out, ng, cfg.nonsym != 0, items, n_split);
    for (auto &b : w.tab) need += b.bytes;
    need += w.rois.bytes + w.counters.bytes;
    if (ws_bytes) *ws_bytes = (int64_t)need;
    if (cap_bytes > 0 && (int64_t)need > cap_bytes)
        return fail(ctx, NYX_ERR_OOM, "workspace needs %llu bytes, cap is %lld", (unsigned long long)need,
                    (long long)cap_bytes);
    HIPC(ctx, w.buckets.alloc((size_t)kClasses * bucket_cap * sizeof(uint2)));
    HIPC(ctx, w.G.alloc(std::max<uint64_t>(g_bytes, 16u)));
    HIPC(ctx, w.dsums.alloc(sums_bytes));
    HIPC(ctx, w.dsums_y.alloc(sums_y_bytes));
    HIPC(ctx, w.split_roi.alloc((size_t)std::max<uint32_t>(n_split, 1u) * 4u));
    HIPC(ctx, w.band_roi.alloc((size_t)std::max<uint32_t>(n_split, 1u) * 4u));
    // two-pass reduction of split matrices: enough row chunks to fill the chip
    const uint64_t mats = (uint64_t)std::max<uint32_t>(n_split, 1u) * K_out;
    const uint32_t chunks = (uint32_t)std::max<uint64_t>(
        1u, std::min<uint64_t>(std::max(1u, ng / 8u), (2u * (uint64_t)std::max(ctx->n_cu, 1) + mats - 1u) / mats));
    HIPC(ctx, w.smarg.alloc((size_t)mats * 4u * ng * 4u));
    HIPC(ctx, w.stot.alloc((size_t)mats * 4u * 8u));
    HIPC(ctx, w.splp.alloc((size_t)mats * chunks * 8u));
    a.buckets = w.buckets.as<uint2>();
    a.bucket_cap = bucket_cap;
    a.G = w.G.as<uint64_t>();
    a.g_cap = n_split;
    a.dsums = w.dsums.as<DirSums>();
    a.dsums_y = w.dsums_y.as<DirSumsY>();
    a.nonsym = cfg.nonsym;
    a.split_roi = w.split_roi.as<uint32_t>();
    a.band_roi = w.band_roi.as<uint32_t>();
    a.smarg = w.smarg.as<uint32_t>();
    a.stot = w.stot.as<uint64_t>();
    a.splp = w.splp.as<double>();
    a.split_chunks = chunks;
    a.band_vox = cfg.band_vox;
    a.band_w = cfg.band_w;
    a.band_dirs = cfg.band_dirs;
    a.band_tile = band_tile(w, cfg, (uint32_t)ctx->n_cu, K);
    for (int k = 0; k < K; ++k) {
        a.off[k][0] = off[k].dz;
        a.off[k][1] = off[k].dy;
        a.off[k][2] = off[k].dx;
    }
    a.K = K;
    a.K_out = K_out;
    a.merged = cfg.merged;
    a.ng = (int32_t)ng;
    a.split_vox = cfg.split_vox;
    a.tile_vox = cfg.tile_vox;
    a.force_split = cfg.force_split;
    a.enqueue = 1;
    a.cls_lo = 0u;
    a.cls_hi = kClasses;
    a.tickets = C_TICKETS;
    a.fp64 = fp64;
    // (ordered counts in volumes and at other distances take the gather: the
    // 3D sweep and the staged ring fold a direction and its reverse together)
    set_sweep(a, w.h_imgs, off, K, cfg.kp);
    if (cfg.nonsym) a.sweep3_ok = 0;
    a.lds = make_layout(cfg, ng, K, !a.sweep_ok && !a.sweep3_ok);
    return NYX_OK;
}

nyx_status set_outputs(nyx_ctx *ctx, StepArgs &a, nyx_roi_table *rois, void *table, uint32_t table_rows) {
    a.table = table;
    a.table_rows = table_rows;
    a.o_label = rois ? rois->label : nullptr;
    a.o_image = rois ? rois->image : nullptr;
    a.o_n = rois ? rois->n_vox : nullptr;
    a.o_min = rois ? rois->vmin : nullptr;
    a.o_max = rois ? rois->vmax : nullptr;
    a.o_bbox = rois ? rois->bbox : nullptr;
    (void)ctx;
    return NYX_OK;
}

void release_streams(nyx_ctx *c) {
    if (c->join_event) (void)hipEventDestroy(c->join_event);
    if (c->fork_event) (void)hipEventDestroy(c->fork_event);
    if (c->side_stream) (void)hipStreamDestroy(c->side_stream);
    if (c->capture_stream) (void)hipStreamDestroy(c->capture_stream);
}

// The batch kernel over the queue: one launch, or one for the larger size
// classes and one, with a layout of its own, for the smaller.
hipError_t launch_batch_main(const nyx_plan *p, hipStream_t st) {
    StepArgs a = p->w.args;
    if (p->small_cls) a.cls_lo = p->small_cls;
    return launch_batch(a, p->grid, p->block, kNone, st);
}

hipError_t launch_batch_small(const nyx_plan *p, hipStream_t st) {
    if (!p->small_cls) return hipSuccess;
    StepArgs a = p->w.args;
    a.cls_lo = 0u;
    a.cls_hi = p->small_cls;
    a.tickets = C_TICKETS2;
    a.lds = p->small_lds;
    nyx_offset off[kMaxOffsets];
    for (int k = 0; k < a.K; ++k) off[k] = nyx_offset{a.off[k][0], a.off[k][1], a.off[k][2]};
    set_sweep(a, p->w.h_imgs, off, a.K, p->small_kp);
    if (a.nonsym) a.sweep3_ok = 0;
    return launch_batch(a, p->small_grid, 256u, kNone, st);
}

hipError_t launch_batches(const nyx_plan *p, hipStream_t st) {
    const hipError_t e = launch_batch_main(p, st);
    return e != hipSuccess ? e : launch_batch_small(p, st);
}

// The counting kernels of a captured step: the small size classes on a branch
// of the graph of their own, beside the banded regions and the main launch
// (they share no counters, and add to matrices and records of different
// regions).  Started first, the work-groups with the large LDS layouts leave
// room for some of the small ones; the other way round they found none.
hipError_t launch_counting_forked(const nyx_plan *p, hipStream_t st) {
    const nyx_ctx *ctx = p->ctx;
    const StepArgs &a = p->w.args;
    hipError_t e = hipEventRecord(ctx->fork_event, st);
    if (e == hipSuccess) e = hipStreamWaitEvent(ctx->side_stream, ctx->fork_event, 0);
    if (e == hipSuccess && p->banded) e = launch_band(a, (uint32_t)ctx->n_cu, st);
    if (e == hipSuccess) e = launch_batch_main(p, st);
    if (e == hipSuccess && !p->banded) e = launch_band(a, (uint32_t)ctx->n_cu, st);
    if (e == hipSuccess) e = launch_batch_small(p, ctx->side_stream);
    if (e == hipSuccess) e = hipEventRecord(ctx->join_event, ctx->side_stream);
    if (e == hipSuccess) e = hipStreamWaitEvent(st, ctx->join_event, 0);
    return e;
}

// Whether a captured step may fork: the branch costs about 10 us of joins, so the
// planned regions outside the small classes have to be worth it.  Step, one
// stream and two, in us: 2000 cells of 100-5000 voxels at 256 levels 292 and
// 248, at 512 levels 380 and 316; 10000 small regions and one of 60 M voxels
// at 1024 levels 996 and 929; 8000 regions all in the small classes 201 and 211.
bool worth_forking(const nyx_plan *p) {
    if (!p->small_cls) return false;
    const StepArgs &a = p->w.args;
    const RoiSizes &rois = p->w.sizes;
    const uint32_t sc = size_class(a.split_vox);
    uint64_t large = 0;
    for (uint32_t cl = p->small_cls; cl < sc; ++cl) large += rois.of_class[cl].vox;
    rois.above((1u << sc) - 1u, [&](const RoiSizes::Box &r) {
        if ((a.band_vox && r.n > a.band_vox) ||
            size_class(item_bound(r.n, r.rows, r.width, tiles_for(r.n, r.rows, r.width, a.split_vox, a.tile_vox))) >= p->small_cls)
            large += r.n;
    });
    return large * 16u > rois.all.vox;
}

// The full step on a stream.  per_roi: one accumulation launch per ROI; fork:
// the counting kernels on two branches (into a capture only).
// scanned: the label statistics are those of the discovery just made on this
// stream (one-shot calls), so the images are not scanned again.
nyx_status enqueue_step(nyx_plan *p, hipStream_t st, bool per_roi, bool scanned = false, bool fork = false) {
    nyx_ctx *ctx = p->ctx;
    const StepArgs &a = p->w.args;
    if (scanned) {
        HIPC(ctx, launch_reset_counters(a, p->w.n_counters, st));
    } else {
        HIPC(ctx, launch_reset(a, p->w.n_counters, st));
        HIPC(ctx, launch_scan(a, st));
    }
    HIPC(ctx, launch_compact(a, 0u, 0xFFFFFFFFu, st));
    HIPC(ctx, launch_zero_split(a, st));
    if (fork) {
        HIPC(ctx, launch_counting_forked(p, st));
    } else if (!per_roi) {
        HIPC(ctx, launch_batches(p, st));
    } else {
        for (uint32_t r = 0; r < p->w.n_rois; ++r) {
            const RoiDesc &d = p->w.h_rois[r];
            const uint32_t nt = tile_count(d.n, d.rows, (uint32_t)(d.x1 - d.x0 + 1), a.split_vox, a.tile_vox, a.band_vox);
            HIPC(ctx, launch_batch(a, nt, p->block, r, st));
        }
    }
    if (!fork) HIPC(ctx, launch_band(a, (uint32_t)ctx->n_cu, st));
    HIPC(ctx, launch_split_finalize(a, st));
    HIPC(ctx, launch_features(a, a.dsums, a.dsums_y, a.roi_cap, a.counters + C_NROIS, st));
    return NYX_OK;
}

void drop_graphs(nyx_plan *p) {
    for (nyx_plan::Graph *g : {&p->plain, &p->forked}) {
        if (g->exec) (void)hipGraphExecDestroy(g->exec);
        if (g->graph) (void)hipGraphDestroy(g->graph);
        *g = nyx_plan::Graph{};
    }
    p->graph_table = nullptr;
}

// A plan's step, with the outputs set, as a graph.
nyx_status capture_step(nyx_plan *p, bool fork, nyx_plan::Graph *to) {
    nyx_ctx *ctx = p->ctx;
    hipStream_t cs = ctx->capture_stream;
    HIPC(ctx, hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    nyx_status s = enqueue_step(p, cs, false, false, fork);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(cs, &g);
    if (s != NYX_OK) { if (g) (void)hipGraphDestroy(g); return s; }
    if (e != hipSuccess) return fail(ctx, NYX_ERR_DEVICE, "graph capture: %s", hipGetErrorString(e));
    to->graph = g;
    HIPC(ctx, hipGraphInstantiate(&to->exec, g, nullptr, nullptr, 0));
    return NYX_OK;
}

nyx_status check_counters(nyx_ctx *ctx, Work &w, hipStream_t st) {
    const uint32_t *h = reinterpret_cast<const uint32_t *>(ctx->pin + kPinUp);
    HIPC(ctx, hipMemcpyAsync(ctx->pin + kPinUp, w.counters.p, 8u * sizeof(uint32_t), hipMemcpyDeviceToHost, st));
    HIPC(ctx, hipStreamSynchronize(st));
    uint32_t e = h[C_ERR];
    if (e & E_LABEL_RANGE) return fail(ctx, NYX_ERR_CAPACITY, "a label exceeds the planned label range");
    if (e & E_ROI_CAP) return fail(ctx, NYX_ERR_CAPACITY, "more ROIs than planned");
    if (e & E_SPLIT_CAP) return fail(ctx, NYX_ERR_CAPACITY, "more split ROIs than planned");
    if (e & E_ITEM_CAP) return fail(ctx, NYX_ERR_CAPACITY, "more work items than planned");
    if (e & E_TABLE_CAP) return fail(ctx, NYX_ERR_CAPACITY, "feature table too small");
    if (e & E_BIN_RANGE) return fail(ctx, NYX_ERR_INVALID, "bin image holds a value outside [1, n_bins]");
    if (e & E_COO_RANGE) return fail(ctx, NYX_ERR_INVALID, "COO entry outside its matrix");
    if (e & (E_LIST_CAP | E_HASH_FULL)) return fail(ctx, NYX_ERR_INTERNAL, "LDS capacity exceeded (error bits %u)", e);
    return NYX_OK;
}

std::string describe(const Config &c, const nyx_plan *p, uint64_t items, uint32_t n_split) {
    uint64_t band_voxels = 0;
    if (c.band_vox) band_voxels = p->w.sizes.all.vox - p->w.sizes.up_to(c.band_vox).vox;
    char buf[640];
    snprintf(buf, sizeof buf,
             "mode=%s kp=%u copies=%u symmetric=%d block=%u grid=%u lds=%uB split_vox=%u tile_vox=%u tile_scale=%g "
             "list_cap=%u hash_cap=%u small_cls=%u small_kp=%u small_cap=%u small_grid=%u small_lds=%uB band_vox=%u band_w=%u band_dirs=%u band_voxels=%llu rois=%u items=%llu split_rois=%u ng=%d K=%d "
             "tuned_ms=%.4f",
             mode_name(c.mode), c.kp, p->w.args.lds.copies, c.nonsym ? 0 : 1, c.block, p->grid, p->w.args.lds.bytes, c.split_vox,
             c.tile_vox, (double)c.tile_scale, c.list_cap, c.hash_cap, p->small_cls, p->small_cls ? c.small_kp : 0u,
             p->small_cls ? c.small_cap : 0u, p->small_cls ? p->small_grid : 0u, p->small_cls ? p->small_lds.bytes : 0u,
             c.band_vox, c.band_w, c.band_dirs,
             (unsigned long long)band_voxels, p->w.n_rois,
             (unsigned long long)items,
             n_split, p->ng, p->K, (double)p->tuned_ms);
    return buf;
}

// Applies a configuration to a plan: scratch, step arguments, grid.
nyx_status configure(nyx_plan *p, const Config &cfg, const nyx_extract_opts *opts) {
    nyx_ctx *ctx = p->ctx;
    nyx_status s = setup_step(ctx, p->w, cfg, opts->offsets_host, p->K, (uint32_t)p->ng, p->prec == NYX_FP64, 0,
                              opts->workspace_cap_bytes, &p->workspace_bytes);
    if (s != NYX_OK) return s;
    if (p->w.args.lds.bytes > kLdsBudget)
        return fail(ctx, NYX_ERR_UNSUPPORTED, "LDS layout of %u bytes exceeds the %u available", p->w.args.lds.bytes,
                    kLdsBudget);
    p->block = cfg.block;
    int occ = 0;
    HIPC(ctx, batch_occupancy(p->w.args, cfg.block, &occ));
    p->grid = (uint32_t)ctx->n_cu * (uint32_t)std::max(occ, 1);
    p->small_cls = cfg.mode == 4 ? cfg.small_cls : 0u;
    if (p->small_cls) {
        Config s = cfg;
        s.block = 256u;
        s.kp = p->small_kp = cfg.small_kp;
        s.hash_cap = cfg.small_cap;
        StepArgs t = p->w.args;
        set_sweep(t, p->w.h_imgs, opts->offsets_host, p->K, s.kp);
        if (cfg.nonsym) t.sweep3_ok = 0;
        p->small_lds = t.lds = make_layout(s, (uint32_t)p->ng, p->K, !t.sweep_ok && !t.sweep3_ok);
        HIPC(ctx, batch_occupancy(t, 256u, &occ));
        p->small_grid = (uint32_t)ctx->n_cu * (uint32_t)std::max(occ, 1);
    }
    uint64_t items;
    uint32_t n_split;
    count_items(p->w.sizes, cfg, &items, &n_split);
    p->banded = cfg.band_vox != 0u && p->w.sizes.all.most > cfg.band_vox;
    p->fork = worth_forking(p);
    p->cfg = nyx_plan::Cfg{cfg.mode, cfg.kp, cfg.block, cfg.split_vox, cfg.tile_vox, cfg.list_cap, cfg.hash_cap,
                           cfg.force_split};
    p->desc = describe(cfg, p, items, n_split);
    return NYX_OK;
}

}  // namespace

// ======================================================================= ABI
extern "C" {

const char *nyx_status_string(nyx_status s) {
    switch (s) {
        case NYX_OK: return "ok";
        case NYX_ERR_INVALID: return "invalid argument";
        case NYX_ERR_OOM: return "out of memory";
        case NYX_ERR_DEVICE: return "device error";
        case NYX_ERR_CAPACITY: return "capacity too small";
        case NYX_ERR_UNSUPPORTED: return "unsupported";
        case NYX_ERR_INTERNAL: return "internal error";
    }
    return "unknown status";
}

nyx_status nyx_create(nyx_ctx **out, int device_ordinal) {
    if (!out) return NYX_ERR_INVALID;
    *out = nullptr;
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || n <= 0) return NYX_ERR_DEVICE;
    if (device_ordinal < 0 || device_ordinal >= n) return NYX_ERR_DEVICE;
    if (hipSetDevice(device_ordinal) != hipSuccess) return NYX_ERR_DEVICE;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device_ordinal) != hipSuccess) return NYX_ERR_DEVICE;
    uint8_t *scr = scratch_address(device_ordinal);
    if (!scr) return NYX_ERR_DEVICE;
    nyx_ctx *c = new nyx_ctx();
    c->device = device_ordinal;
    c->n_cu = prop.multiProcessorCount;
    c->scratch = scr;
    void *pin = nullptr;
    if (hipHostMalloc(&pin, kPinBytes, hipHostMallocDefault) != hipSuccess) {
        delete c;
        return NYX_ERR_DEVICE;
    }
    c->pin = static_cast<uint8_t *>(pin);
    if (hipStreamCreateWithFlags(&c->capture_stream, hipStreamNonBlocking) != hipSuccess ||
        hipStreamCreateWithFlags(&c->side_stream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&c->fork_event, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&c->join_event, hipEventDisableTiming) != hipSuccess) {
        release_streams(c);
        (void)hipHostFree(c->pin);
        delete c;
        return NYX_ERR_DEVICE;
    }
    *out = c;
    return NYX_OK;
}

void nyx_destroy(nyx_ctx *ctx) {
    if (!ctx) return;
    release_streams(ctx);
    if (ctx->pool.base) (void)hipFree(ctx->pool.base);
    if (ctx->pin) (void)hipHostFree(ctx->pin);
    delete ctx;
}

const char *nyx_last_error(const nyx_ctx *ctx) { return ctx ? ctx->err.c_str() : "no context"; }

nyx_status nyx_offsets_default(int32_t dims, int32_t distance, nyx_offset *out_host, int32_t *n) {
    static const int32_t two[4][3] = {{0, 0, 1}, {0, -1, 1}, {0, -1, 0}, {0, -1, -1}};
    static const int32_t three[13][3] = {{0, 0, 1},  {0, 1, 0},  {1, 0, 0},   {0, 1, 1},  {0, 1, -1},
                                         {1, 0, 1},  {1, 0, -1}, {1, 1, 0},   {1, -1, 0}, {1, 1, 1},
                                         {1, 1, -1}, {1, -1, 1}, {1, -1, -1}};
    if (!out_host || !n || distance < 1 || (dims != 2 && dims != 3)) return NYX_ERR_INVALID;
    int k = dims == 2 ? 4 : 13;
    for (int i = 0; i < k; ++i) {
        const int32_t *o = dims == 2 ? two[i] : three[i];
        out_host[i].dz = o[0] * distance;
        out_host[i].dy = o[1] * distance;
        out_host[i].dx = o[2] * distance;
    }
    *n = k;
    return NYX_OK;
}

int32_t nyx_feature_count(void) { return kNumFeat; }

const char *nyx_feature_name(int32_t f) { return (f >= 0 && f < kNumFeat) ? kFeatureNames[f] : nullptr; }

nyx_status nyx_bin_rois(nyx_ctx *ctx, const nyx_image *imgs, int32_t n_images, int32_t n_bins, nyx_roi_table *rois,
                        uint16_t *bins_out, nyx_stream stream) {
    if (!ctx) return NYX_ERR_INVALID;
    if (!rois) return fail(ctx, NYX_ERR_INVALID, "rois is NULL");
    nyx_status s = validate_images(ctx, imgs, n_images);
    if (s != NYX_OK) return s;
    if (n_bins < 2 || n_bins > 65535) return fail(ctx, NYX_ERR_INVALID, "n_bins must be in [2, 65535]");
    hipStream_t st = (hipStream_t)stream;
    HIPC(ctx, hipSetDevice(ctx->device));
    OneShot call(ctx, st);
    Work w;
    w.use_arena(&ctx->pool);
    if ((s = discover(ctx, imgs, n_images, w, st, false)) != NYX_OK) return s;
    if (rois->n_rois_host) *rois->n_rois_host = w.n_rois;
    if (rois->capacity < (int64_t)w.n_rois)
        return fail(ctx, NYX_ERR_CAPACITY, "ROI table capacity %lld < %u ROIs", (long long)rois->capacity, w.n_rois);
    StepArgs a = w.args;
    a.ng = n_bins;
    set_outputs(ctx, a, rois, nullptr, 0);
    HIPC(ctx, launch_roi_out(a, st));
    if (bins_out) HIPC(ctx, launch_bin_image(a, bins_out, w.total_vox, w.vox_base, st));
    HIPC(ctx, hipStreamSynchronize(st));
    return call.end(NYX_OK);
}

nyx_status nyx_glcm_accumulate(nyx_ctx *ctx, const nyx_image *imgs, int32_t n_images, const nyx_roi_table *rois,
                               const uint16_t *bins, const nyx_offset *offsets, int32_t K, int32_t symmetric,
                               int32_t n_bins, nyx_glcm *out, nyx_stream stream) {
    if (!ctx) return NYX_ERR_INVALID;
    if (!out) return fail(ctx, NYX_ERR_INVALID, "out is NULL");
    nyx_status s = validate_images(ctx, imgs, n_images);
    if (s != NYX_OK) return s;
    if ((s = validate_offsets(ctx, imgs, n_images, offsets, K)) != NYX_OK) return s;
    if (n_bins < 2 || n_bins > 65535) return fail(ctx, NYX_ERR_INVALID, "n_bins must be in [2, 65535]");
    if ((s = validate_bins(ctx, n_bins)) != NYX_OK) return s;
    if (symmetric != 0 && symmetric != 1) return fail(ctx, NYX_ERR_INVALID, "symmetric must be 0 or 1");
    const bool nonsym = symmetric == 0;
    hipStream_t st = (hipStream_t)stream;
    HIPC(ctx, hipSetDevice(ctx->device));
    OneShot call(ctx, st);
    Work w;
    w.use_arena(&ctx->pool);
    if ((s = discover(ctx, imgs, n_images, w, st, true)) != NYX_OK) return s;
    if (rois && rois->n_rois_host && *rois->n_rois_host != (int64_t)w.n_rois)
        return fail(ctx, NYX_ERR_INVALID, "ROI table has %lld rows, images have %u ROIs",
                    (long long)*rois->n_rois_host, w.n_rois);
    if (bins && w.n_rois) {   // (without a ROI nothing below waits for the copy)
        uint64_t off = 0;
        for (auto &d : w.h_imgs) { d.B = bins + off; off += d.nvox; }
        HIPC(ctx, copy_up(ctx, w.imgs.p, w.h_imgs.data(), sizeof(ImgDesc) * n_images, 0, st));
    }
    if ((s = fetch_rois(ctx, w, st)) != NYX_OK) return s;
    const uint32_t ng = (uint32_t)n_bins;
    Config cfg;
    if ((s = choose_config(ctx, w, ng, K, 1, 256, cfg, nonsym)) != NYX_OK) return s;
    // ROIs in batches whose global matrices fit a fixed budget
    const uint64_t per_roi = (uint64_t)K * ng * ng * 8u;
    const uint64_t budget = 2ull << 30;
    uint32_t batch = (uint32_t)std::max<uint64_t>(1u, std::min<uint64_t>(w.n_rois ? w.n_rois : 1u, budget / per_roi));
    if ((s = setup_step(ctx, w, cfg, offsets, K, ng, 0, batch, 0, nullptr)) != NYX_OK) return s;
    StepArgs &a = w.args;
    set_outputs(ctx, a, nullptr, nullptr, 0);
    const uint32_t grid = (uint32_t)ctx->n_cu * 2u;
    DevBuf dcount, doff;
    dcount.arena = doff.arena = &ctx->pool;
    HIPC(ctx, dcount.alloc((size_t)batch * K * 8u));
    HIPC(ctx, doff.alloc((size_t)batch * K * 8u));
    std::vector<uint64_t> hcount((size_t)batch * K), hoff((size_t)batch * K);
    uint64_t nnz_total = 0;
    // Phase 0 counts the cells, phase 1 writes them; the matrices of a single
    // batch are still there in phase 1, those of several are made again.
    const bool single = batch >= w.n_rois;
    for (int phase = 0; phase < 2; ++phase) {
        uint64_t written = 0;
        for (uint32_t lo = 0; lo < w.n_rois; lo += batch) {
            uint32_t hi = std::min(w.n_rois, lo + batch);
            uint32_t ns = hi - lo;
            if (phase == 0 || !single) {
                HIPC(ctx, launch_reset_counters(a, w.n_counters, st));
                HIPC(ctx, launch_compact(a, lo, hi, st));
                HIPC(ctx, launch_zero_split(a, st));
                HIPC(ctx, launch_batch(a, grid, cfg.block, kNone, st));
                HIPC(ctx, launch_band(a, (uint32_t)ctx->n_cu, st));
                HIPC(ctx, launch_coo_count(a, ns, dcount.as<uint64_t>(), st));
                HIPC(ctx, hipMemcpyAsync(hcount.data(), dcount.p, (size_t)ns * K * 8u, hipMemcpyDeviceToHost, st));
                if ((s = check_counters(ctx, w, st)) != NYX_OK) return s;   // (synchronises)
            }
            uint64_t acc = written;
            for (size_t i = 0; i < (size_t)ns * K; ++i) { hoff[i] = acc; acc += hcount[i]; }
            if (phase == 1) {
                HIPC(ctx, copy_up(ctx, doff.p, hoff.data(), (size_t)ns * K * 8u, 0, st));
                HIPC(ctx, launch_coo_emit(a, ns, doff.as<uint64_t>(), out->key, out->count, st));
                HIPC(ctx, hipStreamSynchronize(st));
            }
            written = acc;
        }
        if (phase == 0) {
            nnz_total = written;
            if (out->nnz_host) *out->nnz_host = (int64_t)nnz_total;
            out->n_bins = n_bins;
            out->n_offsets = K;
            out->symmetric = symmetric;
            out->n_rois = w.n_rois;
            if (out->capacity < (int64_t)nnz_total)
                return fail(ctx, NYX_ERR_CAPACITY, "COO capacity %lld < %llu nonzero cells", (long long)out->capacity,
                            (unsigned long long)nnz_total);
            if (nnz_total && (!out->key || !out->count)) return fail(ctx, NYX_ERR_INVALID, "COO arrays are NULL");
        }
    }
    return call.end(NYX_OK);
}

int32_t nyx_intensity_feature_count(void) { return kNumIntensityFeat; }

const char *nyx_intensity_feature_name(int32_t f) {
    return (f >= 0 && f < kNumIntensityFeat) ? kIntensityNames[f] : nullptr;
}

nyx_status nyx_intensity_features(nyx_ctx *ctx, const nyx_image *imgs, int32_t n_images, int32_t n_bins,
                                  nyx_precision prec, nyx_roi_table *rois, void *table, int64_t table_capacity_rows,
                                  nyx_stream stream) {
    if (!ctx) return NYX_ERR_INVALID;
    nyx_status s = validate_images(ctx, imgs, n_images);
    if (s != NYX_OK) return s;
    if (n_bins < 2 || n_bins > 65535) return fail(ctx, NYX_ERR_INVALID, "n_bins must be in [2, 65535]");
    if ((s = validate_bins(ctx, n_bins)) != NYX_OK) return s;
    if (prec != NYX_FP32 && prec != NYX_FP64) return fail(ctx, NYX_ERR_INVALID, "bad precision");
    hipStream_t st = (hipStream_t)stream;
    HIPC(ctx, hipSetDevice(ctx->device));
    uint64_t vox = 0;
    for (int i = 0; i < n_images; ++i) vox += (uint64_t)(imgs[i].nz * imgs[i].ny * imgs[i].nx);
    const uint32_t tile = intensity_tile_vox(vox, (uint32_t)ctx->n_cu);
    const TileQueue tq{tile, intensity_split_values(tile)};
    OneShot call(ctx, st);
    Work w;
    w.use_arena(&ctx->pool);
    if ((s = discover(ctx, imgs, n_images, w, st, false, &tq)) != NYX_OK) return s;
    const int64_t n = w.n_rois;
    if (rois && rois->n_rois_host) *rois->n_rois_host = n;
    if (rois && rois->capacity < n)
        return fail(ctx, NYX_ERR_CAPACITY, "ROI table capacity %lld < %lld ROIs", (long long)rois->capacity, (long long)n);
    if (table_capacity_rows < n)
        return fail(ctx, NYX_ERR_CAPACITY, "table capacity %lld < %lld rows", (long long)table_capacity_rows, (long long)n);
    if (n > 0 && !table) return fail(ctx, NYX_ERR_INVALID, "table is NULL");
    StepArgs a = w.args;
    a.ng = n_bins;
    DevBuf slots, sums;
    slots.arena = sums.arena = &ctx->pool;
    HIPC(ctx, slots.alloc(intensity_slot_bytes(w.n_split, w.n_aux)));
    HIPC(ctx, sums.alloc(intensity_sums_bytes(w.n_rois)));
    set_outputs(ctx, a, rois, nullptr, 0);
    HIPC(ctx, launch_roi_out(a, st));
    HIPC(ctx, launch_intensity(a, a.bucket_cap, (uint32_t)ctx->n_cu, prec == NYX_FP64, slots.p, sums.p, table,
                               (uint32_t)std::min<int64_t>(table_capacity_rows, 0xFFFFFFFFll), st));
    return call.end(check_counters(ctx, w, st));
}

int32_t nyx_neighbourhood_feature_count(void) { return kNumNeighbourFeat; }

const char *nyx_neighbourhood_feature_name(int32_t f) {
    return (f >= 0 && f < kNumNeighbourFeat) ? kNeighbourNames[f] : nullptr;
}

nyx_status nyx_neighbourhood_features(nyx_ctx *ctx, const nyx_image *imgs, int32_t n_images, int32_t n_bins,
                                      int32_t alpha, nyx_precision prec, nyx_roi_table *rois, void *table,
                                      int64_t table_capacity_rows, nyx_stream stream) {
    if (!ctx) return NYX_ERR_INVALID;
    nyx_status s = validate_images(ctx, imgs, n_images);
    if (s != NYX_OK) return s;
    if (n_bins < 2 || n_bins > 65535) return fail(ctx, NYX_ERR_INVALID, "n_bins must be in [2, 65535]");
    if (alpha < 0) return fail(ctx, NYX_ERR_INVALID, "alpha must be >= 0");
    if (prec != NYX_FP32 && prec != NYX_FP64) return fail(ctx, NYX_ERR_INVALID, "bad precision");
    int any_volume = 0;
    for (int i = 0; i < n_images; ++i) any_volume |= imgs[i].nz > 1;
    if (neighbourhood_lds_bytes((uint32_t)n_bins, any_volume) > kLdsBudget - 1024u)
        return fail(ctx, NYX_ERR_UNSUPPORTED, "n_bins=%d: the per-ROI %s neighbourhood tables exceed LDS", n_bins,
                    any_volume ? "3D" : "2D");
    hipStream_t st = (hipStream_t)stream;
    HIPC(ctx, hipSetDevice(ctx->device));
    uint64_t vox = 0;
    for (int i = 0; i < n_images; ++i) vox += (uint64_t)(imgs[i].nz * imgs[i].ny * imgs[i].nx);
    const TileQueue tq{neighbourhood_tile_vox(vox, (uint32_t)ctx->n_cu, (uint32_t)n_bins, any_volume), 0};
    OneShot call(ctx, st);
    Work w;
    w.use_arena(&ctx->pool);
    if ((s = discover(ctx, imgs, n_images, w, st, false, &tq)) != NYX_OK) return s;
    const int64_t n = w.n_rois;
    if (rois && rois->n_rois_host) *rois->n_rois_host = n;
    if (rois && rois->capacity < n)
        return fail(ctx, NYX_ERR_CAPACITY, "ROI table capacity %lld < %lld ROIs", (long long)rois->capacity, (long long)n);
    if (table_capacity_rows < n)
        return fail(ctx, NYX_ERR_CAPACITY, "table capacity %lld < %lld rows", (long long)table_capacity_rows, (long long)n);
    if (n > 0 && !table) return fail(ctx, NYX_ERR_INVALID, "table is NULL");
    StepArgs a = w.args;
    a.ng = n_bins;
    DevBuf gtab;
    gtab.arena = &ctx->pool;
    HIPC(ctx, gtab.alloc((size_t)w.n_split * neighbourhood_slot_bytes((uint32_t)n_bins, any_volume)));
    set_outputs(ctx, a, rois, nullptr, 0);
    HIPC(ctx, launch_roi_out(a, st));
    HIPC(ctx, launch_neighbourhood(a, a.bucket_cap, (uint32_t)ctx->n_cu, prec == NYX_FP64, (uint32_t)alpha, any_volume,
                                   gtab.as<uint32_t>(), table,
                                   (uint32_t)std::min<int64_t>(table_capacity_rows, 0xFFFFFFFFll), st));
    return call.end(check_counters(ctx, w, st));
}

nyx_status nyx_glcm_features(nyx_ctx *ctx, const nyx_glcm *glcm, const nyx_roi_table *rois, nyx_precision prec,
                             void *table, int64_t table_capacity_rows, nyx_stream stream) {
    if (!ctx) return NYX_ERR_INVALID;
    if (!glcm || !table) return fail(ctx, NYX_ERR_INVALID, "NULL argument");
    if (rois && rois->n_rois_host && *rois->n_rois_host != glcm->n_rois)
        return fail(ctx, NYX_ERR_INVALID, "ROI table has %lld rows, the COO list %lld ROIs",
                    (long long)*rois->n_rois_host, (long long)glcm->n_rois);
    if (glcm->n_offsets < 1 || glcm->n_offsets > kMaxOffsets) return fail(ctx, NYX_ERR_INVALID, "bad n_offsets");
    nyx_status s = validate_bins(ctx, glcm->n_bins);
    if (s != NYX_OK) return s;
    if (glcm->n_rois < 0 || glcm->n_rois >= (1ll << 26)) return fail(ctx, NYX_ERR_INVALID, "bad n_rois");
    if (table_capacity_rows < glcm->n_rois)
        return fail(ctx, NYX_ERR_CAPACITY, "table capacity %lld < %lld rows", (long long)table_capacity_rows,
                    (long long)glcm->n_rois);
    uint64_t nnz = glcm->nnz_host ? (uint64_t)*glcm->nnz_host : 0u;
    if (nnz && (!glcm->key || !glcm->count)) return fail(ctx, NYX_ERR_INVALID, "COO arrays are NULL");
    if (prec != NYX_FP32 && prec != NYX_FP64) return fail(ctx, NYX_ERR_INVALID, "bad precision");
    if (glcm->symmetric != 0 && glcm->symmetric != 1) return fail(ctx, NYX_ERR_INVALID, "symmetric must be 0 or 1");
    hipStream_t st = (hipStream_t)stream;
    HIPC(ctx, hipSetDevice(ctx->device));
    const uint32_t n_rois = (uint32_t)glcm->n_rois;
    const int K = glcm->n_offsets;
    if (n_rois == 0) return NYX_OK;
    OneShot call(ctx, st);
    DevBuf seg, scratch, scratch_y, counters;
    seg.arena = scratch.arena = scratch_y.arena = counters.arena = &ctx->pool;
    HIPC(ctx, seg.alloc(((size_t)n_rois * K + 1) * 8u));
    HIPC(ctx, scratch.alloc((size_t)n_rois * K * sizeof(DirSums)));
    HIPC(ctx, scratch_y.alloc((size_t)n_rois * K * sizeof(DirSumsY)));
    HIPC(ctx, counters.alloc(256));
    HIPC(ctx, hipMemsetAsync(counters.p, 0, 256, st));
    StepArgs a;
    memset(&a, 0, sizeof a);
    a.K = K;
    a.K_out = K;
    a.ng = glcm->n_bins;
    a.fp64 = prec == NYX_FP64;
    a.table = table;
    a.table_rows = (uint32_t)std::min<int64_t>(table_capacity_rows, 0xFFFFFFFFll);
    a.counters = counters.as<uint32_t>();
    a.nonsym = glcm->symmetric == 0;
    HIPC(ctx, launch_coo_features(a, glcm->key, glcm->count, nnz, n_rois, seg.as<uint64_t>(), scratch.as<DirSums>(),
                                  scratch_y.as<DirSumsY>(), st));
    HIPC(ctx, hipMemcpyAsync(ctx->pin + kPinUp, counters.as<uint32_t>() + C_ERR, 4, hipMemcpyDeviceToHost, st));
    HIPC(ctx, hipStreamSynchronize(st));
    const uint32_t herr = *reinterpret_cast<const uint32_t *>(ctx->pin + kPinUp);
    if (herr & E_COO_RANGE) return fail(ctx, NYX_ERR_INVALID, "COO entry outside its matrix");
    if (herr & E_TABLE_CAP) return fail(ctx, NYX_ERR_CAPACITY, "feature table too small");
    return call.end(NYX_OK);
}

}  // extern "C"

namespace {

// The arguments of a plan or of a whole pass.
nyx_status validate_extract(nyx_ctx *ctx, const nyx_image *imgs, int32_t n_images, const nyx_extract_opts *opts) {
    nyx_status s = validate_images(ctx, imgs, n_images);
    if (s != NYX_OK) return s;
    if ((s = validate_offsets(ctx, imgs, n_images, opts->offsets_host, opts->n_offsets)) != NYX_OK) return s;
    if (opts->n_bins < 2 || opts->n_bins > 65535) return fail(ctx, NYX_ERR_INVALID, "n_bins must be in [2, 65535]");
    if ((s = validate_bins(ctx, opts->n_bins)) != NYX_OK) return s;
    if (opts->symmetric != 0 && opts->symmetric != 1) return fail(ctx, NYX_ERR_INVALID, "symmetric must be 0 or 1");
    if (opts->precision != NYX_FP32 && opts->precision != NYX_FP64) return fail(ctx, NYX_ERR_INVALID, "bad precision");
    if (opts->aggregate != NYX_AGG_PER_OFFSET && opts->aggregate != NYX_AGG_MERGED)
        return fail(ctx, NYX_ERR_INVALID, "aggregate must be NYX_AGG_PER_OFFSET or NYX_AGG_MERGED");
    if (opts->copies != 0 && opts->copies != 1 && opts->copies != 2 && opts->copies != 4)
        return fail(ctx, NYX_ERR_INVALID, "copies must be 0, 1, 2 or 4");
    return NYX_OK;
}

// Bytes that a step's buffers may take: what the caller's cap, or a fixed
// scratch (with room for the buffers' alignment), leaves beside the label
// tables and ROI records; 0: no limit.
uint64_t step_limit(const Work &w, const nyx_extract_opts *opts) {
    uint64_t limit = 0;
    if (opts->workspace_cap_bytes > 0) {
        uint64_t used = w.rois.bytes + w.counters.bytes;
        for (const DevBuf &b : w.tab) used += b.bytes;
        limit = std::max<uint64_t>(1u, (uint64_t)opts->workspace_cap_bytes - std::min<uint64_t>(used, opts->workspace_cap_bytes));
    }
    if (const Arena *ar = w.rois.arena; ar && !ar->spill) {
        const uint64_t used = Arena::up(ar->used) + 16u * 256u, left = used < ar->cap ? ar->cap - used : 1u;
        limit = limit ? std::min(limit, left) : left;
    }
    return limit;
}

// ROI discovery and the untimed default configuration of a plan, of validated
// arguments on the context's device (shared by nyx_plan_create and the whole
// passes).
nyx_status plan_init(nyx_ctx *ctx, const nyx_image *imgs, int32_t n_images, const nyx_extract_opts *opts,
                     nyx_plan *p, hipStream_t st, std::vector<Config> &cands, Config &cfg) {
    nyx_status s = NYX_OK;
    p->ctx = ctx;
    p->imgs.assign(imgs, imgs + n_images);
    p->K = opts->n_offsets;
    p->ng = opts->n_bins;
    p->prec = opts->precision;
    if ((s = discover(ctx, imgs, n_images, p->w, st, true)) != NYX_OK) return s;
    if ((s = fetch_rois(ctx, p->w, st)) != NYX_OK) return s;
    const bool merged = opts->aggregate == NYX_AGG_MERGED;
    // the default plan: one copy (or the forced count) at the load-balance tile size
    const uint32_t copies0 = opts->copies > 0 ? (uint32_t)opts->copies : 1u;
    const bool nonsym = opts->symmetric == 0;
    cands = candidate_configs(ctx, p->w, (uint32_t)p->ng, p->K, 0, 256, merged, copies0, 1.f, nonsym,
                              step_limit(p->w, opts));
    if (cands.empty())
        return fail(ctx, NYX_ERR_UNSUPPORTED, "no LDS configuration fits n_bins=%d with %d offsets%s%s", p->ng, p->K,
                    merged ? " merged in one pass" : "", copies0 > 1u ? " with privatised copies" : "");
    cfg = default_config(cands, p->w, (uint32_t)p->ng, p->K);
    if (opts->accum_mode >= 0) {
        bool found = false;
        for (const Config &c : cands)
            if (is_mode(c, opts->accum_mode, cands)) { cfg = c; found = true; break; }
        if (!found) return fail(ctx, NYX_ERR_UNSUPPORTED, "accumulation mode %d does not fit this workload", opts->accum_mode);
    }
    cfg = widen_block(cfg, (uint32_t)p->ng, p->K, takes_sweep3(p->w, cfg, opts->offsets_host, p->K));
    return NYX_OK;
}

// One eager step of a configured plan, after the capacity checks of the
// caller's buffers; waits for the stream.
nyx_status extract_once(nyx_plan *p, nyx_roi_table *rois, void *table, int64_t table_capacity_rows, hipStream_t st,
                        bool scanned) {
    nyx_ctx *ctx = p->ctx;
    const int64_t n = p->w.n_rois;
    if (rois && rois->n_rois_host) *rois->n_rois_host = n;
    if (table_capacity_rows < n)
        return fail(ctx, NYX_ERR_CAPACITY, "table capacity %lld < %lld rows", (long long)table_capacity_rows, (long long)n);
    if (rois && rois->capacity < n)
        return fail(ctx, NYX_ERR_CAPACITY, "ROI table capacity %lld < %lld", (long long)rois->capacity, (long long)n);
    if (n > 0 && !table) return fail(ctx, NYX_ERR_INVALID, "table is NULL");
    set_outputs(ctx, p->w.args, rois, table, (uint32_t)n);
    nyx_status s = enqueue_step(p, st, false, scanned);
    if (s == NYX_OK) return check_counters(ctx, p->w, st);
    (void)hipStreamSynchronize(st);
    return s;
}

}  // namespace

extern "C" {

nyx_status nyx_plan_create(nyx_ctx *ctx, const nyx_image *imgs, int32_t n_images, const nyx_extract_opts *opts,
                           nyx_plan **out, int64_t *n_rois_host) {
    if (!ctx) return NYX_ERR_INVALID;
    if (!out || !opts) return fail(ctx, NYX_ERR_INVALID, "NULL argument");
    *out = nullptr;
    nyx_status s = validate_extract(ctx, imgs, n_images, opts);
    if (s != NYX_OK) return s;
    // The images may have been written on any stream: the plan's own stream
    // reads them from here on.
    HIPC(ctx, hipSetDevice(ctx->device));
    HIPC(ctx, hipDeviceSynchronize());
    hipStream_t st = ctx->capture_stream;
    std::unique_ptr<nyx_plan> p(new nyx_plan());
    std::vector<Config> cands;
    Config cfg;
    if ((s = plan_init(ctx, imgs, n_images, opts, p.get(), st, cands, cfg)) != NYX_OK) return s;
    const bool merged = opts->aggregate == NYX_AGG_MERGED;
    const uint32_t copies0 = opts->copies > 0 ? (uint32_t)opts->copies : 1u;
    if (opts->autotune) {
        // further axes: privatised copies (when not forced) and the tile size of split ROIs
        for (uint32_t cp : {1u, 2u, 4u}) {
            if (opts->copies > 0 && cp != copies0) continue;
            for (float ts : {0.5f, 1.f, 2.f}) {
                if (cp == copies0 && ts == 1.f) continue;
                for (const Config &c :
                     candidate_configs(ctx, p->w, (uint32_t)p->ng, p->K, 0, 256, merged, cp, ts, opts->symmetric == 0,
                                       step_limit(p->w, opts)))
                    if (cp == 1u || c.copies == cp) cands.push_back(c);
            }
        }
        // and the work-group size: 512 threads where 256 leave one group per CU
        const size_t n256 = cands.size();
        for (size_t i = 0; i < n256; ++i) {
            const Config c = widen_block(cands[i], (uint32_t)p->ng, p->K,
                                         takes_sweep3(p->w, cands[i], opts->offsets_host, p->K));
            if (c.block != cands[i].block) cands.push_back(c);
        }
    }
    if (opts->autotune && cands.size() > 1) {
        // every candidate: one warm-up step, then the median of kTuneSteps timed steps
        constexpr int kTuneSteps = 5;
        DevBuf tmp;
        size_t row_bytes = (size_t)(merged ? 1 : p->K + 1) * kNumFeat * (p->prec == NYX_FP64 ? 8u : 4u);
        HIPC(ctx, tmp.alloc(std::max<size_t>(p->w.n_rois, 1u) * row_bytes));
        hipEvent_t ev[kTuneSteps + 1];
        for (auto &e : ev) HIPC(ctx, hipEventCreate(&e));
        float best = 1e30f;
        for (const Config &c : cands) {
            if (opts->accum_mode >= 0 && !is_mode(c, opts->accum_mode, cands)) continue;
            if (configure(p.get(), c, opts) != NYX_OK) continue;   // (too large for the cap, or for the device)
            set_outputs(ctx, p->w.args, nullptr, tmp.p, p->w.n_rois);
            if ((s = enqueue_step(p.get(), st, false)) != NYX_OK) break;
            hipError_t he = hipEventRecord(ev[0], st);
            for (int k = 0; k < kTuneSteps && he == hipSuccess && s == NYX_OK; ++k) {
                s = enqueue_step(p.get(), st, false);
                he = hipEventRecord(ev[k + 1], st);
            }
            if (s != NYX_OK) break;
            HIPC(ctx, he);
            HIPC(ctx, hipEventSynchronize(ev[kTuneSteps]));
            float t[kTuneSteps];
            for (int k = 0; k < kTuneSteps; ++k) HIPC(ctx, hipEventElapsedTime(&t[k], ev[k], ev[k + 1]));
            std::sort(t, t + kTuneSteps);
            const float ms = t[kTuneSteps / 2];
            if (log_level() > 0)
                fprintf(stderr, "[nyx] autotune %s kp=%u copies=%u tile_scale=%g block=%u: %.3f ms\n", mode_name(c.mode),
                        c.kp, c.copies, (double)c.tile_scale, c.block, ms);
            if (ms < best) { best = ms; cfg = c; }
        }
        for (auto &e : ev) (void)hipEventDestroy(e);
        if (s != NYX_OK) return s;
        p->tuned_ms = best;
    }
    if ((s = configure(p.get(), cfg, opts)) != NYX_OK) return s;
    if (log_level() > 0) fprintf(stderr, "[nyx] plan: %s\n", p->desc.c_str());
    if (n_rois_host) *n_rois_host = p->w.n_rois;
    *out = p.release();
    return NYX_OK;
}

nyx_status nyx_plan_execute(nyx_plan *p, nyx_roi_table *rois, void *table, nyx_stream stream) {
    if (!p) return NYX_ERR_INVALID;
    nyx_ctx *ctx = p->ctx;
    if (!table) return fail(ctx, NYX_ERR_INVALID, "table is NULL");
    if (rois && rois->capacity < (int64_t)p->w.n_rois)
        return fail(ctx, NYX_ERR_CAPACITY, "ROI table capacity too small");
    HIPC(ctx, hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    nyx_roi_table key{};
    if (rois) key = *rois;
    key.n_rois_host = nullptr;
    if (!p->plain.exec || p->graph_table != table || memcmp(&key, &p->graph_rois, sizeof key) != 0) {
        drop_graphs(p);
        set_outputs(ctx, p->w.args, rois, table, p->w.n_rois);
        nyx_status s = capture_step(p, false, &p->plain);
        if (s != NYX_OK) return s;
        p->graph_table = table;
        p->graph_rois = key;
        p->replays = 0;
    } else if (p->fork && p->replays < kForkAfter && ++p->replays == kForkAfter) {
        // (the plain graph stays: a replay of it may still be under way)
        set_outputs(ctx, p->w.args, rois, table, p->w.n_rois);
        nyx_status s = capture_step(p, true, &p->forked);
        if (s != NYX_OK) return s;
    }
    HIPC(ctx, hipGraphLaunch(p->forked.exec ? p->forked.exec : p->plain.exec, st));
    if (rois && rois->n_rois_host) *rois->n_rois_host = p->w.n_rois;
    return NYX_OK;
}

nyx_status nyx_plan_execute_per_roi(nyx_plan *p, nyx_roi_table *rois, void *table, nyx_stream stream) {
    if (!p) return NYX_ERR_INVALID;
    nyx_ctx *ctx = p->ctx;
    if (!table) return fail(ctx, NYX_ERR_INVALID, "table is NULL");
    if (rois && rois->capacity < (int64_t)p->w.n_rois)
        return fail(ctx, NYX_ERR_CAPACITY, "ROI table capacity too small");
    HIPC(ctx, hipSetDevice(ctx->device));
    set_outputs(ctx, p->w.args, rois, table, p->w.n_rois);
    nyx_status s = enqueue_step(p, (hipStream_t)stream, true);
    if (rois && rois->n_rois_host) *rois->n_rois_host = p->w.n_rois;
    return s;
}

nyx_status nyx_plan_profile(nyx_plan *p, void *table, float *ms_host, nyx_stream stream) {
    if (!p) return NYX_ERR_INVALID;
    nyx_ctx *ctx = p->ctx;
    if (!table || !ms_host) return fail(ctx, NYX_ERR_INVALID, "NULL argument");
    HIPC(ctx, hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    set_outputs(ctx, p->w.args, nullptr, table, p->w.n_rois);
    // the graph (if any) was captured with other outputs; drop it
    drop_graphs(p);
    static_assert(NYX_PHASE_COUNT == 8, "one event interval per phase");
    hipEvent_t ev[NYX_PHASE_COUNT + 1];
    for (auto &e : ev) HIPC(ctx, hipEventCreate(&e));
    const StepArgs &a = p->w.args;
    nyx_status s = NYX_OK;
    hipError_t he = hipSuccess;
    he = hipEventRecord(ev[0], st);
    if (he == hipSuccess) he = launch_reset(a, p->w.n_counters, st);
    if (he == hipSuccess) he = hipEventRecord(ev[1], st);
    if (he == hipSuccess) he = launch_scan(a, st);
    if (he == hipSuccess) he = hipEventRecord(ev[2], st);
    if (he == hipSuccess) he = launch_compact(a, 0u, 0xFFFFFFFFu, st);
    if (he == hipSuccess) he = hipEventRecord(ev[3], st);
    if (he == hipSuccess) he = launch_zero_split(a, st);
    if (he == hipSuccess) he = hipEventRecord(ev[4], st);
    if (he == hipSuccess) he = launch_batches(p, st);
    if (he == hipSuccess) he = hipEventRecord(ev[5], st);
    if (he == hipSuccess) he = launch_band(a, (uint32_t)ctx->n_cu, st);
    if (he == hipSuccess) he = hipEventRecord(ev[6], st);
    if (he == hipSuccess) he = launch_split_finalize(a, st);
    if (he == hipSuccess) he = hipEventRecord(ev[7], st);
    if (he == hipSuccess) he = launch_features(a, a.dsums, a.dsums_y, a.roi_cap, a.counters + C_NROIS, st);
    if (he == hipSuccess) he = hipEventRecord(ev[8], st);
    if (he == hipSuccess) he = hipEventSynchronize(ev[8]);
    if (he == hipSuccess)
        for (int i = 0; i < NYX_PHASE_COUNT; ++i) {
            he = hipEventElapsedTime(&ms_host[i], ev[i], ev[i + 1]);
            if (he != hipSuccess) break;
        }
    for (auto &e : ev) (void)hipEventDestroy(e);
    if (he != hipSuccess) s = fail(ctx, NYX_ERR_DEVICE, "profile: %s", hipGetErrorString(he));
    return s;
}

nyx_status nyx_plan_check(nyx_plan *p, nyx_stream stream) {
    if (!p) return NYX_ERR_INVALID;
    return check_counters(p->ctx, p->w, (hipStream_t)stream);
}

const char *nyx_plan_describe(const nyx_plan *p) { return p ? p->desc.c_str() : ""; }

void nyx_plan_destroy(nyx_plan *p) {
    if (!p) return;
    (void)hipSetDevice(p->ctx->device);
    drop_graphs(p);
    delete p;
}

nyx_status nyx_extract_batch(nyx_ctx *ctx, const nyx_image *imgs, int32_t n_images, const nyx_extract_opts *opts,
                             nyx_roi_table *rois, void *table, int64_t table_capacity_rows, nyx_stream stream) {
    if (!ctx) return NYX_ERR_INVALID;
    if (!opts) return fail(ctx, NYX_ERR_INVALID, "NULL argument");
    hipStream_t st = (hipStream_t)stream;
    if (opts->autotune) {
        // timing the candidates runs the step many times: a plan of its own
        nyx_plan *p = nullptr;
        int64_t n = 0;
        nyx_status s = nyx_plan_create(ctx, imgs, n_images, opts, &p, &n);
        if (s != NYX_OK) return s;
        s = extract_once(p, rois, table, table_capacity_rows, st, false);
        nyx_plan_destroy(p);
        return s;
    }
    nyx_status s = validate_extract(ctx, imgs, n_images, opts);
    if (s != NYX_OK) return s;
    HIPC(ctx, hipSetDevice(ctx->device));
    OneShot call(ctx, st);
    nyx_plan p;
    p.w.use_arena(&ctx->pool);
    std::vector<Config> cands;
    Config cfg;
    s = plan_init(ctx, imgs, n_images, opts, &p, st, cands, cfg);
    if (s == NYX_OK) s = configure(&p, cfg, opts);
    if (s != NYX_OK) return s;
    return call.end(extract_once(&p, rois, table, table_capacity_rows, st, true));
}

nyx_status nyx_extract_batch_noalloc(nyx_ctx *ctx, const nyx_image *imgs, int32_t n_images,
                                     const nyx_extract_opts *opts, nyx_roi_table *rois, void *table,
                                     int64_t table_capacity_rows, nyx_stream stream) {
    if (!ctx) return NYX_ERR_INVALID;
    if (!opts) return fail(ctx, NYX_ERR_INVALID, "NULL argument");
    if (!ctx->scratch) return fail(ctx, NYX_ERR_DEVICE, "no scratch address for device %d", ctx->device);
    nyx_status s = validate_extract(ctx, imgs, n_images, opts);
    if (s != NYX_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    HIPC(ctx, hipSetDevice(ctx->device));
    CallGuard call(st);
    // every device buffer of the step is carved from this device's scratch
    Arena ar;
    ar.base = ctx->scratch;
    ar.cap = kScratchBytes;
    nyx_plan p;
    p.w.use_arena(&ar);
    std::vector<Config> cands;
    Config cfg;
    s = plan_init(ctx, imgs, n_images, opts, &p, st, cands, cfg);
    if (s == NYX_OK) s = configure(&p, cfg, opts);
    if (s != NYX_OK) {
        if (ar.wanted > ar.cap)
            return fail(ctx, NYX_ERR_CAPACITY,
                        "batch needs more than the %zu bytes of no-allocation scratch (at least %zu)", ar.cap,
                        ar.wanted);
        return s;
    }
    return call.end(extract_once(&p, rois, table, table_capacity_rows, st, true));
}

}  // extern "C"
