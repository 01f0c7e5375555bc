// host_calls.hip -- test harness (not part of the library): the library's host
// code on a HIP runtime of its own, without a GPU.  Device memory is host
// memory, copies happen at once, and of the kernels only what the host reads
// back takes place: the label maxima, the counters and the ROI descriptors,
// which a check plants.  What the host does -- the current device of every
// allocation, pinned copies that a stream has not been waited for, launches
// and their arguments, captured and instantiated graphs -- is written down and
// looked at by the checks.  Usage: host_calls CHECK; exit status 0: holds.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <algorithm>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "nyx.h"
#include "nyx_types.h"

using nyx::RoiDesc;
using nyx::StepArgs;

struct Launch {
    std::string name;
    const void *fn;
    dim3 grid, block;
    hipStream_t stream;
    bool has_args;
    StepArgs a;
};

namespace host {

int device = 0;
size_t memory_limit = ~(size_t)0;        // of one allocation
hipError_t last_error = hipSuccess;
std::map<void *, size_t> memory;         // device allocations
std::vector<int> alloc_device;           // current device of each
uint8_t *pin = nullptr;
size_t pin_bytes = 0;
std::map<hipStream_t, int> pinned;       // copies from or to pinned memory not waited for
// (a library's kernels are registered before this file's globals are made)
std::map<const void *, std::string> &kernels() {
    static std::map<const void *, std::string> m;
    return m;
}
std::vector<Launch> launches;
std::vector<const void *> occupancy;     // kernels whose occupancy was asked for
hipStream_t capturing = nullptr;
std::set<hipStream_t> captured;          // streams of the launches in the graph being captured
std::vector<size_t> graph_streams;       // streams of each instantiated graph
uint32_t max_label = 0;                  // of the images, at least the number of ROIs
std::vector<RoiDesc> rois;

RoiDesc box(uint32_t n, uint32_t rows, uint32_t width) {
    RoiDesc r{};
    r.n = n; r.rows = rows; r.vmax = 1000u;
    r.x1 = (int)width - 1; r.y1 = (int)rows - 1;
    r.n_tiles = 1u; r.tcols = 1u; r.gslot = nyx::kNone;
    return r;
}

void emulate(const std::string &k, void **args) {
    if (k.find("k_max_label") != std::string::npos) {
        const int n = *static_cast<int *>(args[1]);
        uint32_t *out = *static_cast<uint32_t **>(args[2]);
        for (int i = 0; i < n; ++i) out[i] = std::max(max_label, (uint32_t)rois.size());
    } else if (k.find("k_reset") != std::string::npos) {
        memset(static_cast<StepArgs *>(args[0])->counters, 0, 4u * *static_cast<uint32_t *>(args[1]));
    } else if (k.find("k_compact_write") != std::string::npos) {
        const StepArgs &a = *static_cast<StepArgs *>(args[0]);
        a.counters[nyx::C_NROIS] = (uint32_t)rois.size();
        for (size_t r = 0; r < rois.size() && r < a.roi_cap; ++r) a.rois[r] = rois[r];
    }
}

bool takes_step(const std::string &k) {
    for (const char *s : {"k_batch", "k_band", "k_compact_write", "k_features"})
        if (k.find(s) != std::string::npos) return true;
    return false;
}

void *map_memory(size_t n) {
    void *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    return p == MAP_FAILED ? nullptr : p;
}

bool is_pinned(const void *p) {
    return pin && p >= static_cast<const void *>(pin) && p < static_cast<const void *>(pin + pin_bytes);
}

}  // namespace host

// ------------------------------------------------------------ the runtime
extern "C" {

hipError_t hipGetDeviceCount(int *n) { *n = 2; return hipSuccess; }
hipError_t hipSetDevice(int d) { host::device = d; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError(void) {
    const hipError_t e = host::last_error;
    host::last_error = hipSuccess;
    return e;
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static void *s = host::map_memory(NYX_NOALLOC_SCRATCH_BYTES);
    *p = s;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
    if (n > host::memory_limit || !(*p = host::map_memory(n))) return host::last_error = hipErrorOutOfMemory;
    host::memory[*p] = n;
    host::alloc_device.push_back(host::device);
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    auto it = host::memory.find(p);
    if (it != host::memory.end()) {
        munmap(p, it->second);
        host::memory.erase(it);
    }
    host::pinned.clear();   // (waits for the device)
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned int) {
    host::pin = static_cast<uint8_t *>(*p = calloc(1, n));
    host::pin_bytes = n;
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
    memcpy(d, s, n);
    if (host::is_pinned(d) || host::is_pinned(s)) ++host::pinned[st];
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned int) {
    *s = reinterpret_cast<hipStream_t>(malloc(16));
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { host::pinned.erase(s); return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { host::pinned.clear(); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = reinterpret_cast<hipEvent_t>(malloc(16)); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { host::pinned.clear(); return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int, size_t) {
    host::occupancy.push_back(f);
    *n = 2;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    host::capturing = s;
    host::captured.clear();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    host::capturing = nullptr;
    *g = reinterpret_cast<hipGraph_t>(malloc(16));
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    *e = reinterpret_cast<hipGraphExec_t>(malloc(16));
    host::graph_streams.push_back(host::captured.size());
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { free(e); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { free(g); return hipSuccess; }

struct Config { dim3 grid, block; size_t shared; hipStream_t stream; };
static Config pushed;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t st) {
    pushed = Config{g, b, sh, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *st) {
    *g = pushed.grid; *b = pushed.block; *sh = pushed.shared; *st = pushed.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t, hipStream_t st) {
    const std::string &k = host::kernels()[f];
    Launch l{k, f, g, b, st, host::takes_step(k), StepArgs{}};
    if (l.has_args) l.a = *static_cast<StepArgs *>(args[0]);
    host::launches.push_back(l);
    if (host::capturing) host::captured.insert(st);
    else host::emulate(k, args);
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { static void *m; return &m; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned int, void *, void *, dim3 *, dim3 *,
                           int *) {
    host::kernels()[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

}  // extern "C"

// ----------------------------------------------------------------- checks
namespace {

int failures = 0;
#define EXPECT(c)                                                        \
    do {                                                                 \
        if (!(c)) { printf("%s:%d: %s\n", __FILE__, __LINE__, #c); ++failures; } \
    } while (0)

const hipStream_t kStream = reinterpret_cast<hipStream_t>(0x1000);
uint16_t *const kI = reinterpret_cast<uint16_t *>(0x10000);   // images are not read here
uint32_t *const kL = reinterpret_cast<uint32_t *>(0x20000);
nyx_offset kFlat[4] = {{0, 0, 1}, {0, 1, 0}, {0, 1, 1}, {0, 1, -1}};

nyx_ctx *context(int dev = 0) {
    nyx_ctx *c = nullptr;
    EXPECT(nyx_create(&c, dev) == NYX_OK);
    return c;
}

nyx_image image(int64_t ny, int64_t nx, int64_t nz = 1) {
    nyx_image m{};
    m.intensity = kI; m.labels = kL;
    m.nz = nz; m.ny = ny; m.nx = nx;
    return m;
}

nyx_extract_opts options(int bins, int K = 4) {
    nyx_extract_opts o{};
    o.n_bins = bins;
    o.offsets_host = kFlat;
    o.n_offsets = K;
    o.symmetric = 1;
    o.precision = NYX_FP32;
    o.accum_mode = -1;
    return o;
}

size_t pending() { return host::pinned.size(); }

// The call makes its memory on the context's device, and none for arguments
// that it refuses.
void extract_device() {
    nyx_ctx *c = context(1);
    (void)hipSetDevice(0);
    host::alloc_device.clear();
    nyx_image im = image(64, 64);
    nyx_extract_opts o = options(1);
    nyx_roi_table t{};
    int64_t n = 0;
    t.n_rois_host = &n;
    EXPECT(nyx_extract_batch(c, &im, 1, &o, &t, kI, 100, kStream) == NYX_ERR_INVALID);
    EXPECT(host::alloc_device.empty());
    o.n_bins = 16;
    (void)hipSetDevice(0);
    EXPECT(nyx_extract_batch(c, &im, 1, &o, &t, kI, 100, kStream) == NYX_OK);
    EXPECT(!host::alloc_device.empty());
    for (int d : host::alloc_device) EXPECT(d == 1);
    nyx_destroy(c);
}

// A batch whose label tables outgrow the fixed scratch is refused, and nothing
// of the call is left to run.
void noalloc_wait() {
    nyx_ctx *c = context();
    nyx_image im = image(3000, 3000);
    nyx_extract_opts o = options(16);
    host::max_label = 8000000u;
    EXPECT(nyx_extract_batch_noalloc(c, &im, 1, &o, nullptr, kI, 100, kStream) == NYX_ERR_CAPACITY);
    EXPECT(pending() == 0);
    nyx_destroy(c);
}

// No label anywhere and a bin image: nothing is left to run either.
void accumulate_wait() {
    nyx_ctx *c = context();
    nyx_image im = image(64, 64);
    int64_t nnz = -1;
    nyx_glcm out{};
    out.nnz_host = &nnz;
    EXPECT(nyx_glcm_accumulate(c, &im, 1, nullptr, kI, kFlat, 4, 1, 16, &out, kStream) == NYX_OK);
    EXPECT(nnz == 0 && out.n_rois == 0);
    EXPECT(pending() == 0);
    nyx_destroy(c);
}

bool described(const nyx_plan *p, const char *what) { return strstr(nyx_plan_describe(p), what) != nullptr; }

// Many levels: a hash whose tables hold few voxels splits regions that the
// other configuration takes whole, and every split region costs its matrices
// in global memory.  It is not taken where these outgrow what it saves, nor
// where a limit on the scratch takes the other one only.
void packed_memory() {
    nyx_ctx *c = context();
    nyx_image im = image(2000, 2000);
    int64_t n = 0;
    for (int bins : {1100, 1500, 2048, 4096}) {
        host::rois.assign(1000, host::box(bins == 4096 ? 300u : 1100u, 50u, 24u));
        nyx_extract_opts o = options(bins, 1);
        o.workspace_cap_bytes = 64 << 20;
        nyx_plan *p = nullptr;
        EXPECT(nyx_plan_create(c, &im, 1, &o, &p, &n) == NYX_OK);
        if (p) EXPECT(described(p, "split_rois=0 "));
        nyx_plan_destroy(p);
        nyx_roi_table t{};
        t.capacity = 1000;
        EXPECT(nyx_extract_batch_noalloc(c, &im, 1, &o, &t, kI, 1000, kStream) == NYX_OK);
    }
    // a few split regions among many small ones: taken, but for a limit
    host::rois.assign(20000, host::box(250u, 20u, 20u));
    for (int k = 0; k < 40; ++k) host::rois[500 * k] = host::box(17000u, 160u, 120u);
    nyx_image big[8];
    for (nyx_image &b : big) b = image(2000, 2000);
    for (int k = 0; k < 800; ++k) host::rois.push_back(host::box(16000u, 160u, 120u));
    nyx_extract_opts o = options(256);
    nyx_plan *p = nullptr;
    EXPECT(nyx_plan_create(c, big, 8, &o, &p, &n) == NYX_OK);
    if (p) EXPECT(described(p, "mode=hash") && described(p, "split_rois=40 "));
    nyx_plan_destroy(p);
    o.workspace_cap_bytes = 60 << 20;
    p = nullptr;
    EXPECT(nyx_plan_create(c, big, 8, &o, &p, &n) == NYX_OK);
    if (p) EXPECT(described(p, "mode=dense") && described(p, "split_rois=0 "));
    nyx_plan_destroy(p);
    nyx_destroy(c);
}

// Banded regions more than the CUs: the largest is still cut into its share.
void band_blocks_of_many() {
    nyx_ctx *c = context();
    nyx_image im = image(8000, 10000);
    int64_t n = 0;
    host::rois.assign(300, host::box(40000u, 200u, 200u));
    host::rois.push_back(host::box(60000000u, 8000u, 8000u));
    nyx_extract_opts o = options(1024);
    nyx_plan *p = nullptr;
    EXPECT(nyx_plan_create(c, &im, 1, &o, &p, &n) == NYX_OK);
    EXPECT(nyx_plan_execute(p, nullptr, kI, kStream) == NYX_OK);
    int seen = 0;
    for (const Launch &l : host::launches) {
        if (l.name.find("k_band") == std::string::npos) continue;
        ++seen;
        const uint64_t sets = (4u + l.a.band_dirs - 1u) / l.a.band_dirs;
        EXPECT(nyx::band_blocks(8000u, 8000u, l.a.band_tile) * sets >= 100u);
    }
    EXPECT(seen == 1);
    nyx_plan_destroy(p);
    nyx_destroy(c);
}

// A graph of two branches takes several times as long to instantiate: it is
// made for outputs that come back, not for ones that change with every call.
void forks_when_repeated() {
    nyx_ctx *c = context();
    nyx_image im = image(2000, 2000);
    int64_t n = 0;
    host::rois.assign(6000, host::box(200u, 15u, 15u));
    for (size_t r = 0; r < host::rois.size(); r += 20) host::rois[r] = host::box(3000u, 60u, 55u);
    nyx_extract_opts o = options(256);
    nyx_plan *p = nullptr;
    EXPECT(nyx_plan_create(c, &im, 1, &o, &p, &n) == NYX_OK);
    for (int k = 0; k < 20; ++k) EXPECT(nyx_plan_execute(p, nullptr, kI + 64 * (k & 1), kStream) == NYX_OK);
    for (size_t s : host::graph_streams) EXPECT(s == 1);
    EXPECT(host::graph_streams.size() == 20);
    host::graph_streams.clear();
    for (int k = 0; k < 20; ++k) EXPECT(nyx_plan_execute(p, nullptr, kI, kStream) == NYX_OK);
    EXPECT(host::graph_streams == std::vector<size_t>({1, 2}));
    nyx_plan_destroy(p);
    nyx_destroy(c);
}

uint32_t described_number(const nyx_plan *p, const char *key) {
    const char *at = strstr(nyx_plan_describe(p), key);
    EXPECT(at != nullptr);
    return at ? (uint32_t)strtoul(at + strlen(key), nullptr, 10) : 0u;
}

// The items and split regions of a plan, counted region by region.
void plan_counts() {
    nyx_ctx *c = context();
    nyx_image im = image(8000, 8000);
    int64_t n = 0;
    uint32_t x = 1u;
    const auto next = [&](uint32_t below) {
        x = x * 1664525u + 1013904223u;
        return (x >> 8) % below;
    };
    for (int bins : {16, 100, 256, 700, 2048, 6000}) {
        for (uint32_t count : {1u, 60u, 900u}) {
            host::rois.clear();
            for (uint32_t k = 0; k < count; ++k) {
                const uint32_t rows = 1u + next(k % 9u == 0u ? 3000u : 90u), width = 1u + next(k % 7u == 0u ? 900u : 70u);
                host::rois.push_back(host::box(1u + next(rows * width), rows, width));
            }
            for (uint32_t v : {4095u, 4096u, 4097u, 32767u, 32768u, 32769u}) host::rois.push_back(host::box(v, 190u, 180u));
            nyx_extract_opts o = options(bins);
            nyx_plan *p = nullptr;
            const nyx_status s = nyx_plan_create(c, &im, 1, &o, &p, &n);
            EXPECT(s == NYX_OK || (bins == 6000 && s == NYX_ERR_UNSUPPORTED));   // (too wide a region for its tables)
            if (!p) continue;
            const uint32_t split = described_number(p, "split_vox="), tile = described_number(p, "tile_vox="),
                           band = described_number(p, "band_vox=");
            uint64_t items = 0, n_split = 0, banded = 0;
            for (const RoiDesc &r : host::rois) {
                const uint32_t w = (uint32_t)(r.x1 + 1);
                const nyx::Tiling t = nyx::tiles_for(r.n, r.rows, w, split, tile);
                const bool b = band && r.n > band;
                items += b ? 0u : t.row_blocks * t.col_blocks;
                n_split += b || t.row_blocks * t.col_blocks > 1u;
                banded += b ? r.n : 0u;
            }
            EXPECT(described_number(p, " items=") == items);
            EXPECT(described_number(p, "split_rois=") == n_split);
            EXPECT(described_number(p, "band_voxels=") == banded);
            nyx_plan_destroy(p);
        }
    }
    nyx_destroy(c);
}

// A large image among many small ones is still read by many work-groups.
void label_maximum_of_mixed_sizes() {
    nyx_ctx *c = context();
    std::vector<nyx_image> im(1000, image(64, 64));
    im.push_back(image(6000, 10000));
    nyx_roi_table t{};
    int64_t n = 0;
    t.n_rois_host = &n;
    EXPECT(nyx_bin_rois(c, im.data(), (int32_t)im.size(), 16, &t, nullptr, kStream) == NYX_OK);
    int seen = 0;
    for (const Launch &l : host::launches) {
        if (l.name.find("k_max_label") == std::string::npos) continue;
        ++seen;
        EXPECT(l.grid.x >= 256u && l.grid.y == 1001u);
    }
    EXPECT(seen == 1);
    nyx_destroy(c);
}

// The grid of the batch kernel comes from the occupancy of the kernel that runs.
void occupancy_of_the_kernel_launched() {
    nyx_ctx *c = context();
    nyx_image im = image(2000, 2000), vol = image(200, 200, 100);
    int64_t n = 0;
    int paired = 0;
    for (int bins : {64, 120, 128, 256}) {
        for (int sym : {1, 0}) {
            for (const nyx_image *m : {&im, &vol}) {
                host::rois.assign(2000, host::box(1250u, 40u, 40u));
                host::occupancy.clear();
                host::launches.clear();
                nyx_extract_opts o = options(bins);
                o.symmetric = sym;
                nyx_plan *p = nullptr;
                EXPECT(nyx_plan_create(c, m, 1, &o, &p, &n) == NYX_OK);
                EXPECT(nyx_plan_execute(p, nullptr, kI, kStream) == NYX_OK);
                for (const Launch &l : host::launches) {
                    if (l.name.find("k_batch") == std::string::npos) continue;
                    paired += l.a.lds.marg_pair != 0u;
                    EXPECT(std::count(host::occupancy.begin(), host::occupancy.end(), l.fn) > 0);
                }
                nyx_plan_destroy(p);
            }
        }
    }
    EXPECT(paired > 0);
    nyx_destroy(c);
}

// The tiles of a region: a partition of its box, none with more voxels than the
// bound that its size class and its table are taken from.
void tiles_of_a_box() {
    uint32_t x = 7u;
    const auto next = [&](uint32_t below) {
        x = x * 1664525u + 1013904223u;
        return (x >> 8) % below;
    };
    std::vector<uint8_t> hit;
    for (int k = 0; k < 4000; ++k) {
        const uint32_t rows = 1u + next(k % 5 ? 120u : 3000u), width = 1u + next(k % 3 ? 90u : 700u);
        const uint32_t area = rows * width, n = k % 4 ? 1u + next(area) : area, split = 1u + next(k % 2 ? 64u : 4096u);
        const nyx::Tiling t = nyx::tiles_for(n, rows, width, split, split);
        const uint32_t tiles = t.row_blocks * t.col_blocks, bound = nyx::item_bound(n, rows, width, t);
        hit.assign(area, 0);
        for (uint32_t i = 0; i < tiles; ++i) {
            uint32_t ra, rb, ca, cb;
            nyx::tile_bounds(rows, width, tiles, t.col_blocks, i, &ra, &rb, &ca, &cb);
            if (ra >= rb || ca >= cb) continue;
            EXPECT(rb <= rows && cb <= width);
            EXPECT(std::min(n, (rb - ra) * (cb - ca)) <= bound);
            for (uint32_t r = ra; r < std::min(rb, rows); ++r)
                for (uint32_t c = ca; c < std::min(cb, width); ++c) ++hit[r * width + c];
        }
        EXPECT((size_t)std::count(hit.begin(), hit.end(), 1) == hit.size());
        if (failures) return;
    }
}

// A candidate that outgrows the caller's cap is passed over, also where it is
// the last one that the tuning looks at.
void tuning_under_a_cap() {
    nyx_ctx *c = context();
    nyx_image im = image(6000, 6000);
    int64_t n = 0;
    host::rois.assign(1500, host::box(12000u, 120u, 110u));
    for (int k = 0; k < 100; ++k) host::rois.push_back(host::box(30000u, 180u, 170u));
    nyx_extract_opts o = options(200);
    o.accum_mode = 0;
    o.workspace_cap_bytes = 400 << 20;
    nyx_plan *p = nullptr;
    EXPECT(nyx_plan_create(c, &im, 1, &o, &p, &n) == NYX_OK);
    nyx_plan_destroy(p);
    o.autotune = 1;
    p = nullptr;
    EXPECT(nyx_plan_create(c, &im, 1, &o, &p, &n) == NYX_OK);
    if (p) EXPECT(described_number(p, "split_rois=") == 100u);
    nyx_plan_destroy(p);
    nyx_destroy(c);
}

// A call that runs out of device memory says so, and the next one is none the
// worse: the runtime's last error, which every launch is checked by, is clear.
void out_of_memory_is_over() {
    nyx_ctx *c = context();
    nyx_image im = image(4000, 4000);
    int64_t n = 0;
    host::rois.assign(500, host::box(6000u, 80u, 90u));
    nyx_extract_opts o = options(256);
    nyx_roi_table t{};
    t.capacity = 500;
    host::memory_limit = 100 << 20;
    EXPECT(nyx_extract_batch(c, &im, 1, &o, &t, kI, 500, kStream) == NYX_ERR_OOM);
    EXPECT(hipGetLastError() == hipSuccess);
    nyx_plan *p = nullptr;
    EXPECT(nyx_plan_create(c, &im, 1, &o, &p, &n) == NYX_ERR_OOM);
    EXPECT(hipGetLastError() == hipSuccess);
    host::rois.resize(10);
    EXPECT(nyx_extract_batch(c, &im, 1, &o, &t, kI, 500, kStream) == NYX_OK);
    EXPECT(nyx_plan_create(c, &im, 1, &o, &p, &n) == NYX_OK);
    nyx_plan_destroy(p);
    nyx_destroy(c);
}

struct Check { const char *name; void (*run)(); };
const Check kChecks[] = {
    {"extract_device", extract_device},
    {"noalloc_wait", noalloc_wait},
    {"accumulate_wait", accumulate_wait},
    {"packed_memory", packed_memory},
    {"band_blocks_of_many", band_blocks_of_many},
    {"forks_when_repeated", forks_when_repeated},
    {"plan_counts", plan_counts},
    {"label_maximum_of_mixed_sizes", label_maximum_of_mixed_sizes},
    {"occupancy_of_the_kernel_launched", occupancy_of_the_kernel_launched},
    {"tiles_of_a_box", tiles_of_a_box},
    {"tuning_under_a_cap", tuning_under_a_cap},
    {"out_of_memory_is_over", out_of_memory_is_over},
};

}  // namespace

int main(int argc, char **argv) {
    for (const Check &c : kChecks)
        if (argc == 2 && strcmp(argv[1], c.name) == 0) {
            c.run();
            return failures ? 1 : 0;
        }
    printf("no such check\n");
    return 2;
}
