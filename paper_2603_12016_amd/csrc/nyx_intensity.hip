// nyx_intensity.hip -- first-order intensity features of every ROI.
//
// The intensity group of the paper's feature list (Supplementary Table S1,
// "2-dimensional intensity features", the rows with the NY mark; Table S5
// holds the same statistics for volumes).  The paper names the features and
// states their cost: O(m) in the voxel count m for the moments, O(m, h) for
// the histogram-based ones with h intensity bins (Materials and methods,
// "Feature Control and Tunability").  Each feature is the usual statistical
// definition; the choices the paper leaves open are:
//   * VARIANCE / STDDEV are unbiased (n - 1); a single voxel has variance 0;
//   * SKEWNESS, KURTOSIS, HYPERSKEWNESS, HYPERFLATNESS are the biased central
//     moments m3..m6 over m2^(k/2), 0 for a constant ROI (kurtosis not
//     excess);
//   * percentiles interpolate linearly between the closest ranks: with the n
//     values sorted and h = (n - 1) p / 100, x_(floor h) + frac(h) (x_(floor
//     h + 1) - x_(floor h));
//   * MEDIAN_ABSOLUTE_DEVIATION is the mean distance to the median;
//   * ROBUST_MEAN_ABSOLUTE_DEVIATION is the mean distance to their mean of
//     the values within [P10, P90] (NaN when no value lies there);
//   * MODE, ENTROPY (log2) and UNIFORMITY use the histogram of the
//     fixed-bin-number levels 1..n_bins over the ROI's [min, max] (the same
//     discretisation as the texture features); MODE takes the lowest level
//     among ties;
//   * UNIFORMITY_PIU = 100 (1 - (max - min) / (max + min)), 100 when both are 0;
//   * WEIGHTED_CENTROID_* use image coordinates (column, row, plane), NaN
//     when the intensities sum to 0;
//   * edge voxels are ROI voxels with a face neighbour (4 in a plane, 6 in a
//     volume) outside the image or outside the ROI; EDGE_STDDEV is unbiased.
//
// Work items come from the tile queue of the compaction (nyx_queue.h).  A
// ROI in one tile takes four passes over its values:
//   A  exact integer sums (count, sum, sum of squares, coordinate-weighted
//      sums), edge-voxel sums, a 1024-bucket coarse histogram of (I - min)
//      and the level histogram;
//   B  centred moments about the mean (double) and, when the value range
//      exceeds the coarse buckets, a fine histogram of the few buckets that
//      hold the percentile ranks, so every order statistic is exact;
//   C  distance to the median and the count and sum of the values in
//      [P10, P90];
//   D  distance of those values to their mean.
// Pass A loads a voxel's label, value and face neighbours' labels together
// and leaves the values of a box of at most kFoArea voxels in LDS, with one
// membership bit each, for the other passes (a larger box is read again).
// The tiles of a split ROI add their integer sums and the full histogram of
// their values (one counter per value of the range) to global memory; k_intensity_split
// takes every statistic from the histogram.  Either way the sums of a ROI end
// in a FoSums record, and k_intensity_rows forms the 37 values with one lane
// per ROI.  The family is bound by latency (on eight 2048 x 2048 images the
// vector units are busy 35 % of k_intensity's 355 us and 53 % of
// k_intensity_small's 167, at three wavefronts per SIMD), and for the usual
// small region the cost of a work-group's fixed parts (clearing, rank search,
// reductions) times its wavefronts is most of it: a box of at most kFoSmall
// voxels is taken by one wavefront (k_intensity_small, 16-bit counters, one
// batched reduction per pass), a larger one by 256 threads.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stddef.h>

#include "nyx_device.h"
#include "nyx_features.h"
#include "nyx_launch.h"
#include "nyx_queue.h"

namespace nyx {

namespace {

constexpr int kFoBlock = 256;
constexpr int kFoWaves = kFoBlock / kWave;
constexpr uint32_t kFoCoarse = 1024u;      // coarse buckets of I - min
constexpr int kFoPct = 7;                  // percentiles 1, 10, 25, 50, 75, 90, 99
constexpr int kFoRanks = 2 * kFoPct;       // the two ranks each percentile interpolates between
constexpr uint32_t kFoFine = 64u;          // values per coarse bucket at most (range < 2^16)
constexpr uint32_t kFoArea = 6144u;        // box voxels whose values stay in LDS
constexpr uint32_t kFoSmall = 2048u;       // box voxels of a ROI that one wavefront takes
constexpr int kFoSplitBlock = 512;        // split ROIs: threads of the histogram kernel
constexpr int kFoSplitWaves = kFoSplitBlock / kWave;
constexpr uint32_t kFoMinTile = 4096u;     // voxels per tile of a split ROI, at least

enum FoFeat : int {
    FO_MEAN, FO_MIN, FO_MAX, FO_RANGE, FO_INTEGRATED, FO_ENERGY, FO_RMS, FO_VARIANCE, FO_STDDEV,
    FO_STDERR, FO_SKEWNESS, FO_KURTOSIS, FO_HYPERSKEWNESS, FO_HYPERFLATNESS, FO_MEANAD, FO_MEDIAN,
    FO_MEDIANAD, FO_P01, FO_P10, FO_P25, FO_P75, FO_P90, FO_P99, FO_IQR, FO_ROBUSTMAD, FO_MODE,
    FO_ENTROPY, FO_UNIFORMITY, FO_PIU, FO_WCX, FO_WCY, FO_WCZ, FO_EDGE_INTEGRATED, FO_EDGE_MIN,
    FO_EDGE_MAX, FO_EDGE_MEAN, FO_EDGE_STDDEV, FO_COUNT
};
static_assert(FO_COUNT == kNumIntensityFeat, "column count");

// Percentile i of 1, 10, 25, 50, 75, 90, 99 (one byte each).
__device__ __forceinline__ uint32_t fo_pct(uint32_t i) {
    return (uint32_t)(0x635A4B32190A01ull >> (8u * i)) & 0xFFu;
}

// Scratch of one ROI in one tile; the tiles of split ROIs use the same LDS
// as a window of their value histogram.
struct FoRoi {
    uint32_t coarse[kFoCoarse];
    uint32_t fine[kFoRanks][kFoFine];
    uint16_t val[kFoArea];
    uint64_t in[kFoArea / 64u];            // membership of the box voxels
    uint8_t slot[kFoCoarse];               // coarse bucket -> fine slot + 1 (0: none)
};
constexpr uint32_t kFoWindow = sizeof(FoRoi) / 4u;

struct FoShared {
    union {
        FoRoi r;
        uint32_t window[kFoWindow];
    };
    uint64_t red[kFoWaves * 8];
    uint64_t best;                         // mode: count << 32 | ~level
    uint32_t rank[kFoRanks];               // 0-based rank in sorted order
    uint32_t rank_bucket[kFoRanks], rank_in[kFoRanks], rank_val[kFoRanks];
    uint32_t wave_tot[kFoWaves];
    uint32_t misc[128];                    // queue state (nyx_queue.h)
    uint32_t emin, emax, n_items;
    double pct[kFoPct];
};

// Sums of one ROI, turned into the table row by k_intensity_rows.
struct FoSums {
    uint64_t n, ne, S1, S2, CX, CY, CZ, ES1, ES2;   // n = 0: no voxels, NaN row
    uint32_t emin, emax, vmin, vmax;
    uint64_t mode;
    double m2, m3, m4, m5, m6, mad, dmed, RC, rmad, ent, uni;
    double pct[kFoPct];
};

// A split ROI's slot: the integer sums of its tiles.  The histograms of
// (I - vmin), vmax - vmin + 1 counters each, follow the slots in blocks of 64
// counters, a ROI's at block RoiDesc::aux.
struct FoSlot {
    uint64_t s[8];                         // n | ne << 32, S1, S2, CX, CY, CZ, ES1, ES2
    uint32_t emin, emax, pad[14];
};
static_assert(sizeof(FoSlot) % 128 == 0, "the histograms start on a cache line");
__device__ __forceinline__ uint32_t *fo_hist(FoSlot *slots, uint32_t n_slots, const RoiDesc &rd) {
    return reinterpret_cast<uint32_t *>(slots + n_slots) + 64ull * rd.aux;
}
// (n and ne share a word: a ROI has fewer than 2^31 voxels)

struct Centred {
    double v[6] = {};                      // m2..m6 sums, sum of |d|
    __device__ __forceinline__ void add(double d, double h) {
        const double d2 = d * d;
        v[0] += h * d2;
        v[1] += h * (d2 * d);
        v[2] += h * (d2 * d2);
        v[3] += h * (d2 * d2 * d);
        v[4] += h * (d2 * d2 * d2);
        v[5] += h * fabs(d);
    }
    __device__ __forceinline__ void write(FoSums *out) const {
        out->m2 = v[0]; out->m3 = v[1]; out->m4 = v[2]; out->m5 = v[3]; out->m6 = v[4]; out->mad = v[5];
    }
};

__device__ __forceinline__ double fo_h(uint64_t n, uint32_t k) {
    return (double)((n - 1u) * (uint64_t)fo_pct(k)) / 100.0;
}

// Threads below kFoPct: the two ranks percentile threadIdx.x lies between.
__device__ __forceinline__ void fo_ranks(uint32_t *rank, uint64_t n) {
    if (threadIdx.x < (uint32_t)kFoPct) {
        const uint64_t lo = (uint64_t)floor(fo_h(n, threadIdx.x));
        rank[2 * threadIdx.x] = (uint32_t)lo;
        rank[2 * threadIdx.x + 1] = (uint32_t)min(lo + 1u, n - 1u);
    }
}

// ... and the percentile between the two values.
__device__ __forceinline__ void fo_percentiles(double *pct, const uint32_t *rank_val, uint64_t n) {
    if (threadIdx.x < (uint32_t)kFoPct) {
        const double h = fo_h(n, threadIdx.x), lo = floor(h);
        const double xl = (double)rank_val[2 * threadIdx.x], xh = (double)rank_val[2 * threadIdx.x + 1];
        pct[threadIdx.x] = xl + (h - lo) * (xh - xl);
    }
}

// Level histogram: entropy and uniformity sums (out[0], out[1], this thread's
// part) and the mode into *best (count << 32 | ~level: the highest count,
// then its lowest level).  *best is 0 on entry.
__device__ __forceinline__ void fo_levels(const uint32_t *lev, uint32_t ng, double nd, uint32_t bs, double *out,
                                          uint64_t *best) {
    uint32_t best_c = 0, best_l = 0xFFFFFFFFu;
    for (uint32_t i = threadIdx.x; i < ng; i += bs) {
        const uint32_t c = lev[i];
        if (c > best_c) { best_c = c; best_l = i; }   // i rises: the first maximum is the lowest level
        if (c) {
            const double p = (double)c / nd;
            out[0] -= p * log2(p);
            out[1] += p * p;
        }
    }
    const uint64_t key = wave_max(((uint64_t)best_c << 32) | (uint64_t)(0xFFFFFFFFu - best_l));
    if (lane() == 0) atomicMax(reinterpret_cast<unsigned long long *>(best), (unsigned long long)key);
}

// Integer sums over the voxels of bbox rows [ra, rb) and columns [ca, cb):
// fn(f, x, in) is called by every lane of a wavefront for its box voxel f
// with the voxel's value and whether it belongs to the ROI.  The label, the
// value and the neighbours' labels are loaded at once, so a voxel costs one
// round trip; a neighbour outside the image reads as label 0.
struct FoPart {
    uint64_t v[8] = {};                    // n | ne << 32, S1, S2, CX, CY, CZ, ES1, ES2
    uint32_t emin = 0xFFFFFFFFu, emax = 0u;
};

template <uint32_t BS, class Fn>
__device__ __forceinline__ FoPart fo_scan(const RoiDesc &rd, const ImgDesc &im, uint32_t ra, uint32_t rb, uint32_t ca,
                                          uint32_t cb, Fn &&fn) {
    FoPart s;
    const uint32_t nx = (uint32_t)im.nx, plane = (uint32_t)im.ny * nx, label = rd.label;
    const bool vol = im.nz > 1;
    for (RowWalk<BS> b(cb - ca, (uint32_t)(rd.y1 - rd.y0 + 1), ra, rb); b.ok(); b.next()) {
        const uint32_t X = (uint32_t)rd.x0 + ca + b.x, Y = (uint32_t)rd.y0 + b.y, Z = (uint32_t)rd.z0 + b.z;
        const uint32_t v = Z * plane + Y * nx + X;
        uint32_t l0 = 0u, l1 = 0u, l2 = 0u, l3 = 0u, l4 = label, l5 = label;
        if (X > 0u) l0 = ldg(im.L, v - 1u);
        if (X + 1u < nx) l1 = ldg(im.L, v + 1u);
        if (Y > 0u) l2 = ldg(im.L, v - nx);
        if (Y + 1u < (uint32_t)im.ny) l3 = ldg(im.L, v + nx);
        if (vol) {
            l4 = l5 = 0u;
            if (Z > 0u) l4 = ldg(im.L, v - plane);
            if (Z + 1u < (uint32_t)im.nz) l5 = ldg(im.L, v + plane);
        }
        const uint32_t x = ldg(im.I, v);
        const bool in = ldg(im.L, v) == label;
        fn(b.f, x, in);
        if (!in) continue;
        s.v[0] += 1u;
        s.v[1] += x;
        s.v[2] += (uint64_t)x * x;
        s.v[3] += (uint64_t)x * X;
        s.v[4] += (uint64_t)x * Y;
        s.v[5] += (uint64_t)x * Z;
        if (l0 != label || l1 != label || l2 != label || l3 != label || l4 != label || l5 != label) {
            s.v[0] += 1ull << 32;
            s.v[6] += x;
            s.v[7] += (uint64_t)x * x;
            s.emin = min(s.emin, x);
            s.emax = max(s.emax, x);
        }
    }
    return s;
}

// A ROI in one tile: all its sums, by the whole work-group.
__device__ void fo_roi(const RoiDesc &rd, const ImgDesc &im, uint32_t ng, FoShared &S, uint32_t *lev, FoSums *out) {
    FoRoi &R = S.r;
    const uint32_t W = (uint32_t)(rd.x1 - rd.x0 + 1), H = (uint32_t)(rd.y1 - rd.y0 + 1), area = W * rd.rows;
    const uint32_t nx = (uint32_t)im.nx, plane = (uint32_t)im.ny * nx;
    const uint32_t label = rd.label, vmin = rd.vmin, vmax = rd.vmax, D = vmax - vmin;
    const double rcp = fbn_rcp_up(D ? D : 1u);
    uint32_t sh = 0;
    while ((D >> sh) >= kFoCoarse) ++sh;
    const bool fine_needed = sh > 0, kept = area <= kFoArea;
    for (uint32_t i = threadIdx.x; i < kFoCoarse; i += kFoBlock) R.coarse[i] = 0u;
    if (fine_needed) {
        for (uint32_t i = threadIdx.x; i < kFoCoarse / 4u; i += kFoBlock) reinterpret_cast<uint32_t *>(R.slot)[i] = 0u;
        for (uint32_t i = threadIdx.x; i < kFoRanks * kFoFine; i += kFoBlock) (&R.fine[0][0])[i] = 0u;
    }
    for (uint32_t i = threadIdx.x; i < ng; i += kFoBlock) lev[i] = 0u;
    if (threadIdx.x == 0) { S.emin = 0xFFFFFFFFu; S.emax = 0u; S.best = 0ull; }
    __syncthreads();

    // ---- pass A
    FoPart s = fo_scan<kFoBlock>(rd, im, 0u, rd.rows, 0u, W, [&](uint32_t f, uint32_t x, bool in) {
        if (kept) {
            const uint64_t m = __ballot(in);   // the wavefront's lanes hold 64 consecutive box voxels
            if ((f & 63u) == 0u) R.in[f >> 6] = m;
            R.val[f] = (uint16_t)x;
        }
        if (in) {
            atomicAdd(&R.coarse[(x - vmin) >> sh], 1u);
            atomicAdd(&lev[fbn_level_rd(x, vmin, rcp, ng) - 1u], 1u);
        }
    });
    s.emin = wave_min(s.emin);
    s.emax = wave_max(s.emax);
    if (lane() == 0) { atomicMin(&S.emin, s.emin); atomicMax(&S.emax, s.emax); }
    block_sums<kFoWaves>(s.v, S.red);
    const uint64_t n = s.v[0] & 0xFFFFFFFFu, S1 = s.v[1];
    if (n == 0) {   // (cannot happen for a ROI found by discovery)
        if (threadIdx.x == 0) out->n = 0;
        return;
    }
    // (each group of sums is written as soon as it is formed: nothing is held
    // in registers through the later passes)
    if (threadIdx.x == 0) {
        out->n = n; out->ne = s.v[0] >> 32; out->S1 = S1; out->S2 = s.v[2];
        out->CX = s.v[3]; out->CY = s.v[4]; out->CZ = s.v[5]; out->ES1 = s.v[6]; out->ES2 = s.v[7];
        out->emin = S.emin; out->emax = S.emax; out->vmin = vmin; out->vmax = vmax;
    }
    const double nd = (double)n, mean = (double)S1 / nd;

    // the values of the ROI, from LDS or from the image again, in the same order
    const auto each = [&](auto &&fn) {
        if (kept) {
            for (uint32_t f = threadIdx.x; f < area; f += kFoBlock)
                if (R.in[f >> 6] >> (f & 63u) & 1u) fn((uint32_t)R.val[f]);
        } else {
            for (RowWalk<kFoBlock> b(W, H, 0u, rd.rows); b.ok(); b.next()) {
                const uint32_t v = ((uint32_t)rd.z0 + b.z) * plane + ((uint32_t)rd.y0 + b.y) * nx + (uint32_t)rd.x0 + b.x;
                const uint32_t l = ldg(im.L, v), x = ldg(im.I, v);
                if (l == label) fn(x);
            }
        }
    };

    // ---- order-statistic ranks and the coarse buckets holding them
    fo_ranks(S.rank, n);
    {
        // exclusive prefix of the coarse counts: thread t owns 4 buckets
        static_assert(kFoCoarse == 4u * kFoBlock, "four buckets per thread");
        const uint32_t b0 = 4u * threadIdx.x;
        const uint4 c = *reinterpret_cast<const uint4 *>(&R.coarse[b0]);
        const uint32_t own = c.x + c.y + c.z + c.w, incl = wave_incl_scan(own);
        if (lane() == kWave - 1) S.wave_tot[threadIdx.x / kWave] = incl;
        __syncthreads();
        uint32_t e = incl - own;
        for (uint32_t w = 0; w < threadIdx.x / kWave; ++w) e += S.wave_tot[w];
        if (own) {
            const uint32_t cc[4] = {c.x, c.y, c.z, c.w};
            for (int k = 0; k < kFoRanks; ++k) {
                const uint32_t rk = S.rank[k];
                if (rk < e || rk >= e + own) continue;
                uint32_t in = rk - e;
#pragma unroll
                for (uint32_t j = 0; j < 4u; ++j) {
                    if (in < cc[j]) { S.rank_bucket[k] = b0 + j; S.rank_in[k] = in; break; }
                    in -= cc[j];
                }
            }
        }
    }
    __syncthreads();
    if (!fine_needed) {
        if (threadIdx.x < (uint32_t)kFoRanks) S.rank_val[threadIdx.x] = vmin + S.rank_bucket[threadIdx.x];
    } else if (threadIdx.x == 0) {
        uint32_t ns = 0;
        for (int k = 0; k < kFoRanks; ++k) {
            const uint32_t b = S.rank_bucket[k];
            if (R.slot[b] == 0u) R.slot[b] = (uint8_t)(++ns);
        }
    }
    __syncthreads();

    // ---- pass B: centred moments; fine histograms of the rank buckets
    Centred cm;
    const uint32_t fmask = (1u << sh) - 1u;
    each([&](uint32_t x) {
        cm.add((double)x - mean, 1.0);
        if (fine_needed) {
            const uint32_t q = x - vmin, sl = R.slot[q >> sh];
            if (sl) atomicAdd(&R.fine[sl - 1u][q & fmask], 1u);
        }
    });
    block_sums<kFoWaves>(cm.v, S.red);
    if (threadIdx.x == 0) cm.write(out);
    if (fine_needed && threadIdx.x < (uint32_t)kFoRanks) {
        const uint32_t k = threadIdx.x, b = S.rank_bucket[k], sl = R.slot[b] - 1u;
        uint32_t acc = 0, f = 0;
        for (; f < (1u << sh); ++f) {
            acc += R.fine[sl][f];
            if (acc > S.rank_in[k]) break;
        }
        S.rank_val[k] = vmin + (b << sh) + f;
    }
    __syncthreads();
    fo_percentiles(S.pct, S.rank_val, n);
    __syncthreads();
    const double med = S.pct[3], p10 = S.pct[1], p90 = S.pct[5];

    // ---- pass C: distance to the median; count and sum of the values within
    // [P10, P90] (exact integers below 2^53)
    double c[3] = {};
    each([&](uint32_t xi) {
        const double x = (double)xi;
        c[0] += fabs(x - med);
        if (x >= p10 && x <= p90) { c[1] += 1.0; c[2] += x; }
    });
    block_sums<kFoWaves>(c, S.red);
    const double mus = c[2] / c[1];   // NaN when no value lies in [P10, P90]

    // ---- pass D: distance of the values within [P10, P90] to their mean;
    // level histogram
    double e[3] = {};
    if (c[1] > 0.0)
        each([&](uint32_t xi) {
            const double x = (double)xi;
            if (x >= p10 && x <= p90) e[2] += fabs(x - mus);
        });
    fo_levels(lev, ng, nd, kFoBlock, e, &S.best);
    block_sums<kFoWaves>(e, S.red);   // (its barriers also publish best)
    if (threadIdx.x != 0) return;
    out->mode = 0xFFFFFFFFu - (uint32_t)S.best + 1u;
    out->dmed = c[0]; out->RC = c[1]; out->rmad = e[2]; out->ent = e[0]; out->uni = e[1];
    for (int k = 0; k < kFoPct; ++k) out->pct[k] = S.pct[k];
}

// Scratch of the one-wavefront path: counters of 16 bits, two to a word (a
// box of kFoSmall voxels cannot overflow them).
struct FoWave {
    uint32_t coarse[kFoCoarse / 2u];
    uint32_t fine[kFoRanks][kFoFine / 2u];
    uint16_t val[kFoSmall];
    uint64_t in[kFoSmall / 64u];
    uint8_t slot[kFoCoarse];
    uint32_t rank[kFoRanks], rank_bucket[kFoRanks], rank_in[kFoRanks], rank_val[kFoRanks];
    uint64_t best;
    double pct[kFoPct];
};
__device__ __forceinline__ void add16(uint32_t *h, uint32_t i) { atomicAdd(&h[i >> 1], 1u << ((i & 1u) << 4)); }
__device__ __forceinline__ uint32_t get16(const uint32_t *h, uint32_t i) {
    return (uint32_t)reinterpret_cast<const uint16_t *>(h)[i];
}

// A ROI whose box holds at most kFoSmall voxels, by one wavefront (the
// work-group): the passes of fo_roi.  The integer sums stay below 2^53 here
// (2^11 voxels of 16-bit values at 16-bit coordinates), so they reduce as
// exact doubles, all of a pass in one batch.
__device__ void fo_small(const RoiDesc &rd, const ImgDesc &im, uint32_t ng, FoWave &R, uint32_t *lev, FoSums *out) {
    const uint32_t W = (uint32_t)(rd.x1 - rd.x0 + 1), area = W * rd.rows;
    const uint32_t vmin = rd.vmin, vmax = rd.vmax, D = vmax - vmin, t = threadIdx.x;
    const double rcp = fbn_rcp_up(D ? D : 1u);
    const WaveGrp g;
    uint32_t sh = 0;
    while ((D >> sh) >= kFoCoarse) ++sh;
    const bool fine_needed = sh > 0;
    for (uint32_t i = t; i < kFoCoarse / 2u; i += kWave) R.coarse[i] = 0u;
    if (fine_needed) {
        for (uint32_t i = t; i < kFoCoarse / 4u; i += kWave) reinterpret_cast<uint32_t *>(R.slot)[i] = 0u;
        for (uint32_t i = t; i < kFoRanks * kFoFine / 2u; i += kWave) (&R.fine[0][0])[i] = 0u;
    }
    for (uint32_t i = t; i < ng; i += kWave) lev[i] = 0u;
    if (t == 0) R.best = 0ull;
    __syncthreads();
    // ---- pass A
    const FoPart s = fo_scan<kWave>(rd, im, 0u, rd.rows, 0u, W, [&](uint32_t f, uint32_t x, bool in) {
        const uint64_t m = __ballot(in);
        if ((f & 63u) == 0u) R.in[f >> 6] = m;
        R.val[f] = (uint16_t)x;
        if (in) {
            add16(R.coarse, (x - vmin) >> sh);
            atomicAdd(&lev[fbn_level_rd(x, vmin, rcp, ng) - 1u], 1u);
        }
    });
    const uint32_t emin = wave_min(s.emin), emax = wave_max(s.emax);
    double a[kSumSlots] = {(double)(uint32_t)s.v[0], (double)(uint32_t)(s.v[0] >> 32), (double)s.v[1], (double)s.v[2],
                           (double)s.v[3], (double)s.v[4], (double)s.v[5], (double)s.v[6], (double)s.v[7]};
    const double av = g.reduce_slots(a);
    static_assert(offsetof(FoSums, ES2) == 64, "the first nine words of FoSums are the slots of pass A");
    if (t < 9u) reinterpret_cast<uint64_t *>(out)[t] = (uint64_t)av;
    if (t == 0) { out->emin = emin; out->emax = emax; out->vmin = vmin; out->vmax = vmax; }
    const double nd = g.bcast(av, 0), mean = g.bcast(av, 2) / nd;
    const uint64_t n = (uint64_t)nd;
    if (n == 0) return;   // (cannot happen for a ROI found by discovery)
    const auto each = [&](auto &&fn) {
        for (uint32_t f = t; f < area; f += kWave)
            if (R.in[f >> 6] >> (f & 63u) & 1u) fn((uint32_t)R.val[f]);
    };
    // ---- ranks and their coarse buckets: lane t owns buckets 16 t .. 16 t + 15
    static_assert(kFoCoarse == 16u * kWave, "sixteen buckets per lane");
    fo_ranks(R.rank, n);
    __syncthreads();
    {
        uint32_t w[8], own = 0;
#pragma unroll
        for (uint32_t j = 0; j < 8u; ++j) {
            w[j] = R.coarse[8u * t + j];
            own += (w[j] & 0xFFFFu) + (w[j] >> 16);
        }
        const uint32_t e = wave_incl_scan(own) - own;
        if (own)
            for (int k = 0; k < kFoRanks; ++k) {
                const uint32_t rk = R.rank[k];
                if (rk < e || rk >= e + own) continue;
                uint32_t in = rk - e;
                for (uint32_t j = 0; j < 16u; ++j) {
                    const uint32_t c = get16(R.coarse, 16u * t + j);
                    if (in < c) { R.rank_bucket[k] = 16u * t + j; R.rank_in[k] = in; break; }
                    in -= c;
                }
            }
    }
    __syncthreads();
    if (!fine_needed) {
        if (t < (uint32_t)kFoRanks) R.rank_val[t] = vmin + R.rank_bucket[t];
    } else if (t == 0) {
        uint32_t ns = 0;
        for (int k = 0; k < kFoRanks; ++k) {
            const uint32_t b = R.rank_bucket[k];
            if (R.slot[b] == 0u) R.slot[b] = (uint8_t)(++ns);
        }
    }
    __syncthreads();
    // ---- pass B
    Centred cm;
    const uint32_t fmask = (1u << sh) - 1u;
    each([&](uint32_t x) {
        cm.add((double)x - mean, 1.0);
        if (fine_needed) {
            const uint32_t q = x - vmin, sl = R.slot[q >> sh];
            if (sl) add16(R.fine[sl - 1u], q & fmask);
        }
    });
    double b[kSumSlots] = {cm.v[0], cm.v[1], cm.v[2], cm.v[3], cm.v[4], cm.v[5]};
    const double bv = g.reduce_slots(b);
    if (t < 6u) (&out->m2)[t] = bv;
    __syncthreads();
    if (fine_needed && t < (uint32_t)kFoRanks) {
        const uint32_t bk = R.rank_bucket[t], sl = R.slot[bk] - 1u;
        uint32_t acc = 0, f = 0;
        for (; f < (1u << sh); ++f) {
            acc += get16(R.fine[sl], f);
            if (acc > R.rank_in[t]) break;
        }
        R.rank_val[t] = vmin + (bk << sh) + f;
    }
    __syncthreads();
    fo_percentiles(R.pct, R.rank_val, n);
    __syncthreads();
    const double med = R.pct[3], p10 = R.pct[1], p90 = R.pct[5];
    // ---- pass C
    double c0 = 0.0, c1 = 0.0, c2 = 0.0;
    each([&](uint32_t xi) {
        const double x = (double)xi;
        c0 += fabs(x - med);
        if (x >= p10 && x <= p90) { c1 += 1.0; c2 += x; }
    });
    c0 = wave_sum(c0);
    c1 = wave_sum(c1);
    c2 = wave_sum(c2);
    const double mus = c2 / c1;
    // ---- pass D; level histogram
    double e[2] = {}, rmad = 0.0;
    if (c1 > 0.0)
        each([&](uint32_t xi) {
            const double x = (double)xi;
            if (x >= p10 && x <= p90) rmad += fabs(x - mus);
        });
    fo_levels(lev, ng, nd, kWave, e, &R.best);
    rmad = wave_sum(rmad);
    const double ent = wave_sum(e[0]), uni = wave_sum(e[1]);
    __syncthreads();
    if (t < (uint32_t)kFoPct) out->pct[t] = R.pct[t];
    if (t != 0) return;
    out->mode = 0xFFFFFFFFu - (uint32_t)R.best + 1u;
    out->dmed = c0; out->RC = c1; out->rmad = rmad; out->ent = ent; out->uni = uni;
}

// One tile of a split ROI: integer sums and value histogram into its slot.
// Counts of the first kFoWindow values above the ROI's minimum go through an
// LDS window, wider ones straight to global memory.
__device__ void fo_tile(const RoiDesc &rd, const ImgDesc &im, uint32_t tile, FoShared &S, FoSlot *G, uint32_t *hist) {
    uint32_t ra, rb, ca, cb;
    tile_bounds(rd.rows, (uint32_t)(rd.x1 - rd.x0 + 1), rd.n_tiles, rd.tcols, tile, &ra, &rb, &ca, &cb);
    if (ra >= rb || ca >= cb) return;
    const uint32_t bins = min(rd.vmax - rd.vmin + 1u, kFoWindow);
    for (uint32_t i = threadIdx.x; i < bins; i += kFoBlock) S.window[i] = 0u;
    __syncthreads();
    FoPart s = fo_scan<kFoBlock>(rd, im, ra, rb, ca, cb, [&](uint32_t, uint32_t x, bool in) {
        if (!in) return;
        const uint32_t q = x - rd.vmin;
        atomicAdd(q < kFoWindow ? &S.window[q] : &hist[q], 1u);
    });
    s.emin = wave_min(s.emin);
    s.emax = wave_max(s.emax);
    if (lane() == 0) { atomicMin(&G->emin, s.emin); atomicMax(&G->emax, s.emax); }
    block_sums<kFoWaves>(s.v, S.red);
    if (threadIdx.x < 8u) {
        uint64_t mine = 0;
#pragma unroll
        for (uint32_t k = 0; k < 8u; ++k)
            if (threadIdx.x == k) mine = s.v[k];
        atomicAdd(reinterpret_cast<unsigned long long *>(&G->s[threadIdx.x]), (unsigned long long)mine);
    }
    for (uint32_t i = threadIdx.x; i < bins; i += kFoBlock)
        if (S.window[i]) atomicAdd(&hist[i], S.window[i]);
}

}  // namespace

// Whether k_intensity_small takes the ROI.
__device__ __forceinline__ bool fo_is_small(const RoiDesc &rd) {
    return rd.gslot == kNone && (uint64_t)(uint32_t)(rd.x1 - rd.x0 + 1) * rd.rows <= kFoSmall;
}

__device__ __forceinline__ bool fo_in_image(const RoiDesc &rd, const ImgDesc &im) {
    return !(rd.x0 < 0 || rd.y0 < 0 || rd.z0 < 0 || rd.x1 >= im.nx || rd.y1 >= im.ny || rd.z1 >= im.nz ||
             rd.x0 > rd.x1 || rd.y0 > rd.y1 || rd.z0 > rd.z1 || rd.tcols == 0u);
}

// One wavefront per ROI with a small box.  Dynamic LDS: the level histogram.
__global__ __launch_bounds__(kWave) void k_intensity_small(StepArgs a, FoSums *sums) {
    __shared__ FoWave R;
    extern __shared__ __align__(16) uint8_t smem[];
    const uint32_t r = blockIdx.x;
    if (r >= min(a.counters[C_NROIS], a.roi_cap)) return;
    const RoiDesc rd = a.rois[r];
    if (rd.image >= (uint32_t)a.n_images || !fo_is_small(rd)) return;
    const ImgDesc im = a.imgs[rd.image];
    if (fo_in_image(rd, im)) fo_small(rd, im, (uint32_t)a.ng, R, reinterpret_cast<uint32_t *>(smem), sums + r);
    else if (threadIdx.x == 0) sums[r].n = 0;
}

// Persistent: the other tiles of the queue, one work-group each.  Dynamic
// LDS: the level histogram (ng u32).
__global__ __launch_bounds__(kFoBlock, 5) void k_intensity(StepArgs a, FoSlot *slots, FoSums *sums) {
    __shared__ FoShared S;
    extern __shared__ __align__(16) uint8_t smem[];
    ticket_load(S.misc, a.counters + C_CLASS, a.bucket_cap, threadIdx.x);
    __syncthreads();
    if (threadIdx.x == 0) ticket_prefix(S.misc);
    __syncthreads();
    const uint32_t n_rois = min(a.counters[C_NROIS], a.roi_cap);
    for (;;) {
        if (threadIdx.x == 0) {
            const uint32_t lanes = min(kTicketLanes, gridDim.x), tl = blockIdx.x % lanes;
            S.n_items = ticket_claim(S.misc, &a.counters[C_TICKETS + tl * kTicketStride], tl, lanes, a.buckets,
                                     a.bucket_cap);
        }
        __syncthreads();
        const uint32_t n_items = S.n_items;
        if (n_items == 0u) break;
        for (uint32_t q = 0; q < n_items; ++q) {
            const uint32_t r = S.misc[2u * q], tile = S.misc[2u * q + 1u];
            if (r >= n_rois) continue;
            const RoiDesc rd = a.rois[r];
            if (rd.image >= (uint32_t)a.n_images || tile >= rd.n_tiles || fo_is_small(rd)) continue;
            const ImgDesc im = a.imgs[rd.image];
            if (!fo_in_image(rd, im)) {
                if (threadIdx.x == 0) sums[r].n = 0;
                continue;
            }
            if (rd.gslot == kNone) fo_roi(rd, im, (uint32_t)a.ng, S, reinterpret_cast<uint32_t *>(smem), sums + r);
            else if (rd.gslot < a.g_cap) fo_tile(rd, im, tile, S, slots + rd.gslot, fo_hist(slots, a.g_cap, rd));
            __syncthreads();   // the scratch is reused by the next item
        }
        __syncthreads();       // every thread has read the ticket's entries
    }
}

// Split ROIs: every statistic from the slot's sums and histogram.  Dynamic
// LDS: the level histogram (ng u32).
__global__ __launch_bounds__(kFoSplitBlock) void k_intensity_split(StepArgs a, FoSlot *slots, FoSums *sums) {
    extern __shared__ __align__(16) uint8_t smem[];
    uint32_t *lev = reinterpret_cast<uint32_t *>(smem);
    __shared__ uint64_t red[kFoSplitWaves * 8], best;
    __shared__ uint32_t rank[kFoRanks], rank_val[kFoRanks], wave_tot[kFoSplitWaves];
    __shared__ double pct[kFoPct];
    const uint32_t ng = (uint32_t)a.ng, used = min(a.counters[C_NSPLIT], a.g_cap);
    for (uint32_t slot = blockIdx.x; slot < used; slot += gridDim.x) {
        const uint32_t r = a.split_roi[slot];
        if (r >= a.roi_cap) continue;
        const FoSlot &G = slots[slot];
        const uint32_t *hist = fo_hist(slots, a.g_cap, a.rois[r]);
        const uint32_t vmin = a.rois[r].vmin, vmax = a.rois[r].vmax, D = vmax - vmin;
        const double rcp = fbn_rcp_up(D ? D : 1u);
        const uint64_t n = G.s[0] & 0xFFFFFFFFu, S1 = G.s[1];
        if (n == 0) {
            if (threadIdx.x == 0) sums[r].n = 0;
            continue;
        }
        const double nd = (double)n, mean = (double)S1 / nd;
        for (uint32_t i = threadIdx.x; i < ng; i += kFoSplitBlock) lev[i] = 0u;
        if (threadIdx.x == 0) best = 0ull;
        fo_ranks(rank, n);
        // each thread owns a run of bins; exclusive prefix of the run counts
        const uint32_t per = (D + (uint32_t)kFoSplitBlock) / (uint32_t)kFoSplitBlock;
        const uint32_t b0 = min(threadIdx.x * per, D + 1u), b1 = min(b0 + per, D + 1u);
        uint32_t own = 0;
        for (uint32_t b = b0; b < b1; ++b) own += hist[b];
        const uint32_t incl = wave_incl_scan(own);
        if (lane() == kWave - 1) wave_tot[threadIdx.x / kWave] = incl;
        __syncthreads();
        uint32_t e0 = incl - own;
        for (uint32_t w = 0; w < threadIdx.x / kWave; ++w) e0 += wave_tot[w];
        if (own)
            for (int k = 0; k < kFoRanks; ++k) {
                const uint32_t rk = rank[k];
                if (rk < e0 || rk >= e0 + own) continue;
                uint32_t in = rk - e0, b = b0;
                while (b + 1u < b1 && in >= hist[b]) in -= hist[b++];
                rank_val[k] = vmin + b;
            }
        Centred cm;
        for (uint32_t b = threadIdx.x; b <= D; b += kFoSplitBlock) {
            const uint32_t h = hist[b];
            if (!h) continue;
            cm.add((double)(vmin + b) - mean, (double)h);
            atomicAdd(&lev[fbn_level_rd(vmin + b, vmin, rcp, ng) - 1u], h);
        }
        block_sums<kFoSplitWaves>(cm.v, red);   // (its barriers also publish rank_val and lev)
        fo_percentiles(pct, rank_val, n);
        __syncthreads();
        const double med = pct[3], p10 = pct[1], p90 = pct[5];
        double c[3] = {};
        for (uint32_t b = threadIdx.x; b <= D; b += kFoSplitBlock) {
            const double x = (double)(vmin + b), h = (double)hist[b];
            c[0] += h * fabs(x - med);
            if (x >= p10 && x <= p90) { c[1] += h; c[2] += h * x; }
        }
        block_sums<kFoSplitWaves>(c, red);
        const double mus = c[2] / c[1];
        double e[3] = {};
        if (c[1] > 0.0)
            for (uint32_t b = threadIdx.x; b <= D; b += kFoSplitBlock) {
                const double x = (double)(vmin + b), h = (double)hist[b];
                if (x >= p10 && x <= p90) e[2] += h * fabs(x - mus);
            }
        fo_levels(lev, ng, nd, kFoSplitBlock, e, &best);
        block_sums<kFoSplitWaves>(e, red);
        if (threadIdx.x == 0) {
            FoSums *o = sums + r;
            o->n = n; o->ne = G.s[0] >> 32; o->S1 = S1; o->S2 = G.s[2];
            o->CX = G.s[3]; o->CY = G.s[4]; o->CZ = G.s[5]; o->ES1 = G.s[6]; o->ES2 = G.s[7];
            o->emin = G.emin; o->emax = G.emax; o->vmin = vmin; o->vmax = vmax;
            o->mode = 0xFFFFFFFFu - (uint32_t)best + 1u;
            cm.write(o);
            o->dmed = c[0]; o->RC = c[1]; o->rmad = e[2]; o->ent = e[0]; o->uni = e[1];
            for (int k = 0; k < kFoPct; ++k) o->pct[k] = pct[k];
        }
        __syncthreads();
    }
}

// Clears the sums and the histogram bins in use of the split slots.
__global__ __launch_bounds__(256) void k_intensity_zero(StepArgs a, FoSlot *slots) {
    const uint32_t used = min(a.counters[C_NSPLIT], a.g_cap);
    for (uint32_t slot = blockIdx.y; slot < used; slot += gridDim.y) {
        const uint32_t r = a.split_roi[slot];
        if (r >= a.roi_cap) continue;
        FoSlot &G = slots[slot];
        uint32_t *hist = fo_hist(slots, a.g_cap, a.rois[r]);
        const uint32_t D = a.rois[r].vmax - a.rois[r].vmin, t = blockIdx.x * 256u + threadIdx.x;
        for (uint32_t b = t; b <= D; b += gridDim.x * 256u) hist[b] = 0u;
        if (t < 8u) G.s[t] = 0ull;
        if (t == 8u) { G.emin = 0xFFFFFFFFu; G.emax = 0u; }
    }
}

// The table rows, one lane per ROI, written as one contiguous run per
// work-group.
template <class OutT>
__global__ __launch_bounds__(kWave) void k_intensity_rows(StepArgs a, const FoSums *sums, OutT *table,
                                                          uint32_t table_rows) {
    __shared__ OutT rows[kWave * kNumIntensityFeat];
    const uint32_t n = min(a.counters[C_NROIS], a.roi_cap), row0 = blockIdx.x * (uint32_t)kWave;
    if (row0 >= n) return;
    const uint32_t r = row0 + threadIdx.x;
    OutT *f = rows + threadIdx.x * kNumIntensityFeat;
    const double nan = __builtin_nan("");
    if (r < n && sums[r].n == 0) {
        for (int k = 0; k < FO_COUNT; ++k) f[k] = (OutT)nan;
    } else if (r < n) {
        const FoSums s = sums[r];
        const double nd = (double)s.n, D = (double)(s.vmax - s.vmin);
        f[FO_MEAN] = (OutT)((double)s.S1 / nd);
        f[FO_MIN] = (OutT)(double)s.vmin;
        f[FO_MAX] = (OutT)(double)s.vmax;
        f[FO_RANGE] = (OutT)D;
        f[FO_INTEGRATED] = (OutT)(double)s.S1;
        f[FO_ENERGY] = (OutT)(double)s.S2;
        f[FO_RMS] = (OutT)sqrt((double)s.S2 / nd);
        // unbiased variance from exact integers: (n S2 - S1^2) / (n (n - 1))
        const u128 nvar = (u128)s.n * (u128)s.S2 - (u128)s.S1 * (u128)s.S1;
        const double var = s.n > 1u ? u128_to_double(nvar) / (nd * (nd - 1.0)) : 0.0, sd = sqrt(var);
        f[FO_VARIANCE] = (OutT)var;
        f[FO_STDDEV] = (OutT)sd;
        f[FO_STDERR] = (OutT)(sd / sqrt(nd));
        double k3 = 0.0, k4 = 0.0, k5 = 0.0, k6 = 0.0;
        if (s.vmax > s.vmin) {
            const double c2 = s.m2 / nd, c3 = s.m3 / nd, c4 = s.m4 / nd, c5 = s.m5 / nd, c6 = s.m6 / nd;
            k3 = c3 / (c2 * sqrt(c2));
            k4 = c4 / (c2 * c2);
            k5 = c5 / (c2 * c2 * sqrt(c2));
            k6 = c6 / (c2 * c2 * c2);
        }
        f[FO_SKEWNESS] = (OutT)k3;
        f[FO_KURTOSIS] = (OutT)k4;
        f[FO_HYPERSKEWNESS] = (OutT)k5;
        f[FO_HYPERFLATNESS] = (OutT)k6;
        f[FO_MEANAD] = (OutT)(s.mad / nd);
        f[FO_MEDIAN] = (OutT)s.pct[3];
        f[FO_MEDIANAD] = (OutT)(s.dmed / nd);
        f[FO_P01] = (OutT)s.pct[0];
        f[FO_P10] = (OutT)s.pct[1];
        f[FO_P25] = (OutT)s.pct[2];
        f[FO_P75] = (OutT)s.pct[4];
        f[FO_P90] = (OutT)s.pct[5];
        f[FO_P99] = (OutT)s.pct[6];
        f[FO_IQR] = (OutT)(s.pct[4] - s.pct[2]);
        f[FO_ROBUSTMAD] = (OutT)(s.RC > 0.0 ? s.rmad / s.RC : nan);
        f[FO_MODE] = (OutT)(double)s.mode;
        f[FO_ENTROPY] = (OutT)s.ent;
        f[FO_UNIFORMITY] = (OutT)s.uni;
        const uint32_t tot = s.vmax + s.vmin;
        f[FO_PIU] = (OutT)(tot ? 100.0 * (1.0 - D / (double)tot) : 100.0);
        f[FO_WCX] = (OutT)(s.S1 ? (double)s.CX / (double)s.S1 : nan);
        f[FO_WCY] = (OutT)(s.S1 ? (double)s.CY / (double)s.S1 : nan);
        f[FO_WCZ] = (OutT)(s.S1 ? (double)s.CZ / (double)s.S1 : nan);
        const double ned = (double)s.ne;
        f[FO_EDGE_INTEGRATED] = (OutT)(double)s.ES1;
        f[FO_EDGE_MIN] = (OutT)(s.ne ? (double)s.emin : nan);
        f[FO_EDGE_MAX] = (OutT)(s.ne ? (double)s.emax : nan);
        f[FO_EDGE_MEAN] = (OutT)(s.ne ? (double)s.ES1 / ned : nan);
        const u128 nevar = (u128)s.ne * (u128)s.ES2 - (u128)s.ES1 * (u128)s.ES1;
        f[FO_EDGE_STDDEV] = (OutT)(s.ne > 1u ? sqrt(u128_to_double(nevar) / (ned * (ned - 1.0))) : (s.ne ? 0.0 : nan));
    }
    __syncthreads();
    uint32_t n_out = min((uint32_t)kWave, n - row0);
    if (row0 + n_out > table_rows) {
        if (threadIdx.x == 0) atomicOr(&a.counters[C_ERR], (uint32_t)E_TABLE_CAP);
        n_out = table_rows > row0 ? table_rows - row0 : 0u;
    }
    OutT *out = table + (uint64_t)row0 * kNumIntensityFeat;
    for (uint32_t i = threadIdx.x; i < n_out * (uint32_t)kNumIntensityFeat; i += kWave) out[i] = rows[i];
}

uint64_t intensity_slot_bytes(uint32_t n_split, uint32_t n_aux) {
    return (uint64_t)n_split * sizeof(FoSlot) + 256ull * n_aux;
}
uint64_t intensity_sums_bytes(uint32_t n_rois) { return (uint64_t)n_rois * sizeof(FoSums); }

// Voxels per tile of a split ROI: a sixteenth of a CU's share of the image
// voxels, so that no region's tail outlasts the rest (with regions of up to
// 128 K voxels in one work-group the tail was most of 589 us on eight
// 2048 x 2048 images), but no fewer than a histogram's merge is worth.
uint32_t intensity_tile_vox(uint64_t total_vox, uint32_t n_cu) {
    const uint64_t t = total_vox / (16ull * (n_cu ? n_cu : 1u));
    return (uint32_t)(t > kFoMinTile ? (t < (1u << 20) ? t : (1u << 20)) : kFoMinTile);
}

// Values of its range that a ROI may have per voxel where it is split: its
// histogram is cleared, filled (past the LDS window by global atomics) and
// walked four times, so a region of few voxels and many values is better taken
// whole by one work-group.  Where the image alone does not fill the chip (tiles
// of the least size) the walk competes with the whole region's latency, about
// half of it a value of what it is a voxel; where it does, with its work.  Call
// in us, values from 0 to 65000, split always, then by this rule: one
// 2048 x 2048 image in regions of 4200 voxels 1602 and 311, of 20000 711 and
// 472, of 60000 578 and 698 (whole: 868); eight in regions of 20000 3685 and
// 858, of 60000 2355 and 1121, of 250000 1806 and 1742 (whole: 3381).
uint32_t intensity_split_values(uint32_t tile_vox) { return tile_vox > kFoMinTile ? 1u : 2u; }

hipError_t launch_intensity(const StepArgs &a, uint32_t items, uint32_t n_cu, int fp64, void *slots, void *sums,
                            void *table, uint32_t table_rows, hipStream_t st) {
    if (items == 0u || a.roi_cap == 0u) return hipSuccess;
    const uint32_t lds = (uint32_t)a.ng * 4u;
    FoSlot *sl = reinterpret_cast<FoSlot *>(slots);
    FoSums *sm = reinterpret_cast<FoSums *>(sums);
    if (a.g_cap) {
        const uint32_t gy = a.g_cap < 512u ? a.g_cap : 512u;
        hipLaunchKernelGGL(k_intensity_zero, dim3(8, gy), dim3(256), 0, st, a, sl);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_intensity_small, dim3(a.roi_cap), dim3(kWave), lds, st, a, sm);
    {
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const uint32_t per_cu = 160u * 1024u / (lds + (uint32_t)sizeof(FoShared));
    uint32_t grid = n_cu * (per_cu < 1u ? 1u : (per_cu > 8u ? 8u : per_cu));
    if (grid > items) grid = items;
    hipLaunchKernelGGL(k_intensity, dim3(grid), dim3(kFoBlock), lds, st, a, sl, sm);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.g_cap) {
        const uint32_t fin = a.g_cap < 2u * n_cu ? a.g_cap : 2u * n_cu;
        hipLaunchKernelGGL(k_intensity_split, dim3(fin), dim3(kFoSplitBlock), lds, st, a, sl, sm);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const uint32_t blocks = (a.roi_cap + (uint32_t)kWave - 1u) / (uint32_t)kWave;
    if (fp64)
        hipLaunchKernelGGL(k_intensity_rows<double>, dim3(blocks), dim3(kWave), 0, st, a, sm,
                           reinterpret_cast<double *>(table), table_rows);
    else
        hipLaunchKernelGGL(k_intensity_rows<float>, dim3(blocks), dim3(kWave), 0, st, a, sm,
                           reinterpret_cast<float *>(table), table_rows);
    return hipGetLastError();
}

}  // namespace nyx
