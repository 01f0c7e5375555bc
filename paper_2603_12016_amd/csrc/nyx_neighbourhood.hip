// nyx_neighbourhood.hip -- neighbourhood texture matrices of every ROI.
//
// Three texture families of the paper's feature list (Supplementary Table S3,
// rows with the NY mark) come from one scan of each ROI voxel's
// neighbourhood: the neighbouring grey level dependence matrix (NGLDM, rows
// 175-192), the neighbourhood grey tone difference matrix (NGTDM, rows
// 246-250) and the grey level dependence matrix (GLDM, rows 251-264; the same
// dependence matrix under other names).  The paper names the features; the
// definitions are the usual ones:
//   * levels are the fixed-bin-number levels of the texture features, the
//     neighbourhood is Chebyshev distance 1 (8 neighbours in a plane, 26 in a
//     volume), and only neighbours inside the image and the ROI take part;
//   * dependence k = 1 + the neighbours whose level differs by at most alpha;
//     S(i, k) counts the ROI voxels of level i and dependence k;
//   * NGTDM: n_i counts the voxels of level i with at least one neighbour,
//     s_i sums |i - mean level of their neighbours| over them; the five
//     features use p_i = n_i / sum n over the levels present, with
//     COARSENESS = 1e6, and CONTRAST, BUSYNESS, STRENGTH = 0, where their
//     denominators vanish (a flat texture), and NaN when no voxel has a
//     neighbour.
//
// The queue of the batch kernel hands out tiles: a ROI above a share of the
// voxels is cut into several (blocks of bbox rows), so a few large regions
// fill the chip.  A tile is walked by row blocks: a lane owns a column and
// slides a 3 x 3 (x 3 planes) window of levels down it, so each voxel costs
// one (volume: three) loads and one lane exchange per side instead of a
// gather of 8 (26) labels and values.  A voxel outside the ROI holds
// kNbOut in the window: one sum over the neighbours then gives both their
// count W and their level total.  LDS atomics count S(i, k), the voxels
// without neighbours, and the exact integers A(i, W) = sum |i W - sum of
// the W neighbour levels| per level i and neighbour count W, so
// s_i = sum_W A(i, W) / W needs no floating sum during the scan.  The tables
// of a ROI in one tile become its features at once; those of a split ROI are
// added to its table in global memory, and k_nb_split finishes them.  The
// features come from exact integer moments of S (GLM, GLV, DCM, DCV, the
// non-uniformities, energy) and double sums (the weighted emphases, entropy,
// and the NGTDM pair sums over the levels present).  Bound by latency and by
// instructions (26 compares a voxel): the vector units are busy 46 % of the
// time with two wavefronts per SIMD, LDS conflicts take 1 %.  60 regions of
// 10^3-60^3 voxels in a 128 x 256 x 256 volume at 32 levels took 7.4 ms a call
// with one work-group per region and gathered neighbours (60 work-groups on
// 256 CUs), 0.34 ms so, 0.11 of them in this kernel.
#include <hip/hip_runtime.h>
#include <math.h>

#include "nyx_device.h"
#include "nyx_features.h"
#include "nyx_launch.h"
#include "nyx_queue.h"

namespace nyx {

namespace {

constexpr int kNbBlock = 256;
constexpr int kNbWaves = kNbBlock / kWave;
constexpr int kNbRows = 8;                     // rows a lane's column walk covers per unit
constexpr uint32_t kNbOut = 1u << 20;          // window value of a voxel outside the ROI (26 levels sum below it)
constexpr uint32_t kNbMinTile = 2048u;         // voxels per tile of a split ROI, at least

enum NbFeat : int {
    // NGLDM
    NB_DCENRG, NB_DCENT, NB_DCNU, NB_DCNUN, NB_DCM, NB_DCV, NB_GLNU, NB_GLNUN, NB_GLM, NB_GLV, NB_HDE, NB_HDHGLE,
    NB_HDLGLE, NB_HGLCE, NB_LDE, NB_LDHGLE, NB_LDLGLE, NB_LGLCE,
    // NGTDM
    NB_BUSYNESS, NB_COARSENESS, NB_COMPLEXITY, NB_CONTRAST, NB_STRENGTH,
    // GLDM
    NB_G_SDE, NB_G_LDE, NB_G_GLN, NB_G_DN, NB_G_DNN, NB_G_GLV, NB_G_DV, NB_G_DE, NB_G_LGLE, NB_G_HGLE, NB_G_SDLGLE,
    NB_G_SDHGLE, NB_G_LDLGLE, NB_G_LDHGLE, NB_COUNT
};
static_assert(NB_COUNT == kNumNeighbourFeat, "column count");

// Static LDS: with the dynamic tables it stays below the CU's 160 KB, whose
// last kilobyte the host leaves free.
struct NbShared {
    uint64_t red[kNbWaves * 8];
    uint32_t misc[128];      // queue state (nyx_queue.h)
    uint32_t n_occ;          // levels present in the NGTDM
    uint32_t n_items;
};
static_assert(sizeof(NbShared) <= 1024, "static LDS");

// Words of a ROI's integer tables: A (u64, ng * nn) | S (u32, ng * (nn + 1)) |
// voxels without a neighbour (u32, ng).
__host__ __device__ inline uint32_t nb_tab_words(uint32_t ng, uint32_t nn) { return ng * nn * 2u + ng * (nn + 1u) + ng; }

// The tables in LDS.
struct NbTab {
    uint64_t *A;
    uint32_t *Sd, *iso, *occ;
    double *sl;
    __device__ __forceinline__ NbTab(uint8_t *smem, uint32_t ng, uint32_t nn) {
        A = reinterpret_cast<uint64_t *>(smem);                 // ng * nn
        Sd = reinterpret_cast<uint32_t *>(A + ng * nn);         // ng * (nn + 1) dependence matrix
        iso = Sd + ng * (nn + 1u);                              // ng: voxels without a neighbour, then with one
        occ = iso + ng;                                         // ng: levels present (compacted)
        // (8-byte aligned: the words before it number an even multiple of ng, plus ng (nn + 1))
        uint32_t *e = occ + ng;
        sl = reinterpret_cast<double *>(e + ((ng * (nn + 3u)) & 1u));   // ng: s_i
    }
};

__device__ __forceinline__ uint32_t nb_prev(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x138, 0xF, 0xF, true);   // wave_shr1; lane 0 reads 0
}
__device__ __forceinline__ uint32_t nb_next(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x130, 0xF, 0xF, true);   // wave_shl1; lane 63 reads 0
}

// Counts the voxels of bbox rows [ra, rb) (rows of all planes, flattened) and
// bbox columns [ca, cb) into the LDS tables.  A unit is a strip of columns x
// kNbRows rows of one plane; a wavefront takes 1, 2 or 4 units at a time on
// groups of 64, 32 or 16 lanes (whichever needs the fewest strip steps for
// the width; the first and last lane of a group only supply neighbours).
// Every lane makes every exchange: loads are predicated, not branched.
template <bool VOL>
__device__ void nb_scan(const RoiDesc &rd, const ImgDesc &im, uint32_t ra, uint32_t rb, uint32_t ca, uint32_t cb,
                        uint32_t ng, uint32_t alpha, const NbTab &t) {
    constexpr uint32_t nn = VOL ? 26u : 8u, nk = nn + 1u;
    constexpr int P = VOL ? 3 : 1;
    const uint32_t Wb = (uint32_t)(rd.x1 - rd.x0 + 1), H = (uint32_t)(rd.y1 - rd.y0 + 1),
                   Dz = (uint32_t)(rd.z1 - rd.z0 + 1);
    const uint32_t nx = (uint32_t)im.nx, plane = (uint32_t)im.ny * nx;
    const uint32_t v00 = (uint32_t)rd.z0 * plane + (uint32_t)rd.y0 * nx + (uint32_t)rd.x0;
    const uint32_t label = rd.label, vmin = rd.vmin;
    const double rcp = fbn_rcp_up(rd.vmax > vmin ? rd.vmax - vmin : 1u);
    const uint32_t W = cb - ca;
    uint32_t lg = 0, best = ((W + 61u) / 62u) << 2;
    for (uint32_t q = 1; q <= 2u; ++q) {
        const uint32_t wo = (64u >> q) - 2u, steps = ((W + wo - 1u) / wo) << (2u - q);
        if (steps < best) { best = steps; lg = q; }
    }
    const uint32_t Wl = 64u >> lg, Wo = Wl - 2u, S = 1u << lg;
    const uint32_t ln = (uint32_t)lane(), sub = ln >> (6u - lg), col = ln & (Wl - 1u);
    const uint32_t nstrip = (W + Wo - 1u) / Wo, nch = (H + (uint32_t)kNbRows - 1u) / (uint32_t)kNbRows;
    const uint32_t z_lo = ra / H, z_n = (rb - 1u) / H - z_lo + 1u;
    const uint32_t units = nstrip * nch * z_n;
    const uint32_t w = threadIdx.x / kWave;
    for (uint32_t u0 = w * S; u0 < units; u0 += (uint32_t)kNbWaves * S) {
        const uint32_t u = u0 + sub;
        uint32_t strip = 0u, z = z_lo;
        int32_t y0 = 0, lo = 0, hi = 0;   // owned rows [lo, hi) of the unit's rows [y0, y0 + kNbRows)
        if (u < units) {
            const uint32_t q = u / nstrip, zq = q / nch;
            strip = u - q * nstrip;
            z = z_lo + zq;
            y0 = (int32_t)((q - zq * nch) * (uint32_t)kNbRows);
            lo = max(y0, (int32_t)ra - (int32_t)(z * H));
            hi = min(min(y0 + kNbRows, (int32_t)H), (int32_t)rb - (int32_t)(z * H));
        }
        if (__ballot(lo < hi) == 0ull) continue;
        const int32_t x = (int32_t)(ca + Wo * strip + col) - 1;     // bbox column of the lane
        const bool xin = lo < hi && x >= 0 && x < (int32_t)Wb;
        const bool owner = col >= 1u && col <= Wo && x < (int32_t)cb;
        uint32_t lab[P][kNbRows + 2], val[P][kNbRows + 2];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int32_t zz = VOL ? (int32_t)z + p - 1 : (int32_t)z;
            const bool pin = xin && zz >= 0 && zz < (int32_t)Dz;
#pragma unroll
            for (int j = 0; j < kNbRows + 2; ++j) {
                const int32_t y = y0 + j - 1;
                lab[p][j] = 0u;
                val[p][j] = 0u;
                if (pin && y >= lo - 1 && y <= hi && y >= 0 && y < (int32_t)H) {
                    const uint32_t v = v00 + (uint32_t)zz * plane + (uint32_t)y * nx + (uint32_t)x;
                    lab[p][j] = ldg(im.L, v);
                    val[p][j] = ldg(im.I, v);
                }
            }
        }
        // window rows j - 1, j, j + 1 at index (row mod 3): left, own, right
        uint32_t win[P][3][3], sum[P][3];
#pragma unroll
        for (int j = 0; j < kNbRows + 2; ++j) {
            const int at = j % 3;
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const uint32_t lv = fbn_level_rd(val[p][j], vmin, rcp, ng);
                const uint32_t c = lab[p][j] == label ? lv : kNbOut;   // (label 0 is never a ROI's)
                win[p][at][1] = c;
                win[p][at][0] = nb_prev(c);
                win[p][at][2] = nb_next(c);
                sum[p][at] = c + win[p][at][0] + win[p][at][2];
            }
            if (j < 2) continue;
            const int mid = (j - 1) % 3;
            const uint32_t bv = win[VOL ? 1 : 0][mid][1];
            uint32_t tot = 0u, dep = 0u;
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    tot += sum[p][r];
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const uint32_t o = win[p][r][k];
                        // (the voxel itself counts: k = 1 + its dependent neighbours)
                        dep += (o > bv ? o - bv : bv - o) <= alpha ? 1u : 0u;
                    }
                }
            const int32_t y = y0 + j - 2;
            if (owner && bv < kNbOut && y >= lo && y < hi) {
                tot -= bv;
                const uint32_t wn = nn - (tot >> 20);
                tot &= kNbOut - 1u;
                atomicAdd(&t.Sd[(bv - 1u) * nk + dep - 1u], 1u);
                if (wn) {
                    const uint32_t iw = bv * wn;
                    atomicAdd(reinterpret_cast<unsigned long long *>(&t.A[(bv - 1u) * nn + wn - 1u]),
                              (unsigned long long)(iw > tot ? iw - tot : tot - iw));
                } else {
                    atomicAdd(&t.iso[bv - 1u], 1u);
                }
            }
        }
    }
}

// The 37 features of a ROI from its integer tables in LDS, by the whole
// work-group (thread 0 writes the row).
template <class OutT>
__device__ void nb_features(const NbTab &t, NbShared &S, uint32_t ng, uint32_t nn, OutT *out) {
    const uint32_t nk = nn + 1u;
    if (threadIdx.x == 0) S.n_occ = 0u;
    __syncthreads();
    // ---- dependence matrix: exact integer moments and double emphases
    uint64_t m[8] = {};   // Ns, energy, si, si2, sk, sk2, sik2, rows2
    uint64_t c2[1] = {0};
    double e[6] = {};     // entropy, hdl, lde, ldh, ldl, lgl
    for (uint32_t c = threadIdx.x; c < ng * nk; c += kNbBlock) {
        const uint32_t q = t.Sd[c];
        if (!q) continue;
        const uint32_t i0 = c / nk, k = c - i0 * nk + 1u, i = i0 + 1u;
        const uint64_t ii = (uint64_t)i * i, kk = (uint64_t)k * k;
        m[0] += q;
        m[1] += (uint64_t)q * q;
        m[2] += (uint64_t)i * q;
        m[3] += ii * q;
        m[4] += (uint64_t)k * q;
        m[5] += kk * q;
        m[6] += ii * kk * q;
        const double qd = (double)q, id = (double)ii, kd = (double)kk;
        e[0] += qd * log2(qd);
        e[1] += qd * kd / id;
        e[2] += qd / kd;
        e[3] += qd * id / kd;
        e[4] += qd / (id * kd);
        e[5] += qd / id;
    }
    // rows of S, and with them the voxels with a neighbour, s_i and the list
    // of levels present (one thread per level owns its entries)
    for (uint32_t i = threadIdx.x; i < ng; i += kNbBlock) {
        uint64_t row = 0;
        for (uint32_t k = 0; k < nk; ++k) row += t.Sd[i * nk + k];
        m[7] += row * row;
        const uint32_t with = (uint32_t)row - t.iso[i];
        t.iso[i] = with;
        double s = 0.0;
        for (uint32_t w = 0; w < nn; ++w) {
            const uint64_t a = t.A[i * nn + w];
            if (a) s += (double)a / (double)(w + 1u);
        }
        t.sl[i] = s;
        if (with) t.occ[atomicAdd(&S.n_occ, 1u)] = i;
    }
    // columns of S: eight threads per column
    {
        const uint32_t k = threadIdx.x >> 3;
        uint64_t part = 0;
        if (k < nk)
            for (uint32_t i = threadIdx.x & 7u; i < ng; i += 8u) part += t.Sd[i * nk + k];
        part += __shfl_xor(part, 1);
        part += __shfl_xor(part, 2);
        part += __shfl_xor(part, 4);
        if (k < nk && (threadIdx.x & 7u) == 0u) c2[0] = part * part;
    }
    block_sums<kNbWaves>(m, S.red);
    block_sums<kNbWaves>(e, S.red);
    block_sums<kNbWaves>(c2, S.red);   // (its barriers also publish iso, sl and occ)
    const uint64_t Ns = m[0], e2 = m[1], si = m[2], si2 = m[3], sk = m[4], sk2 = m[5], sik2 = m[6], rows2 = m[7];
    const uint64_t cols2 = c2[0];
    const double ent = e[0], hdl = e[1], lde = e[2], ldh = e[3], ldl = e[4], lgl = e[5];

    // ---- NGTDM over the levels present
    const uint32_t ngp = S.n_occ;
    uint64_t v1[1] = {0};
    for (uint32_t q = threadIdx.x; q < ngp; q += kNbBlock) v1[0] += t.iso[t.occ[q]];
    block_sums<kNbWaves>(v1, S.red);
    const uint64_t nvp = v1[0];
    const double inv_nvp = nvp ? 1.0 / (double)nvp : 0.0;
    double g[6] = {};   // sum p s, sum s, then the pair sums: contrast, busyness denominator, complexity, strength
    for (uint32_t q = threadIdx.x; q < ngp; q += kNbBlock) {
        const uint32_t i = t.occ[q];
        g[0] += (double)t.iso[i] * inv_nvp * t.sl[i];
        g[1] += t.sl[i];
    }
    // pair sums: every term is symmetric and vanishes for i = j, so each
    // unordered pair is visited once (a wavefront per first level) and
    // counted twice; the busyness denominator is summed in voxels, exactly, as
    // it can vanish with several levels present
    for (uint32_t a = threadIdx.x / kWave; a < ngp; a += (uint32_t)kNbWaves) {
        const uint32_t i = t.occ[a];
        const double ni = (double)t.iso[i], pi = ni * inv_nvp, li = (double)(i + 1u), si_ = t.sl[i];
        for (uint32_t c = a + 1u + (uint32_t)lane(); c < ngp; c += (uint32_t)kWave) {
            const uint32_t j = t.occ[c];
            const double nj = (double)t.iso[j], pj = nj * inv_nvp, lj = (double)(j + 1u), d = li - lj;
            g[2] += pi * pj * d * d;
            g[3] += fabs(li * ni - lj * nj);   // whole numbers, below 2^53 in all
            g[4] += fabs(d) * (pi * si_ + pj * t.sl[j]) / (pi + pj);
            g[5] += (pi + pj) * d * d;
        }
    }
    block_sums<kNbWaves>(g, S.red);
    const double ps = g[0], ssum = g[1], con = 2.0 * g[2], bden = nvp ? 2.0 * g[3] / (double)nvp : 0.0, cpx = 2.0 * g[4], str = 2.0 * g[5];
    __syncthreads();   // every thread is done with the tables
    if (threadIdx.x != 0) return;
    double f[NB_COUNT];
    const double nsd = (double)Ns, inv = 1.0 / nsd, ns2 = nsd * nsd;
    f[NB_DCENRG] = (double)e2 / ns2;
    f[NB_DCENT] = log2(nsd) - ent * inv;
    f[NB_DCNU] = (double)cols2 * inv;
    f[NB_DCNUN] = (double)cols2 / ns2;
    f[NB_DCM] = (double)sk * inv;
    f[NB_DCV] = u128_to_double((u128)Ns * sk2 - (u128)sk * sk) / ns2;
    f[NB_GLNU] = (double)rows2 * inv;
    f[NB_GLNUN] = (double)rows2 / ns2;
    f[NB_GLM] = (double)si * inv;
    f[NB_GLV] = u128_to_double((u128)Ns * si2 - (u128)si * si) / ns2;
    f[NB_HDE] = (double)sk2 * inv;
    f[NB_HDHGLE] = (double)sik2 * inv;
    f[NB_HDLGLE] = hdl * inv;
    f[NB_HGLCE] = (double)si2 * inv;
    f[NB_LDE] = lde * inv;
    f[NB_LDHGLE] = ldh * inv;
    f[NB_LDLGLE] = ldl * inv;
    f[NB_LGLCE] = lgl * inv;
    if (nvp == 0) {
        f[NB_BUSYNESS] = f[NB_COARSENESS] = f[NB_COMPLEXITY] = f[NB_CONTRAST] = f[NB_STRENGTH] = __builtin_nan("");
    } else {
        f[NB_COARSENESS] = ps > 0.0 ? 1.0 / ps : 1.0e6;
        f[NB_CONTRAST] = ngp > 1u ? con / ((double)ngp * (double)(ngp - 1u)) * ssum * inv_nvp : 0.0;
        f[NB_BUSYNESS] = bden > 0.0 ? ps / bden : 0.0;
        f[NB_COMPLEXITY] = cpx * inv_nvp;
        f[NB_STRENGTH] = ssum > 0.0 ? str / ssum : 0.0;
    }
    f[NB_G_SDE] = f[NB_LDE];
    f[NB_G_LDE] = f[NB_HDE];
    f[NB_G_GLN] = f[NB_GLNU];
    f[NB_G_DN] = f[NB_DCNU];
    f[NB_G_DNN] = f[NB_DCNUN];
    f[NB_G_GLV] = f[NB_GLV];
    f[NB_G_DV] = f[NB_DCV];
    f[NB_G_DE] = f[NB_DCENT];
    f[NB_G_LGLE] = f[NB_LGLCE];
    f[NB_G_HGLE] = f[NB_HGLCE];
    f[NB_G_SDLGLE] = f[NB_LDLGLE];
    f[NB_G_SDHGLE] = f[NB_LDHGLE];
    f[NB_G_LDLGLE] = f[NB_HDLGLE];
    f[NB_G_LDHGLE] = f[NB_HDHGLE];
    for (int k = 0; k < NB_COUNT; ++k) out[k] = (OutT)f[k];
}

}  // namespace

// LDS bytes of the per-ROI tables for ng levels and nn neighbours.
__host__ __device__ inline uint32_t nb_lds_bytes(uint32_t ng, uint32_t nn) {
    // the integer tables | occupied levels (u32, ng) | s (double, ng), 8-byte aligned
    return nb_tab_words(ng, nn) * 4u + ng * 4u + ng * 8u + 16u;
}

// Persistent: the tiles of the queue, one work-group each.  nn_max:
// neighbours per voxel the LDS tables are laid out for (8 or 26); gtab:
// tables of split ROIs, one per split slot, zero on entry.  At most 168 VGPRs,
// three waves per SIMD: the features of small regions wait for their
// reductions (466489 regions of 3 x 3 at 32 levels, call: 9.87 ms with a
// work-group per region, 11.69 with 169 VGPRs, 8.80 so, 9.02 with 128 and
// spills).
template <class OutT>
__global__ __launch_bounds__(kNbBlock, 3) void k_neighbourhood(StepArgs a, uint32_t alpha, uint32_t nn_max,
                                                            uint32_t *gtab, OutT *table, uint32_t table_rows) {
    __shared__ NbShared S;
    extern __shared__ __align__(16) uint8_t smem[];
    const uint32_t ng = (uint32_t)a.ng;
    uint32_t *const words = reinterpret_cast<uint32_t *>(smem);
    ticket_load(S.misc, a.counters + C_CLASS, a.bucket_cap, threadIdx.x);
    __syncthreads();
    if (threadIdx.x == 0) ticket_prefix(S.misc);
    __syncthreads();
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
            if (r >= min(a.counters[C_NROIS], a.roi_cap)) continue;
            if (r >= table_rows) {
                if (threadIdx.x == 0) atomicOr(&a.counters[C_ERR], (uint32_t)E_TABLE_CAP);
                continue;
            }
            const RoiDesc rd = a.rois[r];
            if (rd.image >= (uint32_t)a.n_images || tile >= rd.n_tiles) continue;
            const ImgDesc im = a.imgs[rd.image];
            if (rd.x0 < 0 || rd.y0 < 0 || rd.z0 < 0 || rd.x1 >= im.nx || rd.y1 >= im.ny || rd.z1 >= im.nz ||
                rd.x0 > rd.x1 || rd.y0 > rd.y1 || rd.z0 > rd.z1 || rd.tcols == 0u)
                continue;
            const bool vol = im.nz > 1;
            const uint32_t nn = vol ? 26u : 8u, nw = nb_tab_words(ng, nn);
            if (nn > nn_max) {
                if (threadIdx.x == 0) atomicOr(&a.counters[C_ERR], (uint32_t)E_LIST_CAP);
                continue;
            }
            for (uint32_t i = threadIdx.x; i < nw; i += kNbBlock) words[i] = 0u;
            __syncthreads();
            const NbTab t(smem, ng, nn);
            uint32_t ra, rb, ca, cb;
            tile_bounds(rd.rows, (uint32_t)(rd.x1 - rd.x0 + 1), rd.n_tiles, rd.tcols, tile, &ra, &rb, &ca, &cb);
            if (ra < rb && ca < cb) {
                if (vol) nb_scan<true>(rd, im, ra, rb, ca, cb, ng, alpha, t);
                else nb_scan<false>(rd, im, ra, rb, ca, cb, ng, alpha, t);
            }
            __syncthreads();
            if (rd.gslot == kNone) {
                nb_features(t, S, ng, nn, table + (uint64_t)r * kNumNeighbourFeat);
            } else if (rd.gslot < a.g_cap) {
                uint32_t *G = gtab + (uint64_t)rd.gslot * nb_tab_words(ng, nn_max);
                const uint32_t n64 = ng * nn;   // leading 64-bit entries
                for (uint32_t i = threadIdx.x; i < n64; i += kNbBlock)
                    if (t.A[i])
                        atomicAdd(reinterpret_cast<unsigned long long *>(G) + i, (unsigned long long)t.A[i]);
                for (uint32_t i = 2u * n64 + threadIdx.x; i < nw; i += kNbBlock)
                    if (words[i]) atomicAdd(&G[i], words[i]);
            }
            __syncthreads();   // the tables are cleared for the next tile
        }
        __syncthreads();       // every thread has read the ticket's entries
    }
}

// Split ROIs: the features from the tables their tiles were added to.
template <class OutT>
__global__ __launch_bounds__(kNbBlock) void k_nb_split(StepArgs a, uint32_t nn_max, const uint32_t *gtab, OutT *table,
                                                       uint32_t table_rows) {
    __shared__ NbShared S;
    extern __shared__ __align__(16) uint8_t smem[];
    const uint32_t ng = (uint32_t)a.ng, used = min(a.counters[C_NSPLIT], a.g_cap);
    uint32_t *const words = reinterpret_cast<uint32_t *>(smem);
    for (uint32_t slot = blockIdx.x; slot < used; slot += gridDim.x) {
        const uint32_t r = a.split_roi[slot];
        if (r >= a.roi_cap || r >= table_rows || a.rois[r].image >= (uint32_t)a.n_images) continue;
        const uint32_t nn = a.imgs[a.rois[r].image].nz > 1 ? 26u : 8u, nw = nb_tab_words(ng, nn);
        if (nn > nn_max) continue;
        const uint32_t *G = gtab + (uint64_t)slot * nb_tab_words(ng, nn_max);
        for (uint32_t i = threadIdx.x; i < nw; i += kNbBlock) words[i] = G[i];
        __syncthreads();
        const NbTab t(smem, ng, nn);
        nb_features(t, S, ng, nn, table + (uint64_t)r * kNumNeighbourFeat);
        __syncthreads();
    }
}

// Zeroes the tables of the split slots in use.
__global__ __launch_bounds__(256) void k_nb_zero(StepArgs a, uint32_t *gtab, uint32_t slot_words) {
    const uint64_t n = (uint64_t)min(a.counters[C_NSPLIT], a.g_cap) * slot_words;
    for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < n; i += gridDim.x * 256ull) gtab[i] = 0u;
}

uint32_t neighbourhood_lds_bytes(uint32_t ng, int any_volume) { return nb_lds_bytes(ng, any_volume ? 26u : 8u); }

uint64_t neighbourhood_slot_bytes(uint32_t ng, int any_volume) {
    return (uint64_t)nb_tab_words(ng, any_volume ? 26u : 8u) * 4u;
}

// Voxels per tile of a split ROI: a sixteenth of a CU's share of the image
// voxels (an even spread whatever part of them is ROI), but no fewer than a
// merge of the tables is worth (a quarter of their bytes).
uint32_t neighbourhood_tile_vox(uint64_t total_vox, uint32_t n_cu, uint32_t ng, int any_volume) {
    const uint64_t share = total_vox / (16ull * (n_cu ? n_cu : 1u));
    const uint64_t least = neighbourhood_slot_bytes(ng, any_volume) / 4u;
    uint64_t t = share > kNbMinTile ? share : kNbMinTile;
    if (t < least) t = least;
    return (uint32_t)(t < (1u << 20) ? t : (1u << 20));
}

template <class OutT>
static hipError_t launch_nb(const StepArgs &a, uint32_t items, uint32_t n_cu, uint32_t alpha, uint32_t nn,
                            uint32_t *gtab, OutT *table, uint32_t table_rows, hipStream_t st) {
    const uint32_t lds = nb_lds_bytes((uint32_t)a.ng, nn);
    // the dynamic tables plus the static NbShared stay within the CU's 160 KB
    for (const void *f : {reinterpret_cast<const void *>(&k_neighbourhood<OutT>),
                          reinterpret_cast<const void *>(&k_nb_split<OutT>)}) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    // levels differ by less than ng: a larger alpha means the same, and stays below kNbOut
    const uint32_t al = alpha < (uint32_t)a.ng ? alpha : (uint32_t)a.ng;
    const uint32_t per_cu = 160u * 1024u / (lds + 1024u);
    uint32_t grid = n_cu * (per_cu < 1u ? 1u : (per_cu > 4u ? 4u : per_cu));
    if (grid > items) grid = items;
    if (a.g_cap) {
        const uint32_t slot_words = nb_tab_words((uint32_t)a.ng, nn);
        hipLaunchKernelGGL(k_nb_zero, dim3(2u * n_cu), dim3(256), 0, st, a, gtab, slot_words);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_neighbourhood<OutT>, dim3(grid), dim3(kNbBlock), lds, st, a, al, nn, gtab, table, table_rows);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !a.g_cap) return e;
    const uint32_t fin = a.g_cap < 4u * n_cu ? a.g_cap : 4u * n_cu;
    hipLaunchKernelGGL(k_nb_split<OutT>, dim3(fin), dim3(kNbBlock), lds, st, a, nn, gtab, table, table_rows);
    return hipGetLastError();
}

hipError_t launch_neighbourhood(const StepArgs &a, uint32_t items, uint32_t n_cu, int fp64, uint32_t alpha,
                                int any_volume, uint32_t *gtab, void *table, uint32_t table_rows, hipStream_t st) {
    if (items == 0u) return hipSuccess;
    const uint32_t nn = any_volume ? 26u : 8u;
    if (fp64)
        return launch_nb(a, items, n_cu, alpha, nn, gtab, reinterpret_cast<double *>(table), table_rows, st);
    return launch_nb(a, items, n_cu, alpha, nn, gtab, reinterpret_cast<float *>(table), table_rows, st);
}

}  // namespace nyx
