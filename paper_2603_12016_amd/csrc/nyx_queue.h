// nyx_queue.h -- work tickets of the persistent kernels: entries of the
// size-class buckets that the compaction fills, largest class first.
#pragma once
#include "nyx_device.h"

namespace nyx {

// Tickets follow ticket_offsets / ticket_range (nyx_types.h).  misc[64 + cl]:
// first ticket of class cl; misc[96 + cl]: its entries (clamped to the bucket
// capacity); misc[63]: number of tickets; misc[62]: shift of
// the most entries of one (ticket_most).  The class counts are loaded by
// lanes 0..kClasses-1 at once (ticket_load, every thread calls it), then one
// thread forms the offsets (ticket_prefix) after a barrier.
// Only the entries of the size classes [lo, hi) are handed out.
__device__ __forceinline__ void ticket_load(uint32_t *misc, const uint32_t *cls_cnt, uint32_t cap, uint32_t tid,
                                            uint32_t lo = 0u, uint32_t hi = (uint32_t)kClasses) {
    if (tid < (uint32_t)kClasses) misc[96 + tid] = tid >= lo && tid < hi ? min(cls_cnt[tid], cap) : 0u;
}

__device__ inline void ticket_prefix(uint32_t *misc) {
    uint32_t items = 0u;
    for (int cl = 0; cl < kClasses; ++cl) items += misc[96 + cl];
    misc[62] = ticket_most(items, gridDim.x);
    misc[63] = ticket_offsets(misc + 96, misc + 64, misc[62]);
}

// Claims ticket `atomicAdd(ctr) * lanes + lane` and writes its entries as
// (roi, tile) pairs to misc[0..); returns how many (0 once the queue is
// drained).  The counters of lanes 0..lanes-1 together hand out every ticket
// once.
__device__ inline uint32_t ticket_claim(uint32_t *misc, uint32_t *ctr, uint32_t lane_, uint32_t lanes, const uint2 *buckets,
                                 uint32_t cap) {
    const uint32_t t = atomicAdd(ctr, 1u) * lanes + lane_;
    if (t >= misc[63]) return 0u;
    int cl;
    uint32_t e0, e1;
    ticket_range(t, misc + 96, misc + 64, &cl, &e0, &e1, misc[62]);
    uint32_t n = 0;
    for (uint32_t e = e0; e < e1; ++e, ++n) {
        const uint2 it = buckets[(uint32_t)cl * cap + e];
        misc[2 * n] = it.x;
        misc[2 * n + 1] = it.y;
    }
    return n;
}

}  // namespace nyx
