// nyx_queue.h -- work tickets of the persistent kernels: entries of the
// size-class buckets that the compaction fills, largest class first.
#pragma once
#include "nyx_device.h"

namespace nyx {

// Tickets follow ticket_offsets / ticket_range (nyx_types.h).  misc[64 + cl]:
// first ticket of class cl; misc[96 + cl]: its entries (clamped to the bucket
// capacity); misc[63]: number of tickets.  The class counts are loaded by
// lanes 0..kClasses-1 at once (ticket_load, every thread calls it), then one
// thread forms the offsets (ticket_prefix) after a barrier.
__device__ __forceinline__ void ticket_load(uint32_t *misc, const uint32_t *cls_cnt, uint32_t cap, uint32_t tid) {
    if (tid < (uint32_t)kClasses) misc[96 + tid] = min(cls_cnt[tid], cap);
}

__device__ inline void ticket_prefix(uint32_t *misc) { misc[63] = ticket_offsets(misc + 96, misc + 64); }

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
    ticket_range(t, misc + 96, misc + 64, &cl, &e0, &e1);
    uint32_t n = 0;
    for (uint32_t e = e0; e < e1; ++e, ++n) {
        const uint2 it = buckets[(uint32_t)cl * cap + e];
        misc[2 * n] = it.x;
        misc[2 * n + 1] = it.y;
    }
    return n;
}

}  // namespace nyx
