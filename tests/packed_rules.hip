// packed_rules.hip -- test harness (not part of the library): the host
// instantiations of the packed hash table's index rules (nyx_types.h).
#include <hip/hip_runtime.h>

#include "nyx_types.h"

extern "C" {

// Largest slot over the keys [0, n) and, per slot, how many keys start there.
uint32_t packed_histogram(uint32_t n, uint32_t slots, uint32_t *hist) {
    uint32_t top = 0;
    for (uint32_t k = 0; k < n; ++k) {
        const uint32_t s = nyx::packed_bucket(k, slots);
        if (s > top) top = s;
        if (s < slots) ++hist[s];
    }
    return top;
}

uint32_t packed_slot_count(uint32_t nb, uint32_t cap) { return nyx::packed_slots(nb, cap); }

uint32_t packed_voxel_count(uint32_t cap) { return nyx::packed_voxels(cap); }

uint32_t packed_item_bound(uint32_t n, uint32_t rows, uint32_t width, uint32_t split) {
    return nyx::item_bound(n, rows, width, nyx::tiles_for(n, rows, width, split, split));
}

int packed_class3d(int dz, int dy, int dx) { return nyx::class3d(dz, dy, dx); }

}  // extern "C"
