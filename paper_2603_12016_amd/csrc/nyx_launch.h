// nyx_launch.h -- host-side launchers of the kernels in nyx_kernels.hip.
#pragma once
#include <hip/hip_runtime.h>

#include "nyx_types.h"

namespace nyx {

hipError_t launch_max_label(const ImgDesc *imgs, int n_images, uint64_t most_vox, uint32_t *out, hipStream_t st);
hipError_t launch_label_collect(const ImgDesc *imgs, int n_images, uint64_t max_vox, uint64_t *list, uint32_t cap,
                                uint32_t *count, hipStream_t st);
hipError_t launch_reset(const StepArgs &a, uint32_t n_counters, hipStream_t st);
hipError_t launch_reset_counters(const StepArgs &a, uint32_t n_counters, hipStream_t st);
hipError_t launch_roi_out(const StepArgs &a, hipStream_t st);
hipError_t launch_fill_u64(uint64_t *p, uint64_t n, uint64_t v, hipStream_t st);
hipError_t launch_zero_split(const StepArgs &a, hipStream_t st);
hipError_t launch_scan(const StepArgs &a, hipStream_t st);
hipError_t launch_compact(const StepArgs &a, uint32_t roi_lo, uint32_t roi_hi, hipStream_t st);
hipError_t launch_bin_image(const StepArgs &a, uint16_t *bins, uint64_t total_vox, const uint64_t *img_vox_base,
                            hipStream_t st);
hipError_t launch_batch(const StepArgs &a, uint32_t grid, uint32_t block, uint32_t direct_roi, hipStream_t st);
hipError_t batch_occupancy(const StepArgs &a, uint32_t block, int *blocks_per_cu);
hipError_t launch_band(const StepArgs &a, uint32_t grid, hipStream_t st);
hipError_t launch_split_finalize(const StepArgs &a, hipStream_t st);
hipError_t launch_features(const StepArgs &a, const DirSums *ds, const DirSumsY *dsy, uint32_t n_cap,
                           const uint32_t *n_ptr, hipStream_t st);
hipError_t launch_coo_count(const StepArgs &a, uint32_t n_slots, uint64_t *counts, hipStream_t st);
hipError_t launch_coo_emit(const StepArgs &a, uint32_t n_slots, const uint64_t *offsets, uint64_t *keys,
                           uint64_t *vals, hipStream_t st);
hipError_t launch_coo_features(const StepArgs &a, const uint64_t *keys, const uint64_t *vals, uint64_t nnz,
                               uint32_t n_rois, uint64_t *seg, DirSums *sums, DirSumsY *sums_y, hipStream_t st);
uint64_t intensity_slot_bytes(uint32_t n_split, uint32_t n_aux);
uint64_t intensity_sums_bytes(uint32_t n_rois);
uint32_t intensity_tile_vox(uint64_t total_vox, uint32_t n_cu);
uint32_t intensity_split_values(uint32_t tile_vox);
hipError_t launch_intensity(const StepArgs &a, uint32_t items, uint32_t n_cu, int fp64, void *slots, void *sums,
                            void *table, uint32_t table_rows, hipStream_t st);
uint32_t neighbourhood_lds_bytes(uint32_t ng, int any_volume);
uint64_t neighbourhood_slot_bytes(uint32_t ng, int any_volume);
uint32_t neighbourhood_tile_vox(uint64_t total_vox, uint32_t n_cu, uint32_t ng, int any_volume);
hipError_t launch_neighbourhood(const StepArgs &a, uint32_t items, uint32_t n_cu, int fp64, uint32_t alpha,
                                int any_volume, uint32_t *gtab, void *table, uint32_t table_rows, hipStream_t st);

}  // namespace nyx
