// Kernels of the tracker, launched by the C ABI (api.hip).
#pragma once

#include "tpc_device.h"
#include "tpc_merge.h"

namespace tpc {

// launchers of the kernels instantiated for a tuning knob (results never
// depend on it): wb = window hits read per round trip (2, 4, 8)
void launch_neighbours(int wb, int blocks, hipStream_t st, const Slot& S, const DevConst& K, int g0,
                       int ns);
// waves that few tracklets / tracks are spread over: measured best of 512,
// 1024, 2048, 4096 (tracklets, us, 32 pp events: 824, 753, 714, 770; one
// peripheral event: 809, 762, 755, 845; tracks: 334, 328, 611, 761; 354, 325,
// 566, 838, where two of the fp64 waves to a SIMD already share its issue)
constexpr uint32_t kTrackletWaves = 2048;
constexpr uint32_t kRefitWaves = 1024;
constexpr uint32_t kFewTracklets = 2 * kTrackletWaves;     // 32 lanes or more a tracklet
constexpr uint32_t kGroupTracklets = 8 * kTrackletWaves;   // eight lanes or more a tracklet
// bound: the most tracklets there can be; blocks: for a lane a tracklet
void launch_tracklets(int wb, int64_t bound, int blocks, int threads, hipStream_t st, const Slot& S,
                      const DevConst& K, int g0);
// stage + grid
__global__ void k_count(Slot S);
__global__ void k_grid_begin(Slot S);
template <bool kTotals>
__global__ void k_rows(Slot S, RowTable X, int n_min_chain, int n_min_track);
__global__ void k_scatter(Slot S);
__global__ void k_row_sort(Slot S, DevConst K);
__global__ void k_row_sort_large(Slot S, DevConst K);
// cellular automaton
__global__ void k_clean_rows(Slot S, int g0, int ns, int n_min_chain);
__global__ void k_start_write(Slot S, int g0, int ns);
// selection (the same grid for both, a multiple of 8 blocks)
__global__ void k_select(Slot S, DevConst K, int g0);
__global__ void k_track_write(Slot S, int g0, int ns);
// Kalman filter
__global__ void k_refit(Slot S, DevConst K, int g0, int ns);
// output
__global__ void k_scan_tiles(const uint32_t* in, const uint32_t* n_dev, int64_t n_host,
                             uint32_t* partial);
__global__ void k_scan_partials(uint32_t* partial, int nb, uint32_t* out, const uint32_t* n_dev,
                                int64_t n_host, uint32_t* total_out, int write_end);
__global__ void k_scan_apply(const uint32_t* in, const uint32_t* n_dev, int64_t n_host,
                             const uint32_t* partial, uint32_t* out);
constexpr int kRowThreadsLaunch = 1024;   // threads of k_rows
constexpr int kSmallPerThread = 16;
constexpr int64_t kSmallScanMax = 1024 * kSmallPerThread;
__global__ void k_scan_small(uint32_t* data, const uint32_t* n_dev, int64_t n_host,
                             uint32_t* total_out, int write_end);
constexpr int kOrderBlocks = 2048;
constexpr int kOrderTile = 1024;    // clusters a block of the output order takes at a time
__global__ void k_out_count(Slot S, int64_t chunk);
__global__ void k_out_order(Slot S, int64_t chunk);
__global__ void k_write_out(Slot S);
// cross-sector merger
__global__ void k_mg_begin(Slot S, MergeSlot M);
__global__ void k_mg_count(Slot S, MergeSlot M);
__global__ void k_mg_scatter(Slot S, MergeSlot M);
__global__ void k_mg_outer(Slot S, DevConst K, MergeSlot M, MergeConst C);
template <bool kFinal>
__global__ void k_mg_pairs(Slot S, DevConst K, MergeSlot M, MergeConst C);
__global__ void k_mg_pair_best(MergeSlot M);
__global__ void k_mg_link(Slot S, MergeSlot M);
__global__ void k_mg_chain(Slot S, DevConst K, MergeSlot M, MergeConst C);
__global__ void k_mg_emit(Slot S, MergeSlot M, int64_t chunk);
__global__ void k_mg_pos(Slot S, MergeSlot M, int64_t chunk);
__global__ void k_mg_write(Slot S, DevConst K, MergeSlot M);
// drift-velocity calibration
__global__ void k_cal_accumulate(Slot S, DevConst K, uint32_t* hist, int n_bins, double z_lo,
                                 double w);
__global__ void k_cal_fit(const uint32_t* hist, int n_bins, double z_lo, double w, double z_max,
                          double eps_t, double* out);
__global__ void k_cal_correct(const uint8_t* sector, float* z, int64_t n, double eps, double z_max);

}  // namespace tpc
