// Kernels of the tracker, launched by the C ABI (api.hip).
#pragma once

#include "tpc_device.h"
#include "tpc_merge.h"

namespace tpc {

// launchers of the kernels instantiated for a tuning knob (results never
// depend on it): wb = window hits read per round trip (2, 4, 8)
void launch_neighbours(int wb, int blocks, hipStream_t st, const Slot& S, const DevConst& K, int g0,
                       int ns);
// Waves that few tracklets (in lane groups, in lanes) and few tracks (refit;
// the merger's outer fits and chains) are spread over.  A call by itself wants
// more of them (its time is that of one wave's chain, and sparse waves are
// shorter), calls in flight on several streams want fewer (a group's lanes do
// the same work, so every wave more is issue that the others wait for).  The
// line lies where calls in flight are not slower than with a lane an item; us
// an event, alone and four in flight, with a lane an item, with 2048 / 2048 /
// 1024 / 1024 / 1024 waves, which is best alone, and so:
//   400 primaries     1540, 418    846, 370    857, 346
//   1000              1540, 452   1028, 540   1090, 407
//   2000              1541, 496   1157, 680   1202, 460
//   4000              1660, 602   1264, 808   1330, 565
//   32 events of 60   1715, 560   1068, 616   1073, 520
//   merger, 2000      1223, 388    685, 376    692, 358
//   merger, 6000      1088, 436    773, 487    788, 407
// Groups where rows are short (a group of 8 tests one with a read a lane or
// two, see short_row) are cheaper and the line is later: 7 events of 400 tracks
// (15000 tracklets, near the most) 1663, 512; 1088, 660; 1092, 550.  32 events of 60
// with a lane each 1278 alone, 617 with three in flight (1073, 582).
// One step to either side, 2000 primaries: lanes on 1152 and 896 waves 1231,
// 481 and 1220, 453; refit on 512 and 320: 1182, 483 and 1188, 455 (but 32
// events of 60 up to 1150 alone with 320, by where its waves fall).  Groups on
// 1536: 1550 primaries 1091, 498 (1588, 477 with a lane a tracklet).
constexpr uint32_t kShortRowWaves = 2048;
constexpr uint32_t kTrackletWaves = 1408;
constexpr uint32_t kLaneWaves = 1024;
constexpr uint32_t kRefitWaves = 384;
constexpr uint32_t kOuterWaves = 512;
constexpr uint32_t kChainWaves = 768;
// tracklets of a wave with 32 lanes or more each, and with eight or more
constexpr uint32_t kWideGroups = 2, kGroups = 8;
// bound: the most tracklets there can be; row_hits: hits of a row on average;
// blocks: for a lane a tracklet
void launch_tracklets(int wb, int64_t bound, int64_t row_hits, int blocks, int threads, hipStream_t st,
                      const Slot& S, const DevConst& K, int g0);
// stage + grid
__global__ void k_count(Slot S);
__global__ void k_grid_begin(Slot S);
constexpr int kRowThreads = 1024;   // threads of k_rows
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
__global__ void k_scan_tiles(const uint32_t* data, uint32_t n, uint32_t* partial);
__global__ void k_scan_partials(uint32_t* partial, int nb, uint32_t* data, uint32_t n, uint32_t* total_out,
                                int write_end);
__global__ void k_scan_apply(uint32_t* data, uint32_t n, const uint32_t* partial);
constexpr int kSmallPerThread = 16;
constexpr int64_t kSmallScanMax = 1024 * kSmallPerThread;
__global__ void k_scan_small(uint32_t* data, uint32_t n, uint32_t* total_out, int write_end);
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
__global__ void k_mg_write(Slot S, MergeSlot M);
// drift-velocity calibration
__global__ void k_cal_accumulate(Slot S, DevConst K, uint32_t* hist, int n_bins, double z_lo,
                                 double w);
__global__ void k_cal_fit(const uint32_t* hist, int n_bins, double z_lo, double w, double z_max,
                          double eps_t, double* out);
__global__ void k_cal_correct(const uint8_t* sector, float* z, int64_t n, double eps, double z_max);

}  // namespace tpc
