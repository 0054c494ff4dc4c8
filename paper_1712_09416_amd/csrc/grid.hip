// Stage and grid: clusters -> per (sector, pad row) hit lists ordered by
// (bin, cluster ID), with a 2-D y x z bin index per row.
//
// This is the input step of the CA tracker: the neighbours finder and the
// Kalman search query "all hits of row r inside a window", and the bins make
// those queries touch a handful of hits.  Results never depend on the bin
// layout: queries scan every bin that can hold a hit of the window and then
// apply the exact window test on each hit.
#include "tpc_device.h"
#include "tpc_kernels.h"

namespace tpc {

// a1: validate, count clusters per (sector, row) and give each its rank
// inside the row (arrival order; the row sort below makes it canonical).
// One block per chunk of kCountChunk clusters of one event (blockIdx.y):
// ranks are taken in an LDS histogram of the event's rows, then one global
// atomic per row and block reserves the block's range.
constexpr int kCountChunk = 4096;
constexpr int kEventRows = kSectorsPerEvent * kRows;
constexpr int kCountThreads = 256;
constexpr int kRowsPerThread = (kEventRows + kCountThreads - 1) / kCountThreads;
constexpr int kCountBatch = 4;

__global__ void __launch_bounds__(kCountThreads) k_count(Slot S) {
  __shared__ uint32_t hist[kEventRows];
  const int e = blockIdx.y;
  const int64_t e0 = S.ev_off[e], e1 = S.ev_off[e + 1];
  const int64_t i0 = e0 + (int64_t)blockIdx.x * kCountChunk;
  if (i0 >= e1) return;
  const int64_t i1 = min(e1, i0 + (int64_t)kCountChunk);
  for (int r = threadIdx.x; r < kEventRows; r += blockDim.x) hist[r] = 0u;
  __syncthreads();
  // clusters kCountBatch per thread at a time: loads first, then the LDS
  // ranks
  for (int64_t ib = i0 + threadIdx.x; ib < i1; ib += kCountBatch * kCountThreads) {
    int sec[kCountBatch], row[kCountBatch];
    float y[kCountBatch], z[kCountBatch];
#pragma unroll
    for (int u = 0; u < kCountBatch; ++u) {
      const int64_t i = ib + u * kCountThreads;
      sec[u] = 0;
      row[u] = 0;
      y[u] = 0.0f;
      z[u] = 0.0f;
      if (i < i1) {
        sec[u] = S.sector[i];
        row[u] = S.row[i];
        y[u] = S.y[i];
        z[u] = S.z[i];
      }
    }
#pragma unroll
    for (int u = 0; u < kCountBatch; ++u) {
      const int64_t i = ib + u * kCountThreads;
      if (i >= i1) continue;
      S.tmap[i] = -1;
      if (sec[u] >= kSectorsPerEvent || row[u] >= kRows || !isfinite(y[u]) || !isfinite(z[u])) {
        atomicAdd(&S.err[0], 1u);
        S.rank[i] = kNoHit;
        continue;
      }
      S.rank[i] = atomicAdd(&hist[sec[u] * kRows + row[u]], 1u);
    }
  }
  __syncthreads();
  // every atomic of the thread is issued before the first result is used
  uint32_t* cnt = S.row_cnt + (size_t)e * kEventRows;
  uint32_t res[kRowsPerThread];
#pragma unroll
  for (int k = 0; k < kRowsPerThread; ++k) {
    const int r = threadIdx.x + k * kCountThreads;
    const uint32_t c = r < kEventRows ? hist[r] : 0u;
    res[k] = c ? atomicAdd(&cnt[r], c) : 0u;
  }
#pragma unroll
  for (int k = 0; k < kRowsPerThread; ++k) {
    const int r = threadIdx.x + k * kCountThreads;
    if (r < kEventRows) hist[r] = res[k];
  }
  __syncthreads();
  for (int64_t ib = i0 + threadIdx.x; ib < i1; ib += kCountBatch * kCountThreads) {
    uint32_t rk[kCountBatch];
    int sr[kCountBatch];
#pragma unroll
    for (int u = 0; u < kCountBatch; ++u) {
      const int64_t i = ib + u * kCountThreads;
      rk[u] = kNoHit;
      sr[u] = 0;
      if (i < i1) {
        rk[u] = S.rank[i];
        sr[u] = S.sector[i] * kRows + S.row[i];
      }
    }
#pragma unroll
    for (int u = 0; u < kCountBatch; ++u) {
      const int64_t i = ib + u * kCountThreads;
      if (i < i1 && rk[u] != kNoHit) S.rank[i] = rk[u] + hist[sr[u]];
    }
  }
}

// Bin layout of one row with n hits: ~bin_target hits per bin, edges at
// least bin_min_edge, at most kBinsPerHit * max(n, 1) bins.
// Its part of the bin table starts where the rows before it would end if all
// were as long as they can be, so no row waits for the others' layouts.
__device__ RowBins make_bins(const DevConst& K, const Slot& S, int sr, uint32_t first, uint32_t n) {
  const int g = sr / kRows;
  const float x_row = S.row_x[sr - g * kRows];
  const bool side_c = (g % kSectorsPerEvent) >= kSectorsPerEvent / 2;
  RowBins b;
  const float ymax = x_row * K.tanh_half + K.medge;
  const float wy = 2.0f * ymax;
  const float wz = K.z_max + 2.0f * K.mz;
  b.y0 = -ymax;
  b.z0 = side_c ? -(K.z_max + K.mz) : -K.mz;
  const float nn = n > 0 ? (float)n : 1.0f;
  float edge = sqrtf(wy * wz * K.bin_target / nn);
  if (edge < K.bin_min_edge) edge = K.bin_min_edge;
  int ny = 1, nz = 1;
  const uint32_t nmax = (uint32_t)kBinsPerHit * (n > 0 ? n : 1u);
  for (int it = 0; it < 32; ++it) {
    ny = (int)ceilf(wy / edge);
    nz = (int)ceilf(wz / edge);
    ny = ny < 1 ? 1 : (ny > 128 ? 128 : ny);
    nz = nz < 1 ? 1 : (nz > 128 ? 128 : nz);
    if ((uint32_t)(ny * nz) <= nmax) break;
    edge *= 1.25f;
  }
  if ((uint32_t)(ny * nz) > nmax) { ny = 1; nz = 1; }
  b.ny = ny;
  b.nz = nz;
  b.iby = (float)ny / wy;
  b.ibz = (float)nz / wz;
  b.base = bin_table_pair(first, (uint32_t)sr);
  b.first = (int32_t)first;
  return b;
}

// The slot's counters and the rows' counts at zero.
__global__ void k_grid_begin(Slot S) {
  const int SR = S.n_sectors * kRows;
  const int stride = gridDim.x * blockDim.x;
  const int t0 = blockIdx.x * blockDim.x + threadIdx.x;
  for (int sr = t0; sr < SR; sr += stride) S.row_cnt[sr] = 0u;
  if (t0 < 4) S.err[t0] = 0u;
  if (t0 < 16) reinterpret_cast<uint32_t*>(S.stats)[t0] = 0u;
  if (t0 == 0) S.range_cnt[2] = 0u;   // rows over 1024 hits, listed by the row sort
}

// Running sum over a block of kRowThreads threads (exclusive, in place);
// returns the block's total.
constexpr int kRowsOfThread = (kEventRows + kRowThreads - 1) / kRowThreads;
__device__ __forceinline__ uint32_t row_block_scan(uint32_t& v) {
  __shared__ uint32_t ws[kRowThreads / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t x = __shfl_up(inc, d, 64);
    if (lane >= d) inc += x;
  }
  __syncthreads();
  if (lane == 63) ws[w] = inc;
  __syncthreads();
  uint32_t before = 0u, tot = 0u;
#pragma unroll
  for (int i = 0; i < kRowThreads / 64; ++i) {
    const uint32_t x = ws[i];
    if (i < w) before += x;
    tot += x;
  }
  v = before + inc - v;
  return tot;
}

// a2: the rows' first hits, and the per-sector regions for start hits /
// tracklets (<= n_g/n_min_chain + 1: each heads its own cleaned chain of >=
// n_min_chain hits, and the chains are disjoint) and tracks
// (<= n_g/n_min_track + 1: each track owns at least n_min_track hits no other
// track owns).  One block per event, its 5724 rows in one pass: as a layout
// kernel and four scans these were the longest part of a small event's grid.
// kTotals: only what the event adds to each of the three tables (S.ev_tot),
// which the other events' blocks start from; not launched for a single event.
template <bool kTotals>
__global__ void __launch_bounds__(kRowThreads) k_rows(Slot S, RowTable X, int n_min_chain,
                                                      int n_min_track) {
  __shared__ uint32_t off[kEventRows + 1];
  const int e = blockIdx.x;
  const int r0 = (int)threadIdx.x * kRowsOfThread;
  uint32_t cnt[kRowsOfThread];
  uint32_t at = 0;
#pragma unroll
  for (int k = 0; k < kRowsOfThread; ++k) {
    cnt[k] = r0 + k < kEventRows ? S.row_cnt[(size_t)e * kEventRows + r0 + k] : 0u;
    if (!kTotals && cnt[k] > (uint32_t)kMaxRowHits) atomicAdd(&S.err[1], 1u);
    at += cnt[k];
  }
  const uint32_t tot = row_block_scan(at);
#pragma unroll
  for (int k = 0; k < kRowsOfThread; ++k) {
    if (r0 + k < kEventRows) off[r0 + k] = at;
    at += cnt[k];
  }
  if (threadIdx.x == 0) off[kEventRows] = tot;
  __syncthreads();
  // the sectors' regions: lane g of every wave the same
  const int lane = threadIdx.x & 63;
  uint2 reg = make_uint2(0u, 0u);
  if (lane < kSectorsPerEvent) {
    const uint32_t ng = off[(lane + 1) * kRows] - off[lane * kRows];
    reg = make_uint2(ng / (uint32_t)n_min_chain + 1u, ng / (uint32_t)n_min_track + 1u);
  }
  uint2 reg_end = reg;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t x = __shfl_up(reg_end.x, d, 64), y = __shfl_up(reg_end.y, d, 64);
    if (lane >= d) {
      reg_end.x += x;
      reg_end.y += y;
    }
  }
  if (kTotals) {
    if (threadIdx.x == 63) {
      uint32_t* t = S.ev_tot + (size_t)e * 4;
      t[0] = tot;
      t[1] = reg_end.x;
      t[2] = reg_end.y;
    }
    return;
  }
  // where this event's tables start: the sums over the events before it
  uint32_t hit0 = 0u, tl0 = 0u, tk0 = 0u;
  if (gridDim.x > 1) {
    uint32_t v0 = 0u, v1 = 0u, v2 = 0u;
    for (int i = threadIdx.x; i < e; i += kRowThreads) {
      const uint32_t* t = S.ev_tot + (size_t)i * 4;
      v0 += t[0];
      v1 += t[1];
      v2 += t[2];
    }
    hit0 = row_block_scan(v0);
    tl0 = row_block_scan(v1);
    tk0 = row_block_scan(v2);
  }
  for (int r = threadIdx.x; r < kEventRows; r += kRowThreads)
    S.row_off[(size_t)e * kEventRows + r] = hit0 + off[r];
  if (threadIdx.x < kSectorsPerEvent) {
    const int g = e * kSectorsPerEvent + lane;
    S.tl_base[g] = tl0 + reg_end.x - reg.x;
    S.tk_base[g] = tk0 + reg_end.y - reg.y;
    if (e == (int)gridDim.x - 1 && lane == kSectorsPerEvent - 1) {
      S.row_off[(size_t)S.n_sectors * kRows] = hit0 + tot;
      S.tl_base[g + 1] = tl0 + reg_end.x;
      S.tk_base[g + 1] = tk0 + reg_end.y;
    }
  }
  // the first event's counts are read (above): the radii go there
  if (e == 0 && threadIdx.x < kRows) const_cast<float*>(S.row_x)[threadIdx.x] = X.x[threadIdx.x];
}
template __global__ void k_rows<true>(Slot, RowTable, int, int);
template __global__ void k_rows<false>(Slot, RowTable, int, int);

// a2: clusters to their row (arrival order within the row), as hit
// records; the row sort then orders each row in place.  The clusters come in
// no order, so a row's line is written 16 bytes at a time: blocks (dealt
// round-robin to the 8 XCDs) take chunks of kCountChunk clusters such that
// each XCD walks a contiguous stretch, and the lines of the one or two events
// of a batch it is in (0.7 MB each) are put together in its own L2.
// Clusters kCountBatch per thread at a time: the batch's fields, then its row
// offsets, are loaded together.
__global__ void __launch_bounds__(kCountThreads) k_scatter(Slot S) {
  const uint32_t xcd = blockIdx.x % 8u, per = gridDim.x / 8u;
  const int64_t i0 = ((int64_t)xcd * per + blockIdx.x / 8u) * kCountChunk;
  const int64_t i1 = min(S.n, i0 + (int64_t)kCountChunk);
  if (i0 >= i1) return;
  int e = 0;                       // event of the chunk's first cluster
  for (int hi = S.n_events - 1; e < hi;) {
    const int mid = (e + hi + 1) >> 1;
    if (S.ev_off[mid] <= i0) e = mid; else hi = mid - 1;
  }
  for (int64_t a = i0; a < i1; ++e) {
    const int64_t b = min(i1, S.ev_off[e + 1]);
    const uint32_t* row_off = S.row_off + (size_t)e * kEventRows;
    for (int64_t ib = a + threadIdx.x; ib < b; ib += kCountBatch * kCountThreads) {
      uint32_t rk[kCountBatch];
      int sr[kCountBatch];
      float y[kCountBatch], z[kCountBatch];
#pragma unroll
      for (int u = 0; u < kCountBatch; ++u) {
        const int64_t i = ib + u * kCountThreads;
        rk[u] = kNoHit;
        sr[u] = 0;
        y[u] = 0.0f;
        z[u] = 0.0f;
        if (i < b) {
          rk[u] = S.rank[i];
          sr[u] = S.sector[i] * kRows + S.row[i];
          y[u] = S.y[i];
          z[u] = S.z[i];
        }
      }
      uint32_t base[kCountBatch];
#pragma unroll
      for (int u = 0; u < kCountBatch; ++u) base[u] = rk[u] != kNoHit ? row_off[sr[u]] : 0u;
#pragma unroll
      for (int u = 0; u < kCountBatch; ++u) {
        if (rk[u] == kNoHit) continue;
        Hit h;                               // one 16-byte store per cluster
        h.y = y[u];
        h.z = z[u];
        h.id = (uint32_t)(ib + u * kCountThreads);
        h.upc = -1;
        S.hit[base[u] + rk[u]] = h;
      }
    }
    a = b;
  }
}

// a2: order a row's hits by (bin, cluster index), write them as Hit records
// with their (sector, row) beside them, and fill the row's bin offsets.
// T threads, PER hits each, held in registers (the row is sorted in place): a
// counting sort by bin in LDS gives each hit its bin's first place, and its
// place inside the bin is the number of smaller indices there, read from the
// bin's indices in LDS (bins hold a hit or two).  Threads of one wave (T = 64)
// need no barrier: their LDS accesses are executed in order.
template <int T, int PER>
struct SortLds {
  uint32_t hist[kBinsPerHit * T * PER + 1];
  uint32_t id[T * PER];
  uint32_t wsum[T / 64];
};
template <int T>
__device__ __forceinline__ void sort_sync() {
  if (T > 64) {
    __syncthreads();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}
template <int T, int PER>
__device__ __forceinline__ void sort_row(const Slot& S, const DevConst& K, int sr, uint32_t off,
                                         uint32_t n, SortLds<T, PER>& L) {
  const uint32_t tid = threadIdx.x & (T - 1);
  const RowBins b = make_bins(K, S, sr, off, n);
  if (tid == 0) S.bins[sr] = b;
  const int nb = b.ny * b.nz;
  Hit h[PER];
  uint32_t bin[PER], rank[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const uint32_t j = tid + k * T;
    if (j < n) h[k] = S.hit[off + j];
  }
  for (int i = tid; i <= nb; i += T) L.hist[i] = 0u;
  sort_sync<T>();
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (tid + k * T < n) {
      bin[k] = (uint32_t)(bin_z(b, h[k].z) * b.ny + bin_y(b, h[k].y));
      rank[k] = atomicAdd(&L.hist[bin[k]], 1u);
    }
  sort_sync<T>();
  // exclusive scan of hist[0, nb) (each thread a contiguous stretch)
  {
    const int per = (nb + T - 1) / T;
    const int a = min(nb, (int)tid * per), z = min(nb, a + per);
    uint32_t sum = 0;
    for (int k = a; k < z; ++k) sum += L.hist[k];
    const int lane = tid & 63, w = tid >> 6;
    uint32_t inc = sum;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t t = __shfl_up(inc, d, 64);
      if (lane >= d) inc += t;
    }
    uint32_t run = inc - sum;
    if (T > 64) {
      if (lane == 63) L.wsum[w] = inc;
      __syncthreads();
      for (int i = 0; i < w; ++i) run += L.wsum[i];
    }
    for (int k = a; k < z; ++k) {
      const uint32_t c = L.hist[k];
      L.hist[k] = run;
      run += c;
    }
    if (tid == 0) L.hist[nb] = n;
  }
  sort_sync<T>();
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (tid + k * T < n) L.id[L.hist[bin[k]] + rank[k]] = h[k].id;
  sort_sync<T>();
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const uint32_t j = tid + k * T;
    if (j >= n) continue;
    const uint32_t p0 = L.hist[bin[k]], p1 = L.hist[bin[k] + 1];
    uint32_t pos = p0;
    if (p1 - p0 > 1u)
      for (uint32_t i = p0; i < p1; ++i) pos += L.id[i] < h[k].id ? 1u : 0u;
    h[k].upc = -1;
    S.hit[off + pos] = h[k];
    S.hit_sr[off + j] = (uint32_t)sr;
  }
  uint32_t* bo = bin_offsets(S, b);
  for (int i = tid; i <= nb; i += T) bo[i] = off + L.hist[i];
  sort_sync<T>();
}

// Four rows a block: rows of at most kTinyRow hits (most rows of small
// events) by a wave each, then the larger ones, up to kMidRow hits, by the
// whole block one after the other; still larger ones are listed.
constexpr int kTinyRow = 256;
constexpr int kMidRow = 1024;
__global__ void __launch_bounds__(256) k_row_sort(Slot S, DevConst K) {
  union Lds {
    SortLds<64, kTinyRow / 64> tiny[4];
    SortLds<256, kMidRow / 256> mid;
  };
  __shared__ Lds L;
  const int SR = S.n_sectors * kRows;
  const int sr0 = (int)blockIdx.x * 4;
  const int w = threadIdx.x >> 6;
  uint32_t off[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) off[k] = S.row_off[min(sr0 + k, SR)];
  uint32_t mine = off[0], end = off[1];
#pragma unroll
  for (int k = 1; k < 4; ++k)
    if (w == k) {
      mine = off[k];
      end = off[k + 1];
    }
  if (sr0 + w < SR && end - mine <= (uint32_t)kTinyRow)
    sort_row<64, kTinyRow / 64>(S, K, sr0 + w, mine, end - mine, L.tiny[w]);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t n = off[k + 1] - off[k];     // 0 past the last row
    if (n <= (uint32_t)kTinyRow) continue;
    if (n > (uint32_t)kMidRow) {                // left to the large instance
      if (threadIdx.x == 0) S.big_rows[atomicAdd(&S.range_cnt[2], 1u)] = sr0 + k;
      continue;
    }
    __syncthreads();                            // the rows before are done with L
    sort_row<256, kMidRow / 256>(S, K, sr0 + k, off[k], n, L.mid);
  }
}

// the listed rows (1025..4096 hits, and the over-full ones)
__global__ void __launch_bounds__(256) k_row_sort_large(Slot S, DevConst K) {
  __shared__ SortLds<256, kMaxRowHits / 256> L;
  const uint32_t nbig = S.range_cnt[2];
  for (uint32_t i = blockIdx.x; i < nbig; i += gridDim.x) {
    const int sr = (int)S.big_rows[i];
    const uint32_t off = S.row_off[sr];
    const uint32_t n = S.row_off[sr + 1] - off;
    if (n <= (uint32_t)kMaxRowHits) {
      sort_row<256, kMaxRowHits / 256>(S, K, sr, off, n, L);
      continue;
    }
    // flagged in k_rows (the slot's result is refused); keep the row harmless
    // for the kernels that still run: no coordinates, empty bins
    const RowBins b = make_bins(K, S, sr, off, n);
    if (threadIdx.x == 0) S.bins[sr] = b;
    const int nb = b.ny * b.nz;
    for (uint32_t j = threadIdx.x; j < n; j += blockDim.x) {
      Hit h;
      h.y = __builtin_nanf("");
      h.z = __builtin_nanf("");
      h.id = S.hit[off + j].id;
      h.upc = -1;
      S.hit[off + j] = h;
      S.hit_sr[off + j] = (uint32_t)sr;
    }
    uint32_t* bo = bin_offsets(S, b);
    for (int k = threadIdx.x; k <= nb; k += blockDim.x) bo[k] = off;
  }
}

}  // namespace tpc
