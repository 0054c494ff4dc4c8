// Device-side building blocks of the TPC sector tracker for gfx950:
// slot layout, pad-row bin geometry and the Kalman-filter transport/update.
//
// Method (paper, Abstract and Section 2): track finding by a cellular
// automaton over pad-row hits followed by Kalman-filter track following.
// The paper gives no formulas; the arithmetic below is the project's written
// definition of those steps (helix in the local sector frame, state
// (y, z, sin phi, tan lambda, q/pT) at the pad-row x).  Float decisions are
// bit-reproducible against a CPU evaluation in the same operation order:
// every kernel is built with -ffp-contract=off and correctly rounded
// division and square root, and each expression below is evaluated left to
// right exactly as written.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bin_table.h"
#include "tpcca.h"

namespace tpc {

constexpr int kRows = 159;
constexpr int kSectorsPerEvent = 36;
constexpr int kMaxRowHits = 4096;         // LDS sort capacity of one pad row
constexpr uint32_t kNoHit = 0xFFFFFFFFu;
constexpr int32_t kStartHit = -2;         // down link of a start hit
constexpr int kRowBlocks = (kRows + 7) / 8;   // a tracklet's hit list in blocks of 8 rows
constexpr uint16_t kNoEntry = 0xFFFFu;        // hit-list entry of a row without hit

// ---------------------------------------------------------------------------
// constants handed to every kernel by value
// ---------------------------------------------------------------------------
struct DevConst {
  float tanh_half;
  float z_max;
  float sy0, sy1, sz0, sz1;
  // error model sigma(z) = sigma_0 + sigma_1 |z| / z_max with sigma_1 / z_max
  // formed once, in float and in double
  float sy1z, sz1z;
  double sy1zd, sz1zd;
  float b;          // curvature per unit q/pT, float
  double bd;        // same, double (refit)
  float nf_w, nf_mmax, chi2max, kwin, wmax, smax, cs0, ct0, cq0, medge, mz;
  int n_gap, n_min_tracklet, n_min_track, n_min_chain;
  float bin_target;  // clusters per grid bin aimed at
  float bin_min_edge;
  float kk, m2;             // scattering law k^2/X0 and mass^2 (0: no scattering), float
  double kkd, m2d;          // the same in double (refit, merger)
};

// Pad-row radii, handed to the kernels that build the grid; they leave them in
// device memory for the others (Slot::row_x).  A lane's read of a kernel
// argument by index goes to the argument buffer, in host memory: over a
// microsecond, more than a filter step, and longer with more waves reading.
struct RowTable {
  float x[kRows + 1];
};

// per (sector, row) grid description
struct RowBins {
  float y0, z0, iby, ibz;   // lower edges and inverse bin sizes
  int32_t ny, nz;           // bins in y and z
  uint32_t base;            // first pair of entries of this row in bin_off (bin_table_pair)
  int32_t first;            // the row's first sorted hit
};

// A sorted hit: coordinates, global cluster index, cleaned up-link (sorted
// index of the next hit of its chain, -1 none).  16 bytes: one load.
struct alignas(16) Hit {
  float y, z;
  uint32_t id;
  int32_t upc;
};

// One slot: a batch of events whose clusters are concatenated; sector g of
// the slot is sector g % 36 of event g / 36.
struct Slot {
  // input (caller device memory, or the slot's own copy)
  const uint8_t* sector;
  const uint8_t* row;
  const float* y;
  const float* z;
  int64_t* ev_off;          // [E+1] cluster offsets of the events
  int32_t n_events;
  int32_t n_sectors;        // 36 * n_events
  int64_t n;                // clusters
  // grid
  uint32_t* row_cnt;        // [SR] clusters of each row, until the rows are laid out
  const float* row_x;       // [kRows] pad-row radii (in the memory of row_cnt, written after it
                            // was last read)
  uint32_t* row_off;        // [SR+1] first sorted hit of each (sector, row)
  RowBins* bins;            // [SR]
  uint32_t* ev_tot;         // [4 E] per event: hits, tracklet and track region entries, spare
  uint32_t* bin_off;        // [2 (n + 2 SR)] per row: its bins' first hits, then the end
  uint32_t* rank;           // [n]
  Hit* hit;                 // [n] sorted by (sector, row, bin, id)
  uint32_t* hit_sr;         // [n] (sector, row) of each sorted hit (slot-wide index)
  // links (sorted-hit indices, -1 none); the cleaned up-link lives in hit[].upc
  int32_t* up;
  int32_t* dn;
  int32_t* dnc;             // cleaned down link; kStartHit for a start hit (which has none)
  // per-sector regions (used by per-sector launches; contiguous for a range)
  uint32_t* tl_base;        // [S+1] tracklet region of each sector
  uint32_t* tk_base;        // [S+1] track region of each sector
  uint32_t* row_nstart;     // [SR+1] start hits per row, then their offsets
  uint32_t* range_cnt;      // [16]: tracklets, tracks of the launched range; rows > 1024 hits
  uint32_t* big_rows;       // [n / 1024 + 1] (sector, row) of the rows over 1024 hits
  int32_t* start_hit;       // [tl capacity] sorted index of the start hit
  int32_t* start_sr;        // [tl capacity] (sector, row) of the start hit
  // tracklets
  uint16_t* tl_hits;        // [tl capacity / 64][kRowBlocks][64][8] per row: the hit's offset in its row, kNoEntry none
  int32_t* tl_info;         // [tl capacity][4]: n, row_in, row_out, valid
  uint32_t* tl_weight;      // [tl capacity]
  float* tl_state;          // [tl capacity][5] inner state (y, z, s, T, Q)
  uint32_t* tl_sel;         // [tl capacity+1] hits owned if selected, else 0 (and chunk counts)
  uint32_t* weight;         // [n] per sorted hit, 0 = unowned
  // tracks (per-sector regions)
  int32_t* tk_tracklet;     // [tk capacity]
  int32_t* tk_own;          // [tk capacity][kRows] owned hits (sorted index), ascending row
  uint8_t* tk_own_row;      // [tk capacity][kRows] their rows
  int32_t* tk_nown;         // [tk capacity]
  int32_t* tk_info;         // [tk capacity][4]: spare, n, row_in, row_out (fitted tracks only)
  double* tk_par;           // [tk capacity][5]
  double* tk_cov;           // [tk capacity][15]
  double* tk_chi2;          // [tk capacity]
  // canonical order
  int32_t* tmap;            // [n] per global cluster: temp track whose innermost hit it is
  uint32_t* scan_a;         // [n+1] scratch: the output order's counts per stretch of clusters
  uint32_t* scan_b;         // [SR / scan tile + 1] block partials of a scan over rows
  uint32_t* out_count;      // [2]: tracks, hits of the slot
  uint32_t* out_ntk;        // [tk capacity+1] first hit of each track, in canonical order
  int32_t* out_order;       // [tk capacity] temporary track of each canonical position
  tpc_track* out_tracks;    // [tk capacity]
  int32_t* out_hits;        // [n]
  uint32_t* ev_track_off;   // [E+1]
  uint32_t* ev_hit_off;     // [E+1]
  uint32_t* err;            // [4]: invalid clusters, dense rows, overflow, spare
  unsigned long long* stats; // [8] work counters
  // capacities
  int64_t cap_n;
  int64_t cap_tl;
  int64_t cap_tk;
  int32_t cap_e;
};

// Row-indexed hit list of tracklet T: per row the hit's offset from its
// row's first sorted hit (rows hold at most 4096 hits), kNoEntry if none.
// Stored in tiles of 64 tracklets; inside a tile, blocks of 8 rows, and in
// a block the 8 entries of each tracklet together (16 bytes): a tracklet
// reads or writes 8 rows with one access, and the lanes of a wave
// (consecutive tracklets) touch one contiguous kilobyte per block.
struct TlList {
  uint16_t* p;              // this tracklet's entries of row block 0
  __device__ __forceinline__ uint4 load_block(int b) const {
    return *reinterpret_cast<const uint4*>(p + (size_t)b * 512);
  }
  __device__ __forceinline__ void store_block(int b, const uint4& v) const {
    *reinterpret_cast<uint4*>(p + (size_t)b * 512) = v;
  }
  __device__ __forceinline__ uint16_t at(int r) const { return p[(size_t)(r >> 3) * 512 + (r & 7)]; }
};
__device__ __forceinline__ TlList tl_list(const Slot& S, uint32_t T) {
  return TlList{S.tl_hits + ((size_t)(T >> 6) * kRowBlocks * 64 + (T & 63u)) * 8};
}
// entry k (0..7) of a block held in registers as two 64-bit halves (a
// shift and a two-way select: no indexed access, which the compiler would
// place in scratch memory)
__device__ __forceinline__ uint32_t block_get(const uint4& v, int k) {
  const uint64_t h = k < 4 ? ((uint64_t)v.y << 32 | v.x) : ((uint64_t)v.w << 32 | v.z);
  return (uint32_t)(h >> ((k & 3) * 16)) & 0xFFFFu;
}
__device__ __forceinline__ void block_set(uint4& v, int k, uint32_t e) {
  const bool lo = k < 4;
  uint64_t h = lo ? ((uint64_t)v.y << 32 | v.x) : ((uint64_t)v.w << 32 | v.z);
  const int sh = (k & 3) * 16;
  h = (h & ~(0xFFFFull << sh)) | ((uint64_t)(e & 0xFFFFu) << sh);
  const uint32_t a = (uint32_t)h, b = (uint32_t)(h >> 32);
  v.x = lo ? a : v.x;
  v.y = lo ? b : v.y;
  v.z = lo ? v.z : a;
  v.w = lo ? v.w : b;
}
// the block moved up by one entry, e (16 bits) the new last one: eight rows
// pushed one after the other stand at their places
__device__ __forceinline__ void block_push(uint4& v, uint32_t e) {
  v.x = __builtin_amdgcn_alignbit(v.y, v.x, 16);
  v.y = __builtin_amdgcn_alignbit(v.z, v.y, 16);
  v.z = __builtin_amdgcn_alignbit(v.w, v.z, 16);
  v.w = __builtin_amdgcn_alignbit(e, v.w, 16);
}
__device__ __forceinline__ uint4 block_empty() {
  return make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
}
// sorted-hit index of an entry of the row whose first hit is `first`
__device__ __forceinline__ int32_t entry_hit(uint32_t e, uint32_t first) {
  return e == kNoEntry ? -1 : (int32_t)(first + e);
}

// the pad-row radii in LDS, for the kernels that walk the rows
__device__ __forceinline__ void load_radii(const Slot& S, RowTable& R) {
  for (int r = threadIdx.x; r < kRows; r += blockDim.x) R.x[r] = S.row_x[r];
  __syncthreads();
}

// ---------------------------------------------------------------------------
// pad-row bins: monotone in y and z, identical in every kernel
// ---------------------------------------------------------------------------
// the row's bin offset table (sorted-hit positions)
__device__ __forceinline__ uint32_t* bin_offsets(const Slot& S, const RowBins& b) {
  return S.bin_off + 2 * (size_t)b.base;
}
// (a NaN coordinate maps to bin 0: every index stays inside the row)
__device__ __forceinline__ int bin_y(const RowBins& b, float y) {
  const float f = (y - b.y0) * b.iby;
  return f >= 0.0f ? (int)fminf(f, (float)(b.ny - 1)) : 0;
}
__device__ __forceinline__ int bin_z(const RowBins& b, float z) {
  const float f = (z - b.z0) * b.ibz;
  return f >= 0.0f ? (int)fminf(f, (float)(b.nz - 1)) : 0;
}

// Hits of one row that can lie inside [yc - wy, yc + wy] x [zc - wz, zc + wz]:
// every bin the window touches, plus a small margin so rounding cannot hide
// a hit; the caller applies the exact window test.  `bo` is the row's bin
// offset table (sorted-hit positions).  The bin ranges of up to four z rows
// are read together, then their hits four at a time across the ranges, so
// a query waits for a few memory round trips rather than one per hit or
// per range.  fn(p, hit) runs in ascending p within a range, ranges in
// ascending z.  WB: hit records read per round trip (a tuning knob).
template <int WB, class Fn>
__device__ __forceinline__ void for_window_hits(const RowBins& b, const uint32_t* bo, const Hit* hit,
                                                float yc, float zc, float wy, float wz, Fn&& fn) {
  const float eps = 1e-3f;
  const int iy0 = bin_y(b, yc - wy - eps), iy1 = bin_y(b, yc + wy + eps);
  const int iz0 = bin_z(b, zc - wz - eps), iz1 = bin_z(b, zc + wz + eps);
  for (int izb = iz0; izb <= iz1; izb += 4) {
    uint32_t lo[4], hi[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      lo[k] = 0u;
      hi[k] = 0u;
      if (izb + k <= iz1) {
        const int first = (izb + k) * b.ny;
        lo[k] = bo[first + iy0];
        hi[k] = bo[first + iy1 + 1];
      }
    }
    // the four ranges as one sequence (same order), read WB hits at a
    // time whichever ranges they fall in
    const uint32_t c0 = hi[0] - lo[0];
    const uint32_t c1 = c0 + (hi[1] - lo[1]);
    const uint32_t c2 = c1 + (hi[2] - lo[2]);
    const uint32_t c3 = c2 + (hi[3] - lo[3]);
    for (uint32_t f = 0; f < c3; f += WB) {
      uint32_t p[WB];
      Hit x[WB];
#pragma unroll
      for (int u = 0; u < WB; ++u) {
        const uint32_t q = f + u;
        p[u] = q < c0 ? lo[0] + q : q < c1 ? lo[1] + (q - c0) : q < c2 ? lo[2] + (q - c1) : lo[3] + (q - c2);
        if (q < c3) x[u] = hit[p[u]];
      }
#pragma unroll
      for (int u = 0; u < WB; ++u)
        if (f + u < c3) fn(p[u], x[u]);
    }
  }
}

__device__ __forceinline__ float sigma_y(const DevConst& k, float z) {
  return k.sy0 + k.sy1z * fabsf(z);
}
__device__ __forceinline__ float sigma_z(const DevConst& k, float z) {
  return k.sz0 + k.sz1z * fabsf(z);
}

// ---------------------------------------------------------------------------
// Kalman filter on the helix state.  Template over float (tracklet phases,
// which take decisions) and double (the output refit).
// Covariance packed as the lower triangle of (y, z, s, T, Q):
//   0:yy 1:zy 2:zz 3:sy 4:sz 5:ss 6:Ty 7:Tz 8:Ts 9:TT 10:Qy 11:Qz 12:Qs 13:QT 14:QQ
// ---------------------------------------------------------------------------
// sum over the wave, then one atomic per wave (all 64 lanes must call)
__device__ __forceinline__ void wave_add_u64(unsigned long long* dst, unsigned long long v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
  if ((threadIdx.x & 63) == 0 && v) atomicAdd(dst, v);
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t t = __shfl_up(x, d, 64);
    if (lane >= d) x += t;
  }
  return x;
}

// exclusive scan of one 256-thread block's values; returns the block total
__device__ __forceinline__ uint32_t block_scan256(uint32_t v, uint32_t* excl) {
  __shared__ uint32_t ws[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t inc = wave_incl_scan(v);
  if (lane == 63) ws[w] = inc;
  __syncthreads();
  uint32_t before = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (i < w) before += ws[i];
    tot += ws[i];
  }
  __syncthreads();
  *excl = before + inc - v;
  return tot;
}

// How a wave's lanes are dealt to `total` items (tracklets, tracks): a lane
// an item where there are many, a group of lanes an item where there are few,
// so that these spread over the idle SIMDs: a wave's step costs what its
// costliest item needs (a search, a second update, the slowest of 64 reads).
// A group's lanes all do the item's work (same addresses, one line read) and
// the first one writes: waves of one or four active lanes issue at half the
// rate of full ones, measured at four to a compute unit.
// per: items of a wave, the fewest (a power of two) that give no more than
// `most` waves.
struct LaneGroup {
  uint32_t per, index;      // items per wave; this lane's item in the wave
  uint32_t size, lane;      // lanes of a group, this lane's place in its own
  unsigned long long mask;  // the group's lanes in the wave
  bool first;               // first lane of its group
};
__device__ __forceinline__ LaneGroup lane_group(uint32_t total, uint32_t most) {
  uint32_t sh = 6;          // log2 of the lanes of an item
  while (sh > 0u && (total + (64u >> sh) - 1u) / (64u >> sh) > most) --sh;
  const uint32_t lane = threadIdx.x & 63u;
  LaneGroup g;
  g.per = 64u >> sh;
  g.index = lane >> sh;
  g.size = 1u << sh;
  g.lane = lane & (g.size - 1u);
  g.mask = (g.size == 64u ? ~0ull : (1ull << g.size) - 1ull) << (lane - g.lane);
  g.first = g.lane == 0u;
  return g;
}

// The same without anything shared by a group's lanes: any number of items to
// a wave, lane l on item l modulo that, the first of each to write.  (Powers of
// two leave up to half of `most` waves unused: 32 events of 60 tracks 1.219 ms
// with them, 1.200 so, on 1024 waves.)
__device__ __forceinline__ LaneGroup lane_deal(uint32_t total, uint32_t most) {
  const uint32_t lane = threadIdx.x & 63u;
  LaneGroup g;
  g.per = min(64u, max(1u, (total + most - 1u) / most));
  g.index = lane % g.per;
  g.size = 1u;
  g.lane = 0u;
  g.mask = 1ull << lane;
  g.first = lane < g.per;
  return g;
}

template <class F>
struct Helix {
  F y, z, s, t, q;
  F c[15];
};

template <class F> __device__ __forceinline__ F fabs_(F v);
template <> __device__ __forceinline__ float fabs_(float v) { return fabsf(v); }
template <> __device__ __forceinline__ double fabs_(double v) { return fabs(v); }
template <class F> __device__ __forceinline__ F sqrt_(F v);
template <> __device__ __forceinline__ float sqrt_(float v) { return sqrtf(v); }
template <> __device__ __forceinline__ double sqrt_(double v) { return sqrt(v); }
// Square root and reciprocal, correctly rounded, for operands that
// the caller knows to be well inside the exponent range: the bits of sqrtf /
// sqrt and of the division without the scaling and special-case steps that
// the compiler adds around them (a filter step has four of these, and its
// lanes are bound by the number of instructions).  Zero, infinity and NaN
// give NaN.  Goldschmidt / Newton steps on the hardware's estimate, the last
// ones on the residual (Markstein 1990).
//  float   5 and 3 instructions instead of 16 and 11; compared with the
//          compiler's operations on every float in [2^-100, 2^100]: equal.
//  double  the residual step that makes the result exact is kept, as the
//          compiler has it: 10 instead of 18, and 7 instead of 11.
__device__ __forceinline__ float sqrt_mid(float x) {
  const float r = __builtin_amdgcn_rsqf(x);
  const float g = x * r, h = 0.5f * r;
  return fmaf(fmaf(-g, g, x), h, g);
}
__device__ __forceinline__ double sqrt_mid(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  double g = x * r, h = 0.5 * r;
  const double e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  g = fma(fma(-g, g, x), h, g);
  return fma(fma(-g, g, x), h, g);
}
__device__ __forceinline__ float rcp_mid(float x) {
  const float y = __builtin_amdgcn_rcpf(x);
  return fmaf(fmaf(-x, y, 1.0f), y, y);
}
__device__ __forceinline__ double rcp_mid(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

// True if |x| lies in [2^-100, 2^100], where the short forms hold (false for NaN).
__device__ __forceinline__ bool mid_range(float x) {
  const float a = fabsf(x);
  return a >= 0x1p-100f && a <= 0x1p100f;
}
// Reciprocal of a residual covariance's determinant.  In float it is tested:
// cluster errors given as tiny numbers reach the ends of the range.  In
// double the squares of four floats stay far from them.
__device__ __forceinline__ float rcp_det(float x) {
  float y = rcp_mid(x);
  if (!mid_range(x)) {
    asm volatile("");        // a branch, not both results and a choice
    y = 1.0f / x;
  }
  return y;
}
__device__ __forceinline__ double rcp_det(double x) { return rcp_mid(x); }

// a*b + c rounded once.  Every sum of products of the filter is a chain of
// these in a fixed order (the CPU checker uses the same chains), so results
// stay bit-identical with contraction switched off for everything else.
template <class F> __device__ __forceinline__ F fma_(F a, F b, F c);
template <> __device__ __forceinline__ float fma_(float a, float b, float c) { return fmaf(a, b, c); }
template <> __device__ __forceinline__ double fma_(double a, double b, double c) { return fma(a, b, c); }

// Move the state by dx along the circle of curvature b*q.  sin(phi) grows
// linearly with x; y advances by dx times the tangent of the mid-angle
// (N/D below); z advances by T times the arc, the arc being the chord
// times asin(u)/u = 1 + u^2/6 + 3u^4/40 (u = half chord * curvature).
// Returns false if |sin phi| would pass smax, leaving the state untouched, or
// (kAlways, for callers that then discard it) of no use: without a branch.
// kCov = false moves the parameters only (the same arithmetic for them),
// for callers that discard the covariance.
// The roots and the reciprocal are the short ones: smax is a float below 1,
// so 1 - s1^2 >= 2^-24 and c1 >= 2^-12, D lies in [2^-12, 2] and 1 + tmid^2
// in [1, 2^27].  (s0 alone may be past smax, as an update without a gate
// leaves it: |s0| > 1 gives NaN here as it does in a general root; |s0| = 1
// makes iD, and with it every entry that iD enters, NaN either way.)
template <class F, bool kCov = true, bool kAlways = false>
__device__ __forceinline__ bool transport(Helix<F>& h, F dx, F b, F smax, F kk = F(0),
                                          F m2 = F(0)) {
  const F one = F(1), half = F(0.5), two = F(2);
  const F bq = b * h.q;
  const F s1 = fma_(bq, dx, h.s);
  const bool ok = fabs_(s1) <= smax;
  if (!kAlways && !ok) return false;
  const F s0 = h.s;
  const F c0 = sqrt_mid(fma_(-s0, s0, one));
  const F c1 = sqrt_mid(fma_(-s1, s1, one));
  const F N = s0 + s1;
  const F D = c0 + c1;
  // one division: the reciprocals of D, c0 and c1 are products with
  // 1/(c0 c1 D)
  const F c01 = c0 * c1;
  const F inv = rcp_mid(c01 * D);
  const F iD = c01 * inv;
  const F ic0 = (c1 * D) * inv;
  const F ic1 = (c0 * D) * inv;
  const F tmid = N * iD;
  // chord and arc with the sign of dx
  const F chord = dx * sqrt_mid(fma_(tmid, tmid, one));
  const F u = half * bq * chord;
  const F u2 = u * u;
  const F arc = chord * fma_(u2, fma_(u2, F(3) / F(40), one / F(6)), one);

  // Jacobian; dz/dQ to leading order, 2 T b N dx^2 / D^3 (the mid-angle
  // cosine taken as D/2)
  const F iD2 = iD * iD;
  const F r0 = s0 * ic0;
  const F r1 = s1 * ic1;
  const F dy_ds = dx * fma_(N, r0 + r1, two * D) * iD2;
  const F dy_dq = b * dx * dx * fma_(N, r1, D) * iD2;
  const F dz_ds = h.t * dx * N * (ic0 * ic1 * iD);
  const F dz_dt = arc;
  const F dz_dq = two * h.t * b * N * dx * dx * (iD2 * iD);
  const F ds_dq = b * dx;

  h.y = fma_(dx, tmid, h.y);
  h.z = fma_(h.t, arc, h.z);
  h.s = s1;
  if (!kCov) return ok;

  F* c = h.c;
  const F yy = c[0], zy = c[1], zz = c[2], sy = c[3], sz = c[4], ss = c[5];
  const F ty = c[6], tz = c[7], ts = c[8], tt = c[9];
  const F qy = c[10], qz = c[11], qs = c[12], qt = c[13], qq = c[14];

  // rows y, z, s of J*C (the columns that the product below reads)
  const F jy_y = fma_(dy_dq, qy, fma_(dy_ds, sy, yy));
  const F jy_s = fma_(dy_dq, qs, fma_(dy_ds, ss, sy));
  const F jy_q = fma_(dy_dq, qq, fma_(dy_ds, qs, qy));
  const F jz_y = fma_(dz_dq, qy, fma_(dz_dt, ty, fma_(dz_ds, sy, zy)));
  const F jz_z = fma_(dz_dq, qz, fma_(dz_dt, tz, fma_(dz_ds, sz, zz)));
  const F jz_s = fma_(dz_dq, qs, fma_(dz_dt, ts, fma_(dz_ds, ss, sz)));
  const F jz_t = fma_(dz_dq, qt, fma_(dz_dt, tt, fma_(dz_ds, ts, tz)));
  const F jz_q = fma_(dz_dq, qq, fma_(dz_dt, qt, fma_(dz_ds, qs, qz)));
  const F js_y = fma_(ds_dq, qy, sy);
  const F js_z = fma_(ds_dq, qz, sz);
  const F js_s = fma_(ds_dq, qs, ss);
  const F js_t = fma_(ds_dq, qt, ts);
  const F js_q = fma_(ds_dq, qq, qs);

  // (J*C)*J^T, lower triangle; TT, QT, QQ unchanged
  c[0] = fma_(dy_dq, jy_q, fma_(dy_ds, jy_s, jy_y));
  c[1] = fma_(dy_dq, jz_q, fma_(dy_ds, jz_s, jz_y));
  c[2] = fma_(dz_dq, jz_q, fma_(dz_dt, jz_t, fma_(dz_ds, jz_s, jz_z)));
  c[3] = fma_(dy_dq, js_q, fma_(dy_ds, js_s, js_y));
  c[4] = fma_(dz_dq, js_q, fma_(dz_dt, js_t, fma_(dz_ds, js_s, js_z)));
  c[5] = fma_(ds_dq, js_q, js_s);
  c[6] = fma_(dy_dq, qt, fma_(dy_ds, ts, ty));
  c[7] = fma_(dz_dq, qt, fma_(dz_dt, tt, fma_(dz_ds, ts, tz)));
  c[8] = fma_(ds_dq, qt, ts);
  c[10] = fma_(dy_dq, qq, fma_(dy_ds, qs, qy));
  c[11] = fma_(dz_dq, qq, fma_(dz_dt, qt, fma_(dz_ds, qs, qz)));
  c[12] = fma_(ds_dq, qq, qs);

  // multiple scattering at the end of the step (kk = k^2/X0 > 0):
  // theta0^2 = kk L (a + m^2 a^2), a = Q^2/(1+T^2), L = |arc| sqrt(1+T^2);
  // var(phi) = theta0^2 (1+T^2), var(lambda) = theta0^2, dQ = Q T dlambda,
  // dT = (1+T^2) dlambda
  if (kk > F(0)) {
    const F t2 = fma_(h.t, h.t, one);
    const F L = fabs_(arc) * sqrt_(t2);
    const F a = (h.q * h.q) / t2;
    const F th2 = kk * L * fma_(m2, a * a, a);
    c[5] = fma_(fma_(-s1, s1, one), th2 * t2, c[5]);
    c[9] = fma_(th2, t2 * t2, c[9]);
    c[13] = fma_(th2, h.q * h.t * t2, c[13]);
    c[14] = fma_(th2, h.q * h.q * (h.t * h.t), c[14]);
  }
  return ok;
}

// Inverse of the 2x2 residual covariance S = C_(y,z) + diag(vy, vz).
template <class F>
struct Resid {
  F w00, w01, w11, s00, s11;
};

template <class F>
__device__ __forceinline__ Resid<F> resid_weights(const Helix<F>& h, F vy, F vz) {
  Resid<F> r;
  const F s00 = h.c[0] + vy;
  const F s01 = h.c[1];
  const F s11 = h.c[2] + vz;
  const F det = fma_(s00, s11, -(s01 * s01));
  const F inv = rcp_det(det);
  r.w00 = s11 * inv;
  r.w01 = -s01 * inv;
  r.w11 = s00 * inv;
  r.s00 = s00;
  r.s11 = s11;
  return r;
}

template <class F>
__device__ __forceinline__ F chi2_of(const Resid<F>& w, F ry, F rz) {
  return fma_(ry, fma_(w.w00, ry, w.w01 * rz), rz * fma_(w.w01, ry, w.w11 * rz));
}

// Kalman update with the measurement (my, mz).  gated: refuse (state
// untouched) when chi2 > chi2max, a variance would not stay positive or
// |sin phi| would reach smax (one test of all of them: a branch of its own
// for each costs a lone wave more than what it skips).
template <class F>
__device__ __forceinline__ bool kalman_update(Helix<F>& h, F my, F mz, F vy, F vz, F chi2max,
                                              F smax, bool gated, F* chi2_out) {
  const Resid<F> w = resid_weights(h, vy, vz);
  const F ry = my - h.y;
  const F rz = mz - h.z;
  const F chi2 = chi2_of(w, ry, rz);
  *chi2_out = chi2;
  const F* c = h.c;
  // covariance column of each state entry with y and with z
  const F cy[5] = {c[0], c[1], c[3], c[6], c[10]};
  const F cz[5] = {c[1], c[2], c[4], c[7], c[11]};
  F ky[5], kz[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    ky[i] = fma_(cy[i], w.w00, cz[i] * w.w01);
    kz[i] = fma_(cy[i], w.w01, cz[i] * w.w11);
  }
  Helix<F> o;
  o.y = fma_(ky[0], ry, fma_(kz[0], rz, h.y));
  o.z = fma_(ky[1], ry, fma_(kz[1], rz, h.z));
  o.s = fma_(ky[2], ry, fma_(kz[2], rz, h.s));
  o.t = fma_(ky[3], ry, fma_(kz[3], rz, h.t));
  o.q = fma_(ky[4], ry, fma_(kz[4], rz, h.q));
  int k = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
#pragma unroll
    for (int j = 0; j <= i; ++j, ++k) o.c[k] = fma_(-ky[i], cy[j], fma_(-kz[i], cz[j], c[k]));
  }
  if (gated) {
    const bool ok = (chi2 <= chi2max) & (o.c[0] > F(0)) & (o.c[2] > F(0)) & (o.c[5] > F(0)) &
                    (o.c[9] > F(0)) & (o.c[14] > F(0)) & (fabs_(o.s) < smax);
    if (!ok) return false;
  }
  h = o;
  return true;
}

// Prior covariance: measurement variances in y and z at the hit, wide
// diagonal for the angles and the curvature.
template <class F>
__device__ __forceinline__ void reset_cov(Helix<F>& h, F vy, F vz, F cs0, F ct0, F cq0) {
#pragma unroll
  for (int i = 0; i < 15; ++i) h.c[i] = F(0);
  h.c[0] = vy;
  h.c[2] = vz;
  h.c[5] = cs0;
  h.c[9] = ct0;
  h.c[14] = cq0;
}

// From x to xt in equal steps of at most step_max (refused beyond 1000 cm,
// longer than any path in the chamber, which also bounds the step count).
template <bool kCov = true>
__device__ __forceinline__ bool transport_to_x(Helix<double>& h, double x, double xt, double b,
                                               double smax, double step_max, double kk = 0.0,
                                               double m2 = 0.0) {
  const double d = xt - x;
  if (!(fabs(d) <= 1000.0)) return false;
  const int n = max(1, (int)ceil(fabs(d) / step_max));
  const double dx = d / (double)n;
  for (int i = 0; i < n; ++i)
    if (!transport<double, kCov>(h, dx, b, smax, kk, m2)) return false;
  return true;
}

}  // namespace tpc
