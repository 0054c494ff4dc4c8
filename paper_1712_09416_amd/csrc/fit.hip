// a6 hit ownership and tracklet selection, a7 output refit.
#include "tpc_device.h"
#include "tpc_kernels.h"

namespace tpc {

__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v = min(v, __shfl_xor(v, d, 64));
  return v;
}
__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v = max(v, __shfl_xor(v, d, 64));
  return v;
}

// a6: selection.  A valid tracklet becomes a track if it owns (holds the
// maximal weight of) at least n_min_track of its hits.
// Few tracklets (up to kSelSparse): 32 lanes a tracklet, each with a block of
// 8 rows of its hit list, so a tracklet costs four memory round trips
// (record, list block, rows' first hits, weights); a lane walking its
// tracklet's rows takes 40, which few tracklets do not hide (a pp event 24 us,
// now 5; a peripheral event 27, now 10).  Many: a lane a tracklet, the wave
// walking the rows its 64 consecutive tracklets span together, so that each
// row's lists and weights are read side by side (a central event 64 us
// against 103 with 32 lanes a tracklet, 64 events 0.48 against 1.62 ms).
// The tracks' lists are written 32 lanes a tracklet either way (five in six
// tracklets are not selected: 47 against 62 us and 0.60 against 0.79 ms).
// Blocks take chunks of consecutive tracklets (in sector order), the chunks
// of one XCD (blocks are dispatched round-robin over the 8) contiguous, so a
// sector's hit lists and weights are read through one XCD's L2.
constexpr uint32_t kSelLanes = 32;
constexpr uint32_t kSelThreads = 256;
constexpr uint32_t kSelRound = kSelThreads / kSelLanes;     // tracklets of a block's round
constexpr uint32_t kSelSparse = 65536;
constexpr int kSelRows = 8;                                 // rows a lane reads together
static_assert(kRowBlocks <= (int)kSelLanes, "a lane per block of a hit list");
struct SelChunk {
  uint32_t size, index;      // index past the last chunk: nothing to do
};
__device__ __forceinline__ SelChunk sel_chunk(uint32_t total) {
  SelChunk c;
  const uint32_t per = (total + gridDim.x - 1) / gridDim.x;
  const uint32_t whole = total > kSelSparse ? kSelThreads : kSelRound;   // a block's round
  c.size = max(whole, (per + whole - 1) / whole * whole);
  const uint32_t chunks = (total + c.size - 1) / c.size;
  const uint32_t of_xcd = max(1u, (chunks + 7u) / 8u), j = blockIdx.x / 8u;
  c.index = j < of_xcd ? blockIdx.x % 8u * of_xcd + j : 0xFFFFFFFFu;
  return c;
}

// The hits that tracklet T owns in the lane's block of 8 rows: a bit per row,
// the hits in hv.  info: its record (row_in, row_out used).
__device__ __forceinline__ uint32_t owned_rows(const Slot& S, uint32_t T, int4 info, uint32_t b,
                                               int32_t (&hv)[8]) {
  const int rin = info.y, rout = info.z;
  const int r0 = (int)b * 8;
  uint32_t own = 0;
  if (r0 <= rout && r0 + 7 >= rin) {
    const uint32_t w = S.tl_weight[T];
    const int gr = S.start_sr[T] / kRows * kRows;
    const uint4 v = tl_list(S, T).load_block((int)b);
    uint32_t first[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) first[u] = S.row_off[gr + min(r0 + u, kRows - 1)];
    uint32_t wv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int r = r0 + u;
      hv[u] = r >= rin && r <= rout ? entry_hit(block_get(v, u), first[u]) : -1;
      wv[u] = hv[u] >= 0 ? S.weight[hv[u]] : 0u;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) own |= hv[u] >= 0 && wv[u] == w ? 1u << u : 0u;
  }
  return own;
}

// Hits that the lane's tracklet T owns (0 if it is not valid), the wave's
// tracklets walked together row by row: the entries of kSelRows rows are read
// together, then the weights of their hits.
__device__ __forceinline__ uint32_t owned_by_lane(const Slot& S, uint32_t T, int4 info) {
  const bool valid = info.w != 0;
  const int rin = valid ? info.y : kRows, rout = valid ? info.z : -1;
  const uint32_t w = valid ? S.tl_weight[T] : 0u;
  const int gr = valid ? S.start_sr[T] / kRows * kRows : 0;
  const int lo = wave_min(rin), hi = wave_max(rout);
  const TlList hits = tl_list(S, T);
  uint32_t n = 0;
  for (int r0 = lo; r0 <= hi; r0 += kSelRows) {
    uint32_t e[kSelRows], f[kSelRows];
#pragma unroll
    for (int u = 0; u < kSelRows; ++u) {
      const int r = r0 + u;
      const bool in = r >= rin && r <= rout;
      e[u] = in ? hits.at(r) : (uint32_t)kNoEntry;
      f[u] = in ? (uint32_t)S.row_off[gr + r] : 0u;
    }
    uint32_t wv[kSelRows];
#pragma unroll
    for (int u = 0; u < kSelRows; ++u)
      wv[u] = e[u] != kNoEntry ? S.weight[entry_hit(e[u], f[u])] : 0u;
#pragma unroll
    for (int u = 0; u < kSelRows; ++u) n += e[u] != kNoEntry && wv[u] == w ? 1u : 0u;
  }
  return n;
}

// Per tracklet of the range the number of hits it owns if it is selected,
// else 0; the first one of a chunk also holds the chunk's selected tracklets
// (above the lowest 8 bits), which place the tracks.
__global__ void __launch_bounds__(kSelThreads) k_select(Slot S, DevConst K, int g0) {
  __shared__ uint32_t selected;
  const uint32_t total = S.range_cnt[0];
  const uint32_t base = S.tl_base[g0];
  const SelChunk c = sel_chunk(total);
  if (c.index >= (total + c.size - 1) / c.size) return;
  const uint32_t t0 = c.index * c.size, t1 = min(total, t0 + c.size);
  if (threadIdx.x == 0) selected = 0;
  __syncthreads();
  const uint32_t b = threadIdx.x % kSelLanes;
  uint32_t mine = 0, first = 0;
  if (total > kSelSparse) {
    for (uint32_t ta = t0; ta < t1; ta += kSelThreads) {
      const uint32_t t = ta + threadIdx.x;
      int4 info = make_int4(0, 0, 0, 0);
      if (t < t1) info = *reinterpret_cast<const int4*>(S.tl_info + (size_t)(base + t) * 4);
      const uint32_t n = owned_by_lane(S, base + t, info);
      const uint32_t s = info.w != 0 && (int)n >= K.n_min_track ? n : 0u;
      mine += s != 0u ? 1u : 0u;
      if (t == t0) first = s; else if (t < t1) S.tl_sel[t] = s;
    }
    if (mine) atomicAdd(&selected, mine);
    __syncthreads();
    if (threadIdx.x == 0) S.tl_sel[t0] = first | selected << 8;
    return;
  }
  for (uint32_t ta = t0; ta < t1; ta += kSelRound) {
    const uint32_t t = ta + threadIdx.x / kSelLanes;
    const uint32_t T = base + t;
    int4 info = make_int4(0, 0, 0, 0);
    if (t < t1) info = *reinterpret_cast<const int4*>(S.tl_info + (size_t)T * 4);
    uint32_t n = 0;
    if (info.w != 0) {
      int32_t hv[8];
      n = (uint32_t)__popc(owned_rows(S, T, info, b, hv));
    }
#pragma unroll
    for (int d = kSelLanes / 2; d > 0; d >>= 1) n += (uint32_t)__shfl_xor((int)n, d, 64);
    if (b == 0 && t < t1) {
      const uint32_t s = info.w != 0 && (int)n >= K.n_min_track ? n : 0u;
      mine += s != 0u ? 1u : 0u;
      if (t == t0) first = s; else S.tl_sel[t] = s;
    }
  }
  if (b == 0 && mine) atomicAdd(&selected, mine);
  __syncthreads();
  if (threadIdx.x == 0) S.tl_sel[t0] = first | selected << 8;
}

// Selected tracklets -> tracks of the range (in tracklet order), each with
// its owned hits compacted (ascending row).  A block adds up the chunks
// before its own, lists its chunk's selected tracklets 256 at a time and
// writes them kSelRound together.  The range's track region holds every track
// its hits allow (each owns >= n_min_track hits of its own); a position
// beyond it is not written and raises the capacity error.
__global__ void __launch_bounds__(kSelThreads) k_track_write(Slot S, int g0, int ns) {
  __shared__ uint32_t list[kSelThreads];
  __shared__ uint32_t wsum[kSelThreads / 64];
  const uint32_t total = S.range_cnt[0];
  const uint32_t tl0 = S.tl_base[g0], tk0 = S.tk_base[g0];
  const uint32_t tk_room = S.tk_base[g0 + ns] - tk0;
  const SelChunk c = sel_chunk(total);
  const uint32_t chunks = max(1u, (total + c.size - 1) / c.size);   // one of no tracklets if there is none
  if (c.index >= chunks) return;
  const bool last = c.index == chunks - 1;
  const uint32_t t0 = c.index * c.size, t1 = min(total, t0 + c.size);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // position of the chunk's first track
  uint32_t pos = 0;
  {
    uint32_t v = 0;
    for (uint32_t i = threadIdx.x; i < c.index; i += kSelThreads) v += S.tl_sel[i * c.size] >> 8;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += (uint32_t)__shfl_xor((int)v, d, 64);
    if (lane == 0) wsum[w] = v;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < (int)kSelThreads / 64; ++i) pos += wsum[i];
  }
  const uint32_t b = threadIdx.x % kSelLanes;
  for (uint32_t ta = t0; ta < t1; ta += kSelThreads) {
    const uint32_t t = ta + threadIdx.x;
    const bool sel = t < t1 && (S.tl_sel[t] & 0xFFu) != 0u;
    const unsigned long long m = __ballot(sel);
    __syncthreads();                                  // wsum and list are free
    if (lane == 0) wsum[w] = (uint32_t)__popcll(m);
    __syncthreads();
    uint32_t before = 0, n_sel = 0;
#pragma unroll
    for (int i = 0; i < (int)kSelThreads / 64; ++i) {
      if (i < w) before += wsum[i];
      n_sel += wsum[i];
    }
    if (sel) list[before + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = t;
    __syncthreads();
    for (uint32_t j0 = 0; j0 < n_sel; j0 += kSelRound) {
      const uint32_t j = j0 + threadIdx.x / kSelLanes;
      const bool act = j < n_sel && pos + j < tk_room;
      if (j < n_sel && !act && b == 0) atomicOr(&S.err[2], 1u);
      uint32_t own = 0, T = 0;
      int32_t hv[8];
      if (act) {
        T = tl0 + list[j];
        const int4 info = *reinterpret_cast<const int4*>(S.tl_info + (size_t)T * 4);
        own = owned_rows(S, T, info, b, hv);
      }
      const uint32_t n = (uint32_t)__popc(own);
      uint32_t end = n;
#pragma unroll
      for (int d = 1; d < (int)kSelLanes; d <<= 1) {
        const uint32_t x = (uint32_t)__shfl_up((int)end, d, kSelLanes);
        if ((int)b >= d) end += x;
      }
      if (act) {
        const uint32_t k = tk0 + pos + j;
        int32_t* o = S.tk_own + (size_t)k * kRows;
        uint8_t* orow = S.tk_own_row + (size_t)k * kRows;
        uint32_t at = end - n;
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (own >> u & 1u) {
            o[at] = hv[u];
            orow[at] = (uint8_t)(b * 8 + u);
            ++at;
          }
        if (b == kSelLanes - 1) {
          S.tk_tracklet[k] = (int32_t)T;
          S.tk_nown[k] = (int32_t)end;
        }
      }
    }
    pos += n_sel;
  }
  if (last && threadIdx.x == 0) S.range_cnt[1] = pos;
}

// The inward walk of one pass over the owned hits own[jmin .. n-1]
// (ascending rows): state reset to the outermost hit with the prior
// covariance, transport row by row, update with every owned hit (no gate).
// True: st is the state after the update with own[jmin], where the walk
// ends.  False: a transport failed below the hit jlast, the last one
// updated; st is of no use then.  Memory reads are issued ahead of their use.
__device__ __forceinline__ bool refit_walk(const Slot& S, const DevConst& K, const RowTable& R, const int32_t* own,
                                           const uint8_t* own_row, int n, int jmin, double s0,
                                           double t0, double q0, Helix<double>& st, double& chi2,
                                           int& jlast) {
  const Hit xo = S.hit[own[n - 1]];
  st.y = (double)xo.y;
  st.z = (double)xo.z;
  st.s = s0;
  st.t = t0;
  st.q = q0;
  const double sy0 = K.sy0, sy1z = K.sy1zd, sz0 = K.sz0, sz1z = K.sz1zd;
  {
    const double sy = sy0 + sy1z * fabs(st.z), sz = sz0 + sz1z * fabs(st.z);
    reset_cov(st, sy * sy, sz * sz, (double)K.cs0, (double)K.ct0, (double)K.cq0);
  }
  chi2 = 0.0;
  jlast = n - 1;
  const double smax = K.smax, chi2max = K.chi2max;
  // row-synchronous walk (every lane moves one row per iteration).  Every
  // memory read of a step is issued at its top and used after the
  // transport: the radius of the next row, the record of the next owned
  // hit (own[j]) and the list entry after it (own[j - 1]); indices clamped
  // into [jmin, n) and row 0 so the reads stay inside the lists.
  const int r_out = own_row[n - 1];
  int j = n - 2;
  int rn = j >= jmin ? (int)own_row[j] : -1;
  int32_t pn = own[max(j, jmin)];
  const int rstop = j >= jmin ? (int)own_row[jmin] : r_out;
  double x_hi = (double)R.x[r_out];
  float x_next = R.x[max(r_out - 1, 0)];
  for (int r = r_out - 1; r >= rstop; --r) {
    const double x_lo = (double)x_next;
    x_next = R.x[max(r - 1, 0)];
    const Hit xh = S.hit[pn];
    const int ja = max(j - 1, jmin);
    const int32_t p_after = own[ja];
    const int r_after = own_row[ja];
    if (!transport(st, x_lo - x_hi, K.bd, smax, K.kkd, K.m2d)) return false;
    x_hi = x_lo;
    if (r != rn) continue;
    const double sy = sy0 + sy1z * fabs(st.z), sz = sz0 + sz1z * fabs(st.z);
    double ch = 0.0;
    kalman_update(st, (double)xh.y, (double)xh.z, sy * sy, sz * sz, chi2max, smax, false, &ch);
    chi2 = chi2 + ch;
    jlast = j;
    --j;
    pn = p_after;
    rn = j >= jmin ? r_after : -1;
  }
  return true;
}

// One pass: a failed transport ends it at the last hit updated.  The state
// there is not kept on the way (20 doubles copied at every update, a seventh
// of a step's instructions, for the few tracks that need it): the walk is
// made again down to that hit, by the same arithmetic, and so ends there.
__device__ __forceinline__ void refit_pass(const Slot& S, const DevConst& K, const RowTable& R, const int32_t* own,
                                           const uint8_t* own_row, int n, int& jmin, double s0,
                                           double t0, double q0, Helix<double>& st, double& chi2) {
  int jlast;
  while (!refit_walk(S, K, R, own, own_row, n, jmin, s0, t0, q0, st, chi2, jlast)) jmin = jlast;
}

// a7: refit of each track over its owned hits, in double, three inward
// passes.  Pass 1 starts from the tracklet's inner (s, T, Q) with s carried
// to the outermost owned row along the circle (sin phi is linear in x);
// each later pass starts from the previous pass's result carried back the
// same way, so the Jacobians are evaluated along the fitted track.  Output
// at the innermost fitted hit; its cluster is marked for the canonical
// ordering.
__global__ void __launch_bounds__(256) k_refit(Slot S, DevConst K, int g0, int ns) {
  __shared__ RowTable R;
  load_radii(S, R);
  const uint32_t tk0 = S.tk_base[g0];
  // tracks past the region were not written (capacity error raised)
  const uint32_t total = min(S.range_cnt[1], S.tk_base[g0 + ns] - tk0);
  // each XCD (blocks are dispatched round-robin over the 8) a contiguous
  // chunk of the tracks, which are in sector order: a sector's hits are read
  // through one XCD's L2
  constexpr uint32_t kXcd = 8;
  const uint32_t xcd = blockIdx.x % kXcd, jb = blockIdx.x / kXcd;
  const uint32_t nbx = (gridDim.x - xcd + kXcd - 1) / kXcd;
  const uint32_t chunk = (total + kXcd - 1) / kXcd;
  const uint32_t c0 = min(total, xcd * chunk);
  const uint32_t c1 = min(total, c0 + chunk);
  unsigned nfit = 0;
  const LaneGroup lg = lane_deal(total, min(kRefitWaves, gridDim.x * (blockDim.x >> 6)));
  const uint32_t waves = blockDim.x >> 6;
  for (uint32_t t = c0 + (jb * waves + (threadIdx.x >> 6)) * lg.per + lg.index; t < c1;
       t += nbx * waves * lg.per) {
    if (lg.first) ++nfit;
    const uint32_t k = tk0 + t;
    const int32_t T = S.tk_tracklet[k];
    const int n = S.tk_nown[k];
    const int32_t* own = S.tk_own + (size_t)k * kRows;
    const uint8_t* own_row = S.tk_own_row + (size_t)k * kRows;
    int32_t* out = S.tk_info + (size_t)k * 4;
    if (n < 1) continue;
    const int ro = own_row[n - 1];
    const int rin_tl = S.tl_info[(size_t)T * 4 + 1];
    const float* sv = S.tl_state + (size_t)T * 5;
    const double smax = K.smax;
    // the three passes: jmin, the innermost hit a pass reached, only grows
    Helix<double> st;
    double chi2 = 0.0;
    int jmin = 0;
    bool ok = true;
    double sin_ = sv[2], tin = sv[3], qin = sv[4];
    int rin = rin_tl;
    for (int pass = 0; ok && pass < 3; ++pass) {
      const double s0 = sin_ + (K.bd * qin) * ((double)R.x[ro] - (double)R.x[rin]);
      if (!(fabs(s0) <= smax)) {
        ok = false;
        break;
      }
      refit_pass(S, K, R, own, own_row, n, jmin, s0, tin, qin, st, chi2);
      sin_ = st.s;
      tin = st.t;
      qin = st.q;
      rin = own_row[jmin];
    }
    const int nfitted = n - jmin;
    if (!ok || nfitted < K.n_min_track || !lg.first) continue;
    out[1] = nfitted;
    out[2] = rin;
    out[3] = ro;
    double* par = S.tk_par + (size_t)k * 5;
    par[0] = st.y;
    par[1] = st.z;
    par[2] = st.s;
    par[3] = st.t;
    par[4] = st.q;
    double* cov = S.tk_cov + (size_t)k * 15;
#pragma unroll
    for (int i = 0; i < 15; ++i) cov[i] = st.c[i];
    S.tk_chi2[k] = chi2;
    S.tmap[S.hit[own[jmin]].id] = (int32_t)k;
  }
  wave_add_u64(&S.stats[3], nfit);
}

}  // namespace tpc
