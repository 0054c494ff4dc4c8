// a5: tracklet construction (paper, Abstract: Kalman-filter track
// following).  One lane per start hit, or a group of lanes where start hits
// are few; float arithmetic; the lane's state and the decisions of its current
// block of 8 rows live in registers, its hit list in global memory
// (row-indexed, a block written when the lane leaves it).
#include <algorithm>

#include "tpc_device.h"
#include "tpc_kernels.h"

namespace tpc {

// Stop rules after a transport to the row at radius xr: left the sector
// sideways, left the drift volume, or crossed the membrane (zsign = -1 on
// the A side, 1 on the C side).
__device__ __forceinline__ bool inside(const DevConst& K, const Helix<float>& h, float xr, float zsign) {
  const bool sector = fabsf(h.y) <= xr * K.tanh_half + K.medge;
  const bool volume = fabsf(h.z) <= K.z_max + K.mz;
  const bool side = !(zsign * h.z > K.mz);
  return sector & volume & side;      // one branch for all of them
}

// The search window around a predicted state: |r_y| <= min(k sqrt(S_yy),
// w_max), |r_z| <= min(k sqrt(S_zz), w_max).
struct Window {
  float wy, wz;
};
__device__ __forceinline__ Window search_window(const DevConst& K, const Resid<float>& w) {
  float ry = sqrt_mid(w.s00), rz = sqrt_mid(w.s11);
  if (!mid_range(fminf(w.s00, w.s11)) || !mid_range(fmaxf(w.s00, w.s11))) {
    asm volatile("");        // a branch, not both results and a choice
    ry = sqrtf(w.s00);
    rz = sqrtf(w.s11);
  }
  Window x;
  x.wy = K.kwin * ry;
  if (x.wy > K.wmax) x.wy = K.wmax;
  x.wz = K.kwin * rz;
  if (x.wz > K.wmax) x.wz = K.wmax;
  return x;
}

// Best hit of row sr for the predicted state: inside the window, smallest
// chi2, ties to the smaller cluster ID.  -1 if none; its place is
// returned in `out` (y and z only).  By one lane; WB: hit records read per round trip.
template <int WB>
__device__ __forceinline__ int32_t search_row(const Slot& S, const DevConst& K, const RowBins& rb,
                                              const Helix<float>& h, float vy, float vz,
                                              unsigned& examined, Hit& out) {
  const Resid<float> w = resid_weights(h, vy, vz);
  const Window win = search_window(K, w);
  const float wy = win.wy, wz = win.wz;
  const float yc = h.y, zc = h.z;
  int32_t best = -1;
  float bchi = 0.0f;
  uint32_t bid = 0;
  for_window_hits<WB>(rb, bin_offsets(S, rb), S.hit, yc, zc, wy, wz, [&](uint32_t p, const Hit& x) {
    const float ry = x.y - yc, rz = x.z - zc;
    if (!(fabsf(ry) <= wy && fabsf(rz) <= wz)) return;
    ++examined;                 // hits inside the window (independent of the binning)
    const float ch = chi2_of(w, ry, rz);
    const uint32_t id = x.id;
    if (best < 0 || ch < bchi || (ch == bchi && id < bid)) {
      best = (int32_t)p;
      bchi = ch;
      bid = id;
      out.y = x.y;
      out.z = x.z;
    }
  });
  return best;
}

// The same search by the lanes of a group, all with the same state: each lane
// tests its own candidates.  A short row (at most two hits a lane) is tested
// whole, the first hit of each lane (hx, valid if the row has it) read before
// the transport, so that the search waits for no memory; a longer one by the
// bins the window touches, a lane taking every (size / 4)-th hit of every
// fourth z row.  In a lone wave every instruction takes 8 cycles and every
// read some 200 to 800: a lane by itself needs some 250 instructions and two
// reads after one another for a search.
__device__ __forceinline__ bool short_row(const LaneGroup& lg, uint32_t n) { return n <= 2u * lg.size; }
__device__ __forceinline__ int32_t search_group(const Slot& S, const DevConst& K, const LaneGroup& lg,
                                                uint32_t first, uint32_t n, const RowBins& rb,
                                                const Hit& hx, const Helix<float>& h, float vy, float vz,
                                                unsigned& examined, Hit& out) {
  const Resid<float> w = resid_weights(h, vy, vz);
  const Window win = search_window(K, w);
  bool have = false;
  float bchi = 0.0f;
  uint32_t bp = 0;
  Hit bx = hx;
  auto test = [&](uint32_t p, const Hit& x) {
    const float ry = x.y - h.y, rz = x.z - h.z;
    if (!(fabsf(ry) <= win.wy && fabsf(rz) <= win.wz)) return;
    ++examined;
    const float ch = chi2_of(w, ry, rz);
    if (!have || ch < bchi || (ch == bchi && x.id < bx.id)) {
      have = true;
      bchi = ch;
      bp = p;
      bx = x;
    }
  };
  if (short_row(lg, n)) {
    if (lg.lane < n) test(first + lg.lane, hx);
    if (lg.size + lg.lane < n) {
      const uint32_t p = first + lg.size + lg.lane;
      test(p, S.hit[p]);
    }
  } else {
    const float eps = 1e-3f;
    const int iy0 = bin_y(rb, h.y - win.wy - eps), iy1 = bin_y(rb, h.y + win.wy + eps);
    const int iz0 = bin_z(rb, h.z - win.wz - eps), iz1 = bin_z(rb, h.z + win.wz + eps);
    const uint32_t* bo = bin_offsets(S, rb);
    for (int izb = iz0; izb <= iz1; izb += 4) {
      const int iz = izb + (int)(lg.lane & 3u);
      uint32_t lo = 0u, hi = 0u;
      if (iz <= iz1) {
        lo = bo[iz * rb.ny + iy0];
        hi = bo[iz * rb.ny + iy1 + 1];
      }
      for (uint32_t p = lo + (lg.lane >> 2); p < hi; p += lg.size >> 2) test(p, S.hit[p]);
    }
  }
  unsigned long long m = __ballot(have) & lg.mask;
  if (m == 0ull) return -1;
  if (__popcll(m) > 1) {
    float c = bchi;
    uint32_t id = bx.id;
    bool any = have;
    for (uint32_t d = lg.size >> 1; d > 0u; d >>= 1) {
      const float co = __shfl_xor(c, (int)d, 64);
      const uint32_t io = (uint32_t)__shfl_xor((int)id, (int)d, 64);
      const bool ho = __shfl_xor((int)any, (int)d, 64) != 0;
      if (ho && (!any || co < c || (co == c && io < id))) {
        c = co;
        id = io;
        any = true;
      }
    }
    const unsigned long long best = __ballot(have && bchi == c && bx.id == id) & lg.mask;
    if (best != 0ull) m = best;      // (0: chi2 is not a number, any hit will be refused)
  }
  const int win_lane = __ffsll((long long)m) - 1;
  out.y = __shfl(bx.y, win_lane, 64);
  out.z = __shfl(bx.z, win_lane, 64);
  return __shfl((int)bp, win_lane, 64);
}

__device__ __forceinline__ bool try_hit(const DevConst& K, Helix<float>& h, const Hit& x, float vy,
                                        float vz, unsigned& tries) {
  float ch;
  ++tries;
  return kalman_update(h, x.y, x.z, vy, vz, K.chi2max, K.smax, true, &ch);
}

// For each start hit h0 (row r0) with cleaned up-link h1:
//  seed  (y, z) = h0, sin phi and tan lambda from h0 -> h1, q/pT = 0, prior
//        covariance (hit variances, wide angles and curvature);
//  out   rows r0+1..158: transport, stop rules; follow the cleaned chain while
//        its hits pass the gate, then (for good) take the best-chi2 hit of
//        each row's window; stop after n_gap consecutive rows without hit;
//  in    restart at the outermost hit with the prior covariance and the
//        outward (s, T, Q); rows down to 0: re-confirm the outward hit, else
//        search; same gap rule.  The inward hits form the tracklet.
// What bounds it is the count of instructions: a wave alone on its SIMD issues
// one every 8 cycles, and some 320 steps follow one another; with four waves
// to a SIMD the vector unit is busy.  So a step has one branch for all its stop
// rules, transports without looking whether it may, and the hit list's block is
// shifted in row by row (four instructions; placing an entry takes 15).
// With these 60 tracks went from 397 to 362 us, 200 in one sector from 473 to
// 436, 2000 from 761 to 703, 15000 from 1255 to 1180.
// kGroup: a group of lg.size >= 8 lanes a tracklet, else a lane each (or a few
// lanes, doing the same).  kSearchFirst: at a row, those without a link to
// follow search before the others try theirs, so that one update serves both;
// a second one is for links that failed.  (A lane each: 1200 and 1249 us for
// 15000 tracks, as some link of a wave fails at nearly every row.)
template <int WB, bool kGroup, bool kSearchFirst>
__device__ __forceinline__ void make_tracklets(const Slot& S, const DevConst& K, const RowTable& R, int g0,
                                               uint32_t total, const LaneGroup& lg) {
  // Tracklets are ordered by (sector, row): give each XCD (blocks are
  // dispatched round-robin over the 8 XCDs) one contiguous chunk, so the
  // hits a chunk's lanes read stay in that XCD's L2.
  const uint32_t base = S.tl_base[g0];
  constexpr uint32_t kXcd = 8;
  const uint32_t xcd = blockIdx.x % kXcd, j = blockIdx.x / kXcd;
  const uint32_t nbx = (gridDim.x - xcd + kXcd - 1) / kXcd;
  const uint32_t chunk = (total + kXcd - 1) / kXcd;
  const uint32_t c0 = xcd * chunk;
  const uint32_t c1 = min(total, c0 + chunk);
  unsigned n_tl = 0, n_visits = 0, n_examined = 0, n_tries = 0, tl_hits = 0;
  const uint32_t waves = blockDim.x >> 6;
  const uint32_t t0 = c0 + (j * waves + (threadIdx.x >> 6)) * lg.per + lg.index;
  for (uint32_t t = t0; t < c1; t += nbx * waves * lg.per) {
    unsigned visits = 0, examined = 0, tries = 0;
    const uint32_t T = base + t;
    const int sr0 = S.start_sr[T];
    const int g = sr0 / kRows;
    const int gr = g * kRows;
    const int r0 = sr0 - gr;
    const float zsign = (g % kSectorsPerEvent) >= kSectorsPerEvent / 2 ? 1.0f : -1.0f;
    const int32_t p0 = S.start_hit[T];
    const Hit x0 = S.hit[p0];
    const Hit x1 = S.hit[x0.upc];
    const TlList hits = tl_list(S, T);
    const uint32_t first0 = S.row_off[sr0];
    // what a tie between tracklets of equal length goes by
    const uint32_t id0 = x0.id - (uint32_t)S.ev_off[g / kSectorsPerEvent];

    // radii of the start row and the next one (r0 <= 157: a start hit has
    // an up link)
    const float x_r0 = R.x[r0], x_r1 = R.x[r0 + 1];
    Helix<float> st;
    {
      const float dx = x_r1 - x_r0;
      const float dy = x1.y - x0.y;
      const float dz = x1.z - x0.z;
      const float L = sqrtf(dx * dx + dy * dy);
      st.y = x0.y;
      st.z = x0.z;
      st.s = dy / L;
      st.t = dz / L;
      st.q = 0.0f;
      const float sy = sigma_y(K, st.z), sz = sigma_z(K, st.z);
      reset_cov(st, sy * sy, sz * sz, K.cs0, K.ct0, K.cq0);
    }
    // the hit list's block of the current row, in registers: the rows are
    // pushed as they are left, up to row `pushed`
    int cb = r0 >> 3;
    uint4 blk = block_empty();
    block_push(blk, (uint32_t)p0 - first0);
    int pushed = r0;

    // outward
    float l_y = st.y, l_z = st.z, l_s = st.s, l_t = st.t, l_q = st.q;   // at the last hit
    int rout = r0;
    float x_rout = x_r0;
    int32_t next = x0.upc;     // cleaned chain link of the last accepted hit
    int32_t p_out = p0;        // the outermost accepted hit
    bool chain = true;
    int miss = 0;
    // row radii: the current one carried in a register, the next one read
    // a step ahead (index clamped to the last row); both start from values
    // the seed has used, so no read before the loop is waited for inside it
    float x_prev = x_r0;
    float x_ahead = x_r1;
    int r = r0;
    // a group's first hits of the current row and the next one, a step ahead
    uint32_t f_lo = 0, f_hi = 0;
    if (kGroup) {
      f_lo = S.row_off[gr + r0 + 1];
      f_hi = S.row_off[gr + r0 + 2];
    }
    bool live = true;
    do {
      ++r;
      const float xr = x_ahead;
      x_ahead = R.x[min(r + 1, kRows - 1)];
      // reads independent of the state, issued before the transport: the
      // row's bin range (a group: its hits, if it is short) and the hit the
      // chain link points to
      RowBins rb;
      Hit hx;
      uint32_t first, nrow = 0;
      if (kGroup) {
        first = f_lo;
        nrow = f_hi - f_lo;
        f_lo = f_hi;
        f_hi = S.row_off[gr + min(r + 2, kRows)];
        if (!short_row(lg, nrow)) rb = S.bins[gr + r];
        else if (lg.lane < nrow) hx = S.hit[first + lg.lane];
      } else {
        rb = S.bins[gr + r];
        first = (uint32_t)rb.first;
      }
      const bool direct = chain & (next >= 0);
      Hit xg;
      if (direct) xg = S.hit[next];
      if ((r & 7) == 0) {          // into the next block of rows
        hits.store_block(cb, blk);
        cb = r >> 3;
        blk = block_empty();
      }
      live = transport<float, true, true>(st, xr - x_prev, K.b, K.smax, K.kk, K.m2);
      const bool in = inside(K, st, xr, zsign);
      live = live & in;
      x_prev = xr;
      if (live) {
        const float sy = sigma_y(K, st.z), sz = sigma_z(K, st.z);
        const float vy = sy * sy, vz = sz * sz;
        int32_t hit = next;
        bool got = false;
        if (kSearchFirst) {
          if (!direct) hit = search_group(S, K, lg, first, nrow, rb, hx, st, vy, vz, examined, xg);
          if (hit >= 0) got = try_hit(K, st, xg, vy, vz, tries);
          chain = direct & got;
          if (direct & !got) {
            hit = search_group(S, K, lg, first, nrow, rb, hx, st, vy, vz, examined, xg);
            if (hit >= 0) got = try_hit(K, st, xg, vy, vz, tries);
          }
        } else {
          if (direct) got = try_hit(K, st, xg, vy, vz, tries);
          if (!got) {
            chain = false;
            hit = kGroup ? search_group(S, K, lg, first, nrow, rb, hx, st, vy, vz, examined, xg)
                         : search_row<WB>(S, K, rb, st, vy, vz, examined, xg);
            if (hit >= 0) got = try_hit(K, st, xg, vy, vz, tries);
          }
        }
        block_push(blk, got ? (uint32_t)hit - first : (uint32_t)kNoEntry);
        pushed = r;
        if (got) {
          if (chain) next = xg.upc;
          p_out = hit;
          miss = 0;
          l_y = st.y;
          l_z = st.z;
          l_s = st.s;
          l_t = st.t;
          l_q = st.q;
          rout = r;
          x_rout = xr;
        } else {
          live = ++miss < K.n_gap;
        }
      }
    } while (live && r < kRows - 1);
    // the last block's entries to their places (unless it is still empty)
    if ((pushed >> 3) == cb)
      for (int k = pushed & 7; k < 7; ++k) block_push(blk, kNoEntry);
    hits.store_block(cb, blk);
    visits += (unsigned)(r - r0);

    // inward, covariance reset at the outermost hit
    const Hit xo = S.hit[p_out];
    st.y = xo.y;
    st.z = xo.z;
    st.s = l_s;
    st.t = l_t;
    st.q = l_q;
    {
      const float sy = sigma_y(K, st.z), sz = sigma_z(K, st.z);
      reset_cov(st, sy * sy, sz * sz, K.cs0, K.ct0, K.cq0);
    }
    int n = 1;
    int rin = rout;
    l_y = st.y;
    l_z = st.z;
    miss = 0;
    // the blocks of the current row and of the one below, in registers (the
    // outward decisions, rewritten as the inward ones are taken; a block is
    // stored back only if an entry changed or the outward phase has not
    // written it); the outward hit of the next row down loaded one step
    // ahead, the first hit of the row below it two steps ahead
    const int cb0 = r0 >> 3;
    cb = max(rout - 1, 0) >> 3;
    bool dirty = cb < cb0;
    blk = dirty ? block_empty() : hits.load_block(cb);
    uint4 blk_dn = cb > cb0 ? hits.load_block(cb - 1) : block_empty();
    const uint32_t f_a = rout - 1 >= r0 ? (uint32_t)S.row_off[gr + rout - 1] : 0u;
    uint32_t f_next = rout - 2 >= r0 ? (uint32_t)S.row_off[gr + rout - 2] : 0u;
    int32_t uh_next = rout - 1 >= r0 ? entry_hit(block_get(blk, (rout - 1) & 7), f_a) : -1;
    Hit xu_next;
    if (uh_next >= 0) xu_next = S.hit[uh_next];
    x_prev = x_rout;
    x_ahead = R.x[max(rout - 1, 0)];
    // wait for these reads here, once: a read still in flight at the loop's
    // entry would make the compiler wait inside every step
    asm volatile("" : "+v"(x_ahead), "+v"(f_next));
    r = rout;
    if (kGroup) {
      f_lo = S.row_off[gr + max(rout - 1, 0)];
      f_hi = S.row_off[gr + rout];
      f_next = S.row_off[gr + max(rout - 2, 0)];
    }
    live = rout > 0;
    while (live) {
      --r;
      const float xr = x_ahead;
      x_ahead = R.x[max(r - 1, 0)];
      RowBins rb;
      Hit hx;
      uint32_t first, nrow = 0;
      if (kGroup) {
        first = f_lo;
        nrow = f_hi - f_lo;
        f_hi = f_lo;
        f_lo = f_next;
        if (!short_row(lg, nrow)) rb = S.bins[gr + r];
        else if (lg.lane < nrow) hx = S.hit[first + lg.lane];
      } else {
        rb = S.bins[gr + r];
        first = (uint32_t)rb.first;
      }
      const int32_t uh = uh_next;
      const Hit xu = xu_next;
      // row r-1: its outward entry (this block or the one below) and the
      // first hit of its row, read a step ago
      uh_next = -1;
      if (r - 1 >= r0)
        uh_next = entry_hit(block_get((r & 7) == 0 ? blk_dn : blk, (r - 1) & 7), f_next);
      if (uh_next >= 0) xu_next = S.hit[uh_next];
      if (kGroup) f_next = S.row_off[gr + max(r - 2, 0)];
      else if (r - 2 >= r0) f_next = (uint32_t)S.row_off[gr + r - 2];
      live = transport<float, true, true>(st, xr - x_prev, K.b, K.smax, K.kk, K.m2);
      const bool in = inside(K, st, xr, zsign);
      live = live & in;
      x_prev = xr;
      if (live) {
        const float sy = sigma_y(K, st.z), sz = sigma_z(K, st.z);
        const float vy = sy * sy, vz = sz * sz;
        int32_t hit = uh;
        bool got = false;
        if (kSearchFirst) {
          Hit xs = xu;
          if (uh < 0) hit = search_group(S, K, lg, first, nrow, rb, hx, st, vy, vz, examined, xs);
          if (hit >= 0) got = try_hit(K, st, xs, vy, vz, tries);
          if ((uh >= 0) & !got) {
            hit = search_group(S, K, lg, first, nrow, rb, hx, st, vy, vz, examined, xs);
            if (hit >= 0) got = try_hit(K, st, xs, vy, vz, tries);
          }
          if (!got) hit = -1;
          if (hit != uh) {              // not what the outward phase found
            block_set(blk, r & 7, got ? (uint32_t)hit - first : (uint32_t)kNoEntry);
            dirty = true;
          }
        } else {
          if (uh >= 0) got = try_hit(K, st, xu, vy, vz, tries);
          if (!got) {
            Hit xs;
            hit = kGroup ? search_group(S, K, lg, first, nrow, rb, hx, st, vy, vz, examined, xs)
                         : search_row<WB>(S, K, rb, st, vy, vz, examined, xs);
            if (hit >= 0) got = try_hit(K, st, xs, vy, vz, tries);
            if (!got) hit = -1;
            if (hit != uh) {
              block_set(blk, r & 7, got ? (uint32_t)hit - first : (uint32_t)kNoEntry);
              dirty = true;
            }
          }
        }
        if (got) {
          ++n;
          miss = 0;
          l_y = st.y;
          l_z = st.z;
          l_s = st.s;
          l_t = st.t;
          l_q = st.q;
          rin = r;
        } else {
          live = ++miss < K.n_gap;
        }
        live = live & (r > 0);
        if (live & ((r & 7) == 0)) {   // into the block below
          if (dirty) hits.store_block(cb, blk);
          --cb;
          dirty = cb < cb0;
          blk = blk_dn;
          blk_dn = cb > cb0 ? hits.load_block(cb - 1) : block_empty();
        }
      }
    }
    if (dirty) hits.store_block(cb, blk);
    visits += (unsigned)(rout - r);
    if (kGroup) n_examined += examined;   // each lane counted its own
    if (!lg.first) continue;         // one lane of the tracklet's group writes
    n_tl += 1u;
    n_visits += visits;
    if (!kGroup) n_examined += examined;
    n_tries += tries;
    tl_hits += (unsigned)n;
    int32_t* info = S.tl_info + (size_t)T * 4;
    const bool valid = n >= K.n_min_tracklet;
    info[0] = n;
    info[1] = rin;
    info[2] = rout;
    info[3] = valid ? 1 : 0;
    const uint32_t w = ((uint32_t)n << 24) | (0xFFFFFFu - id0);
    S.tl_weight[T] = w;
    // a6 (ownership): every hit of a valid tracklet keeps the largest weight
    // of the tracklets holding it; issued here, so the atomics overlap the
    // other lanes' Kalman steps, and only where the weight read is smaller
    if (valid) {
      // the list is read back a block of eight rows per memory round trip
      for (int b = rin >> 3; b <= rout >> 3; ++b) {
        const uint4 v = hits.load_block(b);
        uint32_t f[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) f[u] = (uint32_t)S.row_off[gr + min(8 * b + u, kRows - 1)];
        int32_t h[8];
        uint32_t cur[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int r = 8 * b + u;
          h[u] = (r >= rin && r <= rout) ? entry_hit(block_get(v, u), f[u]) : -1;
          cur[u] = h[u] >= 0 ? S.weight[h[u]] : 0xFFFFFFFFu;
        }
        // a weight already at least w stays so (the maximum only grows)
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (cur[u] < w) atomicMax(&S.weight[h[u]], w);
      }
    }
    float* sv = S.tl_state + (size_t)T * 5;
    sv[0] = l_y;
    sv[1] = l_z;
    sv[2] = l_s;
    sv[3] = l_t;
    sv[4] = l_q;
  }
  wave_add_u64(&S.stats[0], n_tl);
  wave_add_u64(&S.stats[1], n_visits);
  wave_add_u64(&S.stats[2], n_examined);
  wave_add_u64(&S.stats[6], tl_hits);
  wave_add_u64(&S.stats[7], n_tries);
}

// A lane group a tracklet (up to kGroups of them a wave) and a lane a
// tracklet are two kernels: together they would need 145 registers, and the
// second one four waves to a SIMD (at most 128: kept there by the launch
// bound, at 9 spilled words outside of the rows' loops; 8 hits a read need 152).
// Each leaves the other's counts alone.  Where the line lies: on kTrackletWaves
// or kShortRowWaves waves a group has 8 lanes or more.  A 60-track event 443 us
// by the second kernel and 397 by this one, 200 tracks in one sector 496 and
// 473, 2000 tracks 761 and 764; groups of 4 lanes were slower (2000 tracks in
// 1.31 instead of 1.30 ms whole), as every search costs some 40 instructions
// to bring the lanes' results together.
// Of the first kernel there are two: with groups of 32 lanes or more (up to
// kWideGroups of them a wave) a wave has one or two tracklets, and a link that is
// followed needs no search; with smaller groups some tracklet of a wave
// searches at nearly every row, and it costs less to let the others wait with
// their update for it (32 events of 60 tracks 545 us, 480 so; 2000 tracks, then
// in groups of 8, 708 and 662; 60 tracks, a wave each, 361 and 381).
template <bool kSearchFirst>
__global__ void __launch_bounds__(256) k_tracklets_few(Slot S, DevConst K, int g0, uint32_t most) {
  __shared__ RowTable R;
  const uint32_t total = S.range_cnt[0];
  const uint32_t wide = kWideGroups * most;
  if (kSearchFirst ? total <= wide || total > kGroups * most : total > wide) return;
  load_radii(S, R);
  const LaneGroup lg = lane_group(total, min(most, gridDim.x * (blockDim.x >> 6)));
  make_tracklets<1, true, kSearchFirst>(S, K, R, g0, total, lg);
}

template <int WB>
__global__ void __launch_bounds__(256, WB == 8 ? 1 : 4) k_tracklets(Slot S, DevConst K, int g0,
                                                                             uint32_t few) {
  __shared__ RowTable R;
  const uint32_t total = S.range_cnt[0];
  if (total <= few) return;
  load_radii(S, R);
  const LaneGroup lg = lane_deal(total, min(kLaneWaves, gridDim.x * (blockDim.x >> 6)));
  make_tracklets<WB, false, false>(S, K, R, g0, total, lg);
}

// The kernels whose counts the host's bound allows.  A bound of 32 times
// theirs or more leaves the first two out (few = 0, the last kernel takes any
// count): clusters for that many start hits have given four times as many as
// they take, and an idle launch costs 5 us.
void launch_tracklets(int wb, int64_t bound, int64_t row_hits, int blocks, int threads, hipStream_t st,
                      const Slot& S, const DevConst& K, int g0) {
  const uint32_t most = row_hits <= 2 * 64 / kGroups ? kShortRowWaves : kTrackletWaves;
  const uint32_t few = bound < 32 * (int64_t)kGroups * most ? kGroups * most : 0u;
  if (few) {
    const int64_t lanes = std::min<int64_t>(most, bound) * 64;
    const int nb = (int)((lanes + threads - 1) / threads + 7) / 8 * 8;
    k_tracklets_few<false><<<nb, threads, 0, st>>>(S, K, g0, most);
    if (bound > (int64_t)kWideGroups * most) k_tracklets_few<true><<<nb, threads, 0, st>>>(S, K, g0, most);
    if (bound <= (int64_t)few) return;
  }
  switch (wb) {
    case 2: k_tracklets<2><<<blocks, threads, 0, st>>>(S, K, g0, few); break;
    case 8: k_tracklets<8><<<blocks, threads, 0, st>>>(S, K, g0, few); break;
    default: k_tracklets<4><<<blocks, threads, 0, st>>>(S, K, g0, few); break;
  }
}

}  // namespace tpc
