// Cellular-automaton part of the tracker (paper, Abstract: track finding by
// a cellular automaton): per-hit best neighbour pair, mutual-link cleaning
// and start hits of the resulting chains.
#include "tpc_device.h"
#include "tpc_kernels.h"

namespace tpc {

constexpr int kNfThreads = 64;

__device__ __forceinline__ float nf_metric(float yd, float zd, float yu, float zu, float yh, float zh,
                                           float f, float wy, float wz) {
  const float dy = yd + (yu - yd) * f - yh;
  const float dz = zd + (zu - zd) * f - zh;
  return dy * dy * wy + dz * dz * wz;
}

// Running argmin of the pair metric: smaller m, ties to the smaller
// (id_d, id_u).
struct PairBest {
  bool have = false;
  float m = 0.0f;
  uint32_t id_d = 0, id_u = 0;
  int32_t d = -1, u = -1;
  __device__ __forceinline__ void offer(float mm, uint32_t idd, uint32_t idu, int32_t pd, int32_t pu) {
    // (no branches: in a wave some lane takes each of them)
    const bool less = mm < m, same = mm == m;
    const bool id_less = idd < id_d, id_same = idd == id_d, idu_less = idu < id_u;
    const bool better = !have | less | (same & (id_less | (id_same & idu_less)));
    have = true;
    m = better ? mm : m;
    id_d = better ? idd : id_d;
    id_u = better ? idu : id_u;
    d = better ? pd : d;
    u = better ? pu : u;
  }
};

constexpr int kNfCand = 47;      // candidates of both rows listed per hit before a nested scan

// a3: for each hit h of row r (1..157), the
// pair (d in row r-1, u in row r+1) inside the origin-pointing windows
// |y - y_h x_r'/x_r| <= W, |z - z_h x_r'/x_r| <= W whose straight line passes
// closest to h, measured by m = dy^2 / (1.5 sy^2) + dz^2 / (1.5 sz^2);
// ties go to the smaller (id_d, id_u); the pair is kept if m <= m_max.
// Rows 0 and 158 get no links.
// One lane per hit.  The candidates of both rows are listed in LDS
// (thread-minor, so a wave's accesses fall in distinct banks; 16 bits each,
// from the row's first hit: a row has at most 4096) and then paired; a hit
// with more than kNfCand of them pairs the listed up row as it reads the down
// row again, and scans the up window for each down candidate only if the up
// row alone has more.  (Rows of 4096 hits spread over 8 sectors: 1.56 ms, 1.88
// with that scan for every longer list, 2.50 with a list of 32 up hits; 1500
// and a window of 5 cm: 0.49, 0.77, 0.74; 2000 in an eighth of two sectors,
// where nearly every up row is too long: 12.2, 11.3, 12.5.)
// Bound by instructions of waves whose lanes have lists of different lengths,
// each wave issuing one in 8 cycles or so: hence waves on the SIMD count (6 by
// registers and LDS; 4 waves to a block with 32-bit entries had 2.5), and so
// does every branch.  (Nine registers are spilled for 6 waves: two of them once
// a hit, the others in the scans of the longest lists.)  A list is filled without one: each hit of the window's
// bins is written to the next entry, which only a hit inside keeps.  Pairing
// as each down hit is read ran the pair loop for every hit that any lane of
// the wave had inside.
// 15000 tracks 503 us: 16-bit entries 432, one-wave blocks 405, both rows
// listed and no branches 262, registers for 6 waves 255 (64 events of 15000
// tracks 3900, 3080, 2290, 2130; 2000 tracks 27.6, 22).  Measured best: 47
// entries (63: 276; 32 for the up row alone, as before, and 16: 432 and 650),
// 4 pairs at a time (1, 2, 8: 330, 286, 291).  Both rows are read through the
// caches with the batched window reads (faster than staging the rows in LDS).
// This function: sorted hit h, `my` the thread's candidate slots in LDS;
// WB hit records are read per memory round trip (a tuning knob).
template <int WB>
__device__ __forceinline__ void nf_hit(const Slot& S, const DevConst& K, uint32_t h, uint16_t* my) {
  const int sr = (int)S.hit_sr[h];
  const int g = sr / kRows;
  const int row = sr - g * kRows;
  if (row == 0 || row == kRows - 1) {
    S.up[h] = -1;
    S.dn[h] = -1;
    return;
  }
  const RowBins Bd = S.bins[sr - 1], Bu = S.bins[sr + 1];
  const Hit x = S.hit[h];
  const uint32_t* bod = bin_offsets(S, Bd);
  const uint32_t* bou = bin_offsets(S, Bu);
  const float xd = S.row_x[row - 1], xr = S.row_x[row], xu = S.row_x[row + 1];
  const float rho_d = xd / xr;
  const float rho_u = xu / xr;
  const float f = (xr - xd) / (xu - xd);
  const float W = K.nf_w;
  const float yh = x.y, zh = x.z;
  const float ypu = yh * rho_u, zpu = zh * rho_u;
  const float ypd = yh * rho_d, zpd = zh * rho_d;
  // the candidates, up row first, then down row, as distances from the row's
  // first hit; a hit past the list's end lands in the entry after it
  int nu = 0;
  for_window_hits<WB>(Bu, bou, S.hit, ypu, zpu, W, W, [&](uint32_t u, const Hit& c) {
    const bool in_y = fabsf(c.y - ypu) <= W, in_z = fabsf(c.z - zpu) <= W;
    my[min(nu, kNfCand) * kNfThreads] = (uint16_t)(u - (uint32_t)Bu.first);
    nu += in_y & in_z ? 1 : 0;
  });
  PairBest best;
  if (nu > 0) {
    int nc = nu;
    for_window_hits<WB>(Bd, bod, S.hit, ypd, zpd, W, W, [&](uint32_t d, const Hit& c) {
      const bool in_y = fabsf(c.y - ypd) <= W, in_z = fabsf(c.z - zpd) <= W;
      my[min(nc, kNfCand) * kNfThreads] = (uint16_t)(d - (uint32_t)Bd.first);
      nc += in_y & in_z ? 1 : 0;
    });
    const float sy = sigma_y(K, zh), sz = sigma_z(K, zh);
    const float wy = 1.0f / (1.5f * (sy * sy));
    const float wz = 1.0f / (1.5f * (sz * sz));
    // down hit d with the listed up hits, WB records per memory round trip (the
    // last one again past the end: a pair offered twice changes nothing)
    auto pair_listed = [&](uint32_t d, const Hit& hd) {
      for (int k0 = 0; k0 < nu; k0 += WB) {
        uint32_t uu[WB];
        Hit hu[WB];
#pragma unroll
        for (int v = 0; v < WB; ++v) {
          uu[v] = (uint32_t)Bu.first + my[min(k0 + v, nu - 1) * kNfThreads];
          hu[v] = S.hit[uu[v]];
        }
#pragma unroll
        for (int v = 0; v < WB; ++v)
          best.offer(nf_metric(hd.y, hd.z, hu[v].y, hu[v].z, yh, zh, f, wy, wz), hd.id, hu[v].id,
                     (int32_t)d, (int32_t)uu[v]);
      }
    };
    if (nc <= kNfCand) {
      for (int i = nu; i < nc; ++i) {
        const uint32_t d = (uint32_t)Bd.first + my[i * kNfThreads];
        pair_listed(d, S.hit[d]);
      }
    } else if (nu <= kNfCand) {
      for_window_hits<WB>(Bd, bod, S.hit, ypd, zpd, W, W, [&](uint32_t d, const Hit& hd) {
        if (fabsf(hd.y - ypd) <= W && fabsf(hd.z - zpd) <= W) pair_listed(d, hd);
      });
    } else {
      for_window_hits<WB>(Bd, bod, S.hit, ypd, zpd, W, W, [&](uint32_t d, const Hit& hd) {
        if (!(fabsf(hd.y - ypd) <= W && fabsf(hd.z - zpd) <= W)) return;
        for_window_hits<WB>(Bu, bou, S.hit, ypu, zpu, W, W, [&](uint32_t u, const Hit& c) {
          if (!(fabsf(c.y - ypu) <= W && fabsf(c.z - zpu) <= W)) return;
          best.offer(nf_metric(hd.y, hd.z, c.y, c.z, yh, zh, f, wy, wz), hd.id, c.id,
                     (int32_t)d, (int32_t)u);
        });
      });
    }
  }
  const bool ok = best.have && best.m <= K.nf_mmax;
  S.up[h] = ok ? best.u : -1;
  S.dn[h] = ok ? best.d : -1;
}

// The hits of sectors [g0, g0 + ns) as one flat sequence (lane per hit, so
// every wave is full whatever the rows' sizes): blocks are dealt
// round-robin over the 8 XCDs, and the blocks of XCD x stride over the x-th
// contiguous eighth of the hits, so the rows r-1, r+1 its lanes read stay
// in its L2.
template <int WB>
__global__ void __launch_bounds__(kNfThreads, WB == 4 ? 6 : 1) k_neighbours(Slot S, DevConst K, int g0, int ns) {
  __shared__ uint16_t cand[(kNfCand + 1) * kNfThreads];
  const uint32_t h_begin = S.row_off[g0 * kRows];
  const uint32_t h_end = S.row_off[(g0 + ns) * kRows];
  const uint32_t x = blockIdx.x % 8u, nbx = gridDim.x / 8u;
  const uint32_t per = (h_end - h_begin + 7u) / 8u;
  const uint32_t c0 = h_begin + x * per;
  const uint32_t c1 = min(h_end, c0 + per);
  for (uint32_t h = c0 + (blockIdx.x / 8u) * kNfThreads + threadIdx.x; h < c1; h += nbx * kNfThreads)
    nf_hit<WB>(S, K, h, cand + threadIdx.x);
}

void launch_neighbours(int wb, int blocks, hipStream_t st, const Slot& S, const DevConst& K, int g0,
                       int ns) {
  switch (wb) {
    case 2: k_neighbours<2><<<blocks, kNfThreads, 0, st>>>(S, K, g0, ns); break;
    case 8: k_neighbours<8><<<blocks, kNfThreads, 0, st>>>(S, K, g0, ns); break;
    default: k_neighbours<4><<<blocks, kNfThreads, 0, st>>>(S, K, g0, ns); break;
  }
}

// Head of a cleaned chain of >= n_min_chain hits (no cleaned down link; the
// cleaned up links from h reach n_min_chain hits in all), from the links of
// a3 only: a link is cleaned when it is mutual.
__device__ __forceinline__ bool is_start(const Slot& S, uint32_t h, int n_min_chain, int32_t& uc,
                                         int32_t& dc) {
  const int32_t u = S.up[h], d = S.dn[h];
  uc = (u >= 0 && S.dn[u] == (int32_t)h) ? u : -1;
  dc = (d >= 0 && S.up[d] == (int32_t)h) ? d : -1;
  if (uc < 0 || dc >= 0) return false;
  int n = 2;
  for (int32_t k = uc; n < n_min_chain; ++n) {
    const int32_t kk = S.up[k];
    if (kk < 0 || S.dn[kk] != k) break;
    k = kk;
  }
  return n >= n_min_chain;
}

// a4: keep a link only if it is mutual; count the start hits of each row.
// Also clears the hit weights used by the tracklet selection.  One wave per
// row (rows hold ~100 hits), 64 hits at a time.
__global__ void __launch_bounds__(256) k_clean_rows(Slot S, int g0, int ns, int n_min_chain) {
  const int lane = threadIdx.x & 63;
  const int nwaves = (int)(gridDim.x * blockDim.x / 64);
  const int nr = ns * kRows;
  for (int v = (int)((blockIdx.x * blockDim.x + threadIdx.x) / 64); v < nr; v += nwaves) {
    const int sr = g0 * kRows + v;
    const uint32_t h0 = S.row_off[sr], h1 = S.row_off[sr + 1];
    uint32_t count = 0;
    for (uint32_t base = h0; base < h1; base += 64) {
      const uint32_t h = base + lane;
      bool start = false;
      if (h < h1) {
        int32_t uc, dc;
        start = is_start(S, h, n_min_chain, uc, dc);
        S.hit[h].upc = uc;
        S.dnc[h] = start ? kStartHit : dc;
        S.weight[h] = 0u;
      }
      count += (uint32_t)__popcll(__ballot(start));
    }
    if (lane == 0) S.row_nstart[sr] = count;
  }
}

// a4: write the start hits (marked by k_clean_rows) in (sector, row, position)
// order at the offsets given by the scan of the per-row counts over the
// launched sector range.  One wave per row, as in k_clean_rows.
__global__ void __launch_bounds__(256) k_start_write(Slot S, int g0, int ns) {
  const int lane = threadIdx.x & 63;
  const int nwaves = (int)(gridDim.x * blockDim.x / 64);
  const int nr = ns * kRows;
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int v = (int)((blockIdx.x * blockDim.x + threadIdx.x) / 64); v < nr; v += nwaves) {
    const int sr = g0 * kRows + v;
    const uint32_t h0 = S.row_off[sr], h1 = S.row_off[sr + 1];
    uint32_t out = S.tl_base[g0] + S.row_nstart[sr];
    for (uint32_t base = h0; base < h1; base += 64) {
      const uint32_t h = base + lane;
      const bool start = h < h1 && S.dnc[h] == kStartHit;
      const unsigned long long m = __ballot(start);
      if (start) {
        const uint32_t k = out + (uint32_t)__popcll(m & below);
        S.start_hit[k] = (int32_t)h;
        S.start_sr[k] = sr;
      }
      out += (uint32_t)__popcll(m);
    }
  }
}

}  // namespace tpc
