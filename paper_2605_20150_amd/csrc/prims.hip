// Non-template parts of the scan and radix sort (see prims.h).
#include "prims.h"

namespace tide {

__global__ void __launch_bounds__(1024) k_scan_partials(unsigned long long* partial, int64_t nb,
                                                        unsigned long long* total, ScanTail tail, int64_t n_max,
                                                        const unsigned long long* d_n) {
  __shared__ unsigned long long wtot[1024 / kWave];
  __shared__ unsigned long long carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  const int lane = __lane_id(), w = threadIdx.x / kWave;
  for (int64_t b0 = 0; b0 < nb; b0 += 1024) {
    const int64_t i = b0 + threadIdx.x;
    const unsigned long long x = i < nb ? partial[i] : 0ull;
    unsigned long long inc = x;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const unsigned long long y = __shfl_up(inc, off, kWave);
      if (lane >= off) inc += y;
    }
    if (lane == kWave - 1) wtot[w] = inc;
    __syncthreads();
    unsigned long long pre = carry;
    for (int q = 0; q < w; ++q) pre += wtot[q];
    if (i < nb) partial[i] = pre + inc - x;
    __syncthreads();
    if (threadIdx.x == 1023) carry = pre + inc;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *total = carry;
    write_tail(tail, carry, dev_count(n_max, d_n));
  }
}

// Per-tile digit histogram, digit-major for the scan or, by_tile, a tile's 256
// counts together for scatters that add the counts up themselves.  Each wave
// counts into bins of its own, a thread takes four consecutive keys per load (16 bytes when kVec: the keys
// are 16-byte aligned) and adds equal neighbouring digits as one run, and the
// waves' bins are added at the end.  Workgroup b takes tiles b, b + G, ...
// (G the grid), so a grid sized for a large capacity costs little when the
// count on the device is small.
template <bool kVec>
__global__ void __launch_bounds__(kSortThreads) k_radix_hist(const uint32_t* keys, int64_t n_max,
                                                             const unsigned long long* d_n, int shift,
                                                             uint32_t* ghist, int64_t nb,
                                                             unsigned long long* nscan, int by_tile) {
  const int64_t n = dev_count(n_max, d_n);
  // with the count on the device, only its tiles count (the layout's stride
  // is their number, and the scan reads its length from nscan)
  const int64_t nba = d_n ? (n + kSortTile - 1) / kSortTile : nb;
  if (nscan && blockIdx.x == 0 && threadIdx.x == 0) *nscan = 256ull * (unsigned long long)nba;
  __shared__ uint32_t h[kSortWaves][256];
  uint32_t* hw = h[threadIdx.x / kWave];
  for (int64_t tile = blockIdx.x; tile < nba; tile += gridDim.x) {
    for (int k = threadIdx.x; k < kSortWaves * 256; k += kSortThreads) (&h[0][0])[k] = 0;
    __syncthreads();
    const int64_t base = tile * kSortTile;
#pragma unroll
    for (int r = 0; r < kSortRounds / 4; ++r) {
      const int64_t i = base + 4 * ((int64_t)r * kSortThreads + threadIdx.x);
      uint32_t d[4];
      int cnt = 0;   // valid keys of the four (a prefix)
      if (kVec && i + 4 <= n) {
        const uint4 q = *reinterpret_cast<const uint4*>(keys + i);
        d[0] = q.x; d[1] = q.y; d[2] = q.z; d[3] = q.w;
        cnt = 4;
      } else {
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          d[a] = i + a < n ? keys[i + a] : 0u;
          cnt += i + a < n ? 1 : 0;
        }
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) d[a] = (d[a] >> shift) & 255u;
      // runs of equal digits among the valid keys; lanes with none add 0 to
      // their first digit's bin
      uint32_t cur = d[0], run = cnt > 0 ? 1u : 0u;
#pragma unroll
      for (int a = 1; a < 4; ++a) {
        if (a < cnt) {
          if (d[a] == cur) {
            ++run;
          } else {
            atomicAdd(&hw[cur], run);
            cur = d[a];
            run = 1;
          }
        }
      }
      hist_add(hw, cur, run);
    }
    __syncthreads();
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) c += h[w][threadIdx.x];
    ghist[by_tile ? tile * 256 + threadIdx.x : (int64_t)threadIdx.x * nba + tile] = c;
    __syncthreads();
  }
}

// The scatter's 4096-key tiles as eight waves of eight rounds: a tile's
// ranking is a chain of rounds, and eight waves ran the two tile-sort passes
// over 14 M keys in 56.5 + 60.6 us against 61.4 + 66.8 us with four.  Vector
// instructions bound the pass: with 208 per 64 keys it took 815 us over 106.6 M
// keys (tiles of 8192 892 us, with 16 waves 1037 us), with values staged after the
// keys (27 KB of LDS instead of 43 KB, the CU's waves all in flight) 742 us, with
// 101 per 64 keys 489 us, 2.6 TB/s; over 13.2 M keys 63 and now 44 us.
constexpr int kScatterWaves = 8;
constexpr int kScatterRounds = kSortTile / (kWave * kScatterWaves);

// A digit's start for the tile: all counts of lower digits and the earlier
// tiles' of its own.  kScan: from the scan of the digit-major counts (gofs).
// Else gofs holds the counts themselves, tile-major (16-byte aligned), and every
// workgroup adds them up, a wave every eighth row and eight rows in flight: two
// launches fewer per pass, against 1 KB per tile read by every workgroup: at 133
// tiles (543k keys) reduce 4.6 + down 4.7 + scatter 10.2 us before, scatter 12.7
// us now.  Used up to kScatterSumTiles tiles, where it is eight rounds of loads.
constexpr int64_t kScatterSumTiles = 512;

template <bool kScan>
__global__ void __launch_bounds__(kWave * kScatterWaves) k_radix_scatter(const uint32_t* keys_in,
                                                                const uint32_t* vals_in, int64_t n_max,
                                                                const unsigned long long* d_n, int shift,
                                                                const uint32_t* gofs, int64_t nb,
                                                                uint32_t* keys_out, uint32_t* vals_out,
                                                                const uint32_t* gather_src, uint32_t* gather_out,
                                                                int xcd_order) {
  const int64_t n = dev_count(n_max, d_n);
  const int64_t nba = d_n ? (n + kSortTile - 1) / kSortTile : nb;   // the tiles that hold keys
  // with xcd_order, workgroup b (which starts on XCD x = b % 8) takes tile
  // x q + min(x, r) + b / 8 of the nba = 8 q + r tiles that hold keys, if
  // b / 8 is below XCD x's share (q, plus one for x < r; every such b is
  // below nba): each XCD sorts a contiguous eighth of the tiles, so the runs
  // of one digit that consecutive tiles write side by side meet in the same
  // L2.  (One workgroup per tile: taking several tiles per workgroup from a
  // smaller grid was slower, 576 against 663 us per pass over 101 M keys.)
  int64_t tile = blockIdx.x;
  if (xcd_order) {
    const int64_t q = nba / kXcds, r = nba % kXcds, x = blockIdx.x % kXcds, k = blockIdx.x / kXcds;
    if (k >= q + (x < r ? 1 : 0)) return;
    tile = x * q + (x < r ? x : r) + k;
  }
  if (tile >= nba) return;
  const int64_t b0 = tile * kSortTile;
  const int m = (int)(n - b0 < kSortTile ? n - b0 : kSortTile);   // elements of this tile
  __shared__ TileLds<kScatterRounds, kScatterWaves> L;
  for (int k = threadIdx.x; k < kScatterWaves * 256; k += kWave * kScatterWaves) (&L.wcnt[0][0])[k] = 0;
  if (kScan) {
    if (threadIdx.x < 256) L.gofs[threadIdx.x] = gofs[(int64_t)threadIdx.x * nba + tile];
  } else {
    // lane l of wave w: digits 4l .. 4l+3 of tiles w, w + 8, ...
    const int w = threadIdx.x / kWave, lane = __lane_id();
    uint4 tot = make_uint4(0, 0, 0, 0), pre = tot;
    auto add = [](uint4& a, const uint4& c, bool on) {
      a.x += on ? c.x : 0u; a.y += on ? c.y : 0u; a.z += on ? c.z : 0u; a.w += on ? c.w : 0u;
    };
    const uint4* g4 = reinterpret_cast<const uint4*>(gofs) + lane;   // a row is 64 of them
    constexpr int kRows = 8;
    for (int64_t b = w; b < nba; b += kRows * kScatterWaves) {
      uint4 c[kRows];
#pragma unroll
      for (int u = 0; u < kRows; ++u) {   // past the end the last row, not counted
        const int64_t row = b + u * kScatterWaves;
        c[u] = g4[(row < nba ? row : nba - 1) * (256 / 4)];
      }
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        const int64_t row = b + u * kScatterWaves;
        add(tot, c[u], row < nba);
        add(pre, c[u], row < tile);
      }
    }
    // the staging space is free until the keys are ranked
    static_assert(2 * kScatterWaves * 256 <= kSortTile, "both rows of counts per wave fit");
    uint32_t *st = L.stage, *sp = L.stage + kScatterWaves * 256;
    reinterpret_cast<uint4*>(st)[w * (256 / 4) + lane] = tot;
    reinterpret_cast<uint4*>(sp)[w * (256 / 4) + lane] = pre;
    __syncthreads();
    const int d = threadIdx.x;
    uint32_t t = 0, p = 0, inc = 0;
    if (d < 256) {
#pragma unroll
      for (int q = 0; q < kScatterWaves; ++q) {
        t += st[q * 256 + d];
        p += sp[q * 256 + d];
      }
      inc = wave_incl_scan(t);
      if (lane == kWave - 1) L.wsum[w] = inc;
    }
    __syncthreads();
    if (d < 256) {
      uint32_t lower = inc - t;
      for (int q = 0; q < w; ++q) lower += L.wsum[q];
      L.gofs[d] = lower + p;
    }
  }
  __syncthreads();
  uint32_t key[kScatterRounds], val[kScatterRounds], rank[kScatterRounds];
  const bool full = m == kSortTile;
  const uint32_t *kt = keys_in + b0, *vt = vals_in ? vals_in + b0 : nullptr;
  if (full)
    tile_rank<true>(kt, vt, (uint32_t)b0, m, shift, L, key, val, rank);
  else
    tile_rank<false>(kt, vt, (uint32_t)b0, m, shift, L, key, val, rank);
  __syncthreads();
  tile_digit_offsets(L);
  if (threadIdx.x < 256) L.gofs[threadIdx.x] -= L.lstart[threadIdx.x];
  __syncthreads();
  const PairsOut out{keys_out, vals_out, gather_src, gather_out};
  if (full) {
    tile_stage<true>(m, shift, L, key, rank);
    __syncthreads();
    tile_write<true>(m, shift, L, val, rank, out);
  } else {
    tile_stage<false>(m, shift, L, key, rank);
    __syncthreads();
    tile_write<false>(m, shift, L, val, rank, out);
  }
}

void radix_sort_pairs(uint32_t* ka, uint32_t* va, uint32_t* kb, uint32_t* vb, int64_t n, int bits,
                      bool identity_vals, uint32_t* hist, unsigned long long* partial,
                      unsigned long long* total, hipStream_t st, uint32_t** keys_res,
                      uint32_t** vals_res, const unsigned long long* d_n, const uint32_t* gather_src,
                      uint32_t* gather_out, bool xcd_order) {
  uint32_t *ki = ka, *vi = va, *ko = kb, *vo = vb;
  bool ident = identity_vals;
  const int64_t nb = ceil_div(n > 0 ? n : 1, kSortTile);
  // the histogram's grid: one workgroup per tile up to kRadixMaxGrid,
  // beyond that tiles per workgroup (the scatter keeps one per tile)
  const int64_t grid = nb < kRadixMaxGrid ? nb : kRadixMaxGrid;
  const bool scan = nb > kScatterSumTiles || ((uintptr_t)hist & 15) != 0;
  if (n > 0) {
    for (int shift = 0; shift < bits; shift += 8) {
      unsigned long long* nscan = d_n ? total + 1 : nullptr;
      auto count = ((uintptr_t)ki & 15) == 0 ? k_radix_hist<true> : k_radix_hist<false>;
      hipLaunchKernelGGL(count, dim3((uint32_t)grid), dim3(kSortThreads), 0, st, ki, n, d_n, shift, hist, nb, nscan,
                         scan ? 0 : 1);
      if (scan) scan_exclusive(ArrayIn{hist}, 256 * nb, hist, partial, total, st, nscan);
      const bool last = shift + 8 >= bits;
      auto scatter = scan ? k_radix_scatter<true> : k_radix_scatter<false>;
      hipLaunchKernelGGL(scatter, dim3((uint32_t)nb), dim3(kWave * kScatterWaves), 0, st, ki,
                         ident ? nullptr : vi, n,
                         d_n, shift, hist, nb, ko, vo, last ? gather_src : nullptr, last ? gather_out : nullptr,
                         xcd_order ? 1 : 0);
      ident = false;
      uint32_t* t = ki; ki = ko; ko = t;
      t = vi; vi = vo; vo = t;
    }
  }
  *keys_res = ki;
  *vals_res = vi;
}

}  // namespace tide
