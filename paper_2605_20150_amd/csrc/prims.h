// Device-wide exclusive scan and stable LSD radix sort for wave64 (gfx950).
//
// Scan: reduce-then-scan over tiles of 4096 elements (256 lanes x 16
// consecutive items, moved in 16-byte pieces when the arrays are 16-byte
// aligned); with at most 1024 tiles each tile adds up its
// predecessors' sums itself, else one workgroup scans the tile sums.
// Radix sort: 8-bit digits; per tile 256-bin LDS histograms (one per wave,
// added at the end), a bin-major scan of the per-tile histograms, then a
// stable scatter whose in-tile ranks
// come from ballot-based peer masks (a wave sees 64 consecutive keys per
// round, so rank = keys of the same digit in earlier waves + earlier rounds +
// lower lanes).  Equal keys keep their input order, which is what makes the
// (tile, depth, pidx) order of the binning total.
#pragma once

#include "common.h"

namespace tide {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;  // 4096

constexpr int kSortThreads = 256;
constexpr int kSortWaves = kSortThreads / kWave;       // 4
constexpr int kSortRounds = 16;
constexpr int kSortTile = kSortThreads * kSortRounds;  // 4096
constexpr int kXcds = 8;                               // workgroup b starts on XCD b % 8
constexpr int64_t kRadixMaxGrid = 8192;                // radix histogram workgroups at most

// ------------------------------------------------------------------ scan
// Input functors: value of element i as u32; load4 reads elements i..i+3
// with one 16-byte load (i a multiple of 4, used only when aligned() holds).
__device__ inline uint4 ld4(const uint32_t* p) { return *reinterpret_cast<const uint4*>(p); }
struct ArrayIn {
  const uint32_t* a;
  __device__ uint32_t operator()(int64_t i) const { return a[i]; }
  __device__ void load4(int64_t i, uint32_t* v) const {
    const uint4 q = ld4(a + i);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  }
  bool aligned() const { return ((uintptr_t)a & 15) == 0; }
};
struct NonzeroIn {
  const uint32_t* a;
  __device__ uint32_t operator()(int64_t i) const { return a[i] != 0u ? 1u : 0u; }
  __device__ void load4(int64_t i, uint32_t* v) const {
    const uint4 q = ld4(a + i);
    v[0] = q.x != 0u; v[1] = q.y != 0u; v[2] = q.z != 0u; v[3] = q.w != 0u;
  }
  bool aligned() const { return ((uintptr_t)a & 15) == 0; }
};

// Output sinks: element i with exclusive prefix `off` and value v; store4
// writes elements i..i+3 (as load4).
struct OffsetsOut {   // out[i] = off
  uint32_t* out;
  __device__ void operator()(int64_t i, uint32_t off, uint32_t) const { out[i] = off; }
  __device__ void store4(int64_t i, const uint32_t* off, const uint32_t*) const {
    *reinterpret_cast<uint4*>(out + i) = make_uint4(off[0], off[1], off[2], off[3]);
  }
  bool aligned() const { return ((uintptr_t)out & 15) == 0; }
};

// out[i] = off, and mark[b] = i for every multiple of 2^kMarkShift that falls in
// [off, off + v): where a walk over equal pieces of the flattened lists starts.
// mark[0, n_mark) only.
constexpr int kMarkShift = 6;
struct OffsetsMarkOut {
  uint32_t* out;
  uint32_t* mark;
  uint32_t n_mark;
  __device__ void marks(int64_t i, uint32_t off, uint32_t v) const {
    const uint64_t end = (uint64_t)off + v;
    uint64_t b = ((uint64_t)off + ((1u << kMarkShift) - 1)) >> kMarkShift;
    for (; (b << kMarkShift) < end && b < n_mark; ++b) mark[b] = (uint32_t)i;
  }
  __device__ void operator()(int64_t i, uint32_t off, uint32_t v) const {
    out[i] = off;
    marks(i, off, v);
  }
  __device__ void store4(int64_t i, const uint32_t* off, const uint32_t* v) const {
    *reinterpret_cast<uint4*>(out + i) = make_uint4(off[0], off[1], off[2], off[3]);
    for (int k = 0; k < 4; ++k) marks(i + k, off[k], v[k]);
  }
  bool aligned() const { return ((uintptr_t)out & 15) == 0; }
};

// Extras written by whichever block holds the total: a u32 copy of it,
// end[n] = total (the closing offset of an offsets array), and a copy of
// copy_n u64 words from copy_src (read after the total is stored, so it may
// include it) to copy_dst (say, pinned host memory the host reads after an
// event: no copy kernel needed).
struct ScanTail {
  uint32_t* total32 = nullptr;
  uint32_t* end = nullptr;
  const unsigned long long* copy_src = nullptr;
  unsigned long long* copy_dst = nullptr;
  int copy_n = 0;
};

// Element counts: n_max bounds the launch; when d_n is given the kernels
// read the actual count from device memory (n = min(n_max, *d_n)), which
// lets a pipeline size its grids without a host round trip.
__device__ inline int64_t dev_count(int64_t n_max, const unsigned long long* d_n) {
  if (!d_n) return n_max;
  const int64_t n = (int64_t)*d_n;
  return n < n_max ? n : n_max;
}

// A thread's kScanItems consecutive elements: 16-byte loads when kVec and
// the whole run lies below n, else one element at a time (zero past n).
template <bool kVec, typename In>
__device__ inline void scan_items(const In& in, int64_t base, int64_t n, uint32_t* v) {
  if (kVec && base + kScanItems <= n) {
#pragma unroll
    for (int j = 0; j < kScanItems; j += 4) in.load4(base + j, v + j);
  } else {
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) v[k] = (base + k < n) ? in(base + k) : 0u;
  }
}

template <typename In, bool kVec>
__global__ void __launch_bounds__(kScanThreads) k_scan_reduce(In in, int64_t n_max, const unsigned long long* d_n,
                                                              unsigned long long* partial) {
  const int64_t n = dev_count(n_max, d_n);
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  scan_items<kVec>(in, base, n, v);
  unsigned long long s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) s += v[k];
  s = wave_sum(s);
  __shared__ unsigned long long ws[kScanThreads / kWave];
  if (__lane_id() == 0) ws[threadIdx.x / kWave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int w = 0; w < kScanThreads / kWave; ++w) t += ws[w];
    partial[blockIdx.x] = t;
  }
}

// One workgroup scans partial[0..nb) in place (exclusive) and writes the
// total and the tail (n as for dev_count).
__global__ void __launch_bounds__(1024) k_scan_partials(unsigned long long* partial, int64_t nb,
                                                        unsigned long long* total, ScanTail tail, int64_t n_max,
                                                        const unsigned long long* d_n);

__device__ inline void write_tail(const ScanTail& tail, unsigned long long t, int64_t n) {
  if (tail.total32) *tail.total32 = (uint32_t)t;
  if (tail.end) tail.end[n] = (uint32_t)t;
  for (int k = 0; k < tail.copy_n; ++k) tail.copy_dst[k] = tail.copy_src[k];
}

// Where a block of the down-sweep gets the sum of the blocks before it from.
//   kScanned  partial holds the scan of the blocks' sums;
//   kSums     partial holds the blocks' sums, and each block adds up its
//             predecessors' itself (one launch fewer; at most 1024 blocks);
//   kSelf     no sums: each block reads its predecessors' elements itself, for
//             at most kScanSelfBlocks blocks.  A launch fewer; the elements must
//             not be written over by the scan.  Five blocks (reduce + down -> one
//             kernel, us): active rows 2.6 + 3.6 -> 3.1, instance offsets 4.6 +
//             6.1 -> 7.3, visible pairs 3.0 + 5.9 -> 8.3.  A predecessor adds
//             four 16-byte loads per thread; past eight the launch is cheaper.
// The first block writes the total (kSelf: the last one).
enum ScanFrom { kScanned, kSums, kSelf };
constexpr int64_t kScanSelfBlocks = 8;

// The sum of the elements of the blocks before this one, given to every thread
// (wt: one word per wave; synchronises).
template <bool kVec, typename In>
__device__ inline unsigned long long sum_self(const In& in, int64_t n, unsigned long long* wt) {
  const int64_t mine = (int64_t)blockIdx.x * kScanTile, lim = mine < n ? mine : n;
  unsigned long long s = 0;
  int64_t j = 4 * threadIdx.x;
#pragma unroll 4
  for (; j + 4 <= lim; j += 4 * kScanThreads) {
    uint32_t v[4];
    if (kVec) {
      in.load4(j, v);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = in(j + k);
    }
    s += (unsigned long long)v[0] + v[1] + v[2] + v[3];
  }
  for (; j < lim; ++j) s += in(j);   // one thread's last group, where n cuts it
  s = wave_sum(s);
  if (__lane_id() == 0) wt[threadIdx.x / kWave] = s;
  __syncthreads();
  unsigned long long t = 0;
#pragma unroll
  for (int q = 0; q < kScanThreads / kWave; ++q) t += wt[q];
  return t;
}

template <typename In, ScanFrom kFrom, typename Out, bool kVec>
__global__ void __launch_bounds__(kScanThreads) k_scan_down(In in, int64_t n_max, const unsigned long long* d_n,
                                                            const unsigned long long* partial,
                                                            Out out, int64_t nb,
                                                            unsigned long long* total, ScanTail tail) {
  const int64_t n = dev_count(n_max, d_n);
  __shared__ unsigned long long bpre[kScanThreads / kWave + 1];
  if (kFrom == kSums) {
    // predecessors' sums (and, in block 0, all the sums for the total)
    const int64_t upto = blockIdx.x == 0 ? nb : (int64_t)blockIdx.x;
    unsigned long long a = 0;
    for (int64_t q = threadIdx.x; q < upto; q += kScanThreads) a += partial[q];
    a = wave_sum(a);
    if (__lane_id() == 0) bpre[threadIdx.x / kWave] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long t = 0;
      for (int q = 0; q < kScanThreads / kWave; ++q) t += bpre[q];
      if (blockIdx.x == 0) {
        *total = t;
        write_tail(tail, t, n);
      }
      bpre[kScanThreads / kWave] = blockIdx.x == 0 ? 0ull : t;
    }
    __syncthreads();
  }
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  scan_items<kVec>(in, base, n, v);
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) s += v[k];
  unsigned long long bp;
  if (kFrom == kSelf)
    bp = sum_self<kVec>(in, n, bpre);
  else
    bp = kFrom == kSums ? bpre[kScanThreads / kWave] : partial[blockIdx.x];
  // exclusive scan of the 256 thread sums
  const uint32_t inc = wave_incl_scan(s);
  __shared__ uint32_t wtot[kScanThreads / kWave];
  __shared__ unsigned long long wall[kFrom == kSelf ? kScanThreads / kWave : 1];   // the total needs more than 32 bits
  const int w = threadIdx.x / kWave;
  if (__lane_id() == kWave - 1) wtot[w] = inc;
  if (kFrom == kSelf && blockIdx.x == nb - 1) {
    unsigned long long a = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) a += v[k];
    a = wave_sum(a);
    if (__lane_id() == 0) wall[kFrom == kSelf ? w : 0] = a;
  }
  __syncthreads();
  uint32_t wpre = 0;
  for (int q = 0; q < w; ++q) wpre += wtot[q];
  uint32_t run = (uint32_t)bp + wpre + inc - s;
  if (kFrom == kSelf && blockIdx.x == nb - 1 && threadIdx.x == 0) {
    unsigned long long t = bp;
    for (int q = 0; q < kScanThreads / kWave; ++q) t += wall[kFrom == kSelf ? q : 0];
    *total = t;
    write_tail(tail, t, n);
  }
  if (kVec && base + kScanItems <= n) {
    uint32_t o[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      o[k] = run;
      run += v[k];
    }
#pragma unroll
    for (int j = 0; j < kScanItems; j += 4) out.store4(base + j, o + j, v + j);
  } else {
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      if (base + k < n) out(base + k, run, v[k]);
      run += v[k];
    }
  }
}

// Exclusive scan of in(0..n) into the sink out; total (u64, device)
// receives the sum, and the tail its extras.  partial needs
// ceil(n_max/4096) u64 entries; d_n as for dev_count.  in_place: the sink
// writes over the elements.
template <typename In, typename Out>
inline void scan_to(In in, int64_t n, Out out, unsigned long long* partial, unsigned long long* total,
                    hipStream_t st, const unsigned long long* d_n, ScanTail tail, bool in_place) {
  const int64_t nb = ceil_div(n > 0 ? n : 1, kScanTile);
  const bool vec = in.aligned() && out.aligned();
  const dim3 grid((uint32_t)nb), block(kScanThreads);
  if (nb <= kScanSelfBlocks && !in_place) {
    auto down = vec ? k_scan_down<In, kSelf, Out, true> : k_scan_down<In, kSelf, Out, false>;
    hipLaunchKernelGGL(down, grid, block, 0, st, in, n, d_n, (const unsigned long long*)partial, out, nb, total, tail);
    return;
  }
  auto reduce = vec ? k_scan_reduce<In, true> : k_scan_reduce<In, false>;
  hipLaunchKernelGGL(reduce, grid, block, 0, st, in, n, d_n, partial);
  if (nb <= 1024) {
    auto down = vec ? k_scan_down<In, kSums, Out, true> : k_scan_down<In, kSums, Out, false>;
    hipLaunchKernelGGL(down, grid, block, 0, st, in, n, d_n, (const unsigned long long*)partial, out, nb, total, tail);
    return;
  }
  hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(1024), 0, st, partial, nb, total, tail, n, d_n);
  auto down = vec ? k_scan_down<In, kScanned, Out, true> : k_scan_down<In, kScanned, Out, false>;
  hipLaunchKernelGGL(down, grid, block, 0, st, in, n, d_n, (const unsigned long long*)partial, out, nb, total, tail);
}

// Exclusive scan into an offsets array (which may be the elements' own).
inline void scan_exclusive(ArrayIn in, int64_t n, uint32_t* out, unsigned long long* partial,
                           unsigned long long* total, hipStream_t st, const unsigned long long* d_n = nullptr,
                           ScanTail tail = ScanTail{}) {
  scan_to(in, n, OffsetsOut{out}, partial, total, st, d_n, tail, in.a == out);
}

inline size_t scan_partial_count(int64_t n) { return (size_t)ceil_div(n > 0 ? n : 1, kScanTile); }

// The entry that element e of a flattened list of lists falls in: the largest
// s in [0, n) with off[s] <= e (off ascending, off[0] <= e), for a whole wave
// with the same arguments.  64 candidates a round, so five rounds reach 2^30
// entries; ends and stays in bounds whatever off holds.
__device__ inline uint32_t pair_of(const uint32_t* __restrict__ off, uint32_t n, uint32_t e) {
  const uint32_t lane = __lane_id();
  uint32_t lo = 0, hi = n;   // off[lo] <= e, and off[hi] > e where hi < n
  while (hi - lo > 1) {
    const uint32_t step = (hi - lo + kWave - 1) / kWave;
    const uint32_t d = lane * step;
    const bool in = d < hi - lo && (lane == 0 || off[lo + d] <= e);
    const uint32_t top = 63 - __builtin_clzll(__ballot(in));   // lane 0 always counts
    lo += top * step;
    hi = hi - lo > step ? lo + step : hi;
  }
  return lo;
}

// ------------------------------------------------------------- radix sort
inline size_t radix_hist_count(int64_t n) { return 256 * (size_t)ceil_div(n > 0 ? n : 1, kSortTile); }

// Adds this lane's run (digit d, count c) to the wave's bins: one add for
// the whole wave when every lane holds the same digit (the top digits of
// sorted or narrow-range keys), else one LDS atomic per lane.
__device__ __forceinline__ void hist_add(uint32_t* hw, uint32_t d, uint32_t c) {
  const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
  if (__all(d == d0)) {
    const uint32_t t = wave_sum(c);
    if (__lane_id() == 0) atomicAdd(&hw[d0], t);   // atomic: other lanes' earlier runs may add to it too
  } else {
    atomicAdd(&hw[d], c);
  }
}

// Shared LDS of a sort tile's ranking and scatter (tiles of 64 W R keys:
// W waves of R rounds).
template <int R, int W = kSortWaves>
struct TileLds {
  uint32_t wcnt[W][256];
  uint32_t gofs[256], lstart[256], wsum[4];
  alignas(16) uint32_t stage[kWave * W * R];   // the tile's keys, then its values
};

// A tile's phases are bound by the vector instructions they issue (208 per 64 keys
// and pass in the first form, 101 now; k_radix_scatter has the times).  So:
//   - kFull: the tile is full (its m elements are 64 W R), no lane is masked;
//   - indices are 32 bits from the tile's first element;
//   - the lanes of one digit are found by 8 ballots, each taking a bit's sign
//     extension, a comparison and one three-operand instruction per half;
//   - mbcnt gives the lanes below and adds the wave's earlier count.

// Ranks the keys of the tile (its elements from keys, m of them) by digit
// (key >> shift) & 255: wave w holds R rounds of 64 consecutive keys; rank[r] is
// the key's rank among the keys of its digit held by the wave in earlier rounds
// and lower lanes, and L.wcnt[w][d] ends as the wave's count of digit d.  Without
// vals the values are the indices, from first on.
// L.wcnt must be zero on entry; the caller synchronises afterwards.
template <bool kFull, int R, int W>
__device__ __forceinline__ void tile_rank(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals,
                                          uint32_t first, int m, int shift, TileLds<R, W>& L, uint32_t* key,
                                          uint32_t* val, uint32_t* rank) {
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = __lane_id();
  const uint32_t base = w * (kWave * R) + lane;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = base + r * kWave;
    key[r] = kFull || (int)i < m ? keys[i] : 0u;
  }
  if (vals) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t i = base + r * kWave;
      val[r] = kFull || (int)i < m ? vals[i] : 0u;
    }
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) val[r] = first + base + r * kWave;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool ok = kFull || (int)(base + r * kWave) < m;
    const uint32_t d = (key[r] >> shift) & 255u;
    const uint64_t on = kFull ? ~0ull : __ballot(ok);
    uint32_t plo = (uint32_t)on, phi = (uint32_t)(on >> 32);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      // the bit, in all places
      const uint32_t x = (uint32_t)__builtin_amdgcn_sbfe((int)key[r], (uint32_t)(shift + b), 1u);
      const uint64_t mk = __ballot(x != 0u);
      plo = __builtin_amdgcn_bitop3_b32(plo, (uint32_t)mk, x, 0x90);   // a & ~(b ^ c)
      phi = __builtin_amdgcn_bitop3_b32(phi, (uint32_t)(mk >> 32), x, 0x90);
    }
    uint32_t* const c = &L.wcnt[w][d];
    const uint32_t r0 = ok ? *c : 0u;
    rank[r] = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, r0));
    // the lowest lane of each digit group advances the wave's counter
    if (ok && rank[r] == r0) *c = r0 + (uint32_t)(__popc(plo) + __popc(phi));
  }
}

// Thread d < 256: turns L.wcnt[.][d] into the waves' offsets within digit
// d, writes the digit's start in the tile to L.lstart[d] and returns the
// tile's count of digit d (threads from 256 on return 0).  Synchronises.
template <int R, int W>
__device__ __forceinline__ uint32_t tile_digit_offsets(TileLds<R, W>& L) {
  const int d = threadIdx.x, w = threadIdx.x / kWave, lane = __lane_id();
  const bool dig = d < 256;
  uint32_t cnt = 0;
  if (dig) {
#pragma unroll
    for (int q = 0; q < W; ++q) {
      const uint32_t c = L.wcnt[q][d];
      L.wcnt[q][d] = cnt;
      cnt += c;
    }
  }
  const uint32_t inc = wave_incl_scan(cnt);
  if (dig && lane == kWave - 1) L.wsum[w] = inc;
  __syncthreads();
  if (dig) {
    uint32_t pre = 0;
    for (int q = 0; q < w; ++q) pre += L.wsum[q];
    L.lstart[d] = pre + inc - cnt;
  }
  return cnt;
}

// The ranked keys' places in (digit, rank) order, over rank[], and the keys in LDS
// at those places (L.lstart and L.wcnt must be visible; the caller synchronises).
template <bool kFull, int R, int W>
__device__ __forceinline__ void tile_stage(int m, int shift, TileLds<R, W>& L, const uint32_t* key, uint32_t* rank) {
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t base = w * (kWave * R) + __lane_id();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (kFull || (int)(base + r * kWave) < m) {
      const uint32_t dd = (key[r] >> shift) & 255u;
      rank[r] += L.lstart[dd] + L.wcnt[w][dd];
      L.stage[rank[r]] = key[r];
    }
  }
}

// Writes the tile out, the element in place j to L.gofs[digit] + j: its digit's
// start, less the digit's start in the tile, so a digit's run lands on consecutive
// addresses (L.gofs and the staged keys must be visible): out.key(position, key),
// then out.val(position, value).  Keys and values pass through the same LDS one
// after the other: 27 KB instead of 43 KB, so four workgroups run on a CU instead
// of three.
template <bool kFull, int R, int W, typename Out>
__device__ __forceinline__ void tile_write(int m, int shift, TileLds<R, W>& L, const uint32_t* val,
                                           const uint32_t* place, const Out& out) {
  uint32_t pos[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = threadIdx.x + r * (kWave * W);
    if (kFull || j < m) {
      const uint32_t k = L.stage[j];
      pos[r] = L.gofs[(k >> shift) & 255u] + (uint32_t)j;
      out.key(pos[r], k);
    }
  }
  __syncthreads();
  const int base = (int)(threadIdx.x / kWave) * (kWave * R) + (int)__lane_id();
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (kFull || base + r * kWave < m) L.stage[place[r]] = val[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = threadIdx.x + r * (kWave * W);
    if (kFull || j < m) out.val(pos[r], L.stage[j]);
  }
}

// The plain output of a pass: key and value, and with gather_src also
// gather_out[position] = gather_src[value].
struct PairsOut {
  uint32_t* keys;
  uint32_t* vals;
  const uint32_t* gather_src;
  uint32_t* gather_out;
  __device__ void key(uint32_t pos, uint32_t k) const { keys[pos] = k; }
  __device__ void val(uint32_t pos, uint32_t v) const {
    vals[pos] = v;
    if (gather_src) gather_out[pos] = gather_src[v];
  }
};

// Sorts (keys, vals) stably by bits [0, bits) of the key, 8 bits per pass.
// Input in (ka, va); with identity_vals the input values are taken to be
// the input indices and va is only used as storage.  Buffers (ka, va) and
// (kb, vb) ping-pong; the sorted result pointers are returned through
// *keys_res / *vals_res.  hist needs radix_hist_count(n) u32, partial
// scan_partial_count(radix_hist_count(n)) u64, total one u64 (two with d_n:
// then only the tiles that hold the device count's keys are counted,
// scanned and scattered, the second u64 holding the scan's length).  With
// gather_src, the last pass also writes gather_out[j] = gather_src[value j]
// for every sorted position j.  With xcd_order the scatter's tiles are
// assigned so that each XCD writes a contiguous eighth of them.
void radix_sort_pairs(uint32_t* ka, uint32_t* va, uint32_t* kb, uint32_t* vb, int64_t n, int bits,
                      bool identity_vals, uint32_t* hist, unsigned long long* partial,
                      unsigned long long* total, hipStream_t st, uint32_t** keys_res,
                      uint32_t** vals_res, const unsigned long long* d_n = nullptr,
                      const uint32_t* gather_src = nullptr, uint32_t* gather_out = nullptr,
                      bool xcd_order = false);

// ------------------------------------------------- one-sweep radix sort
// The same stable LSD sort with one kernel per 8-bit pass.  A first kernel
// counts every pass's digits over all keys at once (LDS bins per block,
// added to global counts with device-scope atomics).  Each pass kernel then
// ranks its tile of 64 W R keys as k_radix_scatter does, publishes its digit
// counts, and finds the counts of all earlier tiles by walking back over
// their published words until one holds an inclusive prefix (decoupled
// look-back, kOsWindow words per poll).  A tile publishes its own counts
// before it waits on anyone and workgroups start in index order on each
// XCD, so every wait ends; the walk also gives up after kOsSpinLimit polls
// of one word and sets an error word (the output is then wrong, but every
// write stays in bounds), so no kernel spins without end.  Used where the
// keys are few (the depth sort of the visible pairs): there the two
// launches per pass that it saves weigh more than the look-back.
//
// Control words: kOsCtlLen u32 that must read zero when the sort starts
// (an earlier kernel on the stream clears them).  The global digit counts
// are kept in kOsCopies copies (histogram block b adds to copy
// b % kOsCopies, which spreads the atomics), ctl[kOsCtlWords +
// (kOsMaxPasses c + p) 256 + d] being copy c of pass p's count of digit d.
constexpr int kOsCtlWords = 8;
constexpr int kOsMaxPasses = 4;
constexpr int kOsCopies = 8;
constexpr int kOsCtlLen = kOsCtlWords + kOsCopies * kOsMaxPasses * 256;
constexpr int kOsHistBlocks = 1024;
constexpr int kOsWindow = 4;
constexpr uint32_t kOsSpinLimit = 1u << 20;

struct OsWork {
  uint32_t* ctl;                  // kOsCtlLen u32, zero at the start
  unsigned long long* status;     // onesweep_status_count(n, passes)
  uint32_t* err;                  // set to nonzero if a look-back gave up
};

// Look-back words of a sort of n keys in tiles of tile_keys keys.
inline size_t onesweep_status_count(int64_t n, int passes, int64_t tile_keys) {
  return (size_t)passes * 256 * (size_t)ceil_div(n > 0 ? n : 1, tile_keys);
}

// The sort itself: onesweep_sort_pairs in onesweep.h.

}  // namespace tide
