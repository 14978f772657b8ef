// Prefetch-predictor MLP on gfx950: forward, backward and Adam.
//
// Every product runs on the bf16 matrix cores (v_mfma_f32_16x16x32_bf16,
// FP32 accumulation).  Weights are bf16.  An FP32 operand (activations,
// gradients) is split into hi = bf16(a) and lo = bf16(a - hi), and both
// halves are multiplied: W (hi + lo) keeps about 16 significant bits of a,
// against 8 for a plain bf16 cast, for twice the matrix-core work.  The
// weight-gradient product has FP32 on both sides and takes the three
// significant terms hi.hi + lo.hi + hi.lo.
//
// The product kernels share one accumulation order (one chain over K in
// chunks of 32, ascending, the halves in that order), so they give the same
// bits whatever the shape picks: k_gemm_direct feeds the matrix cores straight
// from memory, k_gemm stages square tiles through LDS, k_gemm_chain streams a
// long K past few outputs.
#include <cmath>

#include "common.h"

namespace tide {
namespace {

typedef __bf16 bf16x8 __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBK = 32;

// Nearest bfloat16 (ties to even) of an FP32 value, as its 16-bit pattern.
__device__ inline uint16_t bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// The same rounding of two values at once (v_cvt_pk_bf16_f32: the tests compare
// it with bf16_bits where both halves of a value are normal numbers; a NaN stays
// a NaN).
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// hi / lo halves of eight values, packed in order.  Three instructions per
// value; the integer rounding takes about twelve, which was most of the
// staging's time.
__device__ __forceinline__ void split8(const float (&f)[8], uint4& hi, uint4& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float a = f[2 * j], b = f[2 * j + 1];
    h[j] = bf16_pair(a, b);
    // exact differences
    l[j] = bf16_pair(a - __uint_as_float(h[j] << 16), b - __uint_as_float(h[j] & 0xffff0000u));
  }
  hi = make_uint4(h[0], h[1], h[2], h[3]);
  lo = make_uint4(l[0], l[1], l[2], l[3]);
}
// The low (high) 16-bit halves of x and y as one word, x's first.
__device__ __forceinline__ uint32_t low_halves(uint32_t x, uint32_t y) {
  return __builtin_amdgcn_perm(y, x, 0x05040100u);
}
__device__ __forceinline__ uint32_t high_halves(uint32_t x, uint32_t y) {
  return __builtin_amdgcn_perm(y, x, 0x07060302u);
}
__device__ __forceinline__ bf16x8 frag(const uint4& v) { return __builtin_bit_cast(bf16x8, v); }

enum AKind { kA_KC = 0, kA_MC = 1 };                 // FP32 A contiguous along K / along M
enum BKind { kB_WKC = 0, kB_WNC = 1, kB_FNC = 2 };   // bf16 W [n][k], bf16 W [k][n], FP32 X [k][n]
enum Epi { kE_BIAS = 0, kE_BIAS_RELU = 1, kE_MASK = 2, kE_STORE = 3 };
enum Major { kMajN = 0, kMajM = 1 };                 // the grid dimension spread over the XCDs

// ------------------------------------------------- products straight from memory
// C[m][n] = sum_k A[m][k] W[n][k] + bias[n] (ReLU with kE_BIAS_RELU), A FP32
// and W bf16, both contiguous along K.  A wave owns 16 MT x 16 NT outputs and
// loads each lane's eight operands of U chunks of K at once, so no LDS, no
// barrier and one memory latency per U chunks.  It is the kernel for the
// products that cannot fill the chip with LDS tiles: one row of poses
// (512 -> 65536, 67 MB of weights read once: 13.7 us, 4.9 TB/s) and the hidden
// layers (256 x 512 x 512: 7.6 us, 32 us with 64 x 64 tiles through LDS on 32
// workgroups).  14.8 and 8.7 us with every load behind its own bounds check.
// Requirements (checked by the host): K and the leading dimensions are
// multiples of 8 and the bases 16-byte aligned, so a load is wholly inside
// or wholly outside an operand.
template <int MT, int NT, int U, int EPI>
__global__ __launch_bounds__(256) void k_gemm_direct(const float* __restrict__ A, int64_t lda,
                                                     const uint16_t* __restrict__ W, int64_t ldw,
                                                     float* __restrict__ C, int64_t ldc,
                                                     const float* __restrict__ bias, int M, int N, int K) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r = lane & 15, kc = (lane >> 4) * 8;
  const int n0 = (blockIdx.x * 4 + w) * 16 * NT, m0 = blockIdx.y * 16 * MT;
  if (n0 >= N) return;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // rows past the edges read the last one (their outputs are not stored); k past
  // K, in the last round only, reads the last chunk for zeros
  const uint16_t* pw[NT];
  const float* pa[MT];
#pragma unroll
  for (int j = 0; j < NT; ++j) pw[j] = W + (int64_t)(n0 + 16 * j + r < N ? n0 + 16 * j + r : N - 1) * ldw;
#pragma unroll
  for (int i = 0; i < MT; ++i) pa[i] = A + (int64_t)(m0 + 16 * i + r < M ? m0 + 16 * i + r : M - 1) * lda;
  float4 a[U][MT][2];
  uint4 b[U][NT];
  auto fetch = [&](int k0, bool tail) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k1 = k0 + u * kBK + kc, k = !tail || k1 < K ? k1 : K - 8;
#pragma unroll
      for (int j = 0; j < NT; ++j) b[u][j] = *reinterpret_cast<const uint4*>(pw[j] + k);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        a[u][i][0] = reinterpret_cast<const float4*>(pa[i] + k)[0];
        a[u][i][1] = reinterpret_cast<const float4*>(pa[i] + k)[1];
      }
    }
    if (!tail) return;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = k0 + u * kBK + kc < K;
#pragma unroll
      for (int j = 0; j < NT; ++j)
        b[u][j] = make_uint4(in ? b[u][j].x : 0u, in ? b[u][j].y : 0u, in ? b[u][j].z : 0u, in ? b[u][j].w : 0u);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float4 x = a[u][i][h];
          a[u][i][h] = make_float4(in ? x.x : 0.f, in ? x.y : 0.f, in ? x.z : 0.f, in ? x.w : 0.f);
        }
    }
  };
  for (int k0 = 0; k0 < K; k0 += U * kBK) {
    if (k0 + U * kBK <= K)
      fetch(k0, false);
    else
      fetch(k0, true);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + u * kBK >= K) break;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const float f[8] = {a[u][i][0].x, a[u][i][0].y, a[u][i][0].z, a[u][i][0].w,
                            a[u][i][1].x, a[u][i][1].y, a[u][i][1].z, a[u][i][1].w};
        uint4 hi, lo;
        split8(f, hi, lo);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(hi), frag(b[u][j]), acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(lo), frag(b[u][j]), acc[i][j], 0, 0, 0);
        }
      }
    }
  }
  // accumulator lane layout: row = 4 (lane / 16) + e, column = lane % 16
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + 16 * i + 4 * (lane >> 4) + e, n = n0 + 16 * j + r;
        if (m >= M || n >= N) continue;
        float v = acc[i][j][e] + bias[n];
        if (EPI == kE_BIAS_RELU) v = fmaxf(v, 0.f);
        C[(int64_t)m * ldc + n] = v;
      }
}

// ------------------------------------------------------ products through LDS
// C[m][n] = sum_k A(m, k) B(k, n), then the epilogue:
//   kE_BIAS       C = acc + bias[n]
//   kE_BIAS_RELU  C = max(acc + bias[n], 0)
//   kE_MASK       C = mask[m][n] > 0 ? acc : 0   (ReLU adjoint)
//   kE_STORE      C = acc
// T x T outputs per 256-thread workgroup (four waves in
// a square, (T/2)^2 each), K staged KB (32 or 64) at a time through LDS as bf16
// rows [row][k], so that one 16-byte LDS read gives a lane its eight operands.
// Eight consecutive k of one row are a thread's staging unit: loaded (from
// an operand that is contiguous along the other index as eight coalesced
// loads, one per k, so the transposition costs nothing), rounded in
// registers and written with one conflict-free 16-byte LDS store.  The next
// K step's loads are in flight while the matrix cores work on this one, none
// of them behind a bounds check of its own: rows and k past the edges are read
// from inside and made zeros in the last step only.  T = 128 holds 64
// accumulators per lane and reads each operand half as often as T = 64; T = 32
// is for the products too small to fill the chip, where the staging of a
// workgroup is what it waits for.
// 256 x 512 -> 65536: forward 65 us in a training step and 57 us in scoring (115
// us with 64 x 64 tiles, integer rounding and no loads in flight), weight
// gradient 88 us (335 us, of which 62 us the bias gradient as a kernel of its
// own; 149 us with checked loads).
// Weight gradient 256 x 512 -> 512: 7.4 us (18.7 us with 64 x 64 tiles and
// checked loads, 11.8 us with the tiles alone).
//
// Grid: workgroup ids walk the MAJOR dimension eight at a time, so that the
// workgroups that share its operand tile run on one XCD and meet in its L2.
//
// db (kE_STORE with kA_MC only): the workgroups of the first tile column
// also add up their A rows over k, in FP32 and in k order (the bias
// gradient); the rows pass through LDS in FP32 for that.
//
// Requirements (checked by the host): the contiguous extent of every
// operand (K for kA_KC / kB_WKC, M for kA_MC, N for kB_WNC / kB_FNC) and
// every leading dimension are multiples of 8, and base pointers are 16-byte
// aligned.
template <int T, int KB, int AK, int BK, int EPI, int MAJOR>
__global__ __launch_bounds__(256) void k_gemm(const float* __restrict__ A, int64_t lda, const void* __restrict__ Bv,
                                              int64_t ldb, float* __restrict__ C, int64_t ldc,
                                              const float* __restrict__ bias, const float* __restrict__ mask,
                                              int64_t ldm, float* __restrict__ db, int M, int N, int K, int tm,
                                              int tn) {
  constexpr bool kSplitB = BK == kB_FNC;
  constexpr bool kSumA = AK == kA_MC && EPI == kE_STORE;
  constexpr int WT = T / 32;             // 16 x 16 tiles per wave and side
  constexpr int UN = T * KB / 8 / 256;   // staging units per thread and operand
  constexpr int LD = KB + 8;             // LDS row stride in bf16 (16-byte aligned rows, 4 banks apart)
  static_assert(KB == kBK || (AK == kA_MC && BK == kB_FNC), "deeper stages: operands that are not contiguous along k");
  __shared__ __attribute__((aligned(16))) uint16_t sAh[T][LD];
  __shared__ __attribute__((aligned(16))) uint16_t sAl[T][LD];
  __shared__ __attribute__((aligned(16))) uint16_t sBh[T][LD];
  __shared__ __attribute__((aligned(16))) uint16_t sBl[kSplitB ? T : 1][LD];
  __shared__ float sF[kSumA ? KB : 1][kSumA ? T : 1];

  // id = (major / 8) * 8 * minor-count + minor * 8 + major % 8
  const int n_minor = MAJOR == kMajN ? tm : tn, n_major = MAJOR == kMajN ? tn : tm;
  const int grp = blockIdx.x / (8 * n_minor), rem = blockIdx.x - grp * 8 * n_minor;
  const int major = grp * 8 + (rem & 7), minor = rem >> 3;
  if (major >= n_major) return;
  const int m0 = (MAJOR == kMajN ? minor : major) * T, n0 = (MAJOR == kMajN ? major : minor) * T;

  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wm = (w >> 1) * (T / 2), wn = (w & 1) * (T / 2);
  f32x4 acc[WT][WT];
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // unit u of this thread: row and first k within the tile.  Contiguous
  // along k: four units per row, neighbouring threads on one row.  Else
  // neighbouring threads on neighbouring rows (bf16 W: on row pairs).
  int a_row[UN], a_k[UN], b_row[UN], b_k[UN];
#pragma unroll
  for (int u = 0; u < UN; ++u) {
    const int x = t + u * 256;
    if (AK == kA_KC) { a_row[u] = x >> 2; a_k[u] = (x & 3) * 8; }
    else { a_row[u] = x % T; a_k[u] = (x / T) * 8; }
    if (BK == kB_WKC) { b_row[u] = x >> 2; b_k[u] = (x & 3) * 8; }
    else { b_row[u] = x % T; b_k[u] = (x / T) * 8; }
  }
  // kB_WNC: a unit is a row pair (2 x 8 values in eight dwords), one a
  // thread (T = 64: half the threads)
  const bool p_on = UN > 1 || t < 128;
  const int p_row = 2 * (t % (T / 2)), p_k = (t / (T / 2)) * 8;

  float av[UN][8];
  float bf[kSplitB ? UN : 1][8];
  uint4 bw[BK == kB_WKC ? UN : 1];
  uint32_t bp[BK == kB_WNC ? 8 : 1];
  float dsum = 0.f;
  const bool want_db = kSumA && n0 == 0;

  // Every load is issued whatever the edges (a guarded one costs its own branch
  // or waits): rows past M or N read the last one (their outputs are not
  // stored), k past K the last chunk or k, whose values become zeros.
  const float* pa[UN];
  const float* px[kSplitB ? UN : 1];
  const uint16_t* pw[BK == kB_WKC ? UN : 1];
#pragma unroll
  for (int u = 0; u < UN; ++u) {
    const int m = m0 + a_row[u] < M ? m0 + a_row[u] : M - 1, n = n0 + b_row[u] < N ? n0 + b_row[u] : N - 1;
    pa[u] = AK == kA_KC ? A + (int64_t)m * lda : A + m;
    if (BK == kB_WKC) pw[BK == kB_WKC ? u : 0] = static_cast<const uint16_t*>(Bv) + (int64_t)n * ldb;
    if (BK == kB_FNC) px[kSplitB ? u : 0] = static_cast<const float*>(Bv) + n;
  }
  // eight values of one row or column from k on; tail: k may pass K
  auto along_k = [&](const float* p, int k, bool tail, float (&v)[8]) {   // K and k are multiples of 8
    const bool in = !tail || k < K;
    const float4* q = reinterpret_cast<const float4*>(p + (in ? k : K - 8));
    const float4 x = q[0], y = q[1];
    v[0] = in ? x.x : 0.f; v[1] = in ? x.y : 0.f; v[2] = in ? x.z : 0.f; v[3] = in ? x.w : 0.f;
    v[4] = in ? y.x : 0.f; v[5] = in ? y.y : 0.f; v[6] = in ? y.z : 0.f; v[7] = in ? y.w : 0.f;
  };
  auto across_k = [&](const float* p, int64_t ld, int k, bool tail, float (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = p[(int64_t)(!tail || k + j < K ? k + j : K - 1) * ld];
    if (tail) {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = k + j < K ? v[j] : 0.f;
    }
  };
  auto fetch_from = [&](int k0, bool tail) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (AK == kA_KC)
        along_k(pa[u], k0 + a_k[u], tail, av[u]);
      else
        across_k(pa[u], lda, k0 + a_k[u], tail, av[u]);
      const int k = k0 + b_k[u];
      if (BK == kB_WKC) {
        const bool in = !tail || k < K;
        const uint4 x = *reinterpret_cast<const uint4*>(pw[BK == kB_WKC ? u : 0] + (in ? k : K - 8));
        bw[BK == kB_WKC ? u : 0] = make_uint4(in ? x.x : 0u, in ? x.y : 0u, in ? x.z : 0u, in ? x.w : 0u);
      } else if (BK == kB_FNC) {
        across_k(px[kSplitB ? u : 0], ldb, k, tail, bf[kSplitB ? u : 0]);
      }
    }
    if (BK == kB_WNC) {
      const uint16_t* W = static_cast<const uint16_t*>(Bv);
      const int n = n0 + p_row, k = k0 + p_k;
#pragma unroll
      for (int j = 0; j < 8; ++j)   // N is even: a pair is wholly inside or outside
        bp[BK == kB_WNC ? j : 0] = p_on && n < N && k + j < K
                       ? *reinterpret_cast<const uint32_t*>(W + (int64_t)(k + j) * ldb + n)
                       : 0u;
    }
  };
  auto fetch = [&](int k0) {
    if (k0 + KB <= K)
      fetch_from(k0, false);
    else
      fetch_from(k0, true);
  };
  auto stage = [&]() {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      uint4 hi, lo;
      split8(av[u], hi, lo);
      *reinterpret_cast<uint4*>(&sAh[a_row[u]][a_k[u]]) = hi;
      *reinterpret_cast<uint4*>(&sAl[a_row[u]][a_k[u]]) = lo;
      if (want_db) {
#pragma unroll
        for (int j = 0; j < 8; ++j) sF[kSumA ? a_k[u] + j : 0][kSumA ? a_row[u] : 0] = av[u][j];
      }
    }
    if (BK == kB_WKC) {
#pragma unroll
      for (int u = 0; u < UN; ++u)
        *reinterpret_cast<uint4*>(&sBh[b_row[u]][b_k[u]]) = bw[BK == kB_WKC ? u : 0];
    } else if (BK == kB_WNC) {
      if (p_on) {
        uint32_t e[4], o[4];   // the pair's even and odd row
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t x = bp[BK == kB_WNC ? 2 * j : 0], y = bp[BK == kB_WNC ? 2 * j + 1 : 0];
          e[j] = low_halves(x, y);
          o[j] = high_halves(x, y);
        }
        *reinterpret_cast<uint4*>(&sBh[p_row][p_k]) = make_uint4(e[0], e[1], e[2], e[3]);
        *reinterpret_cast<uint4*>(&sBh[p_row + 1][p_k]) = make_uint4(o[0], o[1], o[2], o[3]);
      }
    } else {
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        uint4 hi, lo;
        split8(bf[kSplitB ? u : 0], hi, lo);
        *reinterpret_cast<uint4*>(&sBh[b_row[u]][b_k[u]]) = hi;
        *reinterpret_cast<uint4*>(&sBl[kSplitB ? b_row[u] : 0][b_k[u]]) = lo;
      }
    }
  };

  fetch(0);
  for (int k0 = 0; k0 < K; k0 += KB) {
    stage();
    __syncthreads();
    if (k0 + KB < K) fetch(k0 + KB);
    if (want_db && t < T) {
#pragma unroll 8
      for (int j = 0; j < KB; ++j) dsum += sF[kSumA ? j : 0][kSumA ? t : 0];   // rows past K hold zeros
    }
    // matrix cores: lane holds row (lane % 16), k = 8 (lane / 16) .. +7 of a chunk of 32
#pragma unroll
    for (int c = 0; c < KB; c += kBK) {
      if (k0 + c >= K) break;
      const int r = lane & 15, kc = c + (lane >> 4) * 8;
      bf16x8 bh[WT], bl[kSplitB ? WT : 1];
#pragma unroll
      for (int j = 0; j < WT; ++j) {
        bh[j] = *reinterpret_cast<const bf16x8*>(&sBh[wn + 16 * j + r][kc]);
        if (kSplitB) bl[kSplitB ? j : 0] = *reinterpret_cast<const bf16x8*>(&sBl[kSplitB ? wn + 16 * j + r : 0][kc]);
      }
#pragma unroll
      for (int i = 0; i < WT; ++i) {
        const bf16x8 ah = *reinterpret_cast<const bf16x8*>(&sAh[wm + 16 * i + r][kc]);
        const bf16x8 al = *reinterpret_cast<const bf16x8*>(&sAl[wm + 16 * i + r][kc]);
#pragma unroll
        for (int j = 0; j < WT; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[j], acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh[j], acc[i][j], 0, 0, 0);
          if (kSplitB)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl[kSplitB ? j : 0], acc[i][j], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }

  // accumulator lane layout: row = 4 (lane / 16) + e, column = lane % 16
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + wm + 16 * i + 4 * (lane >> 4) + e;
        const int n = n0 + wn + 16 * j + (lane & 15);
        if (m >= M || n >= N) continue;
        float v = acc[i][j][e];
        if (EPI == kE_BIAS || EPI == kE_BIAS_RELU) v += bias[n];
        if (EPI == kE_BIAS_RELU) v = fmaxf(v, 0.f);
        if (EPI == kE_MASK) v = mask[(int64_t)m * ldm + n] > 0.f ? v : 0.f;
        C[(int64_t)m * ldc + n] = v;
      }
  if (want_db && t < T && m0 + t < M) db[m0 + t] = dsum;
}

// ------------------------------------------------------ few outputs, a long K
// C[m][n] = mask[m][n] > 0 ? sum_k G[m][k] W[k][n] : 0, G FP32 contiguous
// along K, W bf16 contiguous along N: the input gradient, whose K is the
// layer's output width (65536) while its outputs are batch x 512.  K is not
// split (the sums keep the order of the other kernels), so one chain of matrix
// instructions per output tile is a floor: 2048 chunks of two dependent ones,
// 74 us.  What bounds it above that is feeding the chain, so the roles are
// split: two waves a workgroup multiply (two 16 x 16 tiles each) and do nothing
// else, eight more hold two stages of 256 k in flight in registers, round G
// into its halves and transpose W on the way into LDS.  The tile is 16 x 64
// because 64 columns are whole 128-byte lines of W's rows (16 x 32 on twice
// the CUs measured 285 us).  Batch 256, 65536 -> 512: 215 us (64 x 64 tiles on
// 32 workgroups with a barrier per 32 k: 3980 us); its loads alone take 195 us,
// its staging alone 118 us, its products alone 142 us.
// Grid: super-tiles of 4 x 4 workgroups, one per XCD, that share G rows and W
// columns in its L2.
constexpr int kChK = 256, kChLd = kChK + 8;   // stage depth; LDS row stride of G in bf16 (rows 4 banks apart)
constexpr int kChM = 16, kChN = 64;
constexpr int kChSets = 2;
constexpr int kChMul = 2, kChFeed = 8;        // waves per role
constexpr int kChSup = 4;

__global__ __launch_bounds__(kWave * (kChMul + kChFeed)) void k_gemm_chain(
    const float* __restrict__ G, int64_t ldg, const uint16_t* __restrict__ W, int64_t ldw,
    const float* __restrict__ mask, int64_t ldm, float* __restrict__ C, int64_t ldc, int M, int N, int K, int tm, int tn,
    int sup_m) {
  __shared__ __attribute__((aligned(16))) uint16_t sAh[2][kChM][kChLd], sAl[2][kChM][kChLd], sB[2][kChN][kChK];
  const int inner = (blockIdx.x >> 3) % (kChSup * kChSup);
  const int sup = (blockIdx.x & 7) + 8 * (int)(blockIdx.x / (8 * kChSup * kChSup));
  const int im = (sup % sup_m) * kChSup + inner % kChSup, in = (sup / sup_m) * kChSup + inner / kChSup;
  if (im >= tm || in >= tn) return;
  const int m0 = im * kChM, n0 = in * kChN;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int stages = (K + kChK - 1) / kChK;
  // 16-byte unit g of W column n is kept at unit g ^ h(n): lanes that store
  // parts of columns 8 apart, and those that read a unit of neighbouring
  // columns, each meet all banks once
  auto at = [](int n, int k) {
    const int h = (((n >> 3) & 7) << 1) ^ ((n & 1) | (((n >> 1) & 3) << 2));
    return k ^ (h << 3);
  };

  // Two loops with the same barriers, one per role (in a common loop the
  // compiler carries one role's outstanding loads into the other's waits).
  if (w >= kChMul) {
    const int p = t - kWave * kChMul;   // 0..511
    // a thread's share of a stage: eight k of one G row, and four k of eight
    // W columns.  Every load is unconditional (a guarded one would make the
    // wait for the older stage's loads a wait for all of them): rows, columns
    // and stages past the end read the last ones; such rows and columns are
    // not stored, and k past the end is staged as zero.
    struct Regs {
      float4 a[2];
      uint4 b[4];
    } r[kChSets];
    const int g_row = p >> 5, g_k = (p & 31) * 8;
    const int w_n = (p & 7) * 8, w_k = (p >> 3) * 4;
    const float* gp = G + (int64_t)(m0 + g_row < M ? m0 + g_row : M - 1) * ldg;
    const uint16_t* wp = W + (n0 + w_n < N ? n0 + w_n : N - 8);   // N and K are multiples of 8
    auto fetch = [&](int s, Regs& q) {
      const int ka = s * kChK + g_k, kb = s * kChK + w_k;
      const float4* x = reinterpret_cast<const float4*>(gp + (ka < K ? ka : K - 8));
      q.a[0] = x[0];
      q.a[1] = x[1];
      const uint16_t* y = wp + (int64_t)(kb < K ? kb : K - 4) * ldw;
#pragma unroll
      for (int j = 0; j < 4; ++j) q.b[j] = *reinterpret_cast<const uint4*>(y + j * ldw);
    };
    auto stage = [&](int buf, int s, const Regs& q) {
      const float f[8] = {q.a[0].x, q.a[0].y, q.a[0].z, q.a[0].w, q.a[1].x, q.a[1].y, q.a[1].z, q.a[1].w};
      uint4 hi, lo;
      split8(f, hi, lo);
      const uint32_t c[4][4] = {{q.b[0].x, q.b[0].y, q.b[0].z, q.b[0].w}, {q.b[1].x, q.b[1].y, q.b[1].z, q.b[1].w},
                                {q.b[2].x, q.b[2].y, q.b[2].z, q.b[2].w}, {q.b[3].x, q.b[3].y, q.b[3].z, q.b[3].w}};
      uint2 e[4], o[4];   // k w_k .. w_k + 3 of columns w_n + 2 d and the next
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        e[d] = make_uint2(low_halves(c[0][d], c[1][d]), low_halves(c[2][d], c[3][d]));
        o[d] = make_uint2(high_halves(c[0][d], c[1][d]), high_halves(c[2][d], c[3][d]));
      }
      if ((s + 1) * kChK > K) {   // the last stage, cut by K
        if (s * kChK + g_k >= K) hi = lo = make_uint4(0u, 0u, 0u, 0u);
        if (s * kChK + w_k >= K) {
#pragma unroll
          for (int d = 0; d < 4; ++d) e[d] = o[d] = make_uint2(0u, 0u);
        }
      }
      *reinterpret_cast<uint4*>(&sAh[buf][g_row][g_k]) = hi;
      *reinterpret_cast<uint4*>(&sAl[buf][g_row][g_k]) = lo;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        *reinterpret_cast<uint2*>(&sB[buf][w_n + 2 * d][at(w_n + 2 * d, w_k)]) = e[d];
        *reinterpret_cast<uint2*>(&sB[buf][w_n + 2 * d + 1][at(w_n + 2 * d + 1, w_k)]) = o[d];
      }
    };
    const int last = stages - 1;
    auto upto = [&](int s) { return s < last ? s : last; };
#pragma unroll
    for (int q = 0; q < kChSets; ++q) fetch(upto(q), r[q]);
    stage(0, 0, r[0]);
    __syncthreads();
    for (int s = 0;; s += kChSets) {
#pragma unroll
      for (int q = 0; q < kChSets; ++q) {   // register sets and LDS buffers have fixed names
        fetch(upto(s + q + kChSets), r[q]);
        __builtin_amdgcn_sched_barrier(0);   // the loads go out before the older ones are waited for
        stage((q + 1) & 1, upto(s + q + 1), r[(q + 1) % kChSets]);
        __syncthreads();
        if (s + q + 1 >= stages) return;
      }
    }
  }

  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  const int row = lane & 15, kc = (lane >> 4) * 8, col = 32 * w + row;
  constexpr int kNc = kChK / kBK, kHalf = kNc / 2;
  auto load = [&](int buf, int c, bf16x8& ah, bf16x8& al, bf16x8& b0, bf16x8& b1) {
    ah = *reinterpret_cast<const bf16x8*>(&sAh[buf][row][c * kBK + kc]);
    al = *reinterpret_cast<const bf16x8*>(&sAl[buf][row][c * kBK + kc]);
    b0 = *reinterpret_cast<const bf16x8*>(&sB[buf][col][at(col, c * kBK + kc)]);
    b1 = *reinterpret_cast<const bf16x8*>(&sB[buf][col + 16][at(col + 16, c * kBK + kc)]);
  };
  auto multiply = [&](int buf, int s) {
    const int nc = K - s * kChK < kChK ? (K - s * kChK + kBK - 1) / kBK : kNc;
    if (nc == kNc) {
#pragma unroll
      for (int h = 0; h < kNc; h += kHalf) {
        // half of the stage's operands at a time, so the chains wait for LDS twice a stage
        bf16x8 ah[kHalf], al[kHalf], b0[kHalf], b1[kHalf];
#pragma unroll
        for (int c = 0; c < kHalf; ++c) load(buf, h + c, ah[c], al[c], b0[c], b1[c]);
#pragma unroll
        for (int c = 0; c < kHalf; ++c) {
          acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[c], b0[c], acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[c], b1[c], acc[1], 0, 0, 0);
          acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[c], b0[c], acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[c], b1[c], acc[1], 0, 0, 0);
        }
      }
      return;
    }
    for (int c = 0; c < nc; ++c) {
      bf16x8 ah, al, b0, b1;
      load(buf, c, ah, al, b0, b1);
      acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, b0, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, b1, acc[1], 0, 0, 0);
      acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, b0, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, b1, acc[1], 0, 0, 0);
    }
  };
  __syncthreads();
  for (int s = 0; s < stages; ++s) {
    multiply(s & 1, s);
    __syncthreads();
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int m = m0 + 4 * (lane >> 4) + e;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = n0 + col + 16 * j;
      if (m < M && n < N) C[(int64_t)m * ldc + n] = mask[(int64_t)m * ldm + n] > 0.f ? acc[j][e] : 0.f;
    }
  }
}

template <int T, int KB, int AK, int BK, int EPI, int MAJOR>
void launch_gemm(hipStream_t st, const float* A, int64_t lda, const void* B, int64_t ldb, float* C, int64_t ldc,
                 const float* bias, const float* mask, int64_t ldm, float* db, int M, int N, int K) {
  const int tm = (int)ceil_div(M, T), tn = (int)ceil_div(N, T);
  const int major = MAJOR == kMajN ? tn : tm, minor = MAJOR == kMajN ? tm : tn;
  hipLaunchKernelGGL((k_gemm<T, KB, AK, BK, EPI, MAJOR>), dim3((unsigned)(align_up((size_t)major, 8) * minor)),
                     dim3(256), 0, st, A, lda, B, ldb, C, ldc, bias, mask, ldm, db, M, N, K, tm, tn);
}

template <int MT, int NT, int U, int EPI>
void launch_direct(hipStream_t st, const float* A, int64_t lda, const uint16_t* W, int64_t ldw, float* C, int64_t ldc,
                   const float* bias, int M, int N, int K) {
  hipLaunchKernelGGL((k_gemm_direct<MT, NT, U, EPI>), dim3((unsigned)ceil_div(N, 64 * NT), (unsigned)ceil_div(M, 16 * MT)),
                     dim3(256), 0, st, A, lda, W, ldw, C, ldc, bias, M, N, K);
}

// One forward layer.  Up to 64 rows, and wherever 64 x 64 tiles would give
// fewer than one workgroup per CU, the direct kernel is the faster one (at 256
// x 512 x 512 7.6 us against 32 us); from 512 workgroups on the larger tile is
// (256 x 512 x 65536 65 us against 73 us).  The direct kernel takes several
// row tiles per wave once that leaves two waves per SIMD, so that the weights
// are read once.
template <int EPI>
tide_status layer_fwd(hipStream_t st, const float* A, int64_t lda, const uint16_t* W, int64_t ldw, float* C,
                      int64_t ldc, const float* bias, int M, int N, int K) {
  if (ceil_div(M, 64) * ceil_div(N, 64) >= 256 && M > 64) {
    if (ceil_div(M, 128) * ceil_div(N, 128) >= 512)
      launch_gemm<128, kBK, kA_KC, kB_WKC, EPI, kMajN>(st, A, lda, W, ldw, C, ldc, bias, nullptr, 0, nullptr, M, N, K);
    else
      launch_gemm<64, kBK, kA_KC, kB_WKC, EPI, kMajN>(st, A, lda, W, ldw, C, ldc, bias, nullptr, 0, nullptr, M, N, K);
  } else if (M <= 16 || ceil_div(M, 16) * ceil_div(N, 16) < 2048) {
    launch_direct<1, 1, 8, EPI>(st, A, lda, W, ldw, C, ldc, bias, M, N, K);
  } else if (M <= 32) {
    launch_direct<2, 1, 4, EPI>(st, A, lda, W, ldw, C, ldc, bias, M, N, K);
  } else {
    launch_direct<4, 1, 2, EPI>(st, A, lda, W, ldw, C, ldc, bias, M, N, K);
  }
  TIDE_LAUNCH_CHECK("mlp layer");
  return TIDE_OK;
}

// dW = G^T a and the bias gradient db = column sums of G.  The largest tile from
// 512 workgroups on, as in the forward; 32 x 32 tiles up to four workgroups per
// CU.  The whole backward at batch 256 with a last layer 2048 wide (1024
// workgroups of 32 x 32) 101 us with either tile there, 4096 wide 131 us with
// 64 x 64 and 133 us with 32 x 32.
tide_status weight_grad(hipStream_t st, const float* G, int64_t ldg, const float* a, float* gW, float* gb, int n_out,
                        int n_in, int batch) {
  if (ceil_div(n_out, 128) * ceil_div(n_in, 128) >= 512)
    launch_gemm<128, kBK, kA_MC, kB_FNC, kE_STORE, kMajM>(st, G, ldg, a, n_in, gW, n_in, nullptr, nullptr, 0, gb,
                                                          n_out, n_in, batch);
  else if (ceil_div(n_out, 64) * ceil_div(n_in, 64) <= 256)
    launch_gemm<32, 2 * kBK, kA_MC, kB_FNC, kE_STORE, kMajM>(st, G, ldg, a, n_in, gW, n_in, nullptr, nullptr, 0, gb,
                                                             n_out, n_in, batch);
  else
    launch_gemm<64, kBK, kA_MC, kB_FNC, kE_STORE, kMajM>(st, G, ldg, a, n_in, gW, n_in, nullptr, nullptr, 0, gb,
                                                         n_out, n_in, batch);
  TIDE_LAUNCH_CHECK("mlp weight gradient");
  return TIDE_OK;
}

// Input gradient through the ReLU of the layer's input (act).  Its outputs are
// few and its K long in earnest (the chain kernel, see there); 128 x 128 tiles
// take over where they alone give a workgroup per CU.
tide_status input_grad(hipStream_t st, const float* G, int64_t ldg, const uint16_t* W, const float* act, float* gx,
                       int64_t ldx, int n_out, int n_in, int batch) {
  if (ceil_div(batch, 128) * ceil_div(n_in, 128) >= 256) {
    launch_gemm<128, kBK, kA_KC, kB_WNC, kE_MASK, kMajM>(st, G, ldg, W, n_in, gx, ldx, nullptr, act, n_in, nullptr,
                                                         batch, n_in, n_out);
  } else {
    const int tm = (int)ceil_div(batch, kChM), tn = (int)ceil_div(n_in, kChN);
    const int sup_m = (int)ceil_div(tm, kChSup), sup_n = (int)ceil_div(tn, kChSup);
    const unsigned grid = (unsigned)(align_up((size_t)sup_m * sup_n, 8) * kChSup * kChSup);
    hipLaunchKernelGGL(k_gemm_chain, dim3(grid), dim3(kWave * (kChMul + kChFeed)), 0, st, G, ldg, W, (int64_t)n_in, act,
                       (int64_t)n_in, gx, ldx, batch, n_in, n_out, tm, tn, sup_m);
  }
  TIDE_LAUNCH_CHECK("mlp input gradient");
  return TIDE_OK;
}

// ------------------------------------------------------------------ loss
constexpr int kLossBlocks = 1024;

// G = (sigmoid(z) - y) / denom on valid outputs (0 elsewhere), rows of ldg
// floats; per-block partial sums of the element losses in double, fixed
// order.  denom = batch * (number of valid outputs), which every block counts
// for itself (8 KB of words for 65536 outputs, from L2: one launch fewer); block 0 leaves
// it for k_loss_sum.  A thread takes four neighbouring outputs of a
// 1024-output piece of a row with one 16-byte load and store; blocks take
// pieces grid-stride.  Reads and writes 4 B per output each; the exponential,
// the logarithm and the double-precision sum bound it: 256 x 65536 (134 MB)
// 66 us, 86 us with one output per thread and an index division each.
constexpr int kBcePiece = 1024;
// The logits are the caller's, aligned to their element: moved in 16-byte pieces
// all the same.
typedef float four __attribute__((ext_vector_type(4), aligned(4)));
__global__ __launch_bounds__(256) void k_bce(const float* __restrict__ Z, const uint32_t* __restrict__ lab,
                                             const uint32_t* __restrict__ valid, int batch, int nout,
                                             float* __restrict__ G, int64_t ldg, double* __restrict__ denom,
                                             double* __restrict__ partial) {
  __shared__ double s[256];
  __shared__ int sc[4];
  const int words = nout >> 5;
  int c = 0;
  for (int i = threadIdx.x; i < words; i += 256) c += __popc(valid[i]);
  c = wave_sum(c);
  if (__lane_id() == 0) sc[threadIdx.x / kWave] = c;
  __syncthreads();
  c = sc[0] + sc[1] + sc[2] + sc[3];
  const double d = (double)batch * (double)(c > 0 ? c : 1);
  if (blockIdx.x == 0 && threadIdx.x == 0) *denom = d;
  const float inv = (float)(1.0 / d);
  const int per_row = (nout + kBcePiece - 1) / kBcePiece;
  const int64_t pieces = (int64_t)batch * per_row;
  double acc = 0;
  for (int64_t q = blockIdx.x; q < pieces; q += gridDim.x) {
    const int64_t b = q / per_row;
    const int o = (int)(q - b * per_row) * kBcePiece + 4 * threadIdx.x;
    if (o >= nout) continue;   // nout is a multiple of 32: four outputs share a word
    const f32x4 zz = *reinterpret_cast<const four*>(Z + b * nout + o);
    const uint32_t okw = valid[o >> 5] >> (o & 31), yw = lab[b * words + (o >> 5)] >> (o & 31);
    float g[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float z = zz[j];
      const bool ok = (okw >> j) & 1u;
      const float y = (yw >> j) & 1u ? 1.f : 0.f;
      const float e = __expf(-fabsf(z));
      const float sig = (z >= 0.f ? 1.f : e) / (1.f + e);
      g[j] = ok ? (sig - y) * inv : 0.f;
      if (ok) acc += (double)(fmaxf(z, 0.f) - z * y + log1pf(e));
    }
    *reinterpret_cast<float4*>(G + b * ldg + o) = make_float4(g[0], g[1], g[2], g[3]);
  }
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = s[0];
}

__global__ __launch_bounds__(1024) void k_loss_sum(const double* __restrict__ partial, int n,
                                                   const double* __restrict__ denom, double* __restrict__ out) {
  __shared__ double s[1024];
  s[threadIdx.x] = (int)threadIdx.x < n ? partial[threadIdx.x] : 0.0;
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = s[0] / *denom;
}

// ------------------------------------------------------------------ Adam
__global__ __launch_bounds__(256) void k_mlp_adam(float* __restrict__ p, uint16_t* __restrict__ pb,
                                                  const float* __restrict__ g, float* __restrict__ m,
                                                  float* __restrict__ v, int64_t n, float lr, float b1, float b2,
                                                  float eps, float bc1, float bc2s) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    const float pi = p[i] - lr * (mi * bc1) / (sqrtf(vi) * bc2s + eps);
    m[i] = mi;
    v[i] = vi;
    p[i] = pi;
    pb[i] = bf16_bits(pi);
  }
}

__global__ __launch_bounds__(256) void k_to_bf16(const float* __restrict__ p, uint16_t* __restrict__ pb, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    pb[i] = bf16_bits(p[i]);
}

__global__ __launch_bounds__(256) void k_threshold(const float* __restrict__ Z, int64_t n_words, int nout, float thr,
                                                   uint32_t* __restrict__ out) {
  const int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (w >= n_words) return;
  const int wpr = nout >> 5;
  const int64_t b = w / wpr;
  const int o0 = (int)(w - b * wpr) * 32;
  const float* z = Z + b * nout + o0;
  uint32_t bits = 0;
#pragma unroll 8
  for (int j = 0; j < 32; ++j) bits |= (z[j] >= thr ? 1u : 0u) << j;
  out[w] = bits;
}

// ------------------------------------------------------------------ host
struct Layout {
  int L;
  const int32_t* d;
  int64_t w_off[TIDE_MLP_MAX_LAYERS], b_off[TIDE_MLP_MAX_LAYERS], P;
  int max_out;
};

bool layout(const int32_t* dims, int L, Layout& lay) {
  if (!dims || L < 1 || L > TIDE_MLP_MAX_LAYERS) return false;
  for (int l = 0; l <= L; ++l)
    if (dims[l] <= 0 || dims[l] % 8 != 0) return false;
  if (dims[L] % 32 != 0) return false;
  lay.L = L;
  lay.d = dims;
  int64_t off = 0;
  lay.max_out = 0;
  for (int l = 0; l < L; ++l) {
    lay.w_off[l] = off;
    off += (int64_t)dims[l] * dims[l + 1];
    lay.b_off[l] = off;
    off += dims[l + 1];
    lay.max_out = dims[l + 1] > lay.max_out ? dims[l + 1] : lay.max_out;
  }
  lay.P = off;
  return true;
}

struct Ws {
  float* act[TIDE_MLP_MAX_LAYERS];   // act[l], l = 1..L-1: [batch][dims[l]]
  float* g[2];                       // [batch][grad_ld(width)]
  double* partial;                   // [kLossBlocks]
  double* denom;
  size_t bytes;
};

// Row stride of the backward's gradient buffers.  Widths are powers of two in
// earnest; 256 bytes more per row spread the rows of a tile over the L2's
// channels (k_gemm_chain reads 16 rows 256 KB apart at the same columns).
int64_t grad_ld(int64_t width) { return width + 64; }

Ws carve(void* base, const Layout& lay, int batch) {
  Carver c(base);
  Ws w{};
  for (int l = 1; l < lay.L; ++l) w.act[l] = c.take<float>((size_t)batch * lay.d[l]);
  w.g[0] = c.take<float>((size_t)batch * grad_ld(lay.max_out));
  w.g[1] = c.take<float>((size_t)batch * grad_ld(lay.max_out));
  w.partial = c.take<double>(kLossBlocks);
  w.denom = c.take<double>(1);
  w.bytes = c.used;
  return w;
}

tide_status check_mlp(const tide_mlp* mlp, Layout& lay) {
  TIDE_CHECK_ARG(mlp, "null mlp");
  TIDE_CHECK_ARG(layout(mlp->dims, mlp->n_layers, lay),
                 "bad MLP dims: 1..%d layers, widths positive multiples of 8, output a multiple of 32",
                 TIDE_MLP_MAX_LAYERS);
  TIDE_CHECK_ARG(mlp->params && mlp->params_bf16, "null parameter buffers");
  TIDE_CHECK_ARG(aligned16(mlp->params) && aligned16(mlp->params_bf16), "parameter buffers must be 16-byte aligned");
  return TIDE_OK;
}

int grid_for(int64_t n) { return (int)std::min<int64_t>(ceil_div(n, 256), 4096); }

}  // namespace
}  // namespace tide

using namespace tide;

extern "C" int64_t tide_mlp_param_count(const int32_t* dims, int32_t n_layers) {
  Layout lay;
  return layout(dims, n_layers, lay) ? lay.P : -1;
}

extern "C" size_t tide_mlp_ws_bytes(const tide_mlp* mlp, int32_t batch) {
  Layout lay;
  if (!mlp || !layout(mlp->dims, mlp->n_layers, lay) || batch < 0) return 0;
  return carve(nullptr, lay, batch).bytes;
}

extern "C" tide_status tide_mlp_sync_bf16(const tide_mlp* mlp, void* stream) {
  Layout lay;
  tide_status s = check_mlp(mlp, lay);
  if (s != TIDE_OK) return s;
  hipLaunchKernelGGL(k_to_bf16, dim3(grid_for(lay.P)), dim3(256), 0, (hipStream_t)stream, mlp->params,
                     mlp->params_bf16, lay.P);
  TIDE_LAUNCH_CHECK("mlp to_bf16");
  return TIDE_OK;
}

extern "C" tide_status tide_mlp_fwd(const tide_mlp* mlp, const float* x, int32_t batch, float* logits, void* ws,
                                    size_t ws_bytes, void* stream) {
  Layout lay;
  tide_status s = check_mlp(mlp, lay);
  if (s != TIDE_OK) return s;
  TIDE_CHECK_ARG(batch >= 0, "negative batch");
  if (batch == 0) return TIDE_OK;
  TIDE_CHECK_ARG(x && logits && ws, "null argument");
  TIDE_CHECK_ARG(aligned16(x) && aligned16(ws), "x and ws must be 16-byte aligned");
  const Ws w = carve(ws, lay, batch);
  if (ws_bytes < w.bytes) {
    set_error("mlp workspace too small: %zu < %zu bytes", ws_bytes, w.bytes);
    return TIDE_ECAPACITY;
  }
  hipStream_t st = (hipStream_t)stream;
  const int32_t* d = lay.d;
  const float* in = x;
  timer_mark("mlp_fwd", st, true);
  for (int l = 0; l < lay.L; ++l) {
    const uint16_t* W = mlp->params_bf16 + lay.w_off[l];
    const float* b = mlp->params + lay.b_off[l];
    if (l + 1 < lay.L) {
      s = layer_fwd<kE_BIAS_RELU>(st, in, d[l], W, d[l], w.act[l + 1], d[l + 1], b, batch, d[l + 1], d[l]);
      in = w.act[l + 1];
    } else {
      s = layer_fwd<kE_BIAS>(st, in, d[l], W, d[l], logits, d[l + 1], b, batch, d[l + 1], d[l]);
    }
    if (s != TIDE_OK) return s;
  }
  timer_mark("mlp_fwd", st, false);
  return TIDE_OK;
}

extern "C" tide_status tide_mlp_bwd(const tide_mlp* mlp, const float* x, const float* logits,
                                    const uint32_t* label_bits, const uint32_t* valid_bits, int32_t batch,
                                    double* d_loss, void* ws, size_t ws_bytes, void* stream) {
  Layout lay;
  tide_status s = check_mlp(mlp, lay);
  if (s != TIDE_OK) return s;
  TIDE_CHECK_ARG(batch >= 1, "batch must be positive");
  TIDE_CHECK_ARG(x && logits && label_bits && valid_bits && d_loss && ws && mlp->grad, "null argument");
  TIDE_CHECK_ARG(aligned16(x) && aligned16(ws) && aligned16(mlp->grad), "x, ws and grad must be 16-byte aligned");
  const Ws w = carve(ws, lay, batch);
  if (ws_bytes < w.bytes) {
    set_error("mlp workspace too small: %zu < %zu bytes", ws_bytes, w.bytes);
    return TIDE_ECAPACITY;
  }
  hipStream_t st = (hipStream_t)stream;
  const int32_t* d = lay.d;
  const int L = lay.L, nout = d[L];
  const int nb = (int)std::min<int64_t>(kLossBlocks, batch * ceil_div(nout, kBcePiece));
  TIDE_TIMED("mlp_bce", st,
             hipLaunchKernelGGL(k_bce, dim3(nb), dim3(256), 0, st, logits, label_bits, valid_bits, batch, nout, w.g[0],
                                grad_ld(nout), w.denom, w.partial));
  TIDE_LAUNCH_CHECK("mlp bce");
  hipLaunchKernelGGL(k_loss_sum, dim3(1), dim3(1024), 0, st, w.partial, nb, w.denom, d_loss);
  TIDE_LAUNCH_CHECK("mlp loss_sum");
  int cur = 0;
  timer_mark("mlp_bwd", st, true);
  for (int l = L - 1; l >= 0; --l) {
    const float* G = w.g[cur];                      // dL/d(pre-activation of layer l's output) [batch][d[l+1]]
    const float* a = l == 0 ? x : w.act[l];         // layer input [batch][d[l]]
    float* gW = mlp->grad + lay.w_off[l];
    float* gb = mlp->grad + lay.b_off[l];
    // the input gradient first: G and W are the most recently touched then
    if (l > 0) {
      s = input_grad(st, G, grad_ld(d[l + 1]), mlp->params_bf16 + lay.w_off[l], w.act[l], w.g[cur ^ 1],
                     grad_ld(d[l]), d[l + 1], d[l], batch);
      if (s != TIDE_OK) return s;
    }
    s = weight_grad(st, G, grad_ld(d[l + 1]), a, gW, gb, d[l + 1], d[l], batch);
    if (s != TIDE_OK) return s;
    cur ^= 1;
  }
  timer_mark("mlp_bwd", st, false);
  return TIDE_OK;
}

extern "C" tide_status tide_mlp_adam(tide_mlp* mlp, float lr, float beta1, float beta2, float eps, void* stream) {
  Layout lay;
  tide_status s = check_mlp(mlp, lay);
  if (s != TIDE_OK) return s;
  TIDE_CHECK_ARG(mlp->grad && mlp->exp_avg && mlp->exp_avg_sq, "null Adam buffers");
  TIDE_CHECK_ARG(beta1 >= 0.f && beta1 < 1.f && beta2 >= 0.f && beta2 < 1.f && eps >= 0.f, "bad Adam constants");
  const int64_t t = mlp->step + 1;
  const float bc1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)t)));
  const float bc2s = (float)(1.0 / std::sqrt(1.0 - std::pow((double)beta2, (double)t)));
  hipStream_t st = (hipStream_t)stream;
  TIDE_TIMED("mlp_adam", st,
             hipLaunchKernelGGL(k_mlp_adam, dim3(grid_for(lay.P)), dim3(256), 0, st, mlp->params, mlp->params_bf16,
                                mlp->grad, mlp->exp_avg, mlp->exp_avg_sq, lay.P, lr, beta1, beta2, eps, bc1, bc2s));
  TIDE_LAUNCH_CHECK("mlp adam");
  mlp->step = t;
  return TIDE_OK;
}

extern "C" tide_status tide_mlp_predict_bits(const float* logits, int32_t batch, int32_t n_out, float threshold_logit,
                                             uint32_t* out_bits, void* stream) {
  TIDE_CHECK_ARG(batch >= 0 && n_out > 0 && n_out % 32 == 0, "n_out must be a positive multiple of 32");
  if (batch == 0) return TIDE_OK;
  TIDE_CHECK_ARG(logits && out_bits, "null argument");
  const int64_t words = (int64_t)batch * (n_out / 32);
  hipLaunchKernelGGL(k_threshold, dim3((unsigned)ceil_div(words, 256)), dim3(256), 0, (hipStream_t)stream, logits,
                     words, n_out, threshold_logit, out_bits);
  TIDE_LAUNCH_CHECK("mlp threshold");
  return TIDE_OK;
}
