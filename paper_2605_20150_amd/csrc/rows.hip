// Row-major tables to and from the layouts of the hot path: the (N, 59) table of a
// dense render into block-SoA slots, and the compact column-major gradient back
// into an (N, 59) table.
//
// Both are bound by the launches around them at the sizes they are used at (an
// autograd render of thousands of rows), and by memory beyond: 64 rows per
// workgroup, transposed through LDS, so that both sides are read and written in
// runs of 64 elements or more.  59 is odd: neither side's LDS accesses meet in a
// bank.  In place of fills, copies, transposes, boolean indexing (which waits for
// the GPU) and copies from host memory, some thirty launches: a differentiable
// render of 20k Gaussians at 400x300, forward and backward, 900 us before and
// 460 us after, together with one binning in place of two.
#include "raster.h"

namespace tide {

constexpr int kRowsPerWg = kWave, kRowThreads = 256;

template <typename T>
__global__ void __launch_bounds__(kRowThreads) k_rows_to_blocks(const T* __restrict__ theta, int64_t n, int64_t rows,
                                                                int32_t B, int32_t n_blocks, int32_t n_slots,
                                                                T* __restrict__ params,
                                                                int32_t* __restrict__ slot_block,
                                                                int32_t* __restrict__ slot_rows,
                                                                int32_t* __restrict__ order) {
  __shared__ T s[kRowsPerWg * kD];
  const int64_t r0 = (int64_t)blockIdx.x * kRowsPerWg;
  const int tid = threadIdx.x;
  for (int64_t k = (int64_t)blockIdx.x * kRowThreads + tid; k < n_slots; k += (int64_t)gridDim.x * kRowThreads) {
    const int64_t left = n - k * B;
    slot_block[k] = k < n_blocks ? (int32_t)k : -1;
    slot_rows[k] = left <= 0 ? 0 : (left < B ? (int32_t)left : B);
    if (k < n_blocks) order[k] = (int32_t)k;
  }
  for (int e = tid; e < kRowsPerWg * kD; e += kRowThreads) s[e] = r0 * kD + e < n * kD ? theta[r0 * kD + e] : (T)0;
  __syncthreads();
  const int64_t r = r0 + __lane_id();
  if (r >= rows) return;
  const int64_t slot = r / B;
  T* p = params + slot * kD * B + (r - slot * B);
  for (int d = tid / kWave; d < kD; d += kRowThreads / kWave) p[(int64_t)d * B] = s[__lane_id() * kD + d];
}

// out[i][d] = active[i] ? grad[d][act_idx[i]] : 0
template <typename T>
__global__ void __launch_bounds__(kRowThreads) k_dense_grad(const int32_t* __restrict__ active,
                                                            const int32_t* __restrict__ act_idx,
                                                            const T* __restrict__ grad, int64_t ld, int64_t n,
                                                            T* __restrict__ out) {
  __shared__ T s[kRowsPerWg * kD];
  const int64_t r0 = (int64_t)blockIdx.x * kRowsPerWg;
  const int tid = threadIdx.x, lane = __lane_id();
  const bool on = r0 + lane < n && active[r0 + lane] != 0;
  const T* g = grad + (on ? act_idx[r0 + lane] : 0);
#pragma unroll 5
  for (int d = tid / kWave; d < kD; d += kRowThreads / kWave) s[lane * kD + d] = on ? g[(int64_t)d * ld] : (T)0;
  __syncthreads();
  for (int e = tid; e < kRowsPerWg * kD; e += kRowThreads)
    if (r0 * kD + e < n * kD) out[r0 * kD + e] = s[e];
}

}  // namespace tide

using namespace tide;

extern "C" tide_status tide_rows_to_blocks(const void* theta, int64_t n, int32_t block_rows, int32_t n_slots,
                                           int32_t dtype, void* params, int32_t* slot_block, int32_t* slot_rows,
                                           int32_t* order, void* stream) {
  TIDE_CHECK_ARG(params && slot_block && slot_rows && order && (theta || n == 0), "null argument");
  TIDE_CHECK_ARG(n >= 0 && block_rows > 0 && n_slots > 0, "bad sizes");
  TIDE_CHECK_ARG(dtype == TIDE_F32 || dtype == TIDE_F64, "bad dtype");
  const int64_t rows = (int64_t)n_slots * block_rows, blocks = n > 0 ? ceil_div(n, block_rows) : 1;
  TIDE_CHECK_ARG(blocks <= n_slots, "more rows than the slots hold");
  const int64_t grid = ceil_div(rows, kRowsPerWg);
  TIDE_CHECK_ARG(grid < (1ll << 31), "too many rows");
  hipStream_t st = (hipStream_t)stream;
  if (dtype == TIDE_F32)
    hipLaunchKernelGGL(k_rows_to_blocks<float>, dim3((uint32_t)grid), dim3(kRowThreads), 0, st, (const float*)theta, n,
                       rows, block_rows, (int32_t)blocks, n_slots, (float*)params, slot_block, slot_rows, order);
  else
    hipLaunchKernelGGL(k_rows_to_blocks<double>, dim3((uint32_t)grid), dim3(kRowThreads), 0, st, (const double*)theta,
                       n, rows, block_rows, (int32_t)blocks, n_slots, (double*)params, slot_block, slot_rows, order);
  TIDE_LAUNCH_CHECK("k_rows_to_blocks");
  return TIDE_OK;
}

extern "C" tide_status tide_dense_grad(const tide_proj* proj, const void* grad, int64_t grad_ld, int64_t n, void* out,
                                       void* stream) {
  TIDE_CHECK_ARG(proj && grad && out && proj->active && proj->act_idx, "null argument");
  TIDE_CHECK_ARG(n >= 0 && n <= proj->n_pidx, "more rows than the projection holds");
  TIDE_CHECK_ARG(grad_ld >= proj->n_pidx, "grad_ld too small");
  TIDE_CHECK_ARG(proj->dtype == TIDE_F32 || proj->dtype == TIDE_F64, "bad dtype");
  if (n == 0) return TIDE_OK;
  const int64_t grid = ceil_div(n, kRowsPerWg);
  TIDE_CHECK_ARG(grid < (1ll << 31), "too many rows");
  hipStream_t st = (hipStream_t)stream;
  if (proj->dtype == TIDE_F32)
    hipLaunchKernelGGL(k_dense_grad<float>, dim3((uint32_t)grid), dim3(kRowThreads), 0, st,
                       (const int32_t*)proj->active, (const int32_t*)proj->act_idx, (const float*)grad, grad_ld, n,
                       (float*)out);
  else
    hipLaunchKernelGGL(k_dense_grad<double>, dim3((uint32_t)grid), dim3(kRowThreads), 0, st,
                       (const int32_t*)proj->active, (const int32_t*)proj->act_idx, (const double*)grad, grad_ld, n,
                       (double*)out);
  TIDE_LAUNCH_CHECK("k_dense_grad");
  return TIDE_OK;
}
