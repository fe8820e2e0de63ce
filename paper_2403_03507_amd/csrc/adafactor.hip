// Adafactor with first-order statistics as the optimizer of the projected gradient (the optimizer Sec. 4.3 and Sec. 5 of
// the paper name next to Adam; the paper prints no equations, so this is the published Adafactor update for a matrix,
// with the learning rate left to the caller as in Algorithm 2):
//   rowv_i <- b2 rowv_i + (1 - b2) sum_j (R_ij^2 + eps1),  colv_j <- b2 colv_j + (1 - b2) sum_i (R_ij^2 + eps1),  b2 = 1 - k^-0.8
//   Vhat_ij = rowv_i colv_j / sum_i rowv_i,  U = R / sqrt(Vhat),  Uhat = U / max(1, RMS(U) / d)
//   M <- b1 M + (1 - b1) Uhat,  N = M
// Four or five launches, three passes over R: partial sums of the squares by rows and by columns; the statistics and partial sums of
// the row statistics; partial sums of U^2; for a large matrix their sum; the update.  The total of the row statistics, and for a
// small matrix the sum of U^2, is added by every workgroup that needs it, in the same fixed order, which takes less than the
// launch of a workgroup that would (kAfClipPartials).  No atomics, bit-identical from run to run.  Bound by memory
// traffic: 3 reads of R, one read and write of M, one write of N, transposed where the product that reads it wants it so
// (a transpose of its own took 19 us for 1024 x 11008, the transposed store takes 7).
#include "adafactor.hpp"

namespace galore {
namespace {

constexpr int kAfCols = 256;  // columns per workgroup (one per thread)
constexpr int kAfRows = 32;   // rows per workgroup
// Partial sums of U^2 (one per 32 x 256 tile) up to which every workgroup of the update adds them all itself: that work grows with
// the square of the tiles, a launch of one workgroup that adds them once costs about 3 us.  Update block, us, every workgroup / once:
// 512 tiles (512 x 8192) 27.5 / 29.9, 1024 (1024 x 8192) 42.8 / 43.7, 1376 (1024 x 11008) 58.7 / 57.3, 16000 (4096 x 32000) 602 / 581,
// 65536 (8192 x 65536) 2581 / 2152.
constexpr int64_t kAfClipPartials = 1200;

__device__ __forceinline__ float af_wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// scratch layout (floats): rowpart [cb][rows] | colpart [rb][cols] | blockpart [rb * cb].  The sums of rowv over 256 rows take the
// place of the first row partial of those rows, which only the workgroup that forms the sum reads.
struct AfScratch {
  float* rowpart;
  float* colpart;
  float* blockpart;
  int cb, rb, sb;
};
__host__ __device__ inline AfScratch af_scratch(float* base, int rows, int cols) {
  AfScratch s;
  s.cb = (cols + kAfCols - 1) / kAfCols;
  s.rb = (rows + kAfRows - 1) / kAfRows;
  s.rowpart = base;
  s.colpart = s.rowpart + (size_t)s.cb * rows;
  s.blockpart = s.colpart + (size_t)s.rb * cols;
  s.sb = (rows + 255) / 256;
  return s;
}

// pass 1: sums of R^2 + eps1 over this workgroup's 256 columns for each of its 32 rows, and over its 32 rows for each column.
// A thread owns a column: its 32 loads are independent (clamped addresses, masked afterwards) and all in flight together.
// Column sums stay in the thread; for the row sums the squares cross an LDS tile and 8 threads per row add 32 columns
// each, then each other (fixed order).
__global__ __launch_bounds__(kAfCols) void adafactor_sums_kernel(const AdafactorProblem p) {
  __shared__ float tile[kAfRows][kAfCols + 1];
  const AfScratch s = af_scratch(p.scratch, p.rows, p.cols);
  const int tid = threadIdx.x;
  const int c = blockIdx.x * kAfCols + tid;
  const int row0 = blockIdx.y * kAfRows;
  const bool cok = c < p.cols;
  const int cc = cok ? c : p.cols - 1;
  float x[kAfRows];
#pragma unroll
  for (int rl = 0; rl < kAfRows; ++rl) {
    const int row = row0 + rl < p.rows ? row0 + rl : p.rows - 1;
    x[rl] = p.R[(size_t)row * p.ldr + cc];
  }
  float colacc = 0.f;
#pragma unroll
  for (int rl = 0; rl < kAfRows; ++rl) {
    const float q = (cok && row0 + rl < p.rows) ? x[rl] * x[rl] + p.eps1 : 0.f;
    colacc += q;
    tile[rl][tid] = q;
  }
  if (cok) s.colpart[(size_t)blockIdx.y * p.cols + c] = colacc;
  __syncthreads();
  const int rl = tid >> 3, part = tid & 7;
  float a = 0.f;
#pragma unroll
  for (int j = 0; j < kAfCols / 8; ++j) a += tile[rl][part + 8 * j];
  a += __shfl_xor(a, 1, 64);
  a += __shfl_xor(a, 2, 64);
  a += __shfl_xor(a, 4, 64);
  if (part == 0 && row0 + rl < p.rows) s.rowpart[(size_t)blockIdx.x * p.rows + row0 + rl] = a;
}

// sum over a workgroup of 256 threads, in a fixed order; every thread gets it.  `red`: 4 floats.
__device__ __forceinline__ float af_block_sum(float a, float* red) {
  a = af_wave_sum(a);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

// the total of the row statistics; `red`: 4 floats
__device__ __forceinline__ float af_total(const AfScratch& s, float* red) {
  float a = 0.f;
  for (int i = threadIdx.x; i < s.sb; i += 256) a += s.rowpart[(size_t)i * 256];
  return af_block_sum(a, red);
}

// the statistics: partial sums added in index order (loads in batches of eight), then the decayed averages; one thread per
// row statistic (the first sb workgroups, which also add up theirs) or column statistic
__global__ __launch_bounds__(256) void adafactor_stats_kernel(const AdafactorProblem p) {
  const AfScratch s = af_scratch(p.scratch, p.rows, p.cols);
  __shared__ float red[4];
  const bool is_row = (int)blockIdx.x < s.sb;
  const int i0 = (is_row ? blockIdx.x : blockIdx.x - s.sb) * 256 + threadIdx.x, n = is_row ? p.rows : p.cols;
  const bool ok = i0 < n;
  const int i = ok ? i0 : n - 1;
  const float* part = is_row ? s.rowpart + i : s.colpart + i;
  const size_t stride = is_row ? p.rows : p.cols;
  const int count = is_row ? s.cb : s.rb;
  float a = 0.f;
#pragma unroll 8
  for (int b = 0; b < count; ++b) a += part[(size_t)b * stride];
  float* stat = is_row ? p.rowv + i : p.colv + i;
  const float v = p.beta2t * *stat + (1.f - p.beta2t) * a;
  if (is_row) {  // uniform
    const float sum = af_block_sum(ok ? v : 0.f, red);  // every thread has read its partials before the barrier in here
    if (threadIdx.x == 0) s.rowpart[(size_t)blockIdx.x * 256] = sum;
  }
  if (ok) *stat = v;
}

// U_ij = R_ij / sqrt(rowv_i colv_j / total); the association keeps the quotient colv_j / total (of order 1 / rows) away
// from the underflow that rowv_i colv_j could reach for tiny gradients
__device__ __forceinline__ float af_u(float x, float rv, float cv_over_total) { return x / sqrtf(rv * cv_over_total); }

// pass 2: sum of U^2 over this workgroup's tile
__global__ __launch_bounds__(kAfCols) void adafactor_rms_kernel(const AdafactorProblem p) {
  __shared__ float sm[4], red[4];
  const AfScratch s = af_scratch(p.scratch, p.rows, p.cols);
  const int tid = threadIdx.x;
  const int c = blockIdx.x * kAfCols + tid;
  const int row0 = blockIdx.y * kAfRows;
  float acc = 0.f;
  {
    const bool cok = c < p.cols;
    const int cc = cok ? c : p.cols - 1;
    float x[kAfRows], rv[kAfRows];
#pragma unroll
    for (int rl = 0; rl < kAfRows; ++rl) {        // independent loads from clamped addresses, masked below
      const int row = row0 + rl < p.rows ? row0 + rl : p.rows - 1;
      x[rl] = p.R[(size_t)row * p.ldr + cc];
      rv[rl] = p.rowv[row];
    }
    const float cvt = p.colv[cc] / af_total(s, red);
#pragma unroll
    for (int rl = 0; rl < kAfRows; ++rl) {
      const float u = af_u(x[rl], rv[rl], cvt);
      acc += (cok && row0 + rl < p.rows) ? u * u : 0.f;
    }
  }
  acc = af_block_sum(acc, sm);
  if (tid == 0) s.blockpart[blockIdx.y * s.cb + blockIdx.x] = acc;
}

// the sum of U^2 from `count` partial sums; `red`: 4 floats
__device__ __forceinline__ float af_sum_of_squares(const float* part, int count, float* red) {
  float a = 0.f;
#pragma unroll 8
  for (int i = threadIdx.x; i < count; i += 256) a += part[i];
  return af_block_sum(a, red);
}

// The same for a large matrix, once: the column partials are used up by now, so the first of them takes the sum.
__global__ __launch_bounds__(256) void adafactor_clip_kernel(const AdafactorProblem p) {
  __shared__ float red[4];
  const AfScratch s = af_scratch(p.scratch, p.rows, p.cols);
  const float sum = af_sum_of_squares(s.blockpart, s.rb * s.cb, red);
  if (threadIdx.x == 0) s.colpart[0] = sum;
}

// pass 3: the clipping factor 1 / max(1, RMS(U) / d), Uhat, the momentum, N
// summed: the sum of U^2 is in colpart[0], else every workgroup adds the partial sums
template <class TN>
__global__ __launch_bounds__(kAfCols) void adafactor_update_kernel(const AdafactorProblem p, int summed) {
  constexpr int VEC = 16 / (int)sizeof(TN), PIECES = kAfRows / VEC;
  __shared__ float red[4], red_total[4];
  __shared__ __align__(16) TN turned[kAfCols][kAfRows + VEC];
  const AfScratch s = af_scratch(p.scratch, p.rows, p.cols);
  const int tid = threadIdx.x;
  const int c = blockIdx.x * kAfCols + tid;
  const int row0 = blockIdx.y * kAfRows;
  const bool cok = c < p.cols;
  const int cc = cok ? c : p.cols - 1;
  float x[kAfRows], rv[kAfRows], mo[kAfRows];
#pragma unroll
  for (int rl = 0; rl < kAfRows; ++rl) {          // independent loads from clamped addresses
    const int row = row0 + rl < p.rows ? row0 + rl : p.rows - 1;
    x[rl] = p.R[(size_t)row * p.ldr + cc];
    rv[rl] = p.rowv[row];
    mo[rl] = p.M[(size_t)row * p.cols + cc];
  }
  const float cvt = p.colv[cc] / af_total(s, red_total);
  const float sumsq = summed ? s.colpart[0] : af_sum_of_squares(s.blockpart, s.rb * s.cb, red);
  const float over = sqrtf(sumsq / ((float)p.rows * (float)p.cols)) / p.clip_d;
  const float factor = 1.f / (over > 1.f ? over : 1.f);
  TN* N = static_cast<TN*>(p.N);
#pragma unroll
  for (int rl = 0; rl < kAfRows; ++rl) {
    const int row = row0 + rl;
    const float uhat = af_u(x[rl], rv[rl], cvt) * factor;
    const float m = p.beta1 * mo[rl] + (1.f - p.beta1) * uhat;
    turned[tid][rl] = (TN)m;
    if (cok && row < p.rows) {
      p.M[(size_t)row * p.cols + c] = m;
      if (!p.n_transposed) N[(size_t)row * p.cols + c] = (TN)m;
    }
  }
  if (!p.n_transposed) return;
  // N^T: the 32 entries of a column of the tile leave as 16-byte pieces of neighbouring lanes, at any alignment
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PIECES; ++q) {
    const int col = (tid + 256 * q) / PIECES, i = (tid + 256 * q) % PIECES * VEC;
    if ((int)blockIdx.x * kAfCols + col >= p.cols) continue;
    TN* dst = N + (size_t)(blockIdx.x * kAfCols + col) * p.rows + row0 + i;
    if (row0 + i + VEC <= p.rows) {
      __builtin_memcpy(dst, &turned[col][i], 16);
    } else {
#pragma unroll
      for (int e = 0; e < VEC; ++e)
        if (row0 + i + e < p.rows) dst[e] = turned[col][i + e];
    }
  }
}

}  // namespace

size_t adafactor_scratch_floats(int rows, int cols) {
  const AfScratch s = af_scratch(nullptr, rows, cols);
  return (size_t)(s.blockpart - s.rowpart) + (size_t)s.rb * s.cb + 4;  // the size that galore.h states for galore_adafactor
}

hipError_t launch_adafactor(const AdafactorProblem& p, DType n_dtype, hipStream_t stream) {
  if (p.rows < 1 || p.cols < 1 || p.ldr < p.cols || !p.R || !p.M || !p.rowv || !p.colv || !p.N || !p.scratch) return hipErrorInvalidValue;
  const AfScratch s = af_scratch(p.scratch, p.rows, p.cols);
  if (s.rb > 65535) return hipErrorInvalidValue;   // grid.y
  const dim3 grid(s.cb, s.rb);
  hipLaunchKernelGGL(adafactor_sums_kernel, grid, dim3(kAfCols), 0, stream, p);
  hipLaunchKernelGGL(adafactor_stats_kernel, dim3(s.sb + s.cb), dim3(256), 0, stream, p);
  hipLaunchKernelGGL(adafactor_rms_kernel, grid, dim3(kAfCols), 0, stream, p);
  const int summed = (int64_t)s.rb * s.cb > kAfClipPartials;
  if (summed) hipLaunchKernelGGL(adafactor_clip_kernel, dim3(1), dim3(256), 0, stream, p);
  if (n_dtype == DType::BF16) hipLaunchKernelGGL(adafactor_update_kernel<__bf16>, grid, dim3(kAfCols), 0, stream, p, summed);
  else hipLaunchKernelGGL(adafactor_update_kernel<float>, grid, dim3(kAfCols), 0, stream, p, summed);
  return hipGetLastError();
}

}  // namespace galore
