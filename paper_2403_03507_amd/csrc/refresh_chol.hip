// Orthonormalisation of the iteration block and Cholesky factor of the Rayleigh-Ritz matrix of the subspace refresh
// (Algorithm 2, refresh branch), for the transposed blocks Zt, Qt (r x k).
//
// Qt = L^-1 Zt with L L^T = Zt Zt^T (Cholesky QR), the r x r part in fp64: the Gram matrix squares the condition number
// of Z, which fp64 carries up to 1e7 (all that an fp32 Z can express), and Cholesky does not depend on the scale of the
// columns.  Three steps, each a grid over all tensors of the group:
//   * gram_f64_kernel       Zt Zt^T on the fp64 matrix cores, straight from global memory, lower triangle only;
//   * chol_step_kernel      one launch per 32 columns.  It updates the Schur complement and, in the block columns that
//                           are already eliminated, the rows of L^-1; the workgroup that owns the next diagonal block
//                           goes on to factor it, so no launch waits for a factorisation alone;
//   * an fp32 product       Qt = L^-1 Zt on the small-tile GEMM.
// A column that depends on its predecessors (its squared distance to their span below kDependent of its squared length)
// is taken out of the factorisation and replaced by pseudo-random entries; what that leaves unorthogonal is settled by
// the next pass.  One pass gives a basis of span(Z) that is orthonormal to fp32 rounding times the condition number, which
// is all that the next product with C needs; the last round takes a second pass (see refresh.hip).
// Householder reflectors (refresh_qr.hip) are a serial chain of r reflections; whole refreshes, ms, before and after: 350M layer
// set (k = 1024, r = 256, 4 rounds) 8.48 -> 3.80, 60M (k = 512, r = 128, 6 rounds, with five steps of the optimizer) 6.83 -> 2.46 (3.25 and
// 1.95 since, with the products on small tiles).
// No atomics and fixed summation orders: results are reproducible bit for bit.
#include "refresh_common.hpp"

#include <utility>

namespace galore {
namespace rf {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kCB = 32;      // rows and columns of a block of the factorisation
constexpr int kLP = kCB + 2; // row pitch of a block in LDS

// v_mfma_f64_16x16x4: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator v of lane l is element
// (4 v + l / 16, l % 16) of the product.
__device__ __forceinline__ int out_row(int v, int lane) { return 4 * v + (lane >> 4); }

__device__ __forceinline__ void tri_decode(int x, int& i, int& j) {  // x = i (i + 1) / 2 + j, j <= i
  i = (int)((sqrtf(8.f * (float)x + 1.f) - 1.f) * 0.5f);
  while ((i + 1) * (i + 2) / 2 <= x) ++i;
  while (i * (i + 1) / 2 > x) --i;
  j = x - i * (i + 1) / 2;
}

// The matrices being factored are kept as the 32 x 32 blocks of their lower triangle, each contiguous: block (i, j), j <= i
__host__ __device__ __forceinline__ int tri(int i) { return i * (i + 1) / 2; }
template <class D> __device__ __forceinline__ D* block_at(D* a, int i, int j) { return a + (size_t)(tri(i) + j) * (kCB * kCB); }

// Lower triangle of X Y^T (r x r, contraction k) in fp64 into A0 and its diagonal into diag: X = Y = Zt, or (ritz) X = Qt.
// A workgroup of 4 wavefronts owns 32 x 32 entries, a wavefront 16 x 16: at these ranks there are too few tiles for larger ones.
// The products of one MFMA step take 16 positions of every row as one 16-byte piece per lane, in an order that is the same
// for both operands.  Bound by the serial chain of k / 4 fp64 MFMAs of 64 cycles (7 tensors of k = 1024, r = 256: 23 us).
__global__ __launch_bounds__(256) void gram_f64_kernel(const RefreshGroup* __restrict__ gp, int ritz) {
  const RefreshGroup& grp = *gp;
  constexpr int U = 8;
  const RefreshTensor& t = grp.t[blockIdx.y];
  const int k = t.k, r = grp.r;
  int ti, tj;
  tri_decode(blockIdx.x, ti, tj);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i0 = ti * kCB + (wave & 1) * 16, j0 = tj * kCB + (wave >> 1) * 16;
  if (j0 > i0) return;  // above the diagonal (no barrier below)
  const int i = lane & 15, g = lane >> 4;
  // rows past the matrix repeat the last one; their products are not stored
  const float* x = (ritz ? t.Q : t.Z) + (size_t)min(i0 + i, r - 1) * k;
  const float* y = t.Z + (size_t)min(j0 + i, r - 1) * k;
  d4 acc = {0., 0., 0., 0.};
  auto mma = [&](f4 xa, f4 yb) {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)xa[e], (double)yb[e], acc, 0, 0, 0);
  };
  const int groups = k >> 4;  // of 16 positions
  int s = 0;
  for (; s + U <= groups; s += U) {
    f4 xa[U], yb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      __builtin_memcpy(&xa[u], x + 16 * (s + u) + 4 * g, 16);
      __builtin_memcpy(&yb[u], y + 16 * (s + u) + 4 * g, 16);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) mma(xa[u], yb[u]);
  }
  for (; 16 * s < k; ++s) {  // what is left, element by element
    f4 xa, yb;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int pos = 16 * s + 4 * g + e;
      xa[e] = pos < k ? x[pos] : 0.f;
      yb[e] = pos < k ? y[pos] : 0.f;
    }
    mma(xa, yb);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int row = i0 + out_row(v, lane), col = j0 + i;
    const double e = row < r && col < r ? acc[v] : 0.;
    block_at(t.A0, ti, tj)[(row - ti * kCB) * kCB + col - tj * kCB] = e;
    if (row == col) t.diag[row] = e;
  }
}

__device__ __forceinline__ double lane_value(double x, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// f(0), f(1), .. with the index as a type: a loop that is unrolled whatever its length
template <class F, int... I> __device__ __forceinline__ void each_index(F f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }

// 16 x 16 entries at (i0, j0) of a b^T (BT) or a b, both 32 x 32 in LDS; added to acc
template <bool BT> __device__ __forceinline__ void block_product(d4& acc, const double* a, const double* b, int i0, int j0, int lane) {
  const int i = lane & 15, g = lane >> 4;
#pragma unroll
  for (int kk = 0; kk < kCB; kk += 4) {
    const double x = a[(i0 + i) * kLP + kk + g];
    const double y = BT ? b[(j0 + i) * kLP + kk + g] : b[(kk + g) * kLP + j0 + i];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc, 0, 0, 0);
  }
}

constexpr double kDependent = 1e-12;   // sin^2 to the span of the columns before, in the passes of the last round
constexpr double kDependentRaw = 1e-14;  // in a pass that is followed by a product with C: little above fp64 rounding
constexpr double kZeroColumn = 1e-56;    // squared length below which a column counts as zero: its reciprocal has to fit fp32
constexpr double kRitzShift = 2.4e-7;    // 2^-22

// Step s of the factorisation of the matrix in A0 (blocks of 32; s = -1 only factors block 0).  Steps read one of A0, A1
// and write the other; block (i, j) holds the Schur complement for j > s and a row of L^-1 in the making for j <= s.
//   ritz == 0: S (fp32, r x r) <- L^-1, flag <- dependent columns
//   ritz == 1: Bw (fp32, r x r) <- L^T of the matrix shifted by kRitzShift of its largest diagonal entry.  The shift leaves
//              the eigenvectors alone and keeps every pivot above the fp32 rounding that the matrix carries anyway; so
//              does the power of two that brings the entries near one, whatever the scale of the gradient.
// Bound by latency: about 5 us of launch and block products and 6.5 us of the serial factorisation per launch (7 tensors: 11.8 us; 13.2 with all moves through
// scalar registers and each column's products in the chain of its pivot).
__global__ __launch_bounds__(256) void chol_step_kernel(const RefreshGroup* __restrict__ gp, int s, int ritz, double dependent) {
  const RefreshGroup& grp = *gp;
  __shared__ double D[kCB * kLP], P[kCB * kLP], Q[kCB * kLP];
  __shared__ double wave_max[4];
  __shared__ __align__(16) double column[2][64];
  const RefreshTensor& t = grp.t[blockIdx.y];
  const int r = grp.r, nb = (r + kCB - 1) / kCB, rp = nb * kCB;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool odd = s > 0 && (s & 1);   // s = -1 leaves A0 as it is, step 0 reads it
  const double* __restrict__ src = odd ? t.A1 : t.A0;
  double* __restrict__ dst = odd ? t.A0 : t.A1;
  const int x = blockIdx.x;
  int i, j;
  if (x == 0) {          // first, as the next launch waits for it
    i = j = s + 1;
    if (i >= nb) return;
  } else if (x <= nb) {  // row s of the result
    i = s;
    j = x - 1;
  } else {
    tri_decode(x - 1 - nb + tri(s + 1), i, j);
    if (i == s + 1 && j == s + 1) return;
  }
  // 8 entries of a block per thread pair of rows: thread tid moves columns 4 (tid % 8) .. of row tid / 8
  const int mr = tid >> 3, mc = (tid & 7) * 4;
  auto load = [&](double* lds, const double* from) {
    const d4 v = *reinterpret_cast<const d4*>(from + mr * kCB + mc);
#pragma unroll
    for (int e = 0; e < 4; ++e) lds[mr * kLP + mc + e] = v[e];
  };
  auto block = [&](int bi, int bj) { return block_at(src, bi, bj); };
  const int i0 = (wave & 1) * 16, j0 = (wave >> 1) * 16, oc = lane & 15;
  auto put = [&](double* lds, const d4& v) {
#pragma unroll
    for (int e = 0; e < 4; ++e) lds[(i0 + out_row(e, lane)) * kLP + j0 + oc] = v[e];
  };
  const double* dinv = t.dinv + (size_t)(s & 1) * kCB * kCB;  // inverse of diagonal block s of L
  const d4 zero = {0., 0., 0., 0.};

  if (i == s && s >= 0) {
    float* out = ritz ? t.Bw : t.S;
    d4 v = zero;
    if (j <= s && !ritz) {
      load(D, dinv);
      if (j < s) {
        load(P, block(s, j));
        __syncthreads();
        block_product<false>(v, D, P, i0, j0, lane);
      } else {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = D[(i0 + out_row(e, lane)) * kLP + j0 + oc];
      }
    }
    if (ritz && j >= s) return;  // L^T right of the diagonal is written where it is formed
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = s * kCB + i0 + out_row(e, lane), col = j * kCB + j0 + oc;
      if (row < r && col < r) out[(size_t)row * r + col] = (float)v[e];
    }
    return;
  }
  if (ritz && j < s) return;

  // what is updated, and what the factorisation asks for, requested before anything waits
  const int at0 = (i0 + (lane >> 4)) * kCB + j0 + oc;
  d4 v = zero;
  if (j != s)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = block(i, j)[at0 + 4 * e * kCB];
  double shift = 0., scale = 0., low = 0.;
  if (x == 0) {
    if (ritz && s >= 0) { shift = t.diag[rp]; scale = t.diag[rp + 1]; }
    if (!ritz) low = fmax(dependent * t.diag[i * kCB + (lane & 31)], kZeroColumn);
  }
  d4 upd = zero;
  if (s >= 0) {
    load(D, dinv);
    load(P, block(i, s));
    if (j != s && j != i) load(Q, block(j < s ? s : j, j < s ? j : s));
    __syncthreads();
    d4 l = zero, q = zero;
    block_product<true>(l, P, D, i0, j0, lane);                             // L_is = A_is D^T
    if (j > s && j != i) block_product<true>(q, Q, D, i0, j0, lane);        // L_js
    else if (j < s) block_product<false>(q, D, Q, i0, j0, lane);            // row s of L^-1
    __syncthreads();
    put(P, l);
    if (j != s && j != i) put(Q, q);
    __syncthreads();
    if (j == s) {
      if (ritz) {
        const int row = s * kCB + mr, col = i * kCB + mc;  // row of L^T: 4 entries of a column of L
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < r) t.Bw[(size_t)row * r + col + e] = (float)(t.diag[rp + 1] * P[(mc + e) * kLP + mr]);
        return;
      }
      block_product<false>(upd, P, D, i0, j0, lane);
    } else if (j > s) {
      block_product<true>(upd, P, j == i ? P : Q, i0, j0, lane);
    } else {
      block_product<false>(upd, P, Q, i0, j0, lane);
    }
  }
  v -= upd;
  if (x != 0) {
    double* to = block_at(dst, i, j);
#pragma unroll
    for (int e = 0; e < 4; ++e) to[at0 + 4 * e * kCB] = v[e];
    return;
  }
  put(Q, v);  // Q has not been read since the last barrier (j == i)
  if (ritz && s < 0) {
    double m = 0.;
    for (int c = tid; c < r; c += 256) m = fmax(m, t.diag[c]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
    if (lane == 0) wave_max[wave] = m;
    __syncthreads();
    m = fmin(fmax(fmax(fmax(wave_max[0], wave_max[1]), fmax(wave_max[2], wave_max[3])), 1e-280), 1e280);
    shift = kRitzShift * m;
    scale = ldexp(1., -(ilogb(m) / 2));
    if (tid == 0) { t.diag[rp] = shift; t.diag[rp + 1] = scale; }
  }
  if (ritz) low = shift * 0.0625;
  __syncthreads();
  if (wave != 0) return;
  // One wavefront factors block (s + 1, s + 1): lanes 0 .. 31 hold its rows, lanes 32 .. 63 those of the identity, and the
  // column operations that turn the block into L turn the identity into L^-T.
  const int row = lane & 31;
  const bool mine = lane < 32;
  double a[kCB];
#pragma unroll
  for (int c = 0; c < kCB; ++c) a[c] = mine ? Q[row * kLP + c] + (row == c ? shift : 0.) : (row == c ? 1. : 0.);
  unsigned bad = 0;
  // Column by column: scaled by 1 / sqrt(pivot), then taken out of the columns to its right.  Of the next two that happens at once, with two of
  // its entries moved from lane to scalar registers; of the others while the column after it is worked on, with its entries as
  // broadcast reads from LDS that have had that long to arrive.  What bounds a column is the chain from one pivot to the next, some twenty
  // dependent instructions with the Newton steps of the reciprocal root; the other work is dealt out between them, a part after each.
  double piv, y, w[2][kCB];
  bool out;
  auto pivot = [&](int c) {
    piv = lane_value(a[c], c);
    const double least = lane_value(low, c);
    out = !ritz && piv <= least;  // false for NaN, which is passed on
    if (ritz && piv < least) piv = least;
  };
  pivot(0);
  y = __builtin_amdgcn_rsq(piv);
  y = y * (1.5 - 0.5 * piv * y * y);
  y = y * (1.5 - 0.5 * piv * y * y);
  each_index([&](auto index) {
    constexpr int c = decltype(index)::value;
    if (out) { y = 0.; bad |= 1u << c; }
    a[c] = mine && row == c ? piv * y : a[c] * y;
    if (out) a[c] = 0.;
    if constexpr (c + 1 < kCB) {
      column[c & 1][lane] = a[c];   // lanes 32 .. 63: not read
#pragma unroll
      for (int e = c + 3; e < kCB; ++e) w[c & 1][e] = column[c & 1][e];
      __builtin_amdgcn_sched_barrier(0);
      a[c + 1] = __builtin_fma(-a[c], lane_value(a[c], c + 1), a[c + 1]);
      // column c - 1 out of columns c + 2 .. in 7 parts; column c out of column c + 2 after the first
      constexpr int left = kCB - c - 2;
      auto part = [&](auto i_t) {
        constexpr int i = decltype(i_t)::value, first = c + 2 + (left * i + 6) / 7, last = c + 2 + (left * (i + 1) + 6) / 7;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (c > 0) {
#pragma unroll
          for (int e = first; e < last; ++e) a[e] = __builtin_fma(-a[c - 1], w[(c - 1) & 1][e], a[e]);
        }
        if constexpr (i == 0 && c + 2 < kCB) a[c + 2] = __builtin_fma(-a[c], lane_value(a[c], c + 2), a[c + 2]);
        __builtin_amdgcn_sched_barrier(0);
      };
      using std::integral_constant;
      pivot(c + 1);
      y = __builtin_amdgcn_rsq(piv);
      const double half = 0.5 * piv;
      part(integral_constant<int, 0>{});
      part(integral_constant<int, 1>{});
      double u = half * y;
      part(integral_constant<int, 2>{});
      u = __builtin_fma(-y, u, 1.5);
      part(integral_constant<int, 3>{});
      y = y * u;
      part(integral_constant<int, 4>{});
      u = half * y;
      part(integral_constant<int, 5>{});
      u = __builtin_fma(-y, u, 1.5);
      part(integral_constant<int, 6>{});
      y = y * u;
    }
  }, std::make_integer_sequence<int, kCB>{});
  double* dnext = t.dinv + (size_t)((s + 1) & 1) * kCB * kCB;
#pragma unroll
  for (int c = 0; c < kCB; ++c) {
    if (!mine) dnext[c * kCB + row] = a[c];  // L^-1 = (L^-T)^T; exact zeros above the diagonal
    if (ritz && mine && i * kCB + row < r && i * kCB + c < r) t.Bw[(size_t)(i * kCB + c) * r + i * kCB + row] = row >= c ? (float)(scale * a[c]) : 0.f;
  }
  if (!ritz && mine) t.flag[i * kCB + row] = (bad >> row) & 1;
}

// Replaces the flagged rows of Qt by pseudo-random entries of mean square 1 / k.
__global__ __launch_bounds__(256) void refill_kernel(const RefreshGroup* __restrict__ gp, int pass) {
  const RefreshGroup& grp = *gp;
  const RefreshTensor& t = grp.t[blockIdx.y];
  const int row = blockIdx.x, k = t.k;
  if (!t.flag[row]) return;
  const float scale = 2.f * sqrtf(3.f / (float)k);
  for (int c = threadIdx.x; c < k; c += 256) {
    const uint64_t h = mix64(t.seed ^ mix64(((uint64_t)(pass + 1) << 56) + (uint64_t)row * (uint64_t)k + c));
    t.Q[(size_t)row * k + c] = scale * ((float)(h >> 40) * (1.f / 16777216.f) - 0.5f);
  }
}

hipError_t launch_factor(const RefreshGroup& grp, const RefreshGroup* dgrp, int ritz, double dependent, hipStream_t stream) {
  const int n = grp.count, r = grp.r;
  hipLaunchKernelGGL(gram_f64_kernel, dim3(tri((r + kCB - 1) / kCB), n), dim3(256), 0, stream, dgrp, ritz);
  const int nb = (r + kCB - 1) / kCB;
  for (int s = -1; s < nb; ++s)
    hipLaunchKernelGGL(chol_step_kernel, dim3(s < 0 ? 1 : 1 + nb + tri(nb) - tri(s + 1), n), dim3(256), 0, stream, dgrp, s, ritz, dependent);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_orthonormalise(const RefreshGroup& grp, const RefreshGroup* dgrp, int pass, bool final_round, hipStream_t stream) {
  GALORE_RETURN_IF(launch_factor(grp, dgrp, 0, final_round ? kDependent : kDependentRaw, stream));
  GemmGroup g{};
  g.count = grp.count;
  for (int i = 0; i < grp.count; ++i) {
    const RefreshTensor& t = grp.t[i];
    GemmProblem& p = g.p[i];  // Qt (r x k) = L^-1 Zt
    p.A = t.S; p.lda = grp.r; p.B = t.Z; p.ldb = t.k; p.M = grp.r; p.N = t.k; p.K = grp.r; p.C = t.Q; p.ldc = t.k;
  }
  GALORE_RETURN_IF(launch_product(g, DType::F32, false, stream));
  hipLaunchKernelGGL(refill_kernel, dim3(grp.r, grp.count), dim3(256), 0, stream, dgrp, pass);
  return hipGetLastError();
}

hipError_t launch_ritz_factor(const RefreshGroup& grp, const RefreshGroup* dgrp, hipStream_t stream) {
  return launch_factor(grp, dgrp, 1, 0., stream);
}

}  // namespace rf
}  // namespace galore
