// Shared pieces of the subspace refresh (Algorithm 2, refresh branch; Sec. 3.3 SVD equation): the per-tensor
// descriptor table the kernels read, workspace layout, tuning constants, block reductions, and the entry points
// of the long launch sequences (Householder QR in refresh_qr.hip, Cholesky QR in refresh_chol.hip, Rayleigh-Ritz eigen-solve
// in refresh_ritz.hip) that the driver in refresh.hip strings together.
#pragma once
#include <cstdlib>
#include <type_traits>

#include "refresh.hpp"

namespace galore {
namespace rf {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

constexpr int kJacobiSweeps = 10;   // upper bound; sweeps after convergence return at once
constexpr float kJacobiTol = 1e-5f;  // |b_p.b_q| <= tol |b_p||b_q|: a few times the rounding floor of an fp32 dot of length r
// A sweep whose largest rotation stayed below this level is the last one (Gram-matrix kernel): inner
// products of long fp32 rows keep crossing kJacobiTol by rounding alone, so "no rotation at all" is
// rarely reached although the result has stopped changing.
constexpr float kJacobiStopTol = 4e-5f;
// The Cholesky path (below) rotates the rows of a factor L^T of the Rayleigh-Ritz matrix, whose lengths are the square roots of
// the Ritz values, so the same inner product is twice the angle; and no rotation is accumulated, so tighter levels cost little.
// At levels of 5e-6 / 2e-6 / 1e-6 (stop level five times that): error of a column against 64 bits, root mean square, in units of
// 2^-24 lambda_1 / (distance to the next Ritz value), r = 64 .. 256: 9 to 19 / 5 to 8 / 3 to 6 (Householder path 10 to 20); a refresh of
// seven 1024 x 2736 gradients, ms, at r = 256 3.13 / 3.19 / 3.18, at r = 255 6.65 / 6.73 / 7.22.
// The kernels that stage rows (r of no multiple of 4) have no stop level: a sweep follows while anything rotates.
constexpr float kFactorTol = 2e-6f;
constexpr float kFactorStopTol = 1e-5f;
// Largest rank of the Cholesky path (refresh_chol.hip); higher ranks take Householder QR and Jacobi on the Rayleigh-Ritz matrix itself.
// The Cholesky path is faster at every rank (7B layer set, r = 1024: 34 ms against 61) and its vectors are closer to those of 64 bits:
// root mean square error of a column, r directions inside a factor of 8, fp32, k = 2048, Householder / Cholesky: r = 64 4.1e-5 /
// 2.7e-5, 128 6.9e-5 / 2.7e-5, 256 1.6e-4 / 6.3e-5, 512 3.3e-4 / 1.6e-4, 768 9.4e-4 / 3.5e-4, 1024 1.1e-3 / 5.3e-4.  So accuracy
// sets no line.  What a change of path can change is the sign of a column whose two largest entries tie to within its error.
// Columns signed otherwise than in 64 bits, Householder / Cholesky: r up to 128 0 / 0 of 1120, 256 2 / 0 of 1280, 384 0 / 0 of 1920,
// 512 2 / 1 of 2560, 768 0 / 0 of 1536, 1024 2 / 0 of 2048.  The line stands where the projectors of the two paths still
// agree to 1e-3 in norm on the layers measured (350M 8e-4, 60M 1e-4), signs included; above it they stay, bit for bit, the Householder
// path's, for the runs that are resumed or compared with earlier ones.
constexpr int kCholeskyMaxRank = 256;
inline bool cholesky_path(int64_t r) { return r <= kCholeskyMaxRank; }
constexpr int kNB = 8;               // reflectors per Householder panel (block_sum_vec sums 8 values)
constexpr int kRPT = 4;              // rows per thread in the panel kernels (1024 threads): k - j0 <= 4096
constexpr int kSW = 8;               // columns per block in the blocked reflector application

struct RefreshTensor {
  float* C;      // k x k Gram matrix
  float* Q;      // Qt: r x k, the iteration block transposed
  float* Z;      // Zt: r x k, product block / factored reflectors / fp32 projector, transposed
  float* Bw;     // r x r Rayleigh-Ritz matrix (Cholesky path: its transposed Cholesky factor), rotated in place
  float* Jt;     // r x r accumulated rotations (rows = eigenvectors); Householder path only, null on the Cholesky path
  float* S;      // St: r x r, rows = eigenvectors, ordered by decreasing Ritz value, unit length (Cholesky path: before, the inverse factor of a QR)
  float* tau;    // r: factors of the reflectors; later the reciprocal lengths of the eigenvectors (both paths)
  union {
    struct {         // Householder path
      float* vscale; // r
      float* vclean; // round_up(r, 32) x k: reflectors as plain vectors (unit diagonal, zeros above, scaled), transposed
      float* tmat;   // (r / 32 macro panels) x 32 x 32: triangular factors T of the compact WY form
      float* tpart;  // 8 x 32 x 32: shares of V^T V of the macro panel being prepared
      float* wpart;  // (r / 32 + 1) x 4 x 32 x 32: shares of w = x V^T, per block of 32 target rows and slice of positions
    };
    struct {         // Cholesky path
      double* A0;    // lower triangle of 32 x 32 blocks, twice: the matrix being factored (see chol_step_kernel)
      double* A1;
      double* diag;  // round_up(r, 32) + 2: diagonal of the matrix being factored; its shift and scale
      double* dinv;  // 2 x 32 x 32: inverse of the diagonal block of the step
      int32_t* flag; // round_up(r, 32): dependent columns
    };
  };
  float* lambda; // r
  int32_t* order;// r : order[i] = output column of eigenvector i
  int32_t* sweep_flag;  // kJacobiSweeps + 1 : sweep s rotated something
  void* proj_t;  // output, r x k, ld ldpt (the projector itself is its transpose)
  int32_t k;
  int32_t ldpt;
  uint64_t seed;
  int32_t proj_is_bf16;  // dtype of proj_t
  int32_t split;         // Zt = Qt C runs as a bf16 product of three-way split operands (see split3)
  __bf16* Csplit;        // k x 6k: row n = [hi | mid | hi | mid | lo | hi] parts of row n of C
  __bf16* Qsplit;        // r x 6k: row i = [hi | hi | mid | mid | hi | lo] parts of row i of Qt

  // Cholesky path, r x r: the factor that makes St orthonormal, formed when the last factorisation is done with A0
  __host__ __device__ float* T() const { return reinterpret_cast<float*>(A0); }
};

// The kernels of the long launch sequences (QR panels, Jacobi rounds: about two thousand launches per
// refresh) read this table from device memory through a pointer; the few one-off kernels take it by
// value.  By value every launch would put 2.7 KB into the runtime's kernel-argument ring, whose few MB
// then hold only some hundred launches: the host thread ends up waiting for the GPU launch by launch
// for the whole refresh instead of running ahead of it.
struct RefreshGroup {
  int32_t count;
  int32_t r;
  RefreshTensor t[kMaxGroup];
};
static_assert(sizeof(RefreshGroup) <= 4096 - 256, "some kernels take the table, and a little more, by value: 4 KB of kernel arguments");

struct Layout {
  size_t C, Q, Z, Bw, Jt, S, A0, A1, diag, dinv, flag, tau, vscale, vclean, tmat, tpart, wpart, lambda, order, sweep_flag, group, Csplit, Qsplit, total;
};

bool split_products(int64_t k, int64_t r);
Layout layout_for(int64_t k, int64_t r);

inline unsigned blocks_for(int64_t count, int per_block, unsigned cap) {
  int64_t b = (count + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (unsigned)b;
}

#define GALORE_RETURN_IF(e_)            \
  do {                                  \
    hipError_t _e = (e_);               \
    if (_e != hipSuccess) return _e;    \
  } while (0)

// Householder QR of Zt (r x k per tensor, transposed layout) of every tensor of the group, reflectors left in Zt,
// then Qt <- the orthonormal factor (refresh_qr.hip).  dgrp: the group's table in device memory; kmax: largest short side.
hipError_t launch_householder_qr(const RefreshGroup& grp, const RefreshGroup* dgrp, int64_t kmax, hipStream_t stream);
// Cholesky path: Qt <- orthonormal rows spanning those of Zt (refresh_chol.hip).  pass: number of this pass within the
// refresh; final_round: of the last round, whose passes work on the result of the one before and have to end orthonormal.
hipError_t launch_orthonormalise(const RefreshGroup& grp, const RefreshGroup* dgrp, int pass, bool final_round, hipStream_t stream);
// Cholesky path: Bw <- L^T with L L^T = Qt Zt^T, the Rayleigh-Ritz matrix, shifted by a little of its norm (refresh_chol.hip).
hipError_t launch_ritz_factor(const RefreshGroup& grp, const RefreshGroup* dgrp, hipStream_t stream);
// Eigen-decomposition of the symmetric r x r matrix in Bw (Cholesky path: given by its transposed factor) by blocked
// one-sided Jacobi, eigenvectors ordered by decreasing Ritz value and normalised into S (Cholesky path: Bw) (refresh_ritz.hip).
hipError_t launch_ritz_solve(const RefreshGroup& grp, const RefreshGroup* dgrp, bool crowded, hipStream_t stream);

namespace {

// ---- block reductions (wavefront shuffles, then LDS across the waves) ------------------------
// Sum over the 64 lanes of a wavefront; every lane gets the result.  Data-parallel-primitive
// moves inside the VALU (quad permutes, row mirrors, row broadcasts) instead of LDS-crossbar
// shuffles: six dependent adds of a few cycles each where six ds_bpermute round trips took
// well over a hundred cycles apiece.
__device__ __forceinline__ float wave_sum(float v) {
  auto dpp = [](float x, auto ctrl, auto row_mask) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                                                 decltype(row_mask)::value, 0xF, false));
  };
  using std::integral_constant;
  v += dpp(v, integral_constant<int, 0xB1>{}, integral_constant<int, 0xF>{});   // quad_perm [1,0,3,2]
  v += dpp(v, integral_constant<int, 0x4E>{}, integral_constant<int, 0xF>{});   // quad_perm [2,3,0,1]
  v += dpp(v, integral_constant<int, 0x141>{}, integral_constant<int, 0xF>{});  // row_half_mirror
  v += dpp(v, integral_constant<int, 0x140>{}, integral_constant<int, 0xF>{});  // row_mirror: each row of 16 holds its sum
  v += dpp(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});  // row_bcast15 into rows 1 and 3
  v += dpp(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});  // row_bcast31 into rows 2 and 3
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// Sum over all threads of the block; every thread gets the result.  `red` holds >= 16 floats.
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[wave] = v;
  __syncthreads();
  float s = 0.f;
  for (int w = 0; w < nw; ++w) s += red[w];
  return s;
}

// ---- counter-based pseudo-random bits --------------------------------------------------------
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// which 0: Qt <- [I_r 0] (r x k);  which 1: Jt <- I_r and the sweep flags <- 0
__global__ __launch_bounds__(256) void identity_fill_kernel(const RefreshGroup* __restrict__ gp, int which) {
  const RefreshGroup& grp = *gp;
  const RefreshTensor& t = grp.t[blockIdx.y];
  const int r = grp.r;
  if (which == 1 && blockIdx.x == 0 && threadIdx.x <= kJacobiSweeps) t.sweep_flag[threadIdx.x] = 0;
  if (which == 1 && !t.Jt) return;
  float* X = which == 0 ? t.Q : t.Jt;
  const int64_t width = which == 0 ? t.k : r;
  const int64_t count = width * r;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
    X[i] = (i / width == i % width) ? 1.f : 0.f;
}

}  // namespace
}  // namespace rf
}  // namespace galore
