// Fused low-rank Adam (Algorithm 2, update block): one pass over R, M, V that updates the
// fp32 moments in place, applies the bias correction and writes the normalised update N
// in the dtype the back-projection GEMM consumes.  Pure streaming: 16-byte vectors; R, M and V
// are read and M, V written with non-temporal accesses (each is touched once per step and the
// stack's moments are far larger than the caches), N is written normally because the
// back-projection GEMM reads it next.  Measured at 7B: 0.210 -> 0.204 ms per layer set.
#include <algorithm>

#include "adam_entry.hpp"
#include "common.hpp"

namespace galore {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void store_n(float* N, int64_t i, f32x4 n) { *reinterpret_cast<f32x4*>(N + i) = n; }
__device__ __forceinline__ void store_n(__bf16* N, int64_t i, f32x4 n) {
  bf16x4 o;
  o[0] = (__bf16)n[0]; o[1] = (__bf16)n[1]; o[2] = (__bf16)n[2]; o[3] = (__bf16)n[3];
  *reinterpret_cast<bf16x4*>(N + i) = o;
}

template <class TN>
__global__ __launch_bounds__(256) void adam_group_kernel(const AdamGroup grp) {
  const AdamProblem& pr = grp.p[blockIdx.y];
  const float beta1 = grp.beta1, beta2 = grp.beta2, eps = grp.eps;
  const float ic1 = pr.inv_c1, ic2 = pr.inv_c2;
  const float* __restrict__ R = pr.R;
  float* __restrict__ M = pr.M;
  float* __restrict__ V = pr.V;
  TN* __restrict__ N = static_cast<TN*>(pr.N);
  const int64_t count = pr.count;
  const int64_t nvec = count >> 2;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nvec; q += stride) {
    const int64_t i = q << 2;
    const f32x4 g = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(R + i));
    f32x4 m = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(M + i));
    f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(V + i));
    f32x4 n;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float me = m[e], ve = v[e];
      n[e] = adam_entry(g[e], me, ve, beta1, beta2, eps, ic1, ic2);
      m[e] = me; v[e] = ve;
    }
    __builtin_nontemporal_store(m, reinterpret_cast<f32x4*>(M + i));
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(V + i));
    store_n(N, i, n);
  }
  // ragged tail (count not a multiple of 4)
  if (blockIdx.x == 0) {
    const int64_t i = (nvec << 2) + threadIdx.x;
    if (threadIdx.x < 4 && i < count) {
      float me = M[i], ve = V[i];
      const float n = adam_entry(R[i], me, ve, beta1, beta2, eps, ic1, ic2);
      M[i] = me; V[i] = ve;
      N[i] = (TN)n;
    }
  }
}

// 16-byte access to four floats that are only 4-byte aligned (rows of odd length): the compiler picks
// the widest access the target allows at that alignment
__device__ __forceinline__ f32x4 load4(const float* p) { f32x4 v; __builtin_memcpy(&v, p, sizeof v); return v; }
__device__ __forceinline__ void store4(float* p, f32x4 v) { __builtin_memcpy(p, &v, sizeof v); }

// The update with N transposed (cols x rows) for problems with transpose_n, the back-projection GEMM's layout for a LEFT
// tensor, and row-wise for the others, in one launch.  One workgroup per 64 x 64 tile: R (or the slabs it is the sum of),
// M, V are read and M, V written row-wise in 16-byte pieces at element alignment; all pieces of a thread are requested
// before the first is used (as one piece after the other the kernel was a chain of four memory round trips per tile).
// A transposed N goes through a padded LDS tile and leaves column-wise in 16-byte pieces as well.
template <class TN>
__global__ __launch_bounds__(256) void adam_tile_group_kernel(const AdamGroup grp) {
  constexpr int TS = 64;
  constexpr int VEC = 16 / sizeof(TN);
  __shared__ __align__(16) TN tile[TS][TS + VEC];  // tile[j][i] = N[i][j]
  const AdamProblem& pr = grp.p[blockIdx.y];
  const int rows = pr.rows, cols = pr.cols, ldr = pr.ldr, slabs = pr.slabs;
  const int64_t stride = pr.slab_stride;
  const int tiles_c = (cols + TS - 1) / TS;
  const int ntiles = tiles_c * ((rows + TS - 1) / TS);
  const float beta1 = grp.beta1, beta2 = grp.beta2, eps = grp.eps;
  const float ic1 = pr.inv_c1, ic2 = pr.inv_c2;
  const bool tr = pr.transpose_n != 0;
  const float* __restrict__ R = pr.R;
  float* __restrict__ M = pr.M;
  float* __restrict__ V = pr.V;
  TN* __restrict__ N = static_cast<TN*>(pr.N);
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int i0 = (t / tiles_c) * TS, j0 = (t % tiles_c) * TS;
    const int j = j0 + (threadIdx.x & 15) * 4;
    const bool whole = j + 4 <= cols;
    const int jc = whole ? j : 0;  // lanes without a whole piece read the row's first elements and leave them alone (cols >= 4 there)
    f32x4 g[4], m[4], v[4];
    if (cols >= 4) {
#pragma unroll
      for (int ps = 0; ps < 4; ++ps) {
        const int i = i0 + ps * 16 + (threadIdx.x >> 4), ic = i < rows ? i : rows - 1;
        const float* Ri = R + (size_t)ic * ldr + jc;
        g[ps] = load4(Ri);
        m[ps] = load4(M + (size_t)ic * cols + jc);
        v[ps] = load4(V + (size_t)ic * cols + jc);
      }
      for (int s = 1; s < slabs; s += 2) {  // two slabs of all pieces at a time, added in slab order
        const float* Rs = R + s * stride;
        const int64_t second = s + 1 < slabs ? stride : 0;
        f32x4 x[2][4];
#pragma unroll
        for (int ps = 0; ps < 4; ++ps) {
          const int i = i0 + ps * 16 + (threadIdx.x >> 4), ic = i < rows ? i : rows - 1;
          x[0][ps] = load4(Rs + (size_t)ic * ldr + jc);
          x[1][ps] = load4(Rs + second + (size_t)ic * ldr + jc);
        }
#pragma unroll
        for (int ps = 0; ps < 4; ++ps) {
          g[ps] += x[0][ps];
          if (second) g[ps] += x[1][ps];
        }
      }
    }
#pragma unroll
    for (int ps = 0; ps < 4; ++ps) {
      const int i = i0 + ps * 16 + (threadIdx.x >> 4);
      if (i >= rows || j >= cols) continue;
      float n[4];
      if (whole) {
        f32x4 mo, vo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float me = m[ps][e], ve = v[ps][e];
          n[e] = adam_entry(g[ps][e], me, ve, beta1, beta2, eps, ic1, ic2);
          mo[e] = me; vo[e] = ve;
        }
        store4(M + (size_t)i * cols + j, mo);
        store4(V + (size_t)i * cols + j, vo);
      } else {  // the piece that straddles the end of the row
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          n[e] = 0.f;
          if (j + e < cols) {
            const float* p = R + (size_t)i * ldr + j + e;
            float ge = *p;
            for (int s = 1; s < slabs; ++s) ge += p[s * stride];
            float me = M[(size_t)i * cols + j + e], ve = V[(size_t)i * cols + j + e];
            n[e] = adam_entry(ge, me, ve, beta1, beta2, eps, ic1, ic2);
            M[(size_t)i * cols + j + e] = me;
            V[(size_t)i * cols + j + e] = ve;
          }
        }
        n[3] = 0.f;
      }
      if (tr) {
#pragma unroll
        for (int e = 0; e < 4; ++e) tile[j - j0 + e][i - i0] = (TN)n[e];
      } else {
        TN o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (TN)n[e];
        TN* dst = N + (size_t)i * cols + j;
        if (whole) __builtin_memcpy(dst, o, sizeof o);
        else
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (j + e < cols) dst[e] = o[e];
      }
    }
    if (tr) {
      __syncthreads();
      constexpr int LPR = TS / VEC;        // lanes per output row
      constexpr int RPP = 256 / LPR;       // output rows per pass
#pragma unroll
      for (int ps = 0; ps < TS / RPP; ++ps) {
        const int jj = ps * RPP + threadIdx.x / LPR, i = (threadIdx.x % LPR) * VEC;
        if (j0 + jj >= cols || i0 + i >= rows) continue;
        TN* dst = N + (size_t)(j0 + jj) * rows + i0 + i;
        if (i0 + i + VEC <= rows) {
          const uint4 o = *reinterpret_cast<const uint4*>(&tile[jj][i]);
          __builtin_memcpy(dst, &o, sizeof o);
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e)
            if (i0 + i + e < rows) dst[e] = tile[jj][i + e];
        }
      }
      __syncthreads();
    }
  }
}

// Transposing variant for launches whose tiles are all full and aligned (every LEFT tensor of a large stack) and whose R is
// one matrix: R, M, V row-wise with 16-byte non-temporal accesses, one 16-element trip of a thread at a time.  42 registers
// per lane (bf16 N; allocated in eights: 48), which is what lets a wavefront of it share a SIMD with the two wavefronts of the projection GEMM
// (2 x 232 of the 512 registers per lane): the Adam pass of one call then runs on the CUs that the projection of the next
// call occupies.  The non-temporal loads of R, M and V leave less of N in the L2 for the product that follows (at 7B it reads
// 1205 MB per layer set instead of 1125) and are faster all the same: 1024 x 11008 on data that is not in cache 63 -> 53 us, three 7B
// layers 2990 -> 2953 (resident data, which no step of a model has: 41 -> 48).
template <class TN>
__global__ __launch_bounds__(256) void adam_transpose_group_kernel(const AdamGroup grp) {
  constexpr int TS = 64;
  constexpr int VEC = 16 / sizeof(TN);          // N elements per 16 bytes
  __shared__ __align__(16) TN tile[TS][TS + VEC];  // tile[j][i] = N[i][j]
  const AdamProblem& pr = grp.p[blockIdx.y];
  const int rows = pr.rows, cols = pr.cols, ldr = pr.ldr;
  const int tiles_c = cols / TS;
  const int ntiles = tiles_c * (rows / TS);
  const float beta1 = grp.beta1, beta2 = grp.beta2, eps = grp.eps;
  const float ic1 = pr.inv_c1, ic2 = pr.inv_c2;
  const float* __restrict__ R = pr.R;
  float* __restrict__ M = pr.M;
  float* __restrict__ V = pr.V;
  TN* __restrict__ N = static_cast<TN*>(pr.N);
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int i0 = (t / tiles_c) * TS, j0 = (t % tiles_c) * TS;
    // tile origin as a (wave-uniform) pointer, in-tile offsets in 32 bits: fewer address registers per lane
    const float* __restrict__ Rt = R + ((size_t)i0 * ldr + j0);
    float* __restrict__ Mt = M + ((size_t)i0 * cols + j0);
    float* __restrict__ Vt = V + ((size_t)i0 * cols + j0);
#pragma unroll 1
    for (int ps = 0; ps < 4; ++ps) {
      const int i = ps * 16 + (threadIdx.x >> 4), j = (threadIdx.x & 15) * 4;
      const int idx = i * cols + j;
      const int ridx = i * ldr + j;
      const f32x4 g = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(Rt + ridx));
      f32x4 m = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(Mt + idx));
      f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(Vt + idx));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float me = m[e], ve = v[e];
        tile[j + e][i] = (TN)adam_entry(g[e], me, ve, beta1, beta2, eps, ic1, ic2);
        m[e] = me; v[e] = ve;
      }
      __builtin_nontemporal_store(m, reinterpret_cast<f32x4*>(Mt + idx));
      __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(Vt + idx));
    }
    __syncthreads();
    constexpr int LPR = TS / VEC;        // lanes per output row
    constexpr int RPP = 256 / LPR;       // output rows per pass
#pragma unroll
    for (int ps = 0; ps < TS / RPP; ++ps) {
      const int j = ps * RPP + threadIdx.x / LPR, i = (threadIdx.x % LPR) * VEC;
      *reinterpret_cast<uint4*>(N + (size_t)(j0 + j) * rows + i0 + i) = *reinterpret_cast<const uint4*>(&tile[j][i]);
    }
    __syncthreads();
  }
}

// A launch whose problems are all streams of full, aligned tiles and large enough to be bound by HBM goes to the lean
// kernels, one launch per orientation; everything else runs as one launch of the tile kernel.  On data that is not in cache, us, tile
// kernel / lean kernel: 256 x 4096 (1 Mi entries) transposed 11.3 / 9.5, row-wise 11.4 / 9.0; 512 x 5504 20.3 / 16.0 and 20.4 / 14.2;
// the same within 1 us below.
hipError_t launch_adam_group(const AdamGroup& g, DType n_dtype, hipStream_t stream) {
  if (g.count <= 0) return hipSuccess;
  if (g.count > kMaxGroup) return hipErrorInvalidValue;
  constexpr int64_t ENTRIES_LEAN = (int64_t)1 << 20;
  AdamGroup lean[2] = {}, rest{};
  int64_t entries = 0;
  for (int i = 0; i < g.count; ++i) entries += g.p[i].count;
  for (AdamGroup* x : {&lean[0], &lean[1], &rest}) { x->beta1 = g.beta1; x->beta2 = g.beta2; x->eps = g.eps; }
  for (int i = 0; i < g.count; ++i) {
    const AdamProblem& p = g.p[i];
    if (p.rows < 1 || p.cols < 1) continue;
    if (p.ldr < p.cols || (!p.transpose_n && p.ldr != p.cols)) return hipErrorInvalidValue;  // padded rows of R only with transpose_n
    const bool aligned = ((reinterpret_cast<uintptr_t>(p.R) | reinterpret_cast<uintptr_t>(p.M) | reinterpret_cast<uintptr_t>(p.V) | reinterpret_cast<uintptr_t>(p.N)) & 15) == 0 && p.ldr % 4 == 0;
    const bool full = !p.transpose_n || (p.rows % 64 == 0 && p.cols % 64 == 0);
    AdamGroup& to = entries >= ENTRIES_LEAN && aligned && full && p.slabs <= 1 ? lean[p.transpose_n ? 1 : 0] : rest;
    to.p[to.count++] = p;
  }
  if (lean[1].count > 0) {
    int64_t maxtiles = 0;
    for (int i = 0; i < lean[1].count; ++i) maxtiles = std::max(maxtiles, (int64_t)(lean[1].p[i].rows / 64) * (lean[1].p[i].cols / 64));
    const dim3 grid((unsigned)(maxtiles > 4096 ? 4096 : maxtiles), (unsigned)lean[1].count);
    if (n_dtype == DType::BF16) hipLaunchKernelGGL(adam_transpose_group_kernel<__bf16>, grid, dim3(256), 0, stream, lean[1]);
    else hipLaunchKernelGGL(adam_transpose_group_kernel<float>, grid, dim3(256), 0, stream, lean[1]);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (lean[0].count > 0) {
    int64_t maxcount = 0;
    for (int i = 0; i < lean[0].count; ++i) maxcount = std::max(maxcount, lean[0].p[i].count);
    // 4 elements per thread per trip; enough blocks for ~4 trips each, capped to fill the chip a few times over
    int64_t blocks = (maxcount / 4 + 256 * 4 - 1) / (256 * 4);
    if (blocks < 1) blocks = 1;
    if (blocks > 2048) blocks = 2048;
    const dim3 grid((unsigned)blocks, (unsigned)lean[0].count);
    if (n_dtype == DType::BF16) hipLaunchKernelGGL(adam_group_kernel<__bf16>, grid, dim3(256), 0, stream, lean[0]);
    else hipLaunchKernelGGL(adam_group_kernel<float>, grid, dim3(256), 0, stream, lean[0]);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (rest.count > 0) {
    int64_t maxtiles = 0;
    for (int i = 0; i < rest.count; ++i) maxtiles = std::max(maxtiles, (int64_t)((rest.p[i].rows + 63) / 64) * ((rest.p[i].cols + 63) / 64));
    const dim3 grid((unsigned)(maxtiles > 4096 ? 4096 : maxtiles), (unsigned)rest.count);
    if (n_dtype == DType::BF16) hipLaunchKernelGGL(adam_tile_group_kernel<__bf16>, grid, dim3(256), 0, stream, rest);
    else hipLaunchKernelGGL(adam_tile_group_kernel<float>, grid, dim3(256), 0, stream, rest);
    return hipGetLastError();
  }
  return hipSuccess;
}

// One aligned 16-byte piece of dst per thread and trip; the source piece is read with whatever
// alignment its row has (memcpy lets the compiler pick the widest access the target allows there).
__global__ __launch_bounds__(256) void pad_rows_kernel(const PadGroup grp) {
  const PadProblem& pr = grp.p[blockIdx.y];
  const __bf16* __restrict__ src = static_cast<const __bf16*>(pr.src);
  __bf16* __restrict__ dst = static_cast<__bf16*>(pr.dst);
  const int cols = pr.cols, cpr = pr.ldd / 8;  // pieces per row
  const int64_t pieces = (int64_t)pr.rows * cpr;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < pieces; c += stride) {
    const int64_t row = c / cpr;
    const int col = (int)(c % cpr) * 8;
    const __bf16* s = src + row * pr.lds + col;
    uint4 v;
    if (col + 8 <= cols) {
      __builtin_memcpy(&v, s, sizeof(uint4));
    } else {
      __bf16 tmp[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) tmp[e] = col + e < cols ? s[e] : (__bf16)0.f;
      __builtin_memcpy(&v, tmp, sizeof(uint4));
    }
    *reinterpret_cast<uint4*>(dst + row * pr.ldd + col) = v;
  }
}

hipError_t launch_pad_rows_group(const PadGroup& g, hipStream_t stream) {
  if (g.count <= 0) return hipSuccess;
  if (g.count > kMaxGroup) return hipErrorInvalidValue;
  int64_t most = 0;
  for (int i = 0; i < g.count; ++i) {
    const PadProblem& p = g.p[i];
    if (p.rows < 1 || p.cols < 1 || p.ldd < p.cols || p.ldd % 8 != 0 || p.lds < p.cols || (reinterpret_cast<uintptr_t>(p.dst) & 15))
      return hipErrorInvalidValue;
    const int64_t pieces = (int64_t)p.rows * (p.ldd / 8);
    most = pieces > most ? pieces : most;
  }
  int64_t blocks = (most + 256 * 4 - 1) / (256 * 4);
  if (blocks < 1) blocks = 1;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(pad_rows_kernel, dim3((unsigned)blocks, (unsigned)g.count), dim3(256), 0, stream, g);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void fill_zero_kernel(unsigned char* p, size_t bytes) {
  const size_t nvec = bytes / 16;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const size_t first = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint4* pv = reinterpret_cast<uint4*>(p);
  for (size_t i = first; i < nvec; i += stride) pv[i] = make_uint4(0u, 0u, 0u, 0u);
  const size_t tail = nvec * 16 + first;  // fewer than 16 trailing bytes
  if (tail < bytes) p[tail] = 0;
}

// Zero `bytes` at a 16-byte-aligned pointer with a plain kernel (not a memset node), so the
// call can be recorded in a HIP graph like every other piece of the library's work.
hipError_t launch_fill_zero(void* ptr, size_t bytes, hipStream_t stream) {
  if (bytes == 0) return hipSuccess;
  size_t blocks = (bytes / 16 + 255) / 256;
  if (blocks < 1) blocks = 1;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, stream,
                     static_cast<unsigned char*>(ptr), bytes);
  return hipGetLastError();
}

// dst (cols x rows) = src^T through a padded 64 x 64 LDS tile, any shape, stride and alignment: whole 16-byte pieces are read and written at
// element alignment, the rest of a row element by element.  Bound by the latency of one trip (a tile per workgroup): the projector of
// a 4096 x 11008 weight at r = 1024 (8 MB) takes 7.5 us, element by element 11.6.
template <class T>
__global__ __launch_bounds__(256) void transpose_group_kernel(const TransposeGroup grp) {
  constexpr int TS = 64, VEC = 16 / (int)sizeof(T), PPR = TS / VEC, RPP = 256 / PPR, PASSES = TS / RPP;
  __shared__ T tile[TS][TS + 4 / (int)sizeof(T)];
  const TransposeProblem& pr = grp.p[blockIdx.y];
  const T* __restrict__ src = static_cast<const T*>(pr.src);
  T* __restrict__ dst = static_cast<T*>(pr.dst);
  const int tiles_c = (pr.cols + TS - 1) / TS;
  const int ntiles = tiles_c * ((pr.rows + TS - 1) / TS);
  const int o = threadIdx.x / PPR, x = threadIdx.x % PPR * VEC;
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int i0 = (t / tiles_c) * TS, j0 = (t % tiles_c) * TS;
    T piece[PASSES][VEC];
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      const int i = i0 + o + ps * RPP, j = j0 + x;
      const T* from = src + (size_t)i * pr.lds + j;
      if (i < pr.rows && j + VEC <= pr.cols) {
        __builtin_memcpy(piece[ps], from, 16);
      } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) piece[ps][e] = i < pr.rows && j + e < pr.cols ? from[e] : (T)0.f;
      }
    }
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps)
#pragma unroll
      for (int e = 0; e < VEC; ++e) tile[o + ps * RPP][x + e] = piece[ps][e];
    __syncthreads();
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      const int j = o + ps * RPP;
      T out[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) out[e] = tile[x + e][j];
      if (j0 + j >= pr.cols) continue;
      T* to = dst + (size_t)(j0 + j) * pr.ldd + i0 + x;
      if (i0 + x + VEC <= pr.rows) {
        __builtin_memcpy(to, out, 16);
      } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e)
          if (i0 + x + e < pr.rows) to[e] = out[e];
      }
    }
    __syncthreads();
  }
}

hipError_t launch_transpose_group(const TransposeGroup& g, DType dt, hipStream_t stream) {
  if (g.count <= 0) return hipSuccess;
  if (g.count > kMaxGroup) return hipErrorInvalidValue;
  int64_t maxtiles = 0;
  for (int i = 0; i < g.count; ++i) {
    const int64_t t = (int64_t)((g.p[i].rows + 63) / 64) * ((g.p[i].cols + 63) / 64);
    maxtiles = t > maxtiles ? t : maxtiles;
  }
  if (maxtiles == 0) return hipSuccess;
  const dim3 grid((unsigned)(maxtiles > 2048 ? 2048 : maxtiles), (unsigned)g.count);
  if (dt == DType::BF16) hipLaunchKernelGGL(transpose_group_kernel<__bf16>, grid, dim3(256), 0, stream, g);
  else hipLaunchKernelGGL(transpose_group_kernel<float>, grid, dim3(256), 0, stream, g);
  return hipGetLastError();
}

}  // namespace galore
