// Small-tile grouped MFMA GEMM (gfx950): C = A B with A as [M][K] (or, for Gram matrices, [K][M]) and B as [K][N] or [N][K], bf16 or fp32 operands at
// any element alignment, fp32 accumulate, optionally with the contraction cut into pieces.
//
// The 256 x 256 kernels (gemm_mfma_dl.hpp, gemm_proj_dl.hpp) need hundreds of tiles to fill the chip; a layer of a
// small stack, a single weight or a low rank gives them a few dozen, each a serial chain of K steps at one memory
// latency apiece.  Here a workgroup of 4 wavefronts owns a 64 x 64 (or 128 x 128) tile and several workgroups share a
// CU, so the latency of one is hidden by the others, and a launch has 4 to 16 times as many of them:
//   * operands go global -> registers -> LDS in 16-byte pieces.  The pieces of the next K step are requested before the
//     current one is multiplied.  Pieces are read at element alignment from addresses clamped into the matrix, without a
//     branch; where a tile reaches past an edge the registers are shifted (zeros move in) before they are stored to
//     LDS, so rows of any length and any first element run at the speed of aligned ones.
//   * `splits` pieces of the contraction (StoreF32) go to separate slabs that the consumer adds in slab order: no
//     atomics, no second launch.
//   * the weight update reads its W tile before the K loop and writes it back as 16-byte pieces after a trip of the
//     accumulators through LDS.
// The order of the additions of one element is that of the 256 x 256 kernels (16 k per bf16 MFMA, ascending), so without
// `splits` the results are the same bits whichever kernel a tensor takes.
#pragma once
#include <cstdlib>
#include <type_traits>

#include "adam_entry.hpp"
#include "gemm_mfma_dl.hpp"

namespace galore {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

template <class T, int BX, int BK> struct TileOperand {
  using ET = ElemTraits<T>;
  static constexpr int VEC = ET::VEC;
  static constexpr int PIECES = BX * BK / VEC;
  static constexpr int PER = PIECES / 256;
  static_assert(PIECES % 256 == 0, "pieces divide evenly over the workgroup");
  static constexpr bool SWZ = sizeof(T) == 2 && BX == 64;  // rows of 128 bytes: unpadded, 64-byte halves swapped every other row pair
  static constexpr int PK = BK + ET::PADK;
  static constexpr int PX = SWZ ? BX : BX + ET::PADX;
  static constexpr int LDS_ELEMS = BX * PK > BK * PX ? BX * PK : BK * PX;

  // Requests this thread's pieces of the tile at (x0, k).  X, K: extents (X >= VEC or K >= VEC along the contiguous index).
  template <bool KC>
  static __device__ __forceinline__ void load(u32x4 (&regs)[PER], const T* __restrict__ base, int ld, int x0, int X, int k, int K, int tid) {
    constexpr int CPR = (KC ? BK : BX) / VEC;
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int c = tid + it * 256;
      int o = (KC ? x0 : k) + c / CPR, i = (KC ? k : x0) + (c % CPR) * VEC;
      const int olast = (KC ? X : K) - 1, ilast = (KC ? K : X) - VEC;
      o = o < olast ? o : olast;
      i = i < ilast ? i : ilast;
      __builtin_memcpy(&regs[it], base + (size_t)o * ld + i, sizeof(u32x4));
    }
  }

  // v shifted towards its first element by n elements, zeros shifted in (n >= VEC: all zero)
  static __device__ __forceinline__ u32x4 shift_out(u32x4 v, int n) {
    const int w = sizeof(T) == 2 ? n >> 1 : n;
    if (sizeof(T) == 2) {
      const bool half = n & 1;
      const u32x4 s = {__builtin_amdgcn_alignbit(v.y, v.x, 16), __builtin_amdgcn_alignbit(v.z, v.y, 16),
                       __builtin_amdgcn_alignbit(v.w, v.z, 16), v.w >> 16};
      v = half ? s : v;
    }
    v = (w & 1) ? u32x4{v.y, v.z, v.w, 0u} : v;
    v = (w & 2) ? u32x4{v.z, v.w, 0u, 0u} : v;
    return w >= 4 ? u32x4{0u, 0u, 0u, 0u} : v;
  }

  // Stores the pieces requested by load() with the same arguments.  `edge` (uniform): the tile reaches past the matrix.
  template <bool KC>
  static __device__ __forceinline__ void store(u32x4 (&regs)[PER], T* lds, int x0, int X, int k, int K, bool edge, int tid) {
    constexpr int CPR = (KC ? BK : BX) / VEC;
    if (edge) {
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        const int c = tid + it * 256;
        const int i = (KC ? k : x0) + (c % CPR) * VEC, ilast = (KC ? K : X) - VEC;
        int n = i > ilast ? i - ilast : 0;
        if (!KC && k + c / CPR >= K) n = VEC;  // a row past the end of the contraction
        regs[it] = shift_out(regs[it], n < VEC ? n : VEC);
      }
    }
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int c = tid + it * 256;
      const int o = c / CPR, i = (c % CPR) * VEC;
      T* dst = KC ? lds + o * PK + i : lds + o * PX + (SWZ ? i ^ (32 * ((o >> 1) & 1)) : i);
      *reinterpret_cast<u32x4*>(dst) = regs[it];
    }
  }

  // MFMA operand of the 32 rows (columns) from x on, k = kk .. kk + KSTEP - 1 (see Frag in gemm_mfma.hpp)
  template <bool KC> static __device__ __forceinline__ void frag(Frag<T>& f, const T* lds, int x, int kk, int lane) {
    if constexpr (KC) {
      f.template load_k<PK>(lds, x, kk, lane);
    } else if constexpr (SWZ) {
      const int s = lane & 15, g = lane >> 4;
      const int row = kk + 8 * (g >> 1) + (s >> 2);
      const T* p = lds + row * PX + ((x + 16 * (g & 1) + 4 * (s & 3)) ^ (32 * ((row >> 1) & 1)));
      typedef s16x4 __attribute__((address_space(3))) * lds_v4;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(p + 4 * PX));
      f.v = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
      f.template load_x<PX>(lds, x, kk, lane);
    }
  }
};

template <class T, int BM_, int BN_> struct SmallTile {
  static constexpr int BM = BM_, BN = BN_;
  static constexpr int BK = (BM_ * BN_ <= 64 * 64 ? 256 : 128) / (int)sizeof(T);  // 64 x 64: 128 (bf16) or 64 (fp32); larger tiles: 64 or 32
  using A = TileOperand<T, BM, BK>;
  using B = TileOperand<T, BN, BK>;
  static constexpr int SP = BN + 4;                        // floats per row of the epilogue's staging area
  static constexpr int OPERAND_BYTES = (A::LDS_ELEMS + B::LDS_ELEMS) * (int)sizeof(T);
  static constexpr int ROWS = 64;                          // rows staged at a time
  static constexpr int STAGE_BYTES = ROWS * SP * 4;
  static constexpr int NPITCH = ROWS + 16 / (int)sizeof(T);  // elements per column of the transposed N tile
  static constexpr int NT_BYTES = BN * NPITCH * (int)sizeof(T);
  static constexpr int lds_bytes_groups(int kg) {  // KG groups with the Adam epilogue
    return kg * OPERAND_BYTES > kg * STAGE_BYTES + NT_BYTES ? kg * OPERAND_BYTES : kg * STAGE_BYTES + NT_BYTES;
  }
  static constexpr int lds_bytes(bool adam) {
    return OPERAND_BYTES > STAGE_BYTES + (adam ? NT_BYTES : 0) ? OPERAND_BYTES : STAGE_BYTES + (adam ? NT_BYTES : 0);
  }
};

// The 128 x 128 tile of aligned bf16 operands with direct global -> LDS loads: 8 wavefronts, K steps of 64, a ring of 4, so that three
// steps (96 KB) are on their way to a CU that has one workgroup.  Bound by what a CU draws from L2 (46 GB/s, 2 MB a tile at K = 4096):
// 1024 x 4096 x 4096 44.8 us against 66.6 on 512 register-staged tiles of 128 x 64, 4096 x 1024 x 1024 15.6 against 21.2; the projection of one 350M
// layer with Adam in the epilogue 25.6 against 30.0.
struct DirectTile {
  static constexpr int BK = 64, STAGES = 4, NW = 8;
  static constexpr int STAGE_BYTES = 2 * 128 * BK * 2;
  static constexpr int LDS = STAGES * STAGE_BYTES;
  static constexpr int LOADS = STAGE_BYTES / 1024 / NW;  // per wavefront and step
};

// AKC: A as [M][K]; else (StoreF32 only) as [K][M].  DIRECT: see DirectTile; K is a multiple of 64.
// IN_PLACE (64 x 64, Adam or StoreF32): a workgroup adds the pr.splits K pieces of its tile itself, one after the other, so that a sum is no longer a
// chain than with a slab per piece, and has its bits.  Costs 16 registers of a lane and nothing that shows: see gemm_tile.hip.
// KG (Adam only): the K pieces of a tile are the work of KG groups of 4 wavefronts of one workgroup, which add their products in LDS, in
// the order in which the Adam kernel adds slabs.  A launch and the trip of the slabs through memory less, for the rate at which one CU
// draws the whole contraction's operands.
template <class T, int BM, int BN_, Epilogue EPI, bool AKC = true, bool DIRECT = false, int KG = 1, bool IN_PLACE = false>
__global__ __launch_bounds__(DIRECT ? 512 : 256 * KG, KG > 1 ? KG : 2) void gemm_tile_kernel(const GemmGroup grp) {
  using Cfg = SmallTile<T, BM, BN_>;
  using ET = ElemTraits<T>;
  constexpr int NT = DIRECT ? 512 : 256 * KG;
  static_assert(KG == 1 || (EPI == Epilogue::Adam && BM == 64 && !DIRECT), "");
  static_assert(!IN_PLACE || (KG == 1 && AKC && BM == 64 && BN_ == 64 && !DIRECT && (EPI == Epilogue::Adam || EPI == Epilogue::StoreF32)), "");
  constexpr int BN = Cfg::BN, BK = DIRECT ? DirectTile::BK : Cfg::BK, SP = Cfg::SP, ROWS = Cfg::ROWS;
  constexpr int WM = BM / 2, WN = BN / (DIRECT ? 4 : 2), TM = WM / 32, TN = WN / 32;
  using AOp = typename Cfg::A;
  using BOp = typename Cfg::B;
  static_assert(!DIRECT || (BM == 128 && BN == 128 && AKC && sizeof(T) == 2 && Cfg::STAGE_BYTES + Cfg::NT_BYTES <= DirectTile::LDS), "");
  __shared__ __align__(16) unsigned char smem_static[DIRECT || KG > 1 ? 16 : Cfg::lds_bytes(EPI == Epilogue::Adam)];
  extern __shared__ __align__(1024) unsigned char smem_direct[];
  unsigned char* smem = DIRECT || KG > 1 ? smem_direct : smem_static;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = KG > 1 ? wave >> 2 : 0, gtid = KG > 1 ? tid & 255 : tid, gwave = KG > 1 ? wave & 3 : wave;
  const int wm0 = (gwave & 1) * WM, wn0 = (gwave >> 1) * WN;
  T* As = reinterpret_cast<T*>(smem + group * Cfg::OPERAND_BYTES);
  T* Bs = As + AOp::LDS_ELEMS;

  const int bid = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
  int pi = 0;
  for (int i = 1; i < grp.count; ++i)
    if (bid >= grp.p[i].tile_begin) pi = i;
  const GemmProblem& pr = grp.p[pi];
  const int tiles = pr.tiles_m * pr.tiles_n;
  const int item = bid - pr.tile_begin;
  const int slab = KG > 1 || IN_PLACE ? 0 : item / tiles, piece = KG > 1 ? group : slab;
  int tm, tn;
  tile_coords(item - slab * tiles, pr.tiles_m, pr.tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int M = pr.M, N = pr.N, K = pr.K;
  const int KT = (K + BK - 1) / BK, S = KG > 1 ? KG : !IN_PLACE && pr.splits > 1 ? pr.splits : 1;
  const int first = (int)((long long)piece * KT / S), last = (int)((long long)(piece + 1) * KT / S);
  const T* __restrict__ A = static_cast<const T*>(pr.A);
  const T* __restrict__ B = static_cast<const T*>(pr.B);

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  f32x16 done;  // IN_PLACE: the pieces before the current one; -0 + x is x, also for x = -0
#pragma unroll
  for (int v = 0; v < 16; ++v) done[v] = -0.f;
  int piece_of = 0, piece_end = IN_PLACE ? KT / pr.splits : 0;

  // W pieces of the weight update: piece q of pass ps is row ps * ROWS + q * RPP + tid / CPW, columns WVEC (tid % CPW) ..
  constexpr int WVEC = ET::VEC;
  constexpr int CPW = BN / WVEC, RPP = NT / CPW, NQ = ROWS / RPP, NPASS = BM / ROWS;
  u32x4 wold[EPI == Epilogue::ApplyW ? NPASS * NQ : 1];
  const int wcol = n0 + (tid % CPW) * WVEC;

  auto fetch_w = [&]() {
    if constexpr (EPI == Epilogue::ApplyW) {
      const T* W = static_cast<const T*>(pr.C);
      const int wc = wcol < N - WVEC ? wcol : N - WVEC;
#pragma unroll
      for (int q = 0; q < NPASS * NQ; ++q) {
        const int row = m0 + q * RPP + tid / CPW;
        __builtin_memcpy(&wold[q], W + (size_t)(row < M ? row : M - 1) * pr.ldc + wc, sizeof(u32x4));
      }
    }
  };

  // fp32 pieces of the epilogue: columns 4 (tid % CPC) .. by EPT threads
  constexpr int EPT = KG == 3 ? 512 : NT;
  constexpr int CPC = BN / 4, RPC = EPT / CPC, NC = ROWS / RPC;
  const int pc = (tid % CPC) * 4, col = n0 + pc;
  // The moments are requested before anything waits for them (N >= 4: see tile_problem_fits): of a pass at its start, or with the last
  // products where there is one step more to hide them behind (DIRECT).
  constexpr int HELD = EPI != Epilogue::Adam ? 1 : DIRECT ? NPASS * NC : NC;
  f32x4 mo[HELD], vo[HELD];
  auto fetch_moments = [&](int ps) {
    if constexpr (EPI == Epilogue::Adam) {
      const int cc = col + 4 <= N ? col : 0;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int row = m0 + ps * ROWS + q * RPC + tid / CPC, at = DIRECT ? ps * NC + q : q;
        const size_t e = (size_t)(row < M ? row : M - 1) * N + cc;
        __builtin_memcpy(&mo[at], pr.Mo + e, 16);
        __builtin_memcpy(&vo[at], pr.Vo + e, 16);
      }
    }
  };

  auto run_direct = [&](auto kc) {
    constexpr bool BKC = decltype(kc)::value;
    constexpr int S = DirectTile::STAGES, LOADS = DirectTile::LOADS;
    using DA = DlOperand<true, 128, DirectTile::BK, DirectTile::NW>;
    using DB = DlOperand<BKC, 128, DirectTile::BK, DirectTile::NW>;
    DA da;
    DB db;
    da.plan(pr.lda, m0, M, wave, lane);
    db.plan(pr.ldb, n0, N, wave, lane);
    const unsigned lds0 = (unsigned)(uintptr_t)smem_direct;
    const unsigned char* asrc = static_cast<const unsigned char*>(pr.A);
    const unsigned char* bsrc = static_cast<const unsigned char*>(pr.B);
    const size_t bstep = BKC ? (size_t)DirectTile::BK * 2 : (size_t)DirectTile::BK * pr.ldb * 2;
    auto issue = [&](int kt) {
      const unsigned st = lds0 + ((kt - first) & (S - 1)) * DirectTile::STAGE_BYTES;
      da.template issue<false>(asrc + (size_t)kt * DirectTile::BK * 2, st, wave);
      db.template issue<false>(bsrc + kt * bstep, st + DA::TILE_BYTES, wave);
    };
    for (int kt = first; kt < last && kt < first + S - 1; ++kt) issue(kt);
    fetch_w();
    for (int kt = first; kt < last; ++kt) {
      // this wavefront's pieces of step kt have landed; its LDS reads of the step before have returned
      if (kt + 2 < last) wait_vmcnt<2 * LOADS>();
      else if (kt + 1 < last) wait_vmcnt<LOADS>();
      else wait_vmcnt<0>();
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (kt + S - 1 < last) issue(kt + S - 1);
      if (kt + 1 == last) {  // earlier, the waits for the tiles would wait for these as well (one 350M layer 52.8 us a step instead of 51.5)
#pragma unroll
        for (int ps = 0; ps < NPASS; ++ps) fetch_moments(ps);
      }
      const unsigned char* as = smem_direct + ((kt - first) & (S - 1)) * DirectTile::STAGE_BYTES;
      const unsigned char* bs = as + DA::TILE_BYTES;
      bf16x8 fa[4][TM], fb[4][TN];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[s][i] = DA::frag(as, wm0 + 32 * i, 16 * s, lane);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[s][j] = DB::frag(bs, wn0 + 32 * j, 16 * s, lane);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s][i], fb[s][j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();  // the epilogue takes the ring's place
  };

  auto run = [&](auto kc) {
    constexpr bool BKC = decltype(kc)::value;
    const bool edge_n = !BKC && n0 + BN > N;
    const bool edge_m = !AKC && m0 + BM > M;
    // two register sets: the pieces of the next two K steps are in flight while one is multiplied
    u32x4 ra0[AOp::PER], rb0[BOp::PER], ra1[AOp::PER], rb1[BOp::PER];
    auto load = [&](u32x4 (&ra)[AOp::PER], u32x4 (&rb)[BOp::PER], int kt) {
      AOp::template load<AKC>(ra, A, pr.lda, m0, M, kt * BK, K, gtid);
      BOp::template load<BKC>(rb, B, pr.ldb, n0, N, kt * BK, K, gtid);
    };
    auto step = [&](u32x4 (&ra)[AOp::PER], u32x4 (&rb)[BOp::PER], int kt) {
      const int k = kt * BK;
      const bool tail = k + BK > K;
      if (KG > 1 && kt >= last) {  // a group with a step less keeps the barriers
        __syncthreads();
        __syncthreads();
        return;
      }
      if constexpr (IN_PLACE) {
        if (kt == piece_end) {
          piece_end = (int)((long long)(++piece_of + 1) * KT / pr.splits);
#pragma unroll
          for (int v = 0; v < 16; ++v) { done[v] += acc[0][0][v]; acc[0][0][v] = 0.f; }
        }
      }
      AOp::template store<AKC>(ra, As, m0, M, k, K, tail || edge_m, gtid);
      BOp::template store<BKC>(rb, Bs, n0, N, k, K, tail || edge_n, gtid);
      __syncthreads();
      if (kt + 2 < last) load(ra, rb, kt + 2);
#pragma unroll
      for (int kk = 0; kk < BK; kk += ET::KSTEP) {
        Frag<T> fa[TM], fb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) AOp::template frag<AKC>(fa[i], As, wm0 + 32 * i, kk, lane);
#pragma unroll
        for (int j = 0; j < TN; ++j) BOp::template frag<BKC>(fb[j], Bs, wn0 + 32 * j, kk, lane);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) Frag<T>::mma(acc[i][j], fa[i], fb[j]);
      }
      __syncthreads();
    };
    if (KG == 1 || first < last) load(ra0, rb0, first);
    if (first + 1 < last) load(ra1, rb1, first + 1);
    fetch_w();
    const int end = KG > 1 ? first + (KT + KG - 1) / KG : last;
    for (int kt = first; kt < end; kt += 2) {
      step(ra0, rb0, kt);
      if (kt + 1 < end) step(ra1, rb1, kt + 1);
    }
  };
  if constexpr (DIRECT) {
    if (EPI == Epilogue::ApplyW || pr.b_kcontig) run_direct(std::true_type{});
    else if constexpr (EPI != Epilogue::ApplyW) run_direct(std::false_type{});
  } else if constexpr (EPI == Epilogue::ApplyW) {
    run(std::true_type{});
  } else if constexpr (!AKC) {
    run(std::false_type{});
  } else {
    if (pr.b_kcontig) run(std::true_type{});
    else run(std::false_type{});
  }

  if constexpr (IN_PLACE) {
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][0][v] = done[v] + acc[0][0][v];
  }

  // Epilogue: ROWS rows at a time through LDS, so that global accesses are 16 contiguous bytes per lane.  Accumulator
  // register v of lane l is element (row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32) of a 32 x 32 block.
  float* st = reinterpret_cast<float*>(smem);
  const int ldc = pr.ldc;
#pragma unroll
  for (int ps = 0; ps < NPASS; ++ps) {
    if (ps) __syncthreads();
    if constexpr (!DIRECT) fetch_moments(ps);
    if (wm0 / ROWS == ps) {
      const int wr = wm0 % ROWS;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            st[group * ROWS * SP + (wr + 32 * i + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * SP + wn0 + 32 * j + (lane & 31)] = acc[i][j][v];
    }
    __syncthreads();
    if constexpr (EPI == Epilogue::ApplyW) {
      T* W = static_cast<T*>(pr.C);
      const float s0 = pr.s0, s1 = pr.s1;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int lr = q * RPP + tid / CPW, row = m0 + ps * ROWS + lr;
        if (row >= M || wcol >= N) continue;
        const float* src = st + lr * SP + (tid % CPW) * WVEC;
        T* dst = W + (size_t)row * ldc + wcol;
        if (wcol + WVEC <= N) {
          T o[WVEC], w[WVEC];
          __builtin_memcpy(w, &wold[ps * NQ + q], sizeof(u32x4));
#pragma unroll
          for (int e = 0; e < WVEC; ++e) o[e] = (T)apply_entry(s0, (float)w[e], s1, src[e]);
          __builtin_memcpy(dst, o, sizeof(u32x4));
        } else {  // the piece that straddles the end of the row
#pragma unroll
          for (int e = 0; e < WVEC; ++e)
            if (wcol + e < N) dst[e] = (T)apply_entry(s0, (float)dst[e], s1, src[e]);
        }
      }
    } else if constexpr (EPI == Epilogue::StoreBF16) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int lr = q * RPP + tid / CPW, row = m0 + ps * ROWS + lr;
        if (row >= M || wcol >= N) continue;
        const float* src = st + lr * SP + (tid % CPW) * WVEC;
        T* dst = static_cast<T*>(pr.C) + (size_t)row * ldc + wcol;
        T o[WVEC];
#pragma unroll
        for (int e = 0; e < WVEC; ++e) o[e] = (T)src[e];
        if (wcol + WVEC <= N) {
          __builtin_memcpy(dst, o, sizeof(u32x4));
        } else {
#pragma unroll
          for (int e = 0; e < WVEC; ++e)
            if (wcol + e < N) dst[e] = o[e];
        }
      }
    } else if constexpr (EPI == Epilogue::Adam) {
      constexpr int NP = Cfg::NPITCH;
      T* nt = reinterpret_cast<T*>(smem + KG * Cfg::STAGE_BYTES);  // nt[column][row]
      T* Nout = static_cast<T*>(pr.Nout);
      const bool tr = pr.n_transposed != 0;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int lr = q * RPC + tid / CPC, row = m0 + ps * ROWS + lr;
        if (row >= M || col >= N || (EPT < NT && tid >= EPT)) continue;
        constexpr bool held = DIRECT;
        const int mq = held ? ps * NC + q : q;
        f32x4 g = *reinterpret_cast<const f32x4*>(st + lr * SP + pc);
#pragma unroll
        for (int kg = 1; kg < KG; ++kg) g += *reinterpret_cast<const f32x4*>(st + kg * ROWS * SP + lr * SP + pc);
        float* Mp = pr.Mo + (size_t)row * N + col;
        float* Vp = pr.Vo + (size_t)row * N + col;
        T n[4];
        if (col + 4 <= N) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float me = mo[mq][e], ve = vo[mq][e];
            n[e] = (T)adam_entry(g[e], me, ve, grp.beta1, grp.beta2, grp.eps, pr.inv_c1, pr.inv_c2);
            mo[mq][e] = me; vo[mq][e] = ve;
          }
          __builtin_memcpy(Mp, &mo[mq], 16);
          __builtin_memcpy(Vp, &vo[mq], 16);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            n[e] = (T)0.f;
            if (col + e < N) {
              float me = Mp[e], ve = Vp[e];
              n[e] = (T)adam_entry(g[e], me, ve, grp.beta1, grp.beta2, grp.eps, pr.inv_c1, pr.inv_c2);
              Mp[e] = me; Vp[e] = ve;
            }
          }
        }
        if (tr) {
#pragma unroll
          for (int e = 0; e < 4; ++e) nt[(pc + e) * NP + lr] = n[e];
        } else if (col + 4 <= N) {
          __builtin_memcpy(Nout + (size_t)row * N + col, n, sizeof n);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (col + e < N) Nout[(size_t)row * N + col + e] = n[e];
        }
      }
      if (tr) {  // N^T rows: 16-byte pieces along the tile's rows
        __syncthreads();
        constexpr int LPR = ROWS / WVEC, CPP = EPT / LPR;
#pragma unroll
        for (int q = 0; q < (BN + CPP - 1) / CPP; ++q) {
          const int jc = q * CPP + tid / LPR, i = (tid % LPR) * WVEC, row = m0 + ps * ROWS + i;
          if (n0 + jc >= N || row >= M || jc >= BN || (EPT < NT && tid >= EPT)) continue;
          const u32x4 o = *reinterpret_cast<const u32x4*>(nt + jc * NP + i);
          T* dst = Nout + (size_t)(n0 + jc) * M + row;
          if (row + WVEC <= M) {
            __builtin_memcpy(dst, &o, sizeof o);
          } else {
#pragma unroll
            for (int e = 0; e < WVEC; ++e)
              if (row + e < M) dst[e] = nt[jc * NP + i + e];
          }
        }
      }
    } else {
      float* C = static_cast<float*>(pr.C) + (size_t)slab * pr.slab_stride;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int lr = q * RPC + tid / CPC, row = m0 + ps * ROWS + lr;
        if (row >= M || col >= N) continue;
        const f32x4 x = *reinterpret_cast<const f32x4*>(st + lr * SP + pc);
        float* dst = C + (size_t)row * ldc + col;
        if (col + 4 <= N) {
          __builtin_memcpy(dst, &x, sizeof x);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (col + e < N) dst[e] = x[e];
        }
      }
    }
  }
}

// The fp32 projection of a small weight with the update block: 32 x 32 tiles, and the whole contraction of one in a workgroup of 16 wavefronts
// that cut it among them (4 groups take a run of K steps each, a wavefront a quarter of every step of its group).  The rate of the fp32 MFMA
// on the CUs that have a tile bounds 64 x 64 tiles here (7 us at K = 512); a quarter of the tile is a quarter of that.
struct NarrowTile {
  static constexpr int BM = 32, BN = 32, BK = 64, KG = 4, NT = 256 * KG;
  using Operand = TileOperand<float, 32, BK>;
  static constexpr int GROUP_FLOATS = 2 * Operand::LDS_ELEMS;
  static constexpr int SP = BN + 4, PART = BM * SP;  // floats of one wavefront's partial tile
  static constexpr int NP = BM + 4;                  // floats per column of the transposed N tile
  static constexpr int OPERANDS = KG * GROUP_FLOATS, STAGE = 4 * KG * PART;
  static constexpr int LDS = (OPERANDS > STAGE ? OPERANDS : STAGE) * 4;
  static_assert(BN * NP <= PART, "the transposed N tile takes the place of one partial tile");
};

static __global__ __launch_bounds__(NarrowTile::NT) void narrow_adam_kernel(const GemmGroup grp) {
  using Op = NarrowTile::Operand;
  constexpr int BM = NarrowTile::BM, BN = NarrowTile::BN, BK = NarrowTile::BK, KG = NarrowTile::KG, SP = NarrowTile::SP, PART = NarrowTile::PART;
  extern __shared__ __align__(1024) unsigned char smem_narrow[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave >> 2, gtid = tid & 255, kk0 = (wave & 3) * (BK / 4);
  float* As = reinterpret_cast<float*>(smem_narrow) + group * NarrowTile::GROUP_FLOATS;
  float* Bs = As + Op::LDS_ELEMS;

  const int bid = xcd_contiguous_block_id(blockIdx.x, gridDim.x);
  int pi = 0;
  for (int i = 1; i < grp.count; ++i)
    if (bid >= grp.p[i].tile_begin) pi = i;
  const GemmProblem& pr = grp.p[pi];
  int tm, tn;
  tile_coords(bid - pr.tile_begin, pr.tiles_m, pr.tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN, M = pr.M, N = pr.N, K = pr.K;
  const int KT = (K + BK - 1) / BK, steps = (KT + KG - 1) / KG;
  const int first = (int)((long long)group * KT / KG), last = (int)((long long)(group + 1) * KT / KG);
  const float* __restrict__ A = static_cast<const float*>(pr.A);
  const float* __restrict__ B = static_cast<const float*>(pr.B);

  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;

  // the update's four entries of a thread of the first group; the moments are requested before the products (N >= 4: see tile_problem_fits)
  const int lr = gtid >> 3, pc = (gtid & 7) * 4, row = m0 + lr, col = n0 + pc;
  f32x4 mo = {0.f, 0.f, 0.f, 0.f}, vo = mo;

  auto run = [&](auto kc) {
    constexpr bool BKC = decltype(kc)::value;
    const bool edge_n = !BKC && n0 + BN > N;
    u32x4 ra0[Op::PER], rb0[Op::PER], ra1[Op::PER], rb1[Op::PER];
    auto load = [&](u32x4 (&ra)[Op::PER], u32x4 (&rb)[Op::PER], int kt) {
      Op::load<true>(ra, A, pr.lda, m0, M, kt * BK, K, gtid);
      Op::load<BKC>(rb, B, pr.ldb, n0, N, kt * BK, K, gtid);
    };
    auto step = [&](u32x4 (&ra)[Op::PER], u32x4 (&rb)[Op::PER], int kt) {
      const int k = kt * BK;
      const bool tail = k + BK > K, has = kt < last;  // a group with a step less keeps the barriers
      if (has) {
        Op::store<true>(ra, As, m0, M, k, K, tail, gtid);
        Op::store<BKC>(rb, Bs, n0, N, k, K, tail || edge_n, gtid);
      }
      __syncthreads();
      if (has) {
        if (kt + 2 < last) load(ra, rb, kt + 2);
#pragma unroll
        for (int kk = 0; kk < BK / 4; kk += ElemTraits<float>::KSTEP) {
          Frag<float> fa, fb;
          Op::frag<true>(fa, As, 0, kk0 + kk, lane);
          Op::frag<BKC>(fb, Bs, 0, kk0 + kk, lane);
          Frag<float>::mma(acc, fa, fb);
        }
      }
      __syncthreads();
    };
    if (first < last) load(ra0, rb0, first);
    if (first + 1 < last) load(ra1, rb1, first + 1);
    if (group == 0) {
      const size_t e = (size_t)(row < M ? row : M - 1) * N + (col + 4 <= N ? col : 0);
      __builtin_memcpy(&mo, pr.Mo + e, 16);
      __builtin_memcpy(&vo, pr.Vo + e, 16);
    }
    for (int s = 0; s < steps; s += 2) {
      step(ra0, rb0, first + s);
      if (s + 1 < steps) step(ra1, rb1, first + s + 1);
    }
  };
  if (pr.b_kcontig) run(std::true_type{});
  else run(std::false_type{});

  // the 16 partial tiles, added in the order of the wavefronts
  float* st = reinterpret_cast<float*>(smem_narrow);
#pragma unroll
  for (int v = 0; v < 16; ++v) st[wave * PART + (8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * SP + (lane & 31)] = acc[v];
  __syncthreads();
  f32x4 n = {0.f, 0.f, 0.f, 0.f};
  float* Nout = static_cast<float*>(pr.Nout);
  const bool tr = pr.n_transposed != 0;
  if (group == 0 && row < M && col < N) {
    f32x4 g = *reinterpret_cast<const f32x4*>(st + lr * SP + pc);
#pragma unroll
    for (int w = 1; w < 4 * KG; ++w) g += *reinterpret_cast<const f32x4*>(st + w * PART + lr * SP + pc);
    float* Mp = pr.Mo + (size_t)row * N + col;
    float* Vp = pr.Vo + (size_t)row * N + col;
    if (col + 4 <= N) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float me = mo[e], ve = vo[e];
        n[e] = adam_entry(g[e], me, ve, grp.beta1, grp.beta2, grp.eps, pr.inv_c1, pr.inv_c2);
        mo[e] = me; vo[e] = ve;
      }
      __builtin_memcpy(Mp, &mo, 16);
      __builtin_memcpy(Vp, &vo, 16);
      if (!tr) __builtin_memcpy(Nout + (size_t)row * N + col, &n, 16);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (col + e < N) {
          float me = Mp[e], ve = Vp[e];
          n[e] = adam_entry(g[e], me, ve, grp.beta1, grp.beta2, grp.eps, pr.inv_c1, pr.inv_c2);
          Mp[e] = me; Vp[e] = ve;
          if (!tr) Nout[(size_t)row * N + col + e] = n[e];
        }
    }
  }
  if (!tr) return;  // uniform
  __syncthreads();  // the partial tiles have been read
  constexpr int NP = NarrowTile::NP;
  if (group == 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) st[(pc + e) * NP + lr] = n[e];
  }
  __syncthreads();
  if (group == 0) {  // N^T rows: 16-byte pieces along the tile's rows
    const int jc = gtid >> 3, i = (gtid & 7) * 4, r0 = m0 + i;
    if (n0 + jc >= N || r0 >= M) return;
    const f32x4 o = *reinterpret_cast<const f32x4*>(st + jc * NP + i);
    float* dst = Nout + (size_t)(n0 + jc) * M + r0;
    if (r0 + 4 <= M) {
      __builtin_memcpy(dst, &o, 16);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (r0 + e < M) dst[e] = o[e];
    }
  }
}

}  // namespace galore
