// Host side of the small-tile GEMM (gemm_tile.hpp): choice of the tile, launch, and the choice between it and the
// 256 x 256 kernels.
#include "gemm_mfma_dl.hpp"
#include "gemm_tile.hpp"

namespace galore {

bool tile_problem_fits(const GemmProblem& p, DType dt, bool b_kcontig) {
  const int vec = dt == DType::BF16 ? 8 : 4;  // elements of one piece: clamped pieces have to lie inside a row
  return p.M >= 1 && p.K >= vec && p.N >= vec && (b_kcontig ? p.K : p.N) >= vec;
}

namespace {

long tiles_of(const GemmProblem& p, int bm, int bn) { return (long)((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn) * (p.splits > 1 ? p.splits : 1); }

template <class T, int BM, int BN> hipError_t launch(GemmGroup& g, Epilogue epi, hipStream_t stream, bool a_kcontig = true) {
  long total = 0;
  for (int i = 0; i < g.count; ++i) {
    GemmProblem& p = g.p[i];
    p.tile_begin = (int32_t)total;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    total += tiles_of(p, BM, BN);
  }
  if (total > INT32_MAX) return hipErrorInvalidValue;
  g.total_tiles = (int32_t)total;
  const dim3 grid((unsigned)total);
  if (!a_kcontig) {
    if (epi != Epilogue::StoreF32) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemm_tile_kernel<T, BM, BN, Epilogue::StoreF32, false>), grid, dim3(256), 0, stream, g);
    return hipGetLastError();
  }
  if (epi == Epilogue::StoreF32) hipLaunchKernelGGL((gemm_tile_kernel<T, BM, BN, Epilogue::StoreF32>), grid, dim3(256), 0, stream, g);
  else if (epi == Epilogue::ApplyW) hipLaunchKernelGGL((gemm_tile_kernel<T, BM, BN, Epilogue::ApplyW>), grid, dim3(256), 0, stream, g);
  else if (epi == Epilogue::Adam) hipLaunchKernelGGL((gemm_tile_kernel<T, BM, BN, Epilogue::Adam>), grid, dim3(256), 0, stream, g);
  else if (std::is_same<T, __bf16>::value && epi == Epilogue::StoreBF16) hipLaunchKernelGGL((gemm_tile_kernel<__bf16, BM, BN, Epilogue::StoreBF16>), grid, dim3(256), 0, stream, g);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <Epilogue EPI> hipError_t launch_in_place(GemmGroup& g, hipStream_t stream) {
  long total = 0;
  for (int i = 0; i < g.count; ++i) {
    GemmProblem& p = g.p[i];
    p.tile_begin = (int32_t)total;
    p.tiles_m = (p.M + 63) / 64;
    p.tiles_n = (p.N + 63) / 64;
    if (p.splits < 1) p.splits = 1;
    total += (long)p.tiles_m * p.tiles_n;
  }
  if (total > INT32_MAX) return hipErrorInvalidValue;
  g.total_tiles = (int32_t)total;
  hipLaunchKernelGGL((gemm_tile_kernel<float, 64, 64, EPI, true, false, 1, true>), dim3((unsigned)total), dim3(256), 0, stream, g);
  return hipGetLastError();
}

// Aligned bf16 operands over whole K steps: the problem may run on DirectTile.
bool fits_direct(const GemmProblem& p, DType dt) {
  const bool kc = p.b_kcontig != 0;
  const uintptr_t at = reinterpret_cast<uintptr_t>(p.A) | reinterpret_cast<uintptr_t>(p.B);
  return dt == DType::BF16 && at % 16 == 0 && p.lda % 8 == 0 && p.ldb % 8 == 0 && p.K % DirectTile::BK == 0 && (kc || p.N % 8 == 0) &&
         (int64_t)p.M * p.lda < (1ll << 30) && (kc ? (int64_t)p.N : (int64_t)DirectTile::BK) * p.ldb < (1ll << 30);
}

template <Epilogue EPI> hipError_t direct_instance(const GemmGroup& g, hipStream_t stream) {
  auto kern = gemm_tile_kernel<__bf16, 128, 128, EPI, true, true>;
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, DirectTile::LDS);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)g.total_tiles), dim3(512), DirectTile::LDS, stream, g);
  return hipGetLastError();
}

hipError_t launch_direct(GemmGroup& g, Epilogue epi, hipStream_t stream) {
  long total = 0;
  for (int i = 0; i < g.count; ++i) {
    GemmProblem& p = g.p[i];
    p.tile_begin = (int32_t)total;
    p.tiles_m = (p.M + 127) / 128;
    p.tiles_n = (p.N + 127) / 128;
    total += tiles_of(p, 128, 128);
  }
  if (total > INT32_MAX) return hipErrorInvalidValue;
  g.total_tiles = (int32_t)total;
  switch (epi) {
    case Epilogue::StoreF32: return direct_instance<Epilogue::StoreF32>(g, stream);
    case Epilogue::ApplyW: return direct_instance<Epilogue::ApplyW>(g, stream);
    case Epilogue::Adam: return direct_instance<Epilogue::Adam>(g, stream);
    case Epilogue::StoreBF16: return direct_instance<Epilogue::StoreBF16>(g, stream);
    default: return hipErrorInvalidValue;
  }
}

template <int KG> hipError_t k_groups_instance(GemmGroup& g, hipStream_t stream) {
  using T = __bf16;
  long total = 0;
  for (int i = 0; i < g.count; ++i) {
    GemmProblem& p = g.p[i];
    p.tile_begin = (int32_t)total;
    p.tiles_m = (p.M + 63) / 64;
    p.tiles_n = (p.N + 63) / 64;
    p.splits = 1;
    total += tiles_of(p, 64, 64);
  }
  if (total > INT32_MAX) return hipErrorInvalidValue;
  g.total_tiles = (int32_t)total;
  auto kern = gemm_tile_kernel<T, 64, 64, Epilogue::Adam, true, false, KG>;
  constexpr int lds = SmallTile<T, 64, 64>::lds_bytes_groups(KG);
  static_assert(lds <= 160 * 1024, "");
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(256 * KG), lds, stream, g);
  return hipGetLastError();
}

hipError_t launch_narrow(GemmGroup& g, hipStream_t stream) {
  long total = 0;
  for (int i = 0; i < g.count; ++i) {
    GemmProblem& p = g.p[i];
    p.tile_begin = (int32_t)total;
    p.tiles_m = (p.M + NarrowTile::BM - 1) / NarrowTile::BM;
    p.tiles_n = (p.N + NarrowTile::BN - 1) / NarrowTile::BN;
    p.splits = 1;
    total += tiles_of(p, NarrowTile::BM, NarrowTile::BN);
  }
  if (total > INT32_MAX) return hipErrorInvalidValue;
  g.total_tiles = (int32_t)total;
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(narrow_adam_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, NarrowTile::LDS);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL(narrow_adam_kernel, dim3((unsigned)total), dim3(NarrowTile::NT), NarrowTile::LDS, stream, g);
  return hipGetLastError();
}

// One round of DirectTile, a tile per CU, most CUs with a tile: the deeper ring draws 46 GB/s per CU where the register-staged tiles, several a
// CU, reach 33.  Whole steps, us, on the other tiles / DirectTile:
//   256 tiles at most    one 350M layer at r = 256 (196) 51.8 / 48.9, 4096 x 4096 at r = 1024 (256) 108.7 / 98.2; in more than one round, 258 tiles 139.8 / 147.2,
//                        288 80.1 / 87.2, 386 140.6 / 130.1 but flushed 162.6 / 161.1, 726 246.6 / 228.6 but flushed 275.9 / 275.7
//   150 at least         4096 x 4096 at r = 768 (192) 94.1 / 84.8, r = 512 (128) 68.1 / 73.5
//   K of 2048, or 1024   a 2048 / 5504 layer at r = 128 (193) 99.8 / 91.3, r = 96 (three quarters of the rows used) 93.3 / 84.7; a 350M layer (K = 1024) at r = 192 (three
//   in used tiles        quarters) 44.4 / 46.3; a 768 / 2048 layer (K = 768) at r = 256 36.4 / 39.2
//   the weight update    from 160 tiles: 1024 x 2752 at r = 512 (176) 28.1 / 26.3, to 256: 2560 x 2560 at r = 512 (400) 45.8 / 46.4; from K = 256: 2048 x 2048 (256) at
//                        r = 128 22.3 / 21.6 but flushed 28.6 / 29.1, r = 256 26.5 / 24.9, r = 512 31.8 / 29.6
bool direct_pays(const GemmGroup& g, long items128, bool update) {
  if (items128 > 256 || items128 < (update ? 160 : kDirectItems)) return false;
  double used = 0;
  int shortest = INT32_MAX;
  for (int i = 0; i < g.count; ++i) {
    const GemmProblem& p = g.p[i];
    const int S = p.splits > 1 ? p.splits : 1;
    if (!fits_direct(p, DType::BF16) || (S > 1 && p.K % (128 * S) != 0)) return false;  // pieces end where the other tiles' end
    used += (double)p.M * p.N * S;
    shortest = p.K / S < shortest ? p.K / S : shortest;
  }
  if (update) return shortest >= 256;
  return shortest >= 2048 || (shortest >= 1024 && used >= 0.8 * items128 * 128 * 128);
}

// A larger tile loads fewer bytes per flop through the L2 -> CU path, a smaller one gives more workgroups to hide latency with: the largest that
// still makes a workgroup and a half per CU (128 x 128) or two (128 x 64).  Whole steps, us, with the projection on 64 x 64 / 128 x 64 / 128 x 128 tiles:
//   500 tiles of 128 x 64    one 350M layer (772 / 388 / 196 tiles) 54.0 / 49.0 / 57.2, flushed three of them 183 / 190 / 189 (hence 64 x 64 there)
//   350 tiles of 128 x 128   one 1B layer (3088 / 1544 / 772) 266 / 244 / 230, flushed two of them 502 / 448 / 420; 3805 x 3805 at r = 152 (180 / 120 / 60, two K pieces)
//                            65 / 68 / 83; flushed two 130M layers 99 / 101 / 108
//   half as much again for   two 3329 / 8824 layers at r = 24 451.5 on 64 x 64, 518.8 on 128 x 64, two 3328 / 8824 layers 411 and 423: what a larger tile
//   padding at most          adds in empty rows (or columns) is work; ranks from 129 on fit
//   the weight update        has more tiles and shorter contractions: 128 x 64 from 300 tiles on (r = 54 on a 1105 / 2688 layer 104 / 100 / 103), 128 x 128 from
//                            K = 256 on (r = 401 on 1904 / 3968 232 / 208 / 194)
// Flushed: the caches are written over before each pass; the others are passes repeated on the same tensors.
template <class T> hipError_t launch_typed(GemmGroup& g, Epilogue epi, hipStream_t stream) {
  long items128 = 0, items96 = 0, items64 = 0;
  int longest = 0;
  for (int i = 0; i < g.count; ++i) {
    items128 += tiles_of(g.p[i], 128, 128);
    items96 += tiles_of(g.p[i], 128, 64);
    items64 += tiles_of(g.p[i], 64, 64);
    longest = g.p[i].K > longest ? g.p[i].K : longest;
  }
  if (items128 == 0) return hipSuccess;
  const bool update = epi == Epilogue::ApplyW;
  if (std::is_same<T, __bf16>::value && direct_pays(g, items128, update)) return launch_direct(g, epi, stream);
  if (!update) {  // more than half as much again of a larger tile's work for padding: not that tile
    if (8 * items128 > 3 * items64) items128 = 0;
    if (4 * items96 > 3 * items64) items96 = 0;
  }
  if (items128 >= 350 && (!update || longest >= 256)) return launch<T, 128, 128>(g, epi, stream);
  if (items96 >= (update ? 300 : 500)) return launch<T, 128, 64>(g, epi, stream);
  return launch<T, 64, 64>(g, epi, stream);
}

constexpr long kGramTiles = 4096;  // 16 per CU: beyond, the general kernel has tiles enough and does half the products

bool fits_large(const GemmProblem& p, Epilogue epi, bool b_kcontig, bool w_any) {
  GemmGroup one{};
  one.count = 1;
  one.p[0] = p;
  return group_fits_dl(one, true, b_kcontig, epi) || (w_any && group_fits_dl(one, true, b_kcontig, epi, 64, true));
}

}  // namespace

hipError_t launch_tile_group(GemmGroup& g, DType dt, Epilogue epi, hipStream_t stream) {
  if (g.count <= 0) return hipSuccess;
  if (g.count > kMaxGroup) return hipErrorInvalidValue;
  for (int i = 0; i < g.count; ++i) {
    const GemmProblem& p = g.p[i];
    if (!tile_problem_fits(p, dt, p.b_kcontig != 0)) return hipErrorInvalidValue;
    if (epi != Epilogue::StoreF32 && p.splits > 1) return hipErrorInvalidValue;
    if (epi == Epilogue::ApplyW && !p.b_kcontig) return hipErrorInvalidValue;
    if (epi == Epilogue::Adam && (!p.Mo || !p.Vo || !p.Nout)) return hipErrorInvalidValue;
  }
  return dt == DType::BF16 ? launch_typed<__bf16>(g, epi, stream) : launch_typed<float>(g, epi, stream);
}

// Pieces of the contraction of a single product (not tied to others by the promises of galore_set_concurrency) that fill a round of DirectTile;
// 1 where none do.  `most`: matrices of its size that the caller has room for.
int direct_pieces(const GemmProblem& p, DType dt, bool b_kcontig, int most) {
  GemmProblem q = p;
  q.b_kcontig = b_kcontig;
  if (!fits_direct(q, dt) || !tile_problem_fits(q, dt, b_kcontig)) return 1;
  for (int pieces = most < kMaxTilePieces ? most : kMaxTilePieces; pieces > 1; --pieces) {
    GemmGroup g{};
    g.count = 1;
    g.p[0] = q;
    g.p[0].splits = pieces;
    if (direct_pays(g, tiles_of(g.p[0], 128, 128), false)) return pieces;
  }
  return 1;
}

// Pieces of the contraction for a launch of `tiles` 64 x 64 tiles: enough for two workgroups per CU where the tiles alone
// leave CUs idle, at most 4 (every piece is another fp32 copy of the product to write and to read).  Contractions under
// 512 stay whole.  Whole steps, us, with 1 / 2 / 4 / 8 pieces: 3805 x 3805 at r = 152 (180 tiles) 71.6 / 65.4 / 61.8 /
// 66.9; fp32 512 x 512 at r = 128 (16 tiles) 31.0 / 28.5 / 26.6 / 26.6; 2048 x 2048 at r = 512 (256 tiles) 32.3 / 34.8 / 36.1.
int tile_pieces(long tiles, int64_t K, DType dt) {
  if (tiles < 1 || tiles >= kSplitBelowTiles || K < 512) return 1;
  const int64_t by_k = K / (dt == DType::BF16 ? 256 : 128);
  int64_t pieces = (512 + tiles - 1) / tiles;
  pieces = pieces < by_k ? pieces : by_k;
  return (int)(pieces < kMaxTilePieces ? pieces : kMaxTilePieces);
}

// The launch that adds the slabs, and their trip through memory, against three times as many workgroups.  Whole steps, us, slabs / in place:
//   180 tiles at least      a 512 / 1376 layer at r = 128 (196) 42.7 / 38.6, a 1024 / 2736 layer at r = 64 (193) 79.2 / 66.2, 640 x 5888 at r = 128 (184) 42.8 / 37.4,
//                           11776 x 1024 at r = 64 (184) 60.0 / 55.1; 2048 x 5504 at r = 128 (172) 86.7 / 89.2, 768 x 2048 at r = 256 (128) 36.1 / 38.9
//   8-bit moments, too      (Adam is a launch of its own either way) 512 x 12544 at r = 64 60.7 / 48.5, six 1024 x 2048 at r = 32 80.2 / 64.3
//   kFuseAdamEntries        below, Adam would be one as well: a 1024 / 2736 layer at r = 32 70.7 / 86.7, a 512 / 1376 layer at r = 96 40.7 / 50.2
//   K of 2048               the longer the contraction, the more the balance counts: r = 128, LEFT and RIGHT, K = 1792 83.4 / 83.2, 83.2 / 81.6, K = 2048 88.2 / 90.0,
//                           87.9 / 88.1 (r = 100 RIGHT 91.6 / 90.5), K = 3072 120.3 / 127.7, 120.1 / 125.0
//   any K, LEFT, r <= 64    every panel of G has one reader, and the rate of those reads counts: K = 2048 127.7 / 97.9, 4096 248.8 / 198.5; RIGHT 96.3 / 95.7, 187.8 / 193.5
bool pieces_add_up_in_place(bool left, int64_t K, int64_t ldim, int64_t r) {
  return r * ldim >= kFuseAdamEntries && (left ? K < 2048 || r <= 64 : K <= 2048);
}

// The launch that adds the slabs against one CU that draws a whole contraction's operands (256 KB at K = 1024).  Whole steps of one weight, us, slabs /
// groups, repeated passes and flushed:
//   bf16, K of 1024          512 x 512 at r = 128 15.9 / 11.7, 19.4 / 15.3; 1024 x 1024 at r = 128 16.7 / 12.8, 20.5 / 18.6; 1024 x 2736 at r = 128 22.0 / 16.1, 29.5 / 24.3
//   2048 above rank 128      2048 x 2048 at r = 256 25.1 / 21.8, 35.1 / 31.4; r = 128 21.2 / 19.0 but 28.2 / 30.2; 3072 x 3072 at r = 128 29.7 / 31.5
//   fp32 (NarrowTile), few   512 x 512 at r = 128 19.9 / 14.0, 23.4 / 19.1 (in 64 x 64 tiles, bound by the matrix cores of the CUs that have one, 20.7); 768 x 768 at r = 256
//   enough tiles for 4       23.6 / 19.1, 29.9 / 24.4
//   one round of its tiles   1024 x 1024 at r = 128 22.5 / 17.9, 28.0 / 23.9; 1024 x 2736 at r = 64 28.0 / 22.7, 36.2 / 30.6; 2048 x 2048 at r = 128 39.2 / 37.3, 47.8 / 46.1
//   more to K = 768          768 x 2048 at r = 256 (512) 35.6 / 33.9, 43.6 / 41.6; 1024 x 2736 at r = 192 (516) 47.2 / 51.9, 1536 x 1536 at r = 192 (288) 41.2 / 44.1,
//                            2048 x 5504 at r = 64 (344) 57.3 / 61.7, three 1664 x 1664 at r = 48 in one call (312) 48.0 / 51.0
bool k_groups_pay(int64_t K, DType dt, int rank, int pieces, long tiles32) {
  if (pieces < 2 || pieces > kMaxTilePieces) return false;
  if (dt == DType::F32) return pieces == kMaxTilePieces && (K <= 768 || (K <= 2048 && tiles32 <= 256));
  return K <= 1024 || (K <= 2048 && rank > 128);
}

hipError_t launch_pieces_in_place(GemmGroup& g, Epilogue epi, hipStream_t stream) {
  if (g.count <= 0) return hipSuccess;
  if (g.count > kMaxGroup) return hipErrorInvalidValue;
  for (int i = 0; i < g.count; ++i) {
    const GemmProblem& p = g.p[i];
    if (!tile_problem_fits(p, DType::F32, p.b_kcontig != 0) || p.splits > kMaxTilePieces || (p.splits > 1 && p.K < 64 * p.splits)) return hipErrorInvalidValue;
    if (epi == Epilogue::Adam && (!p.Mo || !p.Vo || !p.Nout)) return hipErrorInvalidValue;
  }
  if (epi == Epilogue::Adam) return launch_in_place<Epilogue::Adam>(g, stream);
  return epi == Epilogue::StoreF32 ? launch_in_place<Epilogue::StoreF32>(g, stream) : hipErrorInvalidValue;
}

hipError_t launch_k_groups(GemmGroup& g, DType dt, hipStream_t stream) {
  if (g.count <= 0) return hipSuccess;
  if (g.count > kMaxGroup) return hipErrorInvalidValue;
  for (int i = 0; i < g.count; ++i) {
    const GemmProblem& p = g.p[i];
    if (!tile_problem_fits(p, dt, p.b_kcontig != 0) || !p.Mo || !p.Vo || !p.Nout || p.splits < 2 || p.splits > kMaxTilePieces) return hipErrorInvalidValue;
  }
  if (dt == DType::F32) return launch_narrow(g, stream);
  for (int pieces = 2; pieces <= kMaxTilePieces; ++pieces) {
    GemmGroup some{};
    some.beta1 = g.beta1; some.beta2 = g.beta2; some.eps = g.eps;
    for (int i = 0; i < g.count; ++i)
      if (g.p[i].splits == pieces) some.p[some.count++] = g.p[i];
    if (some.count == 0) continue;
    const hipError_t e = pieces == 2 ? k_groups_instance<2>(some, stream) : pieces == 3 ? k_groups_instance<3>(some, stream) : k_groups_instance<4>(some, stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_weight_update(GemmGroup& g, DType dt, hipStream_t stream) {
  // The persistent 256 x 256 kernel where its tiles come near filling the CUs (W prefetched across tiles): one 350M
  // layer (196 tiles) 54.3 against 55.5 us per step on the small tiles, a 7B layer at r = 128 305 against 346, at
  // r = 1024 995 against 1290; one 2048 x 2048 weight (64 tiles) 58.2 against 53.5.  With the caches flushed before each pass, three
  // 350M layers 187 against 204, two 1B layers 421 against 448.
  long tiles256 = 0;
  for (int i = 0; i < g.count; ++i) tiles256 += tiles_of(g.p[i], 256, 256);
  GemmGroup large{}, tiles{}, rest{};
  for (int i = 0; i < g.count; ++i) {
    GemmProblem& p = g.p[i];
    p.b_kcontig = 1;
    p.splits = 1;
    GemmGroup& to = dt == DType::BF16 && tiles256 >= 150 && fits_large(p, Epilogue::ApplyW, true, true) ? large : tile_problem_fits(p, dt, true) ? tiles : rest;
    to.p[to.count++] = p;
  }
  hipError_t e = launch_gemm_group(large, dt, true, true, Epilogue::ApplyW, stream);
  if (e == hipSuccess) e = launch_tile_group(tiles, dt, Epilogue::ApplyW, stream);
  if (e == hipSuccess) e = launch_gemm_group(rest, dt, true, true, Epilogue::ApplyW, stream);
  return e;
}

// The two products of the two-sided rule whose results are operands of the next one, 4096 x 4096 at r = 1024: with a copy of the
// fp32 result to bf16 (7 us and a launch each) 174 us per step, rounded in the epilogue 153.
hipError_t launch_product_bf16(GemmGroup& g, bool b_kcontig, hipStream_t stream) {
  long tiles256 = 0;
  for (int i = 0; i < g.count; ++i) tiles256 += tiles_of(g.p[i], 256, 256);
  for (int i = 0; i < g.count; ++i) {
    GemmProblem& p = g.p[i];
    p.b_kcontig = b_kcontig;
    if (p.splits > 1 || !tile_problem_fits(p, DType::BF16, b_kcontig)) return hipErrorNotSupported;
    if (tiles256 >= kLargeProjectionTiles && fits_large(p, Epilogue::StoreF32, b_kcontig, false)) return hipErrorNotSupported;
  }
  return launch_tile_group(g, DType::BF16, Epilogue::StoreBF16, stream);
}

hipError_t launch_product(GemmGroup& g, DType dt, bool b_kcontig, hipStream_t stream) {
  long tiles256 = 0;
  for (int i = 0; i < g.count; ++i) tiles256 += tiles_of(g.p[i], 256, 256);
  GemmGroup large{}, tiles{}, rest{};
  for (int i = 0; i < g.count; ++i) {
    GemmProblem& p = g.p[i];
    p.b_kcontig = b_kcontig;
    GemmGroup& to = dt == DType::BF16 && p.splits <= 1 && tiles256 >= kLargeProjectionTiles && fits_large(p, Epilogue::StoreF32, b_kcontig, false) ? large
                    : tile_problem_fits(p, dt, b_kcontig) ? tiles : rest;
    to.p[to.count++] = p;
  }
  for (int i = 0; i < rest.count; ++i)
    if (rest.p[i].splits > 1) return hipErrorInvalidValue;
  hipError_t e = launch_gemm_group(large, dt, true, b_kcontig, Epilogue::StoreF32, stream);
  if (e == hipSuccess) e = launch_tile_group(tiles, dt, Epilogue::StoreF32, stream);
  if (e == hipSuccess) e = launch_gemm_group(rest, dt, true, b_kcontig, Epilogue::StoreF32, stream);
  return e;
}

// Every tile is computed, also those below the diagonal: C_ij and C_ji are the same sum of the same products, and twice the
// work on 64 x 64 tiles is still less than a handful of 128 x 128 ones.  Whole products of a layer set, us, on the general kernel
// (LEFT and RIGHT tensors) and here: 60M fp32 (k = 512) 136 + 147 -> 58 + 58, 350M bf16 (k = 1024) 101 + 84 -> 73 + 20.
hipError_t launch_gram(GemmGroup& g, DType dt, bool kcontig, hipStream_t stream) {
  long tiles64 = 0;
  for (int i = 0; i < g.count; ++i) tiles64 += tiles_of(g.p[i], 64, 64);
  GemmGroup tiles{}, rest{};
  for (int i = 0; i < g.count; ++i) {
    GemmProblem& p = g.p[i];
    p.b_kcontig = kcontig;
    p.splits = 1;
    const bool fits = tile_problem_fits(p, dt, kcontig) && tile_problem_fits(p, dt, false) && tiles64 <= kGramTiles;
    GemmGroup& to = fits ? tiles : rest;
    to.p[to.count++] = p;
  }
  if (tiles.count > 0) {
    const hipError_t e = dt == DType::BF16 ? launch<__bf16, 64, 64>(tiles, Epilogue::StoreF32, stream, kcontig)
                                           : launch<float, 64, 64>(tiles, Epilogue::StoreF32, stream, kcontig);
    if (e != hipSuccess) return e;
  }
  return launch_gemm_group(rest, dt, kcontig, kcontig, Epilogue::StoreSymF32, stream);
}

}  // namespace galore
