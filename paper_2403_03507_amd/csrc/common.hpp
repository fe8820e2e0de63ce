// Shared declarations of the GaLore HIP library (gfx950 only): grouped-launch
// descriptors passed by value as kernel arguments, and the host launchers the C ABI calls.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace galore {

constexpr int kMaxGroup = 16;  // problems per grouped launch (descriptor table lives in kernarg)

enum class DType : int32_t { F32 = 0, BF16 = 1 };

inline size_t dtype_size(DType d) { return d == DType::F32 ? 4 : 2; }

// ---- grouped GEMM ------------------------------------------------------------------------
// C[M x N] (+epilogue) = A * B, fp32 accumulate.  A is read as a_kcontig ? [M][K] : [K][M],
// B as b_kcontig ? [N][K] : [K][N]; lda/ldb are the strides (elements) of the outer index.
struct GemmProblem {
  const void* A;
  const void* B;
  void* C;        // output / in-place operand of the epilogue
  int64_t slab_stride;  // split contraction (launch_tile_group): elements between the outputs of two pieces
  int32_t splits;       // pieces of the contraction (0 and 1: whole); piece s writes C + s * slab_stride
  int32_t b_kcontig;    // layout of B where it is a field of the problem (launch_tile_group)
  int32_t M, N, K;
  int32_t lda, ldb, ldc;
  int32_t tile_begin;  // first block of this problem in the launch
  int32_t tiles_m;     // tiles along M and N; tile ids are decoded by tile_coords()
  int32_t tiles_n;
  float s0, s1;  // epilogue scalars
  // Epilogue::Adam: fp32 moments with the product's shape (dense, row stride N) and the normalised update in the
  // operands' dtype, n_transposed ? N x M : M x N, dense
  float* Mo;
  float* Vo;
  void* Nout;
  int32_t n_transposed;
  float inv_c1, inv_c2;
};

struct GemmGroup {
  int32_t count;
  int32_t total_tiles;
  float beta1, beta2, eps;  // Epilogue::Adam
  GemmProblem p[kMaxGroup];
};

enum class Epilogue : int32_t {
  StoreF32 = 0,   // C (fp32) = acc
  ApplyW = 1,     // C (T) = s0 * C - s1 * acc            (weight update, s0 = 1 - lr*wd, s1 = lr*alpha)
  StoreSymF32 = 2, // C (fp32) = acc, written to (i,j) and (j,i); tiles with tm > tn skipped (M == N)
  StoreBF16 = 4,  // C (bf16) = acc rounded to nearest even (launch_product_bf16)
  Adam = 3        // the update block of Algorithm 2 on acc: moments in place, N written, the product itself not stored (launch_tile_group)
};

// Launch one grouped GEMM on `stream`.  All problems share dtype / layouts / epilogue.
// Host fills everything except tile_begin / tiles_m / total_tiles.
hipError_t launch_gemm_group(GemmGroup& g, DType dt, bool a_kcontig, bool b_kcontig, Epilogue epi,
                             hipStream_t stream);

// The small-tile GEMM (gemm_tile.hpp): StoreF32 or Adam with A as [M][K] and the layout of B (and, for StoreF32, the
// number of K pieces) as fields of each problem, or ApplyW with both operands contiguous along K.  Any alignment of
// operands and output.
bool tile_problem_fits(const GemmProblem& p, DType dt, bool b_kcontig);
hipError_t launch_tile_group(GemmGroup& g, DType dt, Epilogue epi, hipStream_t stream);
constexpr int kMaxTilePieces = 4;
constexpr long kSplitBelowTiles = 224;  // a launch of as many 64 x 64 tiles keeps its contractions whole
constexpr int64_t kFuseAdamEntries = 65536;  // entries of R from which a whole contraction runs the update block by itself
int tile_pieces(long tiles, int64_t K, DType dt);
// fp32 in 64 x 64 tiles, StoreF32 or Adam, with the `splits` K pieces of a tile added by the workgroup that forms them: the bits of a slab per piece
// in one R.  Where all fp32 tensors that share the chip suit it (pieces_add_up_in_place) and have kInPlaceTiles to kSplitBelowTiles tiles together.
constexpr long kInPlaceTiles = 180;
bool pieces_add_up_in_place(bool left, int64_t K, int64_t ldim, int64_t r);
hipError_t launch_pieces_in_place(GemmGroup& g, Epilogue epi, hipStream_t stream);
// The product in K pieces with the update block of Algorithm 2 on their sum, in one launch: every tile's pieces in one workgroup.  Operands as
// for Epilogue::Adam of launch_tile_group.  bf16: the results are those of `splits` slabs and the Adam kernel, to the bit; fp32: the contraction is cut in 16.
// tiles32: 32 x 32 tiles of the launches that share the chip.
bool k_groups_pay(int64_t K, DType dt, int rank, int pieces, long tiles32);  // for one tensor; whether a call takes them: pieces_of_call
hipError_t launch_k_groups(GemmGroup& g, DType dt, hipStream_t stream);
constexpr long kDirectItems = 150;  // 128 x 128 tiles (times K pieces) from which a product may take the direct-load kernel (gemm_tile.hip)
int direct_pieces(const GemmProblem& p, DType dt, bool b_kcontig, int most);
// A projection launch with at least this many 256 x 256 tiles takes the 256 x 256 kernel (a 7B layer at r = 256, 193 tiles:
// 354 against 390 us per step on the small tiles; one 4096 x 11008 weight at r = 1024, 172 tiles: 256 against 283; one
// 4096 x 4096 weight, 64 tiles: 149 against 102).
constexpr long kLargeProjectionTiles = 160;
// The weight update W = s0 W - s1 A B^T (both operands contiguous along K) and the product C = A B (fp32, optionally in
// K pieces), on whichever kernel suits each problem.
hipError_t launch_weight_update(GemmGroup& g, DType dt, hipStream_t stream);
hipError_t launch_product(GemmGroup& g, DType dt, bool b_kcontig, hipStream_t stream);
// The product rounded to bf16 for the next one to read (bf16 operands): C (bf16) = A B with C's row stride N, on the small-tile
// kernel.  hipErrorNotSupported, with nothing launched, where launch_product would choose another kernel.
hipError_t launch_product_bf16(GemmGroup& g, bool b_kcontig, hipStream_t stream);
// The symmetric product C = A A^T (fp32; M == N, B == A) of A as [M][K] (kcontig) or [K][M], likewise.
hipError_t launch_gram(GemmGroup& g, DType dt, bool kcontig, hipStream_t stream);

// ---- grouped projection GEMM (bf16 operands, fp32 result): R = A * B with A as [M][K] -------------------
// LEFT tensors:  A = the transposed projector (r x m), B = G as [K = m][N = n]  (b_kcontig = 0)
// RIGHT tensors: A = G (m x n),                       B = the transposed projector as [N = r][K = n] (b_kcontig = 1)
struct ProjProblem {
  const void* A;
  const void* B;
  float* R;       // M x N, row stride ldr
  int32_t M, N, K;
  int32_t lda, ldb, ldr;
  int32_t b_kcontig;
  int32_t tile_begin, tiles_m, tiles_n;  // filled by the launcher
  // Adam in the epilogue (launch_proj_group with fuse_adam): R is not stored; the tile's entries go straight
  // into the update block of Algorithm 2.  Mo, Vo: fp32 moments with R's shape (row stride ldm, cols_valid <= N
  // columns: R may carry padded columns); Nout: bf16, n_transposed ? cols_valid x M (row stride ldn) : M x cols_valid.
  float* Mo;
  float* Vo;
  void* Nout;
  int32_t ldm, ldn, cols_valid, n_transposed;
  float inv_c1, inv_c2;
};

struct ProjGroup {
  int32_t count;
  int32_t total_tiles;
  int32_t regular_tiles;  // tiles [0, regular_tiles) run over their whole K range on the persistent grid
  int32_t pieces;         // the remaining tiles are cut into this many K ranges, one work item each
  float* slabs;           // partial tiles of the pieces (tile-local row-major, fp32), summed by the reduce kernel
  float beta1, beta2, eps;  // fused Adam only
  ProjProblem p[kMaxGroup];
};

// True if the problem meets the kernel's rules (16-byte aligned operands and rows, K a multiple of 64, ...);
// problems that do not go through launch_gemm_group.
bool proj_problem_fits(const ProjProblem& p);
// Launch one grouped projection; every problem must fit.  `slabs` (256-byte aligned, slab_bytes long, may be
// NULL / 0) is scratch for the partial tiles; without enough of it the launch simply runs whole tiles only.
// fuse_adam: every problem carries Mo, Vo, Nout, ...; M, V are updated and N written by the GEMM's epilogue (and by
// the kernel that sums the partial tiles), R is left untouched.
hipError_t launch_proj_group(ProjGroup& g, float* slabs, size_t slab_bytes, hipStream_t stream, bool fuse_adam = false);

// ---- grouped low-rank Adam -----------------------------------------------------------------
struct AdamProblem {
  const float* R;
  float* M;
  float* V;
  void* N;        // fp32 or bf16
  int64_t count;  // rows * cols
  int32_t rows;   // shape of R, M, V (M, V dense, row-major)
  int32_t cols;
  int32_t ldr;    // row stride of R, >= cols (padded rows of R only with transpose_n; else ldr == cols)
  int32_t transpose_n;  // 0: N has R's layout; 1: N is stored transposed (cols x rows)
  int32_t slabs;        // R is the sum of this many matrices (0 and 1: R itself), added in order
  int64_t slab_stride;  // elements between them
  float inv_c1;   // 1 / (1 - beta1^k)
  float inv_c2;   // 1 / (1 - beta2^k)
};

struct AdamGroup {
  int32_t count;
  float beta1, beta2, eps;
  AdamProblem p[kMaxGroup];
};

// All problems of a group share n_dtype.
hipError_t launch_adam_group(const AdamGroup& g, DType n_dtype, hipStream_t stream);

// ---- grouped low-rank Adam with 8-bit block-wise moments ------------------------------------------
// Moments are stored as one byte per element plus one fp32 scale per block of 256 consecutive
// elements of the row-major matrix; cols must be a multiple of 256 so that a block never
// straddles two rows.
struct AdamQ8Problem {
  const float* R;
  uint8_t* Mc;     // first-moment codes: sign, 4 exponent bits, 3 mantissa bits
  uint8_t* Vc;     // second-moment codes: 5 exponent bits, 3 mantissa bits
  float* Ms;       // per block: max |m|
  float* Vs;       // per block: max v
  void* N;         // fp32 or bf16
  int32_t rows;    // shape of R and of the code matrices (dense, row-major)
  int32_t cols;
  int32_t transpose_n;
  int32_t slabs;   // R is the sum of this many matrices (0 and 1: R itself), added in order
  int64_t slab_stride;
  float inv_c1, inv_c2;
};

struct AdamQ8Group {
  int32_t count;
  float beta1, beta2;
  float omb1, omb2;  // 1 - beta, formed in fp32 on the host
  float eps;
  AdamQ8Problem p[kMaxGroup];
};

hipError_t launch_adam_q8_group(const AdamQ8Group& g, DType n_dtype, hipStream_t stream);

// ---- grouped matrix transpose (projector k x r -> r x k) ------------------------------------
struct TransposeProblem {
  const void* src;  // rows x cols, leading dimension lds
  void* dst;        // cols x rows, leading dimension ldd
  int32_t rows, cols, lds, ldd;
};
struct TransposeGroup {
  int32_t count;
  TransposeProblem p[kMaxGroup];
};
hipError_t launch_transpose_group(const TransposeGroup& g, DType dt, hipStream_t stream);

// ---- grouped row padding (bf16): dst (rows x ldd, 16-byte aligned, ldd % 8 == 0) <- src (rows x cols, any
// row stride and element alignment), columns cols .. ldd - 1 zero ------------------------------
struct PadProblem {
  const void* src;
  void* dst;
  int32_t rows, cols, lds, ldd;
};
struct PadGroup {
  int32_t count;
  PadProblem p[kMaxGroup];
};
hipError_t launch_pad_rows_group(const PadGroup& g, hipStream_t stream);

// ---- small utilities -----------------------------------------------------------------------
hipError_t launch_fill_zero(void* ptr, size_t bytes, hipStream_t stream);
// dst (rows x cols, leading dimension ldd, dtype dt) <- src (dense fp32), rounded to nearest even
hipError_t launch_cast_rows(const float* src, void* dst, int rows, int cols, int ldd, DType dt, hipStream_t stream);
// the same with every row scaled to unit Euclidean length (a zero row stays zero)
hipError_t launch_normalize_rows(const float* src, void* dst, int rows, int cols, int ldd, DType dt, hipStream_t stream);

}  // namespace galore
