// Complex GEMM on CDNA4 matrix cores: C[b] (=|+=) op(A[b]) * op(B[b]).
#pragma once

#include "common.h"

namespace ephw {

// Weighted |C|^2 epilogue for the loss L = sum w |g|^2 (SplitMix64 weights).
// layout 0: batch b is (il, iq, nu) = (b / (qb nm), (b / nm) % qb, b % nm)
// (k point k0 + il, q point q0 + iq, mode nu) and C's row m and column n are
// band indices.  layout 1: batch b is the pair (il, iq) = (b / qb, b % qb),
// row r of C is (nu, n) = (r / nw, r % nw) and column m is the other band.
// Every workgroup writes the sum of w |c|^2 over its tile to
// partial[b * tiles_per_batch + tile].  With grad_scale the stored value is
// 2 w c (the gradient of L with respect to g) instead of c.
struct LossEpilogue {
  bool on = false;
  bool store = true;        // also store C (plain or scaled)
  bool grad_scale = false;
  int layout = 0;
  uint64_t seed = 0;
  int64_t nk = 0;           // size of the k set (element index stride)
  int nm = 0, nw = 0, qb = 0;
  int64_t q0 = 0, k0 = 0;
  double* partial = nullptr;
};

// Band rotations fused into the epilogue of the Eq. (10) Re-sum GEMM (FP32,
// 128x128 tiles, no transposes, Nw of 4 or 8 so that every Nw x Nw block of a
// (q, nu) lies inside one wave's 64 columns).  C = W[k][(q, nu, m', n')] with
// row r the k point r of the set and column c = (q, nu, m', n') of the batch;
// instead of storing W the tile forms g_nu(k,q) = V(k+q)^dagger W_nu V(k)
// (Eq. (7)'s band factors, U = V^dagger) and applies the epilogues:
//   EPHW_OUT_G        g stored [q][k][nu][m][n]
//   EPHW_OUT_BAND_SUM T_nu = sum_mn |g|^2 stored [q][k][nu]
//   EPHW_OUT_LOSS     sum of w |g|^2 over the tile -> loss_partial[tile]
//   lw_partial        linewidth terms of every element (the weights of
//                     ephw_linewidth) summed over the (q, nu, m) of a column
//                     group -> lw_partial[group][k][n], cgemm_band_lw_groups
//                     groups of 64 or 128 columns
struct BandEpilogue {
  bool on = false;
  int nw = 0, nm = 0;
  int64_t nk = 0;                 // k points of the set (rows of C; stride of kq_index, g_out, band_sum)
  int64_t q_global0 = 0;          // position of the batch's first q in the caller's list (loss index)
  const void* Vk = nullptr;       // [nk][nw][nw] c64, eigenvector columns V(k)
  const void* Vkq = nullptr;      // [qb][nk][nw][nw] c64 V(k+q), or NULL: taken through kq_index
  const int32_t* kq_index = nullptr;  // [qb][nk], offset to the batch
  uint32_t flags = 0;             // EPHW_OUT_G / EPHW_OUT_BAND_SUM / EPHW_OUT_LOSS
  void* g_out = nullptr;          // [qb][nk][nm][nw][nw] c64, offset to the batch
  double* band_sum = nullptr;     // [qb][nk][nm], offset to the batch
  double* loss_partial = nullptr; // [tiles of the launch]
  uint64_t loss_seed = 0;
  double* lw_partial = nullptr;   // [groups][nk][nw], or NULL: no linewidth terms
  const double* eps_k = nullptr;  // [nk][nw]
  const double* eps_kq = nullptr; // [qb][nk][nw]
  const double* omega = nullptr;  // [qb][nm]
  LwParams lw;
  uint32_t* status = nullptr;     // kStatusIndex for an index outside [0, nk)
};

// Least K of a product on the 16-bit matrix cores: with few slabs per tile the
// first load and the store are the larger part of it, and an FP32 sum of few
// terms has few roundings to save.
constexpr int kSplitMinK = 64;

// The 16-bit matrix instructions do not round their running sum to nearest:
// what they drop has one sign, whatever that of the sum.  A product whose
// columns are summed next (Eq. (9) before Eq. (10)) would carry it into that
// sum coherently where the phases agree, near k or q = 0.  So the columns are
// multiplied with pseudo-random signs, taken out of the result again, which
// costs nothing: at q = 0 of the dense-Si window the error of |g|^2 was 1.28e-6
// (2.26e-6 after a first sum on BF16 parts) against 6.9e-7 over all q, and is
// 5.5e-7 with the signs (9.3e-7 in FP32 instructions).
__device__ __forceinline__ bool column_negated(int64_t col) { return (uint32_t)col * 0x9E3779B1u >> 31; }

// Packed operands of an FP32 product C = A B (pack.hip): rows of A and columns
// of B scaled by powers of two and held as two binary16 values per real value.
struct PackedOperands {
  bool on = false;
  const void* A = nullptr;
  const void* B = nullptr;
  int64_t lda = 0, ldb = 0;        // packed_ld of M and N
  float inv_a = 1.f;               // 1 / the scale of A's values
  const float* inv_b = nullptr;    // [N], 1 / the scale of each column, whose sign is column_negated's
  // grouped products: the rows of A are picked by each problem's index list
  // from `nrows` kept row by row (pack.hip), packed_row_bytes each
  int64_t nrows = 0;
  uint32_t* status = nullptr;      // kStatusIndex for an index outside [0, nrows)
};
// rows a packed operand is padded to, its groups of eight k, its bytes
inline int64_t packed_ld(int64_t rows) { return ceil_div(rows, 128) * 128; }
inline int64_t packed_groups(int64_t K) { return ceil_div(K, 16) * 2; }
inline int64_t packed_bytes(int64_t rows, int64_t K) { return packed_groups(K) * 4 * packed_ld(rows) * 16; }
inline int64_t packed_row_bytes(int64_t K) { return packed_groups(K) * 64; }

// All sizes, leading dimensions, strides and offsets count complex elements.
// Operands are interleaved complex (T re, T im), T = double (prec 0) or float
// (prec 1).  "trans" means the operand is stored transposed (A as [K][M],
// B as [N][K]); "conj" conjugates it on load.  Batch b is decomposed as
// b = (i0 * n1 + i1) * n2 + i2 and uses
//   A + (offA ? offA[b] : i0 * strideA + i1 * strideA1 + i2 * strideA2),
// likewise for B and C (n1 = n2 = 1 gives the plain stride b * strideA).
struct GemmParams {
  int64_t M = 0, N = 0, K = 0, batch = 1;
  const void* A = nullptr;
  int64_t lda = 0, strideA = 0;
  const int64_t* offA = nullptr;
  const void* B = nullptr;
  int64_t ldb = 0, strideB = 0;
  const int64_t* offB = nullptr;
  void* C = nullptr;
  int64_t ldc = 0, strideC = 0;
  const int64_t* offC = nullptr;
  bool transA = false, conjA = false, transB = false, conjB = false;
  bool accumulate = false;
  // FP32 only: K-blocked accumulation (fresh accumulators every 32 k, block
  // sums added in FP32), the compensated form of EPHW_FP32_COMP
  bool compensated = false;
  // the order of the sum and its roundings are free.  FP32: the product may run
  // on the 16-bit matrix cores with every value split (gemm_split.h), its error
  // against 64 bits no larger; FP64: on tiles that sum in another order.  Set
  // for FP64 results, and for FP32 ones where only complex64 values are
  // returned.  Sums returned in double precision (band sums, losses,
  // linewidths, gradients) keep the FP32 instructions, and the eigenproblems
  // they depend on their solver, so that their values do not move by more than
  // 1e-9; they are no more accurate for it (against 64 bits their errors are
  // some 1e-7 either way).
  bool any_rounding = false;
  int64_t n1 = 1, n2 = 1;
  int64_t strideA1 = 0, strideA2 = 0, strideB1 = 0, strideB2 = 0, strideC1 = 0, strideC2 = 0;
  // tblock > 0: C is stored in blocks of tblock rows, each block transposed:
  // element (r, c) goes to (r / tblock) * ldc + c * tblock + r % tblock
  // (ldc is then the block stride).
  int64_t tblock = 0;
  LossEpilogue loss;
  BandEpilogue band;
  PackedOperands packed;   // used in place of A and B where on
  int64_t batch_base = 0;  // internal: first batch index of this launch
};
// whether cgemm can run the fused band epilogue for this Re-sum shape (FP32,
// nw 4 or 8; always on 128x128 tiles, ceil(M/128) * ceil(N/128) of them);
// otherwise the caller stores W and rotates
bool cgemm_band_fusable(int prec, int64_t M, int64_t N, int nw, int64_t lda, int64_t ldb);
// column groups of the fused epilogue's linewidth partials for N columns
int64_t cgemm_band_lw_groups(int nw, int nm, int64_t N);
// workgroup tiles per batch entry of a GEMM (size of the loss partial block)
int64_t cgemm_tiles(int prec, int64_t M, int64_t N);

// whether an FP32 product of this shape runs on packed operands (both within
// 32-bit byte offsets)
bool cgemm_packable(int64_t M, int64_t N, int64_t K);

// prec: 0 = complex128 on FP64 MFMA, 1 = complex64 on FP32 MFMA, or on the 16-bit
// ones with split values (any_rounding, packed)
ephw_status cgemm(int prec, const GemmParams& p, hipStream_t stream);

// Many independent GEMMs C = A B (row-major, no transposes) in one persistent
// launch: `grid` workgroups take tiles of the concatenated tile lists from a
// work queue (per-XCD ranges, then the others).  All
// problems of one launch share a tile configuration `cfg` (0 = large,
// 1 = small 64x64; FP32 also 2 and 3, cgemm_grouped_split_cfg).
struct GroupProblem {
  int64_t M = 0, N = 0, K = 0;
  const void* A = nullptr;
  int64_t lda = 0;
  const void* B = nullptr;
  int64_t ldb = 0;
  void* C = nullptr;
  int64_t ldc = 0;
  int32_t cfg = 0;
  int64_t tiles_m = 0, tiles_n = 0, tile_base = 0;  // set by cgemm_grouped_layout
  int32_t flat = 0;   // set by cgemm_grouped_layout: both operands' extents fit 32-bit byte offsets
  // packed products (in place of A and B): the problem's M row indices, its first column of B
  const int32_t* rows = nullptr;
  int64_t col0 = 0;
};
void cgemm_tile_shape(int prec, int cfg, int* bm, int* bn);
// workgroups of the grouped kernel one CU holds at once (its persistent grid
// is this times the CU count)
int cgemm_grouped_blocks_per_cu(int prec, int cfg);
// FP32 tile configuration of a grouped product that may be split (see
// GemmParams::any_rounding; 2 = 128x128, 3 = 64x128 tiles) for problems of
// start[i + 1] - start[i] rows and depth K, or -1 where they are not split
int cgemm_grouped_split_cfg(int64_t K, int64_t lda, int64_t ldb, const int64_t* start, int64_t n);
// whether the grouped kernel can address operands with these leading dimensions
bool cgemm_grouped_fits(int prec, int64_t lda, int64_t ldb);
// fills tiles_m/tiles_n/tile_base of every problem; returns the total tile count
int64_t cgemm_grouped_layout(int prec, GroupProblem* probs, int n);
// `queue` points at kGroupQueues ints that must be zero when the launch
// starts (cgemm_grouped_reset zeroes many with one kernel, so a captured graph
// holds no memset node); the launch leaves them nonzero.
constexpr int kGroupQueues = 8;
ephw_status cgemm_grouped(int prec, int cfg, const GroupProblem* d_probs, int n, int64_t total_tiles, int grid,
                          int* queue, hipStream_t stream);
// The same for FP32 problems on packed operands, one K for all, laid out with
// cfg 2 (tiles of 128 x 128): C = A[rows] B[:, col0 : col0 + N]
bool cgemm_grouped_packable(int64_t nrows, int64_t columns, int64_t K);
ephw_status cgemm_grouped_packed(const PackedOperands& P, int64_t K, const GroupProblem* d_probs, int n,
                                 int64_t total_tiles, hipStream_t stream);
ephw_status cgemm_grouped_reset(int* queues, int count, hipStream_t stream);

}  // namespace ephw
