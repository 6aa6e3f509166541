// FP32-accurate complex GEMM tile on the 16-bit matrix cores.
//
// The FP32 matrix instructions reach 157 TFLOP/s, the BF16 ones 2.5 PFLOP/s.
// An FP32 value is exactly the sum of three bfloat16 values (each the rest
// rounded to 8 bits), so a product x y of two FP32 values is the sum of nine
// BF16 products, each exact in FP32.  Six of them are kept,
//   x0 y0 + (x0 y1 + x1 y0) + (x0 y2 + x1 y1 + x2 y0);
// with |x1| <= 2^-8 |x| and |x2| <= 2^-16 |x| of either sign (rounded, not cut
// off: the parts dropped would otherwise all have one sign) the others are
// below 2^-23 of |x y| and average out.  A 32x32x16 instruction accumulates 16
// products at a time in FP32, so a sum over K rounds less often than with the
// FP32 instructions' K steps of 4.
//
// This file is part of gemm.hip (included inside its anonymous namespace).

typedef float Acc32 __attribute__((ext_vector_type(16)));
typedef __bf16 Bf8 __attribute__((ext_vector_type(8)));
typedef float F2 __attribute__((ext_vector_type(2)));
typedef __bf16 Bf2 __attribute__((ext_vector_type(2)));
typedef uint32_t U4 __attribute__((ext_vector_type(4)));
typedef uint32_t U2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ Acc32 mma32(U4 a, U4 b, Acc32 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(Bf8, a), __builtin_bit_cast(Bf8, b), c, 0, 0, 0);
}
// row of register v in a 32x32 result (column lane % 32)
__device__ __forceinline__ int row32(int lane, int v) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }

constexpr int kSplitNp = 3, kSplitK = 16;

// WM x WN waves of FM x FN blocks of 32x32 outputs
template <int WM_, int WN_, int FM_, int FN_>
struct SplitShape {
  static constexpr int WM = WM_, WN = WN_, FM = FM_, FN = FN_;
  static constexpr int BM = 32 * WM * FM, BN = 32 * WN * FN;
  static_assert(WM * WN == 4 && BM % 64 == 0 && BN % 64 == 0, "four waves, whole 64-row groups");
  // one stage: per operand [2 groups of 8 k][kSplitNp re planes, kSplitNp im planes][rows] of eight
  // bfloat16; sizes in 16-byte units
  static constexpr int group_a = 2 * kSplitNp * BM, group_b = 2 * kSplitNp * BN, base_b = 2 * group_a;
  static constexpr size_t stage_bytes = (size_t)2 * (group_a + group_b) * 16;
  // 64-row x 8-k pieces of the A and B slabs, dealt to the waves in turn
  static constexpr int GA = BM / 64 * 2, GB = BN / 64 * 2, NG = (GA + GB + 3) / 4;
};
typedef SplitShape<2, 2, 2, 2> Split128;   // 128x128
typedef SplitShape<2, 2, 1, 2> Split64;    // 64x128, for M <= 64

// x[0..15] = eight complex values (re, im); writes the planes of the eight re
// and the eight im values to dst[p * plane]
// (sign bits flipped by re_sign and im_sign)
__device__ __forceinline__ void split_store(const float (&x)[16], uint32_t re_sign, uint32_t im_sign, U4* dst,
                                            int plane) {
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    U4 pl[kSplitNp];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      float a = x[4 * h + part], b = x[4 * h + 2 + part];
#pragma unroll
      for (int p = 0; p < kSplitNp; ++p) {
        const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(F2{a, b}, Bf2));
        pl[p][h] = w ^ (part == 1 ? im_sign : re_sign);
        if (p + 1 < kSplitNp) {   // the rest, exact
          a -= __uint_as_float(w << 16);
          b -= __uint_as_float(w & 0xffff0000u);
        }
      }
    }
#pragma unroll
    for (int p = 0; p < kSplitNp; ++p) dst[(part * kSplitNp + p) * plane] = pl[p];
  }
}

// One BM x BN tile at (m0, n0) of job j by 256 threads.  Per 16-deep slab a
// thread loads eight k values of a row of A or a column of B, NG times
// (k-contiguous operands as four 16-byte loads, the others as eight 8-byte
// loads that are contiguous across lanes; the buffer range check pads the
// tails with zeros), splits them and writes the planes to LDS as 16-byte
// values, so that an MFMA operand is one 16-byte LDS read.  The loads of slab
// s + 1 are in flight while slab s is multiplied; one LDS stage (48 KB at
// 128x128) and two barriers per slab let two workgroups share a CU, each
// converting while the other multiplies.
// FOLD: the 16-deep partial products start from zero and are added to the sum
// in FP32 (the compensated form: one rounding of the running sum per 16 k).
template <typename S, bool TA, bool TB, bool FOLD>
__device__ __forceinline__ void split_mainloop(const TileJob<float>& j, int64_t m0, int64_t n0, U4* smem,
                                               Acc32 (&acc_r)[S::FM][S::FN], Acc32 (&acc_i)[S::FM][S::FN]) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % S::WM, wn = wave / S::WM;
  const int64_t K = j.K;
  float x[S::NG][16];

  // rows contiguous in k (element (row, k) at row * ld + k), 64 rows from `first` of `rows`, 8 k from kk
  auto load_kc = [&](float (&v)[16], const float* base, int64_t ld, int64_t rows, int64_t first, int64_t kk) {
    const int64_t left = rows - first;
    const __amdgpu_buffer_rsrc_t rs =
        make_rsrc(base + 2 * (first * ld + kk), left > 0 && kk < K ? ((left - 1) * ld + (K - kk)) * 8 : 0);
    const uint32_t off = (uint32_t)lane * ((uint32_t)ld * 8u);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const U4 w = __builtin_bit_cast(U4, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16 * i, 0, 0));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * i + e] = __uint_as_float(w[e]);
    }
  };
  // contiguous in the row index (element (row, k) at k * ld + row): rows past
  // the last read the next k's (they only enter outputs that are not stored),
  // k past K reads zero
  auto load_rc = [&](float (&v)[16], const float* base, int64_t ld, int64_t rows, int64_t first, int64_t kk) {
    const int64_t left = rows - first;
    const __amdgpu_buffer_rsrc_t rs =
        make_rsrc(base + 2 * (kk * ld + first), left > 0 && kk < K ? ((K - kk - 1) * ld + left) * 8 : 0);
    const uint32_t step = (uint32_t)ld * 8u;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const U2 w = __builtin_bit_cast(U2, __builtin_amdgcn_raw_buffer_load_b64(rs, lane * 8 + i * step, 0, 0));
      v[2 * i] = __uint_as_float(w[0]);
      v[2 * i + 1] = __uint_as_float(w[1]);
    }
  };
  auto load = [&](int64_t k0) {
#pragma unroll
    for (int t = 0; t < S::NG; ++t) {
      const int g = wave + 4 * t;
      if (g < S::GA) {
        const int64_t first = m0 + (g >> 1) * 64, kk = k0 + (g & 1) * 8;
        if constexpr (TA) load_rc(x[t], j.A, j.lda, j.M, first, kk);
        else load_kc(x[t], j.A, j.lda, j.M, first, kk);
      } else if (g < S::GA + S::GB) {
        const int64_t first = n0 + ((g - S::GA) >> 1) * 64, kk = k0 + (g & 1) * 8;
        if constexpr (TB) load_kc(x[t], j.B, j.ldb, j.N, first, kk);
        else load_rc(x[t], j.B, j.ldb, j.N, first, kk);
      }
    }
  };
  static_assert(S::GA % 2 == 0, "the k half of a piece is its low bit for both operands");
  const uint32_t sa = j.sa < 0.f ? 0x80008000u : 0u, sb = j.sb < 0.f ? 0x80008000u : 0u;
  auto stash = [&](int64_t k0) {
#pragma unroll
    for (int t = 0; t < S::NG; ++t) {
      const int g = wave + 4 * t;
      const bool is_a = g < S::GA;
      // the K tail of k-contiguous rows: the next row's values must not enter
      const int64_t left = K - (k0 + (g & 1) * 8);
      if ((is_a ? !TA : TB) && left < 8) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (i >= left) x[t][2 * i] = x[t][2 * i + 1] = 0.f;
      }
      if (is_a)
        split_store(x[t], 0u, sa, smem + (g & 1) * S::group_a + (g >> 1) * 64 + lane, S::BM);
      else if (g < S::GA + S::GB) {
        const int col = ((g - S::GA) >> 1) * 64 + lane;
        const uint32_t flip = column_negated(n0 + col) ? 0x80008000u : 0u;
        split_store(x[t], flip, sb ^ flip, smem + S::base_b + (g & 1) * S::group_b + col, S::BN);
      }
    }
  };
#pragma unroll
  for (int i = 0; i < S::FM; ++i)
#pragma unroll
    for (int c = 0; c < S::FN; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc_r[i][c][v] = acc_i[i][c][v] = 0.f;

  auto compute = [&]() {
    constexpr int NP = kSplitNp;
    const U4* ap = smem + (lane >> 5) * S::group_a + wm * 32 * S::FM + (lane & 31);
    const U4* bp = smem + S::base_b + (lane >> 5) * S::group_b + wn * 32 * S::FN + (lane & 31);
#pragma unroll
    for (int i = 0; i < S::FM; ++i) {
      U4 a[2 * NP], na[NP];
#pragma unroll
      for (int p = 0; p < 2 * NP; ++p) a[p] = ap[p * S::BM + 32 * i];
#pragma unroll
      for (int p = 0; p < NP; ++p) na[p] = a[NP + p] ^ 0x80008000u;   // -im
#pragma unroll
      for (int c = 0; c < S::FN; ++c) {
        U4 b[2 * NP];
#pragma unroll
        for (int p = 0; p < 2 * NP; ++p) b[p] = bp[p * S::BN + 32 * c];
        Acc32 cr, ci;
        if constexpr (FOLD) {
#pragma unroll
          for (int v = 0; v < 16; ++v) cr[v] = ci[v] = 0.f;
        } else {
          cr = acc_r[i][c];
          ci = acc_i[i][c];
        }
        // smallest terms first; re and im chains alternate
#pragma unroll
        for (int o = NP - 1; o >= 0; --o)
#pragma unroll
          for (int p = 0; p <= o; ++p) {
            const int q = o - p;
            cr = mma32(a[p], b[q], cr);
            ci = mma32(a[p], b[NP + q], ci);
            cr = mma32(na[p], b[NP + q], cr);
            ci = mma32(a[NP + p], b[q], ci);
          }
        if constexpr (FOLD) {
          acc_r[i][c] += cr;
          acc_i[i][c] += ci;
        } else {
          acc_r[i][c] = cr;
          acc_i[i][c] = ci;
        }
        // one block's operands in registers at a time (reads hoisted over
        // several blocks spilled the accumulators)
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  load(0);
  stash(0);
  __syncthreads();
  for (int64_t k0 = 0; k0 < K; k0 += kSplitK) {
    const bool more = k0 + kSplitK < K;
    if (more) load(k0 + kSplitK);
    compute();
    __syncthreads();
    if (more) {
      stash(k0 + kSplitK);
      __syncthreads();
    }
  }
#pragma unroll
  for (int c = 0; c < S::FN; ++c) {
    const float sign = column_negated(n0 + wn * 32 * S::FN + c * 32 + (lane & 31)) ? -1.f : 1.f;
#pragma unroll
    for (int i = 0; i < S::FM; ++i) {
      acc_r[i][c] = acc_r[i][c] * sign;
      acc_i[i][c] = acc_i[i][c] * sign;
    }
  }
}

// C of a finished tile: plain, accumulated or block-transposed store (see
// GemmParams; products with the loss epilogue do not come here).
template <typename S>
__device__ __forceinline__ void split_epilogue(const TileJob<float>& j, int64_t m0, int64_t n0,
                                               const Acc32 (&acc_r)[S::FM][S::FN],
                                               const Acc32 (&acc_i)[S::FM][S::FN]) {
  typedef float V2 __attribute__((ext_vector_type(2)));
  typedef float V4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % S::WM, wn = wave / S::WM;
  const int64_t M = j.M, N = j.N, tb = j.tblock, cstep = tb > 0 ? tb : 1;
  auto row_off = [&](int64_t row) -> int64_t {
    if (tb > 0) {
      const int64_t blk = row / tb;
      return blk * j.ldc + (row - blk * tb);
    }
    return row * j.ldc;
  };
  // block-transposed: the lane's four consecutive rows are consecutive in C
  if (tb > 0 && tb % 4 == 0 && j.ldc % 4 == 0 && (reinterpret_cast<uintptr_t>(j.C) & 31) == 0 && !j.accumulate) {
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t row0 = m0 + wm * 32 * S::FM + i * 32 + row32(lane, 4 * u);
        if (row0 >= M) continue;
        const int64_t ro = row_off(row0);
#pragma unroll
        for (int c = 0; c < S::FN; ++c) {
          const int64_t col = n0 + wn * 32 * S::FN + c * 32 + (lane & 31);
          if (col >= N) continue;
          float* p = j.C + 2 * (ro + col * cstep);
          const Acc32 &cr = acc_r[i][c], &ci = acc_i[i][c];
          if (row0 + 3 < M) {
            reinterpret_cast<V4*>(p)[0] = V4{cr[4 * u], ci[4 * u], cr[4 * u + 1], ci[4 * u + 1]};
            reinterpret_cast<V4*>(p)[1] = V4{cr[4 * u + 2], ci[4 * u + 2], cr[4 * u + 3], ci[4 * u + 3]};
          } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (row0 + v < M) reinterpret_cast<V2*>(p)[v] = V2{cr[4 * u + v], ci[4 * u + v]};
          }
        }
      }
    return;
  }
#pragma unroll
  for (int i = 0; i < S::FM; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t row = m0 + wm * 32 * S::FM + i * 32 + row32(lane, v);
      if (row >= M) continue;
      const int64_t ro = row_off(row);
#pragma unroll
      for (int c = 0; c < S::FN; ++c) {
        const int64_t col = n0 + wn * 32 * S::FN + c * 32 + (lane & 31);
        if (col < N) {
          V2* p = reinterpret_cast<V2*>(j.C + 2 * (ro + col * cstep));
          V2 val{acc_r[i][c][v], acc_i[i][c][v]};
          if (j.accumulate) val += *p;
          *p = val;
        }
      }
    }
}

// BANDNW: 0 plain epilogues, 16 the Nw = 8 rotations on the matrix cores (see
// BandEpilogue)
template <typename S, int BANDNW>
__device__ __forceinline__ void split_finish(const TileJob<float>& j, int64_t m0, int64_t n0, float* smem,
                                             const BandEpilogue* band, const Acc32 (&acc_r)[S::FM][S::FN],
                                             const Acc32 (&acc_i)[S::FM][S::FN]) {
  if constexpr (BANDNW > 0) {
    static_assert(BANDNW == 16 && S::FM == 2 && S::FN == 2 && S::WM == 2, "the band epilogues take 64x64 outputs per wave");
    const int lane = threadIdx.x & 63;
    // W rows of half h (32 k points) of the wave's 64x64 block, [row][ldw] complex
    auto put_rows = [&](const Acc32 (&r)[2], const Acc32 (&i)[2], float* wl, int ldw) {
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          *reinterpret_cast<float2*>(wl + 2 * (row32(lane, v) * ldw + c * 32 + (lane & 31))) =
              make_float2(r[c][v], i[c][v]);
    };
    auto put = [&](int h, float* wl, int ldw) {
      if (h == 0)
        put_rows(acc_r[0], acc_i[0], wl, ldw);
      else
        put_rows(acc_r[1], acc_i[1], wl, ldw);
    };
    band_epilogue_mfma8(j, *band, m0, n0, put, smem);
  } else {
    split_epilogue<S>(j, m0, n0, acc_r, acc_i);
  }
}

template <typename S, bool TA, bool TB, bool FOLD, int BANDNW>
__device__ __forceinline__ void split_tile(const TileJob<float>& j, int64_t m0, int64_t n0, float* smem,
                                           const BandEpilogue* band) {
  Acc32 acc_r[S::FM][S::FN], acc_i[S::FM][S::FN];
  split_mainloop<S, TA, TB, FOLD>(j, m0, n0, reinterpret_cast<U4*>(smem), acc_r, acc_i);
  split_finish<S, BANDNW>(j, m0, n0, smem, band, acc_r, acc_i);
}

// the band epilogues stage 4 x 32 rows of 65 complex values
constexpr size_t kBandSmem = 4 * 32 * 65 * 2;
static_assert(kBandSmem * 4 >= Split128::stage_bytes, "stage and epilogue share the LDS");

template <typename S, bool TA, bool TB, bool FOLD, int BANDNW>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
    cgemm_split_kernel(GemmParams p, int64_t tiles_m, int64_t tiles_n) {
  __shared__ __align__(16) float smem[BANDNW > 0 ? kBandSmem : S::stage_bytes / 4];
  const int64_t logical = xcd_remap(blockIdx.x, tiles_m * tiles_n);
  int64_t tm, tn;
  tile_coords(logical, tiles_m, tiles_n, &tm, &tn);
  TileJob<float> j = job_of<float>(p, p.batch_base + blockIdx.y);
  j.tile = tm * tiles_n + tn;
  j.ntiles = tiles_m * tiles_n;
  split_tile<S, TA, TB, FOLD, BANDNW>(j, tm * S::BM, tn * S::BN, smem, &p.band);
}

// A wave's piece of an operand (64 k-contiguous rows, or 8 k of 64 contiguous
// rows) is addressed with 32-bit offsets.
inline bool split_fits(bool trans_a, bool trans_b, int64_t lda, int64_t ldb) {
  constexpr int64_t bytes = ((int64_t)1 << 32) - 4096;
  return lda >= 0 && ldb >= 0 && lda < bytes / (8 * (trans_a ? 8 : 64)) && ldb < bytes / (8 * (trans_b ? 64 : 8));
}

template <typename S, bool TA, bool TB, bool FOLD, int BANDNW = 0>
ephw_status launch_split(const GemmParams& p0, hipStream_t stream) {
  const int64_t tiles_m = ceil_div(p0.M, S::BM), tiles_n = ceil_div(p0.N, S::BN), ntiles = tiles_m * tiles_n;
  if (ntiles > 0x7fffffff) {
    set_error("cgemm: too many tiles");
    return EPHW_EUNSUPPORTED;
  }
  GemmParams p = p0;
  for (int64_t b0 = 0; b0 < p0.batch; b0 += 65535) {
    const int64_t nb = (p0.batch - b0) < 65535 ? (p0.batch - b0) : 65535;
    p.batch_base = b0;
    hipLaunchKernelGGL((cgemm_split_kernel<S, TA, TB, FOLD, BANDNW>), dim3((unsigned)ntiles, (unsigned)nb), dim3(256),
                       0, stream, p, tiles_m, tiles_n);
    EPHW_CHECK_LAUNCH();
  }
  return EPHW_OK;
}

template <typename S, bool FOLD>
ephw_status dispatch_split(const GemmParams& p, hipStream_t s) {
  if (!p.transA && !p.transB) return launch_split<S, false, false, FOLD>(p, s);
  if (p.transA && !p.transB) return launch_split<S, true, false, FOLD>(p, s);
  if (!p.transA && p.transB) return launch_split<S, false, true, FOLD>(p, s);
  return launch_split<S, true, true, FOLD>(p, s);
}

// ---------------------------------------------------------------------------
// Products of packed operands (pack.hip): every value scaled by a power of two
// and held as two binary16 values, so a product is x0 y0 + (x0 y1 + x1 y0),
// three FP16 matrix products instead of the six of the BF16 form.  The parts
// kept hold 22 to 24 bits of a value and the dropped x1 y1 is below 2^-22 of
// |x y| (rms 2^-23.6), an error that averages out over K, while the sum over
// 16 products per instruction rounds K / 16 x 3 times instead of K times.
// ---------------------------------------------------------------------------
typedef _Float16 Hf8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ Acc32 mma32h(U4 a, U4 b, Acc32 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(Hf8, a), __builtin_bit_cast(Hf8, b), c, 0, 0, 0);
}

// One 128x128 tile, four waves of 64x64 outputs.  A stage is 16 k of both
// operands as they lie in memory, [2 groups of 8 k][4 planes][128 rows] of 16
// bytes (16 KB per operand), copied straight to LDS by the loads; two stages,
// one barrier per slab: the operands of slab s go to registers, then the loads
// of slab s + 1 are issued into the other stage and complete while slab s is
// multiplied.
constexpr int kPackStage = 2 * 2 * 4 * 128;   // 16-byte units, both operands
constexpr size_t kPackSmem = 2 * (size_t)kPackStage * 4;   // floats
static_assert(kPackSmem <= kBandSmem, "the band epilogue's LDS holds both stages");

// ROWS: A's rows at the byte offsets row_off (the lane's rows of both halves)
// of the row-by-row form; a load's 64 lanes then touch 64 lines, and the eight
// loads of a slab's planes the same ones.
template <bool ROWS>
__device__ __forceinline__ void packed_mainloop(const PackedOperands& P, int64_t K, int64_t m0, int64_t n0,
                                                const uint32_t (&row_off)[2], U4* smem, Acc32 (&acc_r)[2][2],
                                                Acc32 (&acc_i)[2][2]) {
  typedef __attribute__((address_space(3))) void* LdsPtr;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const int64_t slabs = (K + 15) / 16;
  const uint32_t row_a = (uint32_t)P.lda * 16u, row_b = (uint32_t)P.ldb * 16u;   // bytes of one plane
  const __amdgpu_buffer_rsrc_t rsa = make_rsrc(P.A, slabs * 8 * (ROWS ? P.nrows : P.lda) * 16),
                               rsb = make_rsrc(P.B, slabs * 8 * P.ldb * 16);
  // the wave's four 1 KB pieces of each operand: planes 2 wave, 2 wave + 1 of the slab's eight, both row halves
  auto issue = [&](int64_t s, U4* st) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t pl = 2 * wave + (c >> 1), h = c & 1;
      const uint32_t oa = ROWS ? ((uint32_t)s * 8u + pl) * 16u : ((uint32_t)s * 8u + pl) * row_a + (uint32_t)(m0 + h * 64) * 16u;
      const uint32_t ob = ((uint32_t)s * 8u + pl) * row_b + (uint32_t)(n0 + h * 64) * 16u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsa, (LdsPtr)(st + pl * 128 + h * 64), 16, ROWS ? row_off[h] : lane * 16, oa, 0,
                                               0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsb, (LdsPtr)(st + 1024 + pl * 128 + h * 64), 16, lane * 16, ob, 0, 0);
    }
  };
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc_r[i][c][v] = acc_i[i][c][v] = 0.f;
  issue(0, smem);
  for (int64_t s = 0; s < slabs; ++s) {
    U4* st = smem + (s & 1) * kPackStage;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's pieces of slab s are in LDS
    __syncthreads();                                    // everyone's are, and the other stage has been read
    const U4* ap = st + (lane >> 5) * 512 + wm * 64 + (lane & 31);
    const U4* bp = st + 1024 + (lane >> 5) * 512 + wn * 64 + (lane & 31);
    U4 a[2][4], b[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        a[i][p] = ap[p * 128 + 32 * i];
        b[i][p] = bp[p * 128 + 32 * i];
      }
    if (s + 1 < slabs) issue(s + 1, smem + ((s + 1) & 1) * kPackStage);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const U4 nh = a[i][2] ^ 0x80008000u, nl = a[i][3] ^ 0x80008000u;   // -im
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        Acc32 cr = acc_r[i][c], ci = acc_i[i][c];
        cr = mma32h(a[i][1], b[c][0], cr);
        ci = mma32h(a[i][1], b[c][2], ci);
        cr = mma32h(a[i][0], b[c][1], cr);
        ci = mma32h(a[i][0], b[c][3], ci);
        cr = mma32h(nl, b[c][2], cr);
        ci = mma32h(a[i][3], b[c][0], ci);
        cr = mma32h(nh, b[c][3], cr);
        ci = mma32h(a[i][2], b[c][1], ci);
        cr = mma32h(a[i][0], b[c][0], cr);
        ci = mma32h(a[i][0], b[c][2], ci);
        cr = mma32h(nh, b[c][2], cr);
        ci = mma32h(a[i][2], b[c][0], ci);
        acc_r[i][c] = cr;
        acc_i[i][c] = ci;
      }
    }
  }
}

// the scales taken out again, exactly: A's first, so that no step overflows
// (column n0 + i of the output is column b0 + i of B)
__device__ __forceinline__ void packed_unscale(const PackedOperands& P, int64_t n0, int64_t b0, int64_t N,
                                               Acc32 (&acc_r)[2][2], Acc32 (&acc_i)[2][2]) {
  const int lane = threadIdx.x & 63, wn = threadIdx.x >> 7;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int col = wn * 64 + c * 32 + (lane & 31);
    const float sb = n0 + col < N ? P.inv_b[b0 + col] : 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      acc_r[i][c] = acc_r[i][c] * P.inv_a * sb;
      acc_i[i][c] = acc_i[i][c] * P.inv_a * sb;
    }
  }
}

template <int BANDNW>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
    cgemm_packed_kernel(GemmParams p, int64_t tiles_m, int64_t tiles_n) {
  __shared__ __align__(16) float smem[BANDNW > 0 ? kBandSmem : kPackSmem];
  const int64_t logical = xcd_remap(blockIdx.x, tiles_m * tiles_n);
  int64_t tm, tn;
  tile_coords(logical, tiles_m, tiles_n, &tm, &tn);
  TileJob<float> j = job_of<float>(p, 0);
  j.tile = tm * tiles_n + tn;
  j.ntiles = tiles_m * tiles_n;
  const int64_t m0 = tm * 128, n0 = tn * 128;
  Acc32 acc_r[2][2], acc_i[2][2];
  const uint32_t unused[2] = {0, 0};
  packed_mainloop<false>(p.packed, p.K, m0, n0, unused, reinterpret_cast<U4*>(smem), acc_r, acc_i);
  packed_unscale(p.packed, n0, n0, p.N, acc_r, acc_i);
  split_finish<Split128, BANDNW>(j, m0, n0, smem, &p.band, acc_r, acc_i);
}

// A workgroup per tile of the problems' concatenated tile lists (see
// cgemm_grouped): the tiles of a problem share its columns of B and its picked
// rows, so neighbours run on one XCD.  500 problems of about 640 rows, N = 384,
// K = 1000: 2.76 ms; with the BF16 split on gathered rows 5.29 and 1.05 ms for
// the gather, the packing of B counted here 0.70.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
    cgemm_packed_grouped_kernel(PackedOperands packed, int64_t K, const GroupProblem* __restrict__ probs, int n,
                                int64_t total) {
  __shared__ __align__(16) float smem[kPackSmem];
  const int64_t t = xcd_remap(blockIdx.x, total);
  const int lane = threadIdx.x & 63;
  int cnt = 0;                                   // problems that start at or before tile t
  for (int i0 = 0; i0 < n; i0 += 64) cnt += __popcll(__ballot(i0 + lane < n && probs[i0 + lane].tile_base <= t));
  const GroupProblem P = probs[cnt - 1];
  int64_t tm, tn;
  tile_coords(t - P.tile_base, P.tiles_m, P.tiles_n, &tm, &tn);
  const int64_t m0 = tm * 128, n0 = tn * 128;
  uint32_t row_off[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int64_t m = m0 + h * 64 + lane;        // rows past the last repeat it: their outputs are not stored
    int64_t r = P.rows[m < P.M ? m : P.M - 1];
    if (r < 0 || r >= packed.nrows) {
      if (threadIdx.x < 64) atomicOr(packed.status, kStatusIndex);
      r = 0;
    }
    row_off[h] = (uint32_t)r * (uint32_t)((K + 15) / 16 * 128);
  }
  TileJob<float> j;
  j.A = j.B = nullptr;
  j.C = static_cast<float*>(P.C);
  j.M = P.M;
  j.N = P.N;
  j.K = K;
  j.lda = j.ldb = 0;
  j.ldc = P.ldc;
  j.sa = j.sb = 1.f;
  j.accumulate = false;
  j.tblock = 0;
  j.loss = LossEpilogue();
  j.batch = 0;
  j.tile = 0;
  j.ntiles = 1;
  Acc32 acc_r[2][2], acc_i[2][2];
  packed_mainloop<true>(packed, K, m0, P.col0 + n0, row_off, reinterpret_cast<U4*>(smem), acc_r, acc_i);
  packed_unscale(packed, n0, P.col0 + n0, P.N, acc_r, acc_i);
  split_finish<Split128, 0>(j, m0, n0, smem, nullptr, acc_r, acc_i);
}

template <int BANDNW>
ephw_status launch_packed(const GemmParams& p, hipStream_t stream) {
  const int64_t tiles_m = ceil_div(p.M, 128), tiles_n = ceil_div(p.N, 128);
  if (tiles_m * tiles_n > 0x7fffffff) {
    set_error("cgemm: too many tiles");
    return EPHW_EUNSUPPORTED;
  }
  hipLaunchKernelGGL((cgemm_packed_kernel<BANDNW>), dim3((unsigned)(tiles_m * tiles_n)), dim3(256), 0, stream, p,
                     tiles_m, tiles_n);
  EPHW_CHECK_LAUNCH();
  return EPHW_OK;
}
