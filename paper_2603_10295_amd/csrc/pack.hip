// Operands of the packed FP32 products (cgemm_packed_kernel in gemm_split.h):
// every real value x of a row or column is scaled by a power of two and kept
// as two binary16 values, hi = rn(x), lo = rn(x - hi), which hold its first 22
// to 24 bits (the two round to nearest, so lo's sign is one more bit).  Four
// planes (re hi, re lo, im hi, im lo) of eight consecutive k each:
//   [k / 8][plane][row][k % 8],
// rows padded to a multiple of 128 (their contents are never stored) and k to
// a multiple of 16 with zeros.  The 8 bytes a complex value takes are those of
// complex64.  Phases whose rows a product picks through an index list are kept
// row by row instead, [row][k / 8][plane][k % 8]: the eight planes of a 16-deep
// slab are then the 128 bytes of one cache line, where rows picked from the
// planes would each take a line of their own.
#include "gemm.h"
#include "kernels.h"

namespace ephw {
namespace {

typedef uint32_t U4 __attribute__((ext_vector_type(4)));
typedef _Float16 H2 __attribute__((ext_vector_type(2)));

// the planes of eight complex values, re (part 0) and im (part 1) in x[2 i + part]
__device__ __forceinline__ void store_planes(const float (&x)[16], uint4* dst, int64_t plane) {
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    U4 hi, lo;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const float a = x[4 * h + part], b = x[4 * h + 2 + part];
      const H2 t = {(_Float16)a, (_Float16)b};
      const H2 r = {(_Float16)(a - (float)t[0]), (_Float16)(b - (float)t[1])};
      hi[h] = __builtin_bit_cast(uint32_t, t);
      lo[h] = __builtin_bit_cast(uint32_t, r);
    }
    dst[(2 * part) * plane] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    dst[(2 * part + 1) * plane] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
  }
}

// w_R exp(2 pi i p.R) of eight R per thread (phase.hip's phase, computed in
// FP64 and not rounded to complex64 in between), times `scale`
__global__ void pack_phase_kernel(const double* __restrict__ pts, int64_t n, const int32_t* __restrict__ R,
                                  const double* __restrict__ w, int64_t nr, float scale, uint4* __restrict__ out,
                                  int64_t plane, int64_t row, int64_t group) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, k8 = blockIdx.y;
  if (i >= n) return;
  const double px = pts[3 * i], py = pts[3 * i + 1], pz = pts[3 * i + 2];
  H2 hi[2][4], lo[2][4];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t r = k8 * 8 + e;
    double sn = 0.0, cs = 0.0;
    if (r < nr) {
      const double t = px * (double)R[3 * r] + py * (double)R[3 * r + 1] + pz * (double)R[3 * r + 2];
      sincospi(2.0 * (t - rint(t)), &sn, &cs);
      const double f = w[r] * (double)scale;
      sn *= f;
      cs *= f;
    }
    const _Float16 hc = (_Float16)(float)cs, hs = (_Float16)(float)sn;
    hi[0][e / 2][e & 1] = hc;
    lo[0][e / 2][e & 1] = (_Float16)(float)(cs - (double)hc);
    hi[1][e / 2][e & 1] = hs;
    lo[1][e / 2][e & 1] = (_Float16)(float)(sn - (double)hs);
  }
  uint4* dst = out + k8 * group + i * row;
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    dst[(2 * part) * plane] = __builtin_bit_cast(uint4, hi[part]);
    dst[(2 * part + 1) * plane] = __builtin_bit_cast(uint4, lo[part]);
  }
}

// 2^e with |m| 2^e in [2^14, 2^15) (FP16 goes to 65504), e limited so that 2^e
// and 2^-e are normal floats; 1 for a zero or non-finite m
__device__ __forceinline__ float column_scale(float m) {
  const uint32_t ex = __float_as_uint(m) >> 23;      // m >= 0: biased exponent
  if (m == 0.f || ex == 255u) return 1.f;
  int e = 14 + 127 - (int)ex;
  if (e > 126) e = 126;
  return __uint_as_float((uint32_t)(127 + e) << 23);
}

// Columns of row-major complex64 matrices [K][N] (N contiguous).  A workgroup
// takes 64 columns: its waves first find each column's largest component (the
// second read of the columns is then served by the caches), then scale and
// pack eight k at a time.  Memory bound: src is read twice, once from HBM.
__global__ void __launch_bounds__(256)
    pack_columns_kernel(const float* __restrict__ src, int64_t K, int64_t N, int64_t ld_src, int64_t stride_src,
                        uint4* __restrict__ out, int64_t ld, float* __restrict__ inv_scale) {
  __shared__ float red[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t blocks = (N + 63) / 64, b = blockIdx.x / blocks, n = (blockIdx.x % blocks) * 64 + lane;
  const bool ok = n < N;
  src += 2 * b * stride_src;
  out += b * N;
  inv_scale += b * N;
  const float2* col = reinterpret_cast<const float2*>(src) + (ok ? n : N - 1);
  float m = 0.f;
  bool bad = false;
#pragma unroll 8
  for (int64_t k = wave; k < K; k += 4) {
    const float2 v = col[k * ld_src];
    m = fmaxf(m, fmaxf(fabsf(v.x), fabsf(v.y)));
    bad = bad || !(fabsf(v.x) <= 3.4e38f) || !(fabsf(v.y) <= 3.4e38f);
  }
  red[wave][lane] = bad ? __builtin_inff() : m;   // fmaxf drops a NaN
  __syncthreads();
  m = fmaxf(fmaxf(red[0][lane], red[1][lane]), fmaxf(red[2][lane], red[3][lane]));
  const float sc = column_negated(b * N + n) ? -column_scale(m) : column_scale(m);
  if (wave == 0 && ok) inv_scale[n] = 1.f / sc;
  const int64_t groups = (K + 15) / 16 * 2;
  for (int64_t g = wave; g < groups; g += 4) {
    float x[16];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t k = g * 8 + i;
      const float2 v = k < K ? col[k * ld_src] : make_float2(0.f, 0.f);
      x[2 * i] = v.x * sc;
      x[2 * i + 1] = v.y * sc;
    }
    if (ok) store_planes(x, out + g * 4 * ld + n, ld);
  }
}

}  // namespace

ephw_status pack_phases(const double* pts, int64_t n, const int32_t* R, const double* w, int64_t nr, float scale,
                        void* out, hipStream_t s, bool by_row) {
  if (n <= 0 || nr <= 0) return EPHW_OK;
  const int64_t groups = packed_groups(nr);
  const int64_t plane = by_row ? 1 : packed_ld(n), row = by_row ? 4 * groups : 1, group = 4 * plane;
  for (int64_t g0 = 0; g0 < groups; g0 += 65535) {
    // nr past the groups of this launch is cut by the group index itself
    const int64_t ng = groups - g0 < 65535 ? groups - g0 : 65535;
    hipLaunchKernelGGL(pack_phase_kernel, dim3((unsigned)ceil_div(n, 256), (unsigned)ng), dim3(256), 0, s, pts, n,
                       R + 3 * 8 * g0, w + 8 * g0, nr - 8 * g0, scale,
                       static_cast<uint4*>(out) + g0 * group, plane, row, group);
    EPHW_CHECK_LAUNCH();
  }
  return EPHW_OK;
}

ephw_status pack_columns(const void* src, int64_t K, int64_t N, int64_t ld_src, void* out, float* inv_scale,
                         hipStream_t s, int64_t batch, int64_t stride_src) {
  if (K <= 0 || N <= 0 || batch <= 0) return EPHW_OK;
  if (batch * ceil_div(N, 64) > 0x7fffffff) {
    set_error("pack_columns: too many columns for one launch");
    return EPHW_EUNSUPPORTED;
  }
  hipLaunchKernelGGL(pack_columns_kernel, dim3((unsigned)(batch * ceil_div(N, 64))), dim3(256), 0, s,
                     static_cast<const float*>(src), K, N, ld_src, stride_src, static_cast<uint4*>(out),
                     packed_ld(batch * N), inv_scale);
  EPHW_CHECK_LAUNCH();
  return EPHW_OK;
}

}  // namespace ephw
