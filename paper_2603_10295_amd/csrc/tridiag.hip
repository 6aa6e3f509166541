// Batched Hermitian eigensolver in FP64 for orders up to 256 by Householder
// tridiagonalisation and implicit QL, for solves whose last bits are free
// (those of jacobi.hip keep theirs): about 10 n^3 operations a matrix, where
// the Jacobi sweeps take about 6 n rounds of all n^2 / 2 blocks.
//
// Up to order 32, reduction (reduce_kernel): a wavefront takes 64 / L matrices, L lanes each
// (the order rounded up to 8, 16 or 32), lane r holding row r of A and of Q in
// registers.  For each column, v and tau of H = I - tau v v^H with H x = e e1,
// A <- H A H as a rank-2 update and Q <- Q H; v and w pass through LDS, where
// every lane reads them as a broadcast.  The off-diagonals' phases go into Q's
// columns.  The matrix is scaled by a power of two to entries near 1 first, so
// no square under- or overflows.
//
// QL (ql_kernel; the classical implicit shifts, Bowdler, Martin, Reinsch and
// Wilkinson 1968): the recurrence is one serial chain of some 25 dependent FP64
// operations per rotation and about 0.9 n^2 rotations, the rotations of Q are
// wide.  So one lane runs a matrix's recurrence for a few steps and logs them
// in LDS, then a thread per row of Q applies the log to its row in registers.
// (With all lanes of a group computing the recurrence alike, in one kernel with
// the reduction, the recurrence was most of the time.)
// 131 072 matrices (us, reduction + QL, Jacobi): n = 8: 103 + 242, 761; n = 11:
// 333 + 535, 2347; n = 16: 667 + 1277, 7325.  32 768 of n = 24: 929 + 1082,
// 11 454; of n = 32: 1734 + 2814, 33 783.  The QL of a few matrices is its chain
// alone (n = 16: 105 us).
#include "kernels.h"

namespace ephw {
namespace {

// Reduction: N padded order, L lanes per matrix
template <int N, int L>
struct TriShape {
  static constexpr int G = 64 / L;              // matrices per wavefront
  static constexpr int waves = 4;               // per workgroup
  static constexpr size_t wave_elems = (size_t)G * 3 * N;   // double2: v, w, column phases
};

// QL: M matrices per workgroup, a thread per row; T steps per log
template <int N>
struct QlShape {
  static constexpr int M = N <= 16 ? 16 : 8;
  static constexpr int T = N <= 16 ? 8 : 4;
  static constexpr int CB = 4;                  // columns per block of the phase search
  static constexpr size_t log_elems = (size_t)M * T * N, stage_elems = (size_t)M * N * CB;
  static constexpr size_t shared = log_elems > stage_elems ? log_elems : stage_elems;
};

template <int L>
__device__ __forceinline__ double group_sum(double v) {
#pragma unroll
  for (int off = 1; off < L; off <<= 1) v += __shfl_xor(v, off, 64);
  return v;
}
template <int L>
__device__ __forceinline__ double group_max(double v) {
#pragma unroll
  for (int off = 1; off < L; off <<= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// 1/sqrt(x) for x > 0 in the normal range: the hardware estimate and one step
// of third order (e is the estimate's relative error doubled, near 2^-25)
__device__ __forceinline__ double rsqrt_nr(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// 1/x, |x| in the normal range, likewise
__device__ __forceinline__ double rcp_nr(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, y, 1.0);
  return fma(y * e, 1.0 + e, y);
}

// the power of two that takes the largest entry to [1, 2)
__device__ __forceinline__ int scale_exponent(double big) {
  const int ex = big > 0.0 && big < 1.7e308 ? ilogb(big) : 0;
  return ex < -1000 ? -1000 : ex;
}

// the off-diagonal e between d0 and d1 (of a matrix scaled to entries near 1) counts as zero
__device__ __forceinline__ bool negligible(double e, double d0, double d1) {
  return fabs(e) <= fmax(2.220446049250313e-16 * (fabs(d0) + fabs(d1)), 1e-140);
}

// Where |e| and the scale's exponent stay between the kernels, in doubles of the
// matrix in H: the first n + 1 of it, or (KEEP: the Jacobi kernels may take the
// matrix) the imaginary parts of its diagonal, which no solver reads; |e| of the
// last index is not used
template <bool KEEP>
struct EdgeSlots {
  static __device__ __forceinline__ int e(int n, int i) { return KEEP ? 2 * i * (n + 1) + 1 : i; }
  static __device__ __forceinline__ int exponent(int n) { return KEEP ? e(n, n - 1) : n; }
};

// H -> d in eps, |e| and the scale's exponent in H (EdgeSlots), Q in V
template <int N, int L, bool KEEP>
__global__ void __launch_bounds__((64 * TriShape<N, L>::waves))
    reduce_kernel(double2* __restrict__ H, int64_t batch, int n, double* __restrict__ eps, double2* __restrict__ V) {
  using S = TriShape<N, L>;
  __shared__ double2 lds[S::waves * S::wave_elems];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane % L, g = lane / L;          // row, matrix of the wave
  double2* sv = lds + wave * S::wave_elems + g * 3 * N;   // v
  double2* sw = sv + N;
  double2* sd = sw + N;
  const int64_t b = ((int64_t)blockIdx.x * S::waves + wave) * S::G + g;
  const bool live = b < batch;                   // a group past the end reduces a zero matrix
  double2* h = H + (live ? b : 0) * n * n;
  double* off = reinterpret_cast<double*>(h);

  double2 a[N], q[N];
  double big = 0.0;
#pragma unroll
  for (int c = 0; c < N; ++c) {
    // the matrix of jacobi.hip's small solves: the upper triangle and its conjugate
    a[c] = live && r < n && c < n ? h[c < r ? c * n + r : r * n + c] : make_double2(0.0, 0.0);
    if (c <= r) a[c].y = c == r ? 0.0 : -a[c].y;
    big = fmax(big, fmax(fabs(a[c].x), fabs(a[c].y)));
    q[c] = make_double2(c == r ? 1.0 : 0.0, 0.0);
  }
  big = group_max<L>(big);
  const int ex = scale_exponent(big);
  const double scale = ldexp(1.0, -ex);
#pragma unroll
  for (int c = 0; c < N; ++c) a[c] = make_double2(a[c].x * scale, a[c].y * scale);

  double2 delta = make_double2(1.0, 0.0);        // phase of Q's column k
  double dr = 0.0, er = 0.0;                     // d and |e| of this lane's index
#pragma unroll 1
  for (int k = 0; k < n; ++k) {
    // row k in LDS: lane r reads A[r][k] as its conjugate
    wave_sync();
    if (r == k) {
#pragma unroll
      for (int c = 0; c < N; ++c) sv[c] = a[c];
    }
    wave_sync();
    const double2 row = r < N ? sv[r] : make_double2(0.0, 0.0);
    const double2 alpha = k + 1 < n ? make_double2(sv[k + 1].x, -sv[k + 1].y) : make_double2(0.0, 0.0);
    double2 v = make_double2(0.0, 0.0);
    if (r > k + 1 && r < n) v = make_double2(row.x, -row.y);
    const double rest = group_sum<L>(v.x * v.x + v.y * v.y);
    const double a2 = alpha.x * alpha.x + alpha.y * alpha.y;
    // columns below 1e-140 of the matrix count as zero: their squares are near
    // the end of the range
    const bool has = a2 > 1e-280, reflect = rest > 1e-280;
    const double ia = has ? rsqrt_nr(a2) : 0.0, aabs = a2 * ia;
    const double2 ph = has ? make_double2(alpha.x * ia, alpha.y * ia) : make_double2(1.0, 0.0);
    double norm = aabs, tau = 0.0, sgn = 1.0;
    if (reflect) {
      const double t = a2 + rest, in = rsqrt_nr(t);
      norm = t * in;
      tau = in * rcp_nr(norm + aabs);
      sgn = -1.0;
      if (r == k + 1) v = make_double2(alpha.x + ph.x * norm, alpha.y + ph.y * norm);
    } else {
      v = make_double2(0.0, 0.0);
    }
    if (r == k) {
      dr = row.x;
      er = k + 1 < n ? norm : 0.0;               // |e|: e = sgn ph norm
      sd[k] = delta;
    }
    // delta_{k+1} = delta_k e / |e|
    delta = make_double2(sgn * (delta.x * ph.x - delta.y * ph.y), sgn * (delta.x * ph.y + delta.y * ph.x));
    wave_sync();                                 // everyone has read row k
    if (r < N) sv[r] = v;
    wave_sync();
    // v is zero up to row k: blocks of columns before it are left out
    double2 p = make_double2(0.0, 0.0), s = make_double2(0.0, 0.0);
#pragma unroll
    for (int c0 = 0; c0 < N; c0 += 4) {
      if (c0 + 3 <= k) continue;
#pragma unroll
      for (int c = c0; c < c0 + 4; ++c) {
        const double2 vc = sv[c];
        p.x = fma(a[c].x, vc.x, fma(-a[c].y, vc.y, p.x));
        p.y = fma(a[c].x, vc.y, fma(a[c].y, vc.x, p.y));
        s.x = fma(q[c].x, vc.x, fma(-q[c].y, vc.y, s.x));
        s.y = fma(q[c].x, vc.y, fma(q[c].y, vc.x, s.y));
      }
    }
    p = make_double2(tau * p.x, tau * p.y);
    s = make_double2(tau * s.x, tau * s.y);
    const double kk = 0.5 * tau * group_sum<L>(v.x * p.x + v.y * p.y);
    const double2 w = make_double2(p.x - kk * v.x, p.y - kk * v.y);
    if (r < N) sw[r] = w;
    wave_sync();
#pragma unroll
    for (int c0 = 0; c0 < N; c0 += 4) {
      if (c0 + 3 <= k) continue;
#pragma unroll
      for (int c = c0; c < c0 + 4; ++c) {
        const double2 vc = sv[c], wc = sw[c];
        // a -= v conj(w_c) + w conj(v_c); q -= s conj(v_c)
        a[c].x = fma(-v.x, wc.x, fma(-v.y, wc.y, fma(-w.x, vc.x, fma(-w.y, vc.y, a[c].x))));
        a[c].y = fma(-v.y, wc.x, fma(v.x, wc.y, fma(-w.y, vc.x, fma(w.x, vc.y, a[c].y))));
        q[c].x = fma(-s.x, vc.x, fma(-s.y, vc.y, q[c].x));
        q[c].y = fma(-s.y, vc.x, fma(s.x, vc.y, q[c].y));
      }
    }
  }
  wave_sync();
  if (!live || r >= n) return;
  using Edge = EdgeSlots<KEEP>;
  eps[b * n + r] = dr;
  if (!KEEP || r + 1 < n) off[Edge::e(n, r)] = er;
  if (r == 0) off[Edge::exponent(n)] = (double)ex;   // n = 1: the matrix has two doubles
  double2* out = V + (b * n + r) * n;
#pragma unroll
  for (int c = 0; c < N; ++c) {
    const double2 del = sd[c];
    if (c < n) out[c] = make_double2(q[c].x * del.x - q[c].y * del.y, q[c].x * del.y + q[c].y * del.x);
  }
}

// (d, e, Q) -> eigenvalues ascending (ties by index) and their vectors, each
// with its largest entry real positive.  KEEP: the imaginary part of H's first
// entry becomes 1 where eigenvalues are closer than `close` of the largest, else 0
template <int N, bool KEEP>
__global__ void __launch_bounds__((QlShape<N>::M * N))
    ql_kernel(double2* __restrict__ H, int64_t batch, int n, double* __restrict__ eps, double2* __restrict__ V,
              uint32_t* status, double close) {
  using S = QlShape<N>;
  constexpr int M = S::M, T = S::T, CB = S::CB;
  __shared__ double2 shared[S::shared];
  __shared__ double sdp[(N + 1) * M], sep[(N + 1) * M];   // [index][matrix], index -1 is read and not used
  double *const sd = sdp + M, *const se = sep + M;
  __shared__ uint32_t steps[M * T];              // l | m << 16 of each logged step
  __shared__ int rank[M * N];
  __shared__ double2 fix[M * CB];
  __shared__ int near[M];
  using Edge = EdgeSlots<KEEP>;
  const int tid = threadIdx.x;
  const int r = tid % n, mt = tid / n;           // row, matrix of the workgroup
  const int64_t b0 = (int64_t)blockIdx.x * M, b = b0 + mt;
  const bool live = mt < M && b < batch;
  double2 z[N];
  if (live) {
    sd[r * M + mt] = eps[b * n + r];
    se[r * M + mt] = reinterpret_cast<const double*>(H + b * n * n)[Edge::e(n, r)];
    if (KEEP && r == 0) near[mt] = 0;
    const double2* in = V + (b * n + r) * n;
#pragma unroll
    for (int c = 0; c < N; ++c) z[c] = c < n ? in[c] : make_double2(0.0, 0.0);
  }
  __syncthreads();

  // the recurrence's state: matrix tid of the workgroup
  const bool owner = tid < M && b0 + tid < batch;
  double* d = sd + tid;
  double* e = se + tid;
  double2* log = shared + tid * T * N;
  uint32_t small = 1u << (n - 1);                // bit i: e[i] is negligible
  if (owner)
    for (int i = 0; i + 1 < n; ++i) small |= negligible(e[i * M], d[i * M], d[(i + 1) * M]) ? 1u << i : 0u;
  const int limit = sweep_limit(status);
  int l = owner ? 0 : n, iter = 0;
  for (;;) {
    int count = 0;
    while (l < n && count < T) {
      // past the eigenvalues that are done (up to 32), in the same pass of the
      // loop: its passes last as long as the longest lane's
      const int skip = __builtin_ctzll(~(uint64_t)(small >> l));
      l += skip;
      iter = skip > 0 ? 0 : iter;
      if (l >= n) break;
      if (iter >= limit) {
        atomicOr(status, kStatusNoConv);
        ++l;
        iter = 0;
        continue;
      }
      const int m = l + __builtin_ctz(small >> l);
      ++iter;
      const double dl = d[l * M], el = e[l * M];
      double gg = 0.5 * (d[(l + 1) * M] - dl) * rcp_nr(el);
      double dn = d[m * M];                      // d[i + 1]
      const double h2 = fma(gg, gg, 1.0);
      gg = dn - dl + el * rcp_nr(gg + copysign(h2 * rsqrt_nr(h2), gg));
      double s = 1.0, c = 1.0, p = 0.0;
      double ei = e[(m - 1) * M], di = d[(m - 1) * M], above = 0.0;   // above: d[i + 2] after this step
      uint32_t hits = 0;
      asm volatile("" : "+v"(di), "+v"(ei), "+v"(dn), "+v"(gg));   // the loop begins with nothing in flight
#pragma unroll 1
      for (int i = m - 1; i >= l; --i) {
        // the next step's operands while this one's chain runs
        double en = e[(i - 1) * M], dp = d[(i - 1) * M];
        const double f = s * ei, bb = c * ei;
        const double t = fma(f, f, gg * gg);
        const bool zero = t < 1e-290;            // underflowed: no rotation
        const double inv = rsqrt_nr(zero ? 1.0 : t), eo = t * inv;
        s = f * inv;
        c = zero ? 1.0 : gg * inv;
        gg = dn - p;
        const double rr = fma(di - gg, s, 2.0 * c * bb);
        p = s * rr;
        const double dw = gg + p;
        gg = fma(c, rr, -bb);
        d[(i + 1) * M] = dw;
        e[(i + 1) * M] = eo;                     // e[m] is negligible and not read again
        hits |= (negligible(eo, dw, above) ? 1u : 0u) << (i + 1);
        log[count * N + i] = make_double2(c, s);
        above = dw;
        dn = di;
        // (not copied before this step's results are there: the copy would wait for LDS)
        asm volatile("" : "+v"(dp), "+v"(en) : "v"(gg), "v"(p));
        di = dp;
        ei = en;
      }
      const double dw = dn - p;
      d[l * M] = dw;
      e[l * M] = gg;
      hits |= (negligible(gg, dw, above) ? 1u : 0u) << l;
      const uint32_t inner = ((1u << m) - 1) & ~((1u << l) - 1);
      small = (small & ~inner) | (hits & inner);
      steps[tid * T + count] = (uint32_t)l | (uint32_t)m << 16;
      ++count;
    }
    if (tid < M)
      for (int t = count; t < T; ++t) steps[tid * T + t] = 0;
    const bool more = __syncthreads_or(l < n);
    if (live) {
#pragma unroll 1
      for (int t = 0; t < T; ++t) {
        const uint32_t lm = steps[mt * T + t];
        const int lo = lm & 0xffff, hi = lm >> 16;
        const double2* cs = shared + (mt * T + t) * N;
#pragma unroll
        for (int i0 = N - 4; i0 >= 0; i0 -= 4) {
          if (!__any(lo < i0 + 4 && hi > i0)) continue;
#pragma unroll
          for (int i = i0 + 3; i >= i0; --i) {
            if (i == N - 1) continue;
            // outside the step's range the log is another step's: no rotation
            double2 x = cs[i];
            const bool in = i >= lo && i < hi;
            x.x = in ? x.x : 1.0;
            x.y = in ? x.y : 0.0;
            const double2 z0 = z[i], z1 = z[i + 1];
            z[i + 1] = make_double2(fma(x.y, z0.x, x.x * z1.x), fma(x.y, z0.y, x.x * z1.y));
            z[i] = make_double2(fma(x.x, z0.x, -(x.y * z1.x)), fma(x.x, z0.y, -(x.y * z1.y)));
          }
        }
      }
    }
    __syncthreads();
    if (!more) break;
  }

  // ascending order
  if (live) {
    const int place = ascending_place([&](int j) { return sd[j * M + mt]; }, n, r);
    rank[mt * N + r] = place;
    const double* edge = reinterpret_cast<const double*>(H + b * n * n);
    eps[b * n + place] = ldexp(sd[r * M + mt], (int)edge[Edge::exponent(n)]);
    if constexpr (KEEP) {
      double top = 0.0, gap = HUGE_VAL;
      for (int j = 0; j < n; ++j) {
        const double o = sd[j * M + mt];
        top = fmax(top, fabs(o));
        if (j != r) gap = fmin(gap, fabs(o - sd[r * M + mt]));
      }
      if (gap <= close * top) near[mt] = 1;      // every lane that writes, the same value
    }
  }
  // phases, CB columns at a time: rows to LDS, a thread per column
#pragma unroll
  for (int c0 = 0; c0 < N; c0 += CB) {
    __syncthreads();
    if (live) {
#pragma unroll
      for (int c = 0; c < CB; ++c) shared[(mt * N + r) * CB + c] = z[c0 + c];
    }
    __syncthreads();
    if (tid < M * CB && b0 + tid / CB < batch) {
      double best = -1.0;
      double2 bv = make_double2(1.0, 0.0);
      for (int j = 0; j < n; ++j) {
        const double2 x = shared[(tid / CB * N + j) * CB + tid % CB];
        const double m2 = x.x * x.x + x.y * x.y;
        if (m2 > best) {
          best = m2;
          bv = x;
        }
      }
      if constexpr (N > 16)
        for (int j = 0; j < n; ++j) {
          const double2 x = shared[(tid / CB * N + j) * CB + tid % CB];
          const double m2 = x.x * x.x + x.y * x.y;
          if (m2 >= kTied * best) {
            best = m2;
            bv = x;
            break;
          }
        }
      const double mag = sqrt(best);
      fix[tid] = mag > 0.0 ? make_double2(bv.x / mag, -bv.y / mag) : make_double2(1.0, 0.0);
    }
    __syncthreads();
    if (live) {
      double2* out = V + (b * n + r) * n;
#pragma unroll
      for (int c = 0; c < CB; ++c) {
        const double2 x = z[c0 + c], y = fix[mt * CB + c];
        if (c0 + c < n) out[rank[mt * N + c0 + c]] = make_double2(x.x * y.x - x.y * y.y, x.x * y.y + x.y * y.x);
      }
    }
  }
  if (KEEP && live && r == 0) H[b * n * n].y = near[mt] ? 1.0 : 0.0;
}

// ---------------------------------------------------------------------------
// Orders 33 to 256: the same method over a workspace, one matrix per workgroup
// in the serial parts.  The reduction works in V's place (from L2: n^2 complex
// values do not fit the LDS above n = 100) and leaves v_k in row k; QL runs on
// the real tridiagonal with its rotations logged to memory; the rotations are
// applied to the rows of a real Z, 64 rows per wavefront; the reflectors, last
// first, take the columns of Z back, a wavefront per column.  Bound by the QL
// chain (about 0.85 n^2 rotations in a row) and the reduction's n steps of five
// barriers.  8 matrices of n = 150: reduction 1.19 ms,
// QL 2.90, rotations 1.25, back 0.12, launches that find nothing left to the
// Jacobi kernels 0.08; Jacobi 9.9.
// ---------------------------------------------------------------------------
constexpr int kBigThreads = 1024, kBigMax = 256, kBigRounds = 3;

// A matrix's part of the workspace: jacobi_work_doubles' share, 4 n (n - 1)
// doubles or more, holds the 3 n^2 + 9 n + 4 of these for n >= 33.
struct BigWork {
  double2 *log, *delta;       // [n^2] rotations (c, s) of a round; [n] phases of Q's columns
  double *zt, *d, *e, *tau;   // Z transposed [col][row]; [n] each
  uint2* step;                // [4 n] of a round: l | m << 16, first rotation
  int* state;                 // scale exponent, next eigenvalue, steps of the round, whether Jacobi takes over
  __device__ BigWork(double* base, int n) {
    const int64_t n2 = (int64_t)n * n;
    log = reinterpret_cast<double2*>(base);
    delta = log + n2;
    zt = reinterpret_cast<double*>(delta + n);
    d = zt + n2;
    e = d + n;
    tau = e + n;
    step = reinterpret_cast<uint2*>(tau + n);
    state = reinterpret_cast<int*>(step + 4 * n);
  }
};

// sum of v over the workgroup; red: 16 values no one reads any more
__device__ __forceinline__ double block_sum(double v, double* red) {
  v = group_sum<64>(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int i = 0; i < kBigThreads / 64; ++i) t += red[i];
  return t;
}

__global__ void __launch_bounds__(kBigThreads)
    reduce_big_kernel(const double2* __restrict__ H, int n, double2* __restrict__ V, double* __restrict__ work,
                      int64_t wstride) {
  __shared__ double2 sv[kBigMax], sw[kBigMax], part[kBigThreads];
  __shared__ double red[2][kBigThreads / 64];
  const int tid = threadIdx.x, W = (n + 63) / 64 * 64, G = kBigThreads / W;
  const int c = tid % W, g = tid / W;            // column; thread g takes the rows r = g modulo G
  const bool own = g < G && c < n;
  const double2* h = H + (int64_t)blockIdx.x * n * n;
  double2* A = V + (int64_t)blockIdx.x * n * n;
  const BigWork w(work + (int64_t)blockIdx.x * wstride, n);

  // a matrix that is not Hermitian to 1e-14 of its norm is left to the Jacobi
  // kernels, which do not converge on it
  double big = 0.0, tot = 0.0, skew = 0.0;
  if (own)
    for (int r = g; r < n; r += G) {
      const double2 x = h[(int64_t)r * n + c], y = h[(int64_t)c * n + r];
      big = fmax(big, fmax(fabs(x.x), r == c ? 0.0 : fabs(x.y)));
      tot += x.x * x.x + x.y * x.y;
      skew += 0.25 * ((x.x - y.x) * (x.x - y.x) + (x.y + y.y) * (x.y + y.y));
    }
  tot = block_sum(tot, red[0]);
  __syncthreads();
  skew = block_sum(skew, red[1]);
  big = group_max<64>(big);
  if ((tid & 63) == 0) red[0][tid >> 6] = big;   // tot has been read
  __syncthreads();
  for (int i = 0; i < kBigThreads / 64; ++i) big = fmax(big, red[0][i]);
  const int ex = scale_exponent(big);
  const double scale = ldexp(1.0, -ex);
  if (tid == 0) {
    w.state[0] = ex;
    w.state[1] = 0;
    w.state[3] = skew > 1e-28 * tot ? 1 : 0;
  }
  if (own)
    for (int r = g; r < n; r += G) {
      const double2 x = h[(int64_t)r * n + c];
      A[(int64_t)r * n + c] = make_double2(x.x * scale, r == c ? 0.0 : x.y * scale);
    }
  __syncthreads();

  double2 delta = make_double2(1.0, 0.0);
#pragma unroll 1
  for (int k = 0; k < n; ++k) {
    const double2* row = A + (int64_t)k * n;
    const double dk = row[k].x;
    double2 alpha = make_double2(0.0, 0.0), v = make_double2(0.0, 0.0);
    if (k + 1 < n) alpha = make_double2(row[k + 1].x, -row[k + 1].y);
    if (g == 0 && c > k + 1 && c < n) v = make_double2(row[c].x, -row[c].y);
    const double rest = block_sum(v.x * v.x + v.y * v.y, red[0]);
    const double a2 = alpha.x * alpha.x + alpha.y * alpha.y;
    const bool has = a2 > 1e-280, reflect = rest > 1e-280;   // see reduce_kernel
    const double ia = has ? rsqrt_nr(a2) : 0.0, aabs = a2 * ia;
    const double2 ph = has ? make_double2(alpha.x * ia, alpha.y * ia) : make_double2(1.0, 0.0);
    double norm = aabs, tau = 0.0;
    if (reflect) {
      const double t = a2 + rest, in = rsqrt_nr(t);
      norm = t * in;
      tau = in * rcp_nr(norm + aabs);
      if (g == 0 && c == k + 1) v = make_double2(alpha.x + ph.x * norm, alpha.y + ph.y * norm);
    }
    if (tid == 0) {
      w.d[k] = dk;
      w.e[k] = k + 1 < n ? norm : 0.0;
      w.tau[k] = tau;
      w.delta[k] = delta;
    }
    const double sgn = reflect ? -1.0 : 1.0;
    delta = make_double2(sgn * (delta.x * ph.x - delta.y * ph.y), sgn * (delta.x * ph.y + delta.y * ph.x));
    if (!reflect) {
      __syncthreads();                           // red is free again
      continue;
    }
    if (g == 0 && c < n) sv[c] = v;
    __syncthreads();
    if (g == 0 && c > k && c < n) A[(int64_t)k * n + c] = v;
    const int r0 = k + 1 + (g + G - (k + 1) % G) % G;   // first own row past k
    double2 p = make_double2(0.0, 0.0);
    if (own && c > k) {
#pragma unroll 8
      for (int r = r0; r < n; r += G) {          // A[c][r] is the conjugate of A[r][c]
        const double2 x = A[(int64_t)r * n + c], vr = sv[r];
        p.x = fma(x.x, vr.x, fma(x.y, vr.y, p.x));
        p.y = fma(x.x, vr.y, fma(-x.y, vr.x, p.y));
      }
    }
    part[tid] = p;
    __syncthreads();
    double dot = 0.0;
    if (g == 0) {
      for (int i = 1; i < G; ++i) {
        p.x += part[i * W + c].x;
        p.y += part[i * W + c].y;
      }
      p = make_double2(tau * p.x, tau * p.y);
      dot = v.x * p.x + v.y * p.y;
    }
    const double kk = 0.5 * tau * block_sum(dot, red[1]);
    if (g == 0 && c < n) sw[c] = make_double2(p.x - kk * v.x, p.y - kk * v.y);
    __syncthreads();
    if (own && c > k) {
      const double2 vc = sv[c], wc = sw[c];
#pragma unroll 8
      for (int r = r0; r < n; r += G) {
        double2 x = A[(int64_t)r * n + c];
        const double2 vr = sv[r], wr = sw[r];
        x.x = fma(-vr.x, wc.x, fma(-vr.y, wc.y, fma(-wr.x, vc.x, fma(-wr.y, vc.y, x.x))));
        x.y = fma(-vr.y, wc.x, fma(vr.x, wc.y, fma(-wr.y, vc.x, fma(wr.x, vc.y, x.y))));
        if (r == c) x.y = 0.0;
        A[(int64_t)r * n + c] = x;
      }
    }
    __syncthreads();
  }
}

// One wavefront per matrix runs the recurrence, every lane alike, until the
// log of the round is full or all eigenvalues are done.
__global__ void __launch_bounds__(64)
    ql_big_kernel(int n, double* __restrict__ work, int64_t wstride, uint32_t* status, bool last) {
  __shared__ double dpad[kBigMax + 1], epad[kBigMax + 1];   // index -1 is read and not used
  double *const d = dpad + 1, *const e = epad + 1;
  const int lane = threadIdx.x;
  const BigWork w(work + (int64_t)blockIdx.x * wstride, n);
  int l = w.state[1], steps = 0, t = 0, iter = 0;
  if (l < n) {
    for (int i = lane; i < n; i += 64) {
      d[i] = w.d[i];
      e[i] = w.e[i];
    }
    const int limit = sweep_limit(status), room = n * n;
    wave_sync();
#pragma unroll 1
    while (l < n) {
      int m = n - 1;
      for (int i0 = l;; i0 += 64) {
        const int i = i0 + lane;
        const uint64_t mask = __ballot(i >= n - 1 || negligible(e[i], d[i], d[i + 1]));
        if (mask != 0) {
          m = i0 + __builtin_ctzll(mask);
          break;
        }
      }
      m = __builtin_amdgcn_readfirstlane(m);
      if (m == l || iter >= limit) {
        if (m != l && lane == 0) atomicOr(status, kStatusNoConv);
        ++l;
        iter = 0;
        continue;
      }
      if (steps == 4 * n || t + (m - l) > room) break;
      if (lane == 0) w.step[steps] = make_uint2((uint32_t)l | (uint32_t)m << 16, (uint32_t)t);
      ++steps;
      ++iter;
      const double dl = d[l], el = e[l];
      double gg = 0.5 * (d[l + 1] - dl) * rcp_nr(el);
      double dn = d[m];
      const double h2 = fma(gg, gg, 1.0);
      gg = dn - dl + el * rcp_nr(gg + copysign(h2 * rsqrt_nr(h2), gg));
      double s = 1.0, c = 1.0, p = 0.0, ei = e[m - 1], di = d[m - 1];
      asm volatile("" : "+v"(di), "+v"(ei), "+v"(dn), "+v"(gg));   // see ql_kernel
#pragma unroll 1
      for (int i = m - 1; i >= l; --i) {
        double en = e[i - 1], dp = d[i - 1];
        const double f = s * ei, bb = c * ei;
        const double q = fma(f, f, gg * gg);
        const bool zero = q < 1e-290;
        const double inv = rsqrt_nr(zero ? 1.0 : q), eo = q * inv;
        s = f * inv;
        c = zero ? 1.0 : gg * inv;
        gg = dn - p;
        const double rr = fma(di - gg, s, 2.0 * c * bb);
        p = s * rr;
        d[i + 1] = gg + p;
        e[i + 1] = eo;
        gg = fma(c, rr, -bb);
        w.log[t] = make_double2(c, s);           // every lane the same value: no branch in the chain
        ++t;
        dn = di;
        asm volatile("" : "+v"(dp), "+v"(en) : "v"(gg), "v"(p));
        di = dp;
        ei = en;
      }
      d[l] = dn - p;
      e[l] = gg;
      e[m] = 0.0;
      wave_sync();
    }
    for (int i = lane; i < n; i += 64) {
      w.d[i] = d[i];
      w.e[i] = e[i];
    }
    if (last && l < n && lane == 0) atomicOr(status, kStatusNoConv);
  }
  if (lane == 0) {
    w.state[1] = l;
    w.state[2] = steps;
  }
}

__device__ __forceinline__ double read_lane(double x, int lane) {
  const int2 v = __builtin_bit_cast(int2, x);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(v.x, lane), __builtin_amdgcn_readlane(v.y, lane)));
}

// The round's rotations on 64 rows of Z (identity before the first round),
// a lane per row, columns in LDS.
__global__ void __launch_bounds__(64) rotate_big_kernel(int n, double* __restrict__ work, int64_t wstride, bool first) {
  extern __shared__ double tri_z[];              // [n][64]
  const int lane = threadIdx.x, r = blockIdx.x * 64 + lane;
  const BigWork w(work + (int64_t)blockIdx.y * wstride, n);
  const int steps = w.state[2];
  if (steps == 0 && !first) return;
  double* z = tri_z + lane;
  for (int c = 0; c < n; ++c) z[c * 64] = first ? (c == r ? 1.0 : 0.0) : r < n ? w.zt[(int64_t)c * n + r] : 0.0;
#pragma unroll 1
  for (int k = 0; k < steps; ++k) {
    const uint2 st = w.step[k];
    const int lo = __builtin_amdgcn_readfirstlane(st.x & 0xffff), hi = __builtin_amdgcn_readfirstlane(st.x >> 16);
    const int t0 = __builtin_amdgcn_readfirstlane(st.y), len = hi - lo;
    double zc = z[hi * 64];
    int i = hi - 1;
#pragma unroll 1
    for (int b = 0; b < len; b += 64) {
      const double2 x = w.log[t0 + (b + lane < len ? b + lane : len - 1)];
      const int cnt = len - b < 64 ? len - b : 64;
      int j = 0;
#pragma unroll 1
      for (; j + 4 <= cnt; j += 4, i -= 4) {
        double z0[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) z0[u] = z[(i - u) * 64];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double c = read_lane(x.x, j + u), s = read_lane(x.y, j + u);
          z[(i - u + 1) * 64] = fma(s, z0[u], c * zc);
          zc = fma(c, z0[u], -(s * zc));
        }
      }
#pragma unroll 1
      for (; j < cnt; ++j, --i) {
        const double c = read_lane(x.x, j), s = read_lane(x.y, j), z0 = z[i * 64];
        z[(i + 1) * 64] = fma(s, z0, c * zc);
        zc = fma(c, z0, -(s * zc));
      }
    }
    z[lo * 64] = zc;
  }
  if (r < n)
    for (int c = 0; c < n; ++c) w.zt[(int64_t)c * n + r] = z[c * 64];
}

// Column j of V = H_0 .. H_{n-2} diag(delta) z_j, its phase and its place, to
// the workspace in place of the log (V still holds the reflectors)
__global__ void __launch_bounds__(256)
    back_big_kernel(const double2* __restrict__ V, int n, double* __restrict__ work, int64_t wstride,
                    double* __restrict__ eps, double close) {
  constexpr int NX = kBigMax / 64;
  const int lane = threadIdx.x & 63, j = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= n) return;
  const int64_t b = blockIdx.y;
  const BigWork w(work + b * wstride, n);
  const double2* A = V + b * n * n;
  double2 x[NX], v[NX];
#pragma unroll
  for (int u = 0; u < NX; ++u) {
    const int r = lane + 64 * u;
    const double z = r < n ? w.zt[(int64_t)j * n + r] : 0.0;
    const double2 del = r < n ? w.delta[r] : make_double2(0.0, 0.0);
    x[u] = make_double2(z * del.x, z * del.y);
  }
  auto load = [&](int k) {
#pragma unroll
    for (int u = 0; u < NX; ++u) {
      const int r = lane + 64 * u;
      v[u] = k >= 0 && r > k && r < n ? A[(int64_t)k * n + r] : make_double2(0.0, 0.0);
    }
  };
  load(n - 2);
#pragma unroll 1
  for (int k = n - 2; k >= 0; --k) {
    double2 y[NX];
#pragma unroll
    for (int u = 0; u < NX; ++u) y[u] = v[u];
    const double tau = w.tau[k];
    load(k - 1);
    if (tau == 0.0) continue;                    // row k holds no reflector
    double2 s = make_double2(0.0, 0.0);
#pragma unroll
    for (int u = 0; u < NX; ++u) {
      s.x = fma(y[u].x, x[u].x, fma(y[u].y, x[u].y, s.x));
      s.y = fma(y[u].x, x[u].y, fma(-y[u].y, x[u].x, s.y));
    }
    s.x = tau * group_sum<64>(s.x);
    s.y = tau * group_sum<64>(s.y);
#pragma unroll
    for (int u = 0; u < NX; ++u) {
      x[u].x = fma(-y[u].x, s.x, fma(y[u].y, s.y, x[u].x));
      x[u].y = fma(-y[u].x, s.y, fma(-y[u].y, s.x, x[u].y));
    }
  }
  // the first entry that is as large as any (see kTied)
  double best = 0.0;
#pragma unroll
  for (int u = 0; u < NX; ++u) best = fmax(best, x[u].x * x[u].x + x[u].y * x[u].y);
  best = group_max<64>(best);
  int at = n;
  double2 bv = make_double2(1.0, 0.0);
#pragma unroll
  for (int u = NX - 1; u >= 0; --u)
    if (lane + 64 * u < n && x[u].x * x[u].x + x[u].y * x[u].y >= kTied * best) {
      at = lane + 64 * u;
      bv = x[u];
    }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double ox = __shfl_xor(bv.x, off, 64), oy = __shfl_xor(bv.y, off, 64);
    const int oa = __shfl_xor(at, off, 64);
    if (oa < at) {
      at = oa;
      bv = make_double2(ox, oy);
    }
  }
  const double mag = sqrt(bv.x * bv.x + bv.y * bv.y);
  const double2 fix = mag > 0.0 ? make_double2(bv.x / mag, -bv.y / mag) : make_double2(1.0, 0.0);
  // ascending order (ties by index)
  const double mine = w.d[j];
  int place = 0;
  bool order = true;
  double top = 0.0, gap = HUGE_VAL;
  for (int i = lane; i < n; i += 64) {
    const double o = w.d[i];
    order = order && o == o;
    place += (o < mine) || (o == mine && i < j);
    top = fmax(top, fabs(o));
    if (i != j) gap = fmin(gap, fabs(o - mine));
  }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) place += __shfl_xor(place, off, 64);
  if (-group_max<64>(-gap) <= close * group_max<64>(top)) w.state[3] = 1;
  if (!__all(order)) place = j;                  // NaN eigenvalues (a matrix that is not finite) would share places
  if (lane == 0) eps[b * n + place] = ldexp(mine, w.state[0]);
#pragma unroll
  for (int u = 0; u < NX; ++u) {
    const int r = lane + 64 * u;
    if (r < n)
      w.log[r * n + place] = make_double2(x[u].x * fix.x - x[u].y * fix.y, x[u].x * fix.y + x[u].y * fix.x);
  }
}

// V out of the workspace, and which matrices the Jacobi kernels leave out
__global__ void __launch_bounds__(256)
    store_big_kernel(int n, double* __restrict__ work, int64_t wstride, double2* __restrict__ V,
                     int* __restrict__ state) {
  const int64_t b = blockIdx.y, i = (int64_t)blockIdx.x * 256 + threadIdx.x, nn = (int64_t)n * n;
  const BigWork w(work + b * wstride, n);
  if (i < nn) V[b * nn + i] = w.log[i];
  if (i == 0) state[3 * b] = w.state[3] ? 0 : kLeaveOut;
}

ephw_status launch_big(double* H, int64_t batch, int n, double* eps, double* V, double* work, uint32_t* status,
                       double close, hipStream_t s) {
  if (!work) {
    set_error("tridiag_modes_eigh: orders above 32 need a workspace");
    return EPHW_EINVAL;
  }
  constexpr int64_t kChunk = 1024;               // that of jacobi_work_doubles
  const int64_t chunk = batch < kChunk ? batch : kChunk;
  const int64_t wstride = jacobi_work_doubles(n, chunk) / chunk & ~(int64_t)1;
  const size_t lds = (size_t)n * 64 * sizeof(double);
  EPHW_HIP(hipFuncSetAttribute((const void*)rotate_big_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  for (int64_t b0 = 0; b0 < batch; b0 += chunk) {
    const unsigned nb = (unsigned)(batch - b0 < chunk ? batch - b0 : chunk);
    double2 *h = reinterpret_cast<double2*>(H) + b0 * n * n, *v = reinterpret_cast<double2*>(V) + b0 * n * n;
    hipLaunchKernelGGL(reduce_big_kernel, dim3(nb), dim3(kBigThreads), 0, s, h, n, v, work, wstride);
    EPHW_CHECK_LAUNCH();
    for (int round = 0; round < kBigRounds; ++round) {
      hipLaunchKernelGGL(ql_big_kernel, dim3(nb), dim3(64), 0, s, n, work, wstride, status, round + 1 == kBigRounds);
      EPHW_CHECK_LAUNCH();
      hipLaunchKernelGGL(rotate_big_kernel, dim3((unsigned)ceil_div(n, 64), nb), dim3(64), lds, s, n, work, wstride,
                         round == 0);
      EPHW_CHECK_LAUNCH();
    }
    hipLaunchKernelGGL(back_big_kernel, dim3((unsigned)ceil_div(n, 4), nb), dim3(256), 0, s, v, n, work, wstride,
                       eps + b0 * n, close);
    EPHW_CHECK_LAUNCH();
    hipLaunchKernelGGL(store_big_kernel, dim3((unsigned)ceil_div((int64_t)n * n, 256), nb), dim3(256), 0, s, n, work,
                       wstride, v, jacobi_large_state(work, n, nb));
    EPHW_CHECK_LAUNCH();
    EPHW_TRY(jacobi_eigh_some(reinterpret_cast<double*>(h), nb, n, eps + b0 * n, reinterpret_cast<double*>(v), work,
                              status, s));
  }
  return EPHW_OK;
}

template <int N, int L, bool KEEP = false>
ephw_status launch(double* H, int64_t batch, int n, double* eps, double* V, uint32_t* status, hipStream_t s,
                   double close = 0.0) {
  using S = TriShape<N, L>;
  const int64_t grid = ceil_div(batch, (int64_t)S::waves * S::G), gridq = ceil_div(batch, QlShape<N>::M);
  if (grid > 0x7fffffff || gridq > 0x7fffffff) {
    set_error("tridiag_eigh: too many matrices for one launch");
    return EPHW_EUNSUPPORTED;
  }
  // every column's phase needs a thread as well as every row
  const int rows = QlShape<N>::M * (n > QlShape<N>::CB ? n : QlShape<N>::CB);
  hipLaunchKernelGGL((reduce_kernel<N, L, KEEP>), dim3((unsigned)grid), dim3(64 * S::waves), 0, s,
                     reinterpret_cast<double2*>(H), batch, n, eps, reinterpret_cast<double2*>(V));
  EPHW_CHECK_LAUNCH();
  hipLaunchKernelGGL((ql_kernel<N, KEEP>), dim3((unsigned)gridq), dim3((unsigned)((rows + 63) / 64 * 64)), 0, s,
                     reinterpret_cast<double2*>(H), batch, n, eps, reinterpret_cast<double2*>(V), status, close);
  EPHW_CHECK_LAUNCH();
  return EPHW_OK;
}

}  // namespace

// By the order alone: states of degenerate bands are the solver's own choice, and
// must not depend on how the points are divided over calls, q batches or ranks.
// Up to order 6 the two are level (n = 3: 82 us by Jacobi and 99 here at 131 072
// matrices, n = 6: 280 and 261).  From 7 on this one is ahead where there are
// thousands of matrices (4096 of n = 8: 54 and 50 us, n = 11: 108 and 77, n = 16:
// 291 and 142, n = 24: 1731 and 369); 64 matrices are level up to order 12 (n = 11:
// 77 and 73), up to 30 us behind from 13 to 17 (n = 14: 93 and 115, n = 17: 126
// and 158), where the Jacobi rounds are the shorter chain, and ahead again at 24
// (457 and 266).
bool tridiag_better(int n) { return n > 6 && n <= 32; }

ephw_status tridiag_eigh(double* H, int64_t batch, int n, double* eps, double* V, uint32_t* status, hipStream_t s) {
  if (batch <= 0) return EPHW_OK;
  if (n < 1 || n > 32) {
    set_error("tridiag_eigh: matrix order must be in [1, 32]");
    return EPHW_EUNSUPPORTED;
  }
  if ((reinterpret_cast<uintptr_t>(H) | reinterpret_cast<uintptr_t>(V)) & 15) {
    set_error("tridiag_eigh: matrices and eigenvectors must be 16-byte aligned complex128 arrays");
    return EPHW_EINVAL;
  }
  if (n <= 8) return launch<8, 8>(H, batch, n, eps, V, status, s);
  if (n <= 12) return launch<12, 16>(H, batch, n, eps, V, status, s);
  if (n <= 16) return launch<16, 16>(H, batch, n, eps, V, status, s);
  if (n <= 24) return launch<24, 32>(H, batch, n, eps, V, status, s);
  return launch<32, 32>(H, batch, n, eps, V, status, s);
}

// Up to 22 the Jacobi rounds of few matrices are the shorter chain (whole calls,
// n = 18, 64 matrices: 155 by Jacobi and 227 us here; 2048: 392 and 404, 4096: 751
// and 684; n = 21, 64: 230 and 272, 2048: 560 and 476; n = 24, one: 460 and 260).
// From 33 to 63 few
// matrices are level (n = 33: 469 by Jacobi and 445 us here, n = 48: 680 and 750),
// 512 are not (n = 48: 2824 and 1371); n = 66, one matrix: 1362 and 1270, n = 150:
// 9913 and 5409, n = 255, 64 matrices: 73 500 and 18 140.
bool tridiag_modes_better(int n, int64_t batch) {
  if (n <= 32) return n > 22 || (n > 16 && batch >= 2048);
  return n <= kBigMax && (n >= 64 || batch >= 256);
}

ephw_status tridiag_modes_eigh(double* H, int64_t batch, int n, double* eps, double* V, double* work, uint32_t* status,
                               double close, hipStream_t s) {
  if (batch <= 0) return EPHW_OK;
  if (n <= 16 || n > kBigMax) {
    set_error("tridiag_modes_eigh: matrix order must be in [17, 256]");
    return EPHW_EUNSUPPORTED;
  }
  if ((reinterpret_cast<uintptr_t>(H) | reinterpret_cast<uintptr_t>(V)) & 15) {
    set_error("tridiag_modes_eigh: matrices and eigenvectors must be 16-byte aligned complex128 arrays");
    return EPHW_EINVAL;
  }
  if (n > 32) return launch_big(H, batch, n, eps, V, work, status, close, s);
  if (n <= 24)
    EPHW_TRY((launch<24, 32, true>(H, batch, n, eps, V, status, s, close)));
  else
    EPHW_TRY((launch<32, 32, true>(H, batch, n, eps, V, status, s, close)));
  return jacobi_eigh_some(H, batch, n, eps, V, nullptr, status, s);
}

}  // namespace ephw
