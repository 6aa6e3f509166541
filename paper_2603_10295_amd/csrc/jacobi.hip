// Batched Hermitian eigensolver in FP64: cyclic two-sided Jacobi with the
// round-robin (tournament) ordering, so every step rotates n/2 disjoint
// (p, q) planes at once.
//
// Rotation of plane (p, q) with a = A_pp, d = A_qq, b = A_pq = |b| e^{i phi}:
//   tau = (d - a) / (2|b|), t = sign(tau) / (|tau| + sqrt(1 + tau^2)),
//   c = 1/sqrt(1 + t^2), s = t c,
//   J = [[c, s e^{i phi}], [-s e^{-i phi}, c]]  (unitary; J^H A J zeroes A_pq).
// A <- A J (columns), V <- V J, then A <- J^H A (rows).  A sweep visits every
// plane once; sweeps repeat until the off-diagonal Frobenius norm is below
// 1e-14 of the total norm.
//
// Small matrices (n <= 32) live in LDS sized to the order (4 KB per solve at
// n = 11) so that a CU holds as many solves as its registers allow; each lane
// owns one 2x2 block of the round (below), a wavefront runs one solve, or
// several up to n = 12.  Large matrices (n > 32) live in a global workspace,
// one 1024-thread workgroup per matrix (the rotation parameters stay in LDS).
#include "kernels.h"

namespace ephw {
namespace {

constexpr double kOffTol2 = 1e-28;  // (off-diagonal norm / total norm)^2 at convergence

__device__ __forceinline__ int player_at(int pos, int round, int n2) {
  return pos == 0 ? 0 : 1 + ((pos - 1 + round) % (n2 - 1));
}

// the pair of a round that holds the missing player n2 - 1 of an odd order
__device__ __forceinline__ int missing_pair(int round, int n2) {
  // position of player n2 - 1: 1 + (n2 - 2 - round) mod (n2 - 1)
  const int d = n2 - 2 - round, pos = 1 + (d < 0 ? d + n2 - 1 : d);
  return pos < n2 - 1 - pos ? pos : n2 - 1 - pos;
}

template <int NT>
__device__ double block_sum(double v, double* red) {
  // wave reduction then across waves through LDS
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double tot = 0;
  for (int w = 0; w < NT / 64; ++w) tot += red[w];
  return tot;
}

constexpr int kSmallN = 32;
constexpr int kSmallPerBlock = 4;  // small solves (wavefronts) per workgroup

// ---------------------------------------------------------------------------
// Small solves (n <= 32): a 64-lane wavefront per matrix (several matrices
// up to n = 12, below), A and V in LDS as
// interleaved complex with the order padded to N2 = 2 NP (a zero row and
// column for odd n, whose pair is then the identity).  In each round of the
// tournament the NP disjoint planes cut A and V into NP^2 2x2 blocks, rows
// {p_i, q_i} x columns {p_j, q_j}.  J_i^H A J_j and V J_j touch only block
// (i, j), so one lane updates a block with no other lane's data.  A stays
// exactly Hermitian: only its upper triangle is kept (an entry below the
// diagonal is read as the conjugate of its transpose) and only blocks with
// i <= j are computed.  The
// NP (NP + 1) / 2 blocks of A and the NP^2 of V are one list of tasks of the
// same shape (V's left rotation is the identity), 57 of them at n = 11, so
// the round is a single pass over the wave.  The sweep's last round sums
// |A|^2 (total and off-diagonal) over the blocks it wrote, so the stopping
// test costs one wave reduction per sweep.
//
// Rotation parameters without divisions, for x = d - a, y = 2|b|:
//   r = sqrt(x^2 + y^2), w = |x| + r, z = 1/sqrt(w^2 + y^2),
//   c = w z, s = sign(x) y z, sigma = s b/|b| = sign(x) 2 z b,
// which are the t = sign(tau)/(|tau| + sqrt(1 + tau^2)) formulas above with
// the common factors cleared; J = [[c, sigma], [-conj(sigma), c]].
// ---------------------------------------------------------------------------
template <int NP>
struct SmallLayout {
  static constexpr int N2 = 2 * NP;
  static constexpr int NA = NP * (NP + 1) / 2;                   // blocks of A (i <= j)
  static constexpr int NT = NA + NP * NP;                         // tasks: A blocks, then V blocks
  static constexpr int TPL = (NT + 63) / 64;                      // tasks per lane
  static constexpr size_t a_elems = (size_t)N2 * N2;            // complex
  // A and V: the full squares, or, where the solve keeps per-lane offsets
  // (one task per lane), task-major: entry e of task t's block at e RS + t,
  // the regions RS apart (an odd stride above 32 tasks, which spreads the
  // scattered stores to the moved positions over more LDS banks)
  static constexpr bool kTaskMajor = TPL == 1;
  static constexpr int RS = NT > 32 ? 63 : NT;
  static constexpr size_t data_elems = kTaskMajor ? 3 * (size_t)RS + NT : 2 * a_elems;
  static constexpr size_t prm_elems = 2 * (size_t)NP;            // per pair (c, 0), sigma; task-major: sigma[NP], c[NP]
  static constexpr size_t fix_elems = (size_t)N2;                // phase fix per column
  static constexpr size_t bytes = (data_elems + prm_elems + fix_elems) * 16 + (size_t)N2 * 4;
  static constexpr size_t slice_elems = (bytes + 15) / 16;       // one wavefront's share, 16-byte units
  // per-round task descriptors and plane pairs, shared by the workgroup's
  // solves (which all have this padded order), when they fit
  static constexpr size_t table_bytes = (size_t)(N2 - 1) * NT * 8 + (size_t)(N2 - 1) * NP * 4;
  static constexpr bool kTable = TPL > 1 && table_bytes <= 32768;
  static constexpr size_t table_elems = kTable ? (table_bytes + 15) / 16 : 0;
};

template <int NP>
__host__ __device__ __forceinline__ void decode_task(int t, bool& is_v, int& i, int& j) {
  constexpr int NA = SmallLayout<NP>::NA;
  if (t < NA) {
    int r = 0, rest = t;
    while (rest >= NP - r) {
      rest -= NP - r;
      ++r;
    }
    is_v = false;
    i = r;
    j = r + rest;
  } else {
    const int v = t - NA;
    is_v = true;
    i = v / NP;
    j = v % NP;
  }
}

// plane of pair k in a round: p | q << 8 with p < q
__device__ __forceinline__ int pair_pq(int k, int round, int n2) {
  const int u = player_at(k, round, n2), v = player_at(n2 - 1 - k, round, n2);
  return u < v ? (u | v << 8) : (v | u << 8);
}

// The four entries of task t's block in a round, as offsets into the solve's
// slice (A at 0, V after it); bit 15 marks an entry of A below the diagonal,
// held as the conjugate of its transpose.
template <int NP>
__device__ __forceinline__ uint2 task_entries(int t, int round) {
  using L = SmallLayout<NP>;
  constexpr int N2 = L::N2;
  bool is_v;
  int i, j;
  decode_task<NP>(t, is_v, i, j);
  const int pqi = pair_pq(i, round, N2), pqj = pair_pq(j, round, N2);
  const int rr[2] = {pqi & 0xff, pqi >> 8}, cc[2] = {pqj & 0xff, pqj >> 8};
  uint32_t d[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = rr[e >> 1], c = cc[e & 1];
    d[e] = is_v ? (uint32_t)(L::a_elems + r * N2 + c)
                : (r <= c ? (uint32_t)(r * N2 + c) : (uint32_t)(c * N2 + r) | 0x8000u);
  }
  return make_uint2(d[0] | d[1] << 16, d[2] | d[3] << 16);
}

template <int NP>
__device__ void build_tables(uint2* ent, int* pq) {
  using L = SmallLayout<NP>;
  constexpr int N2 = L::N2;
  for (int e = threadIdx.x; e < (N2 - 1) * L::NT; e += blockDim.x) ent[e] = task_entries<NP>(e % L::NT, e / L::NT);
  for (int e = threadIdx.x; e < (N2 - 1) * NP; e += blockDim.x) pq[e] = pair_pq(e % NP, e / NP, N2);
}

// Position order.  A and V are held with their rows and columns (V: columns)
// in tournament-position order: pair k of every round is positions k and
// N2 - 1 - k, and after each round the indices move to the positions they take
// in the next one.  The move is the same every round (the index at position 1
// goes to the last position, those above 1 move down by one, position 0
// stays), so a lane's block has fixed load addresses and fixed store
// addresses (the moved positions) in every round; after a whole sweep of
// N2 - 1 rounds every index is back at its own position.
__host__ __device__ __forceinline__ int next_pos(int pos, int n2) {
  return pos == 0 ? 0 : (pos == 1 ? n2 - 1 : pos - 1);
}

// Where entries live in the one-task-per-lane solves: entry e (0..3, row
// bit then column bit) of task t's block at e RS + t, so that each of a
// round's four loads reads consecutive lanes' entries from consecutive
// addresses (no LDS bank conflicts).  In position order the entry (r, c)
// belongs to the planes pr(r), pr(c) of its row and column (pr(x) = x below
// NP, else N2 - 1 - x), at row bit r >= NP and column bit c >= NP.  A keeps
// one slot per entry of its upper triangle: an entry below the diagonal is
// read and written as the conjugate of its transpose (bit 15 of the offset).
// V: task NA + pr(r) NP + pr(c).  A, (r, c) with r <= c, a = pr(r), b = pr(c):
// a < b: block (a, b); a > b: block (b, a), whose entry (c, r) lies below
// the diagonal and so holds this one; a = b: the diagonal block (a, a), whose
// entries (a, N2-1-a) and (N2-1-a, a) share slot 1.
template <int NP>
__host__ __device__ __forceinline__ uint32_t entry_offset(bool is_v, int r, int c) {
  using L = SmallLayout<NP>;
  constexpr int N2 = L::N2, RS = L::RS, NA = L::NA;
  const auto pr = [](int x) { return x < NP ? x : N2 - 1 - x; };
  const auto hi = [](int x) { return x >= NP ? 1 : 0; };
  // task of A block (a, b), a <= b: the blocks are numbered row by row
  const auto task_a = [](int a, int b) { return a * NP - a * (a - 1) / 2 + (b - a); };
  if (is_v) return (uint32_t)((2 * hi(r) + hi(c)) * RS + NA + pr(r) * NP + pr(c));
  uint32_t flag = 0;
  if (r > c) {
    const int t = r;
    r = c;
    c = t;
    flag = 0x8000u;
  }
  const int a = pr(r), b = pr(c);
  int e, t;
  if (a < b) {
    e = 2 * hi(r) + hi(c);
    t = task_a(a, b);
  } else if (a > b) {
    e = 2 * hi(c) + hi(r);
    t = task_a(b, a);
  } else {
    e = r == c ? 3 * hi(r) : 1;
    t = task_a(a, a);
  }
  return (uint32_t)(e * RS + t) | flag;
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// x' = c x - conj(sg) y ; y' = sg x + c y   (one row of [x y] J)
__device__ __forceinline__ void rot_right(double2& x, double2& y, double c, double2 sg) {
  const double2 nx = make_double2(fma(c, x.x, -fma(sg.x, y.x, sg.y * y.y)), fma(c, x.y, -fma(sg.x, y.y, -sg.y * y.x)));
  const double2 ny = make_double2(fma(c, y.x, fma(sg.x, x.x, -sg.y * x.y)), fma(c, y.y, fma(sg.x, x.y, sg.y * x.x)));
  x = nx;
  y = ny;
}

// x' = c x - sg y ; y' = conj(sg) x + c y   (one column of J^H [x; y])
__device__ __forceinline__ void rot_left(double2& x, double2& y, double c, double2 sg) {
  const double2 nx = make_double2(fma(c, x.x, -fma(sg.x, y.x, -sg.y * y.y)), fma(c, x.y, -fma(sg.x, y.y, sg.y * y.x)));
  const double2 ny = make_double2(fma(c, y.x, fma(sg.x, x.x, sg.y * x.y)), fma(c, y.y, fma(sg.x, x.y, -sg.y * x.x)));
  x = nx;
  y = ny;
}

__device__ __forceinline__ double norm2(double2 v) { return v.x * v.x + v.y * v.y; }

// entry descriptor (15-bit offset, conjugate flag in bit 15) -> value
__device__ __forceinline__ double flip_sign(double v, uint32_t d) {
  return __longlong_as_double(__double_as_longlong(v) ^ ((long long)(d & 0x8000u) << 48));
}
__device__ __forceinline__ double2 ld_entry(const double2* X, uint32_t d) {
  const double2 v = X[d & 0x7fffu];
  return make_double2(v.x, flip_sign(v.y, d));
}
__device__ __forceinline__ void st_entry(double2* X, uint32_t d, double2 v) {
  X[d & 0x7fffu] = make_double2(v.x, flip_sign(v.y, d));
}

// the solve of a matrix is one wavefront's (wave_sync, no workgroup barrier)

template <int NP>
__device__ __forceinline__ void jacobi_small_body(const double* __restrict__ H, int n, double* __restrict__ eps,
                                                  double* __restrict__ Vout, uint32_t* status, double tol2, int64_t b,
                                                  double2* slice, int lane, const uint2* ent, const int* pqt) {
  using L = SmallLayout<NP>;
  constexpr int N2 = L::N2;
  double2* A = slice;
  double2* V = A + L::a_elems;
  double2* prm = V + L::a_elems;
  double2* fix = prm + L::prm_elems;
  int* perm = reinterpret_cast<int*>(fix + L::fix_elems);
  const double2* h = reinterpret_cast<const double2*>(H) + b * n * n;
  const double2 zero = make_double2(0.0, 0.0);

  // this lane's tasks, packed as (is_v << 16) | (i << 8) | j; the list does not change between rounds
  int task[L::TPL];
#pragma unroll
  for (int k = 0; k < L::TPL; ++k) {
    const int t = lane + 64 * k;
    int code = -1;
    if (t < L::NT) {
      bool is_v;
      int i, j;
      decode_task<NP>(t, is_v, i, j);
      code = (is_v ? 1 << 16 : 0) | (i << 8) | j;
    }
    task[k] = code;
  }

  double off = 0.0, tot = 0.0;
  for (int e = lane; e < N2 * N2; e += 64) {
    const int r = e / N2, c = e % N2;
    double2 v = (r < n && c < n) ? h[r * n + c] : zero;
    if (r == c) v.y = 0.0;  // Hermitian: a real diagonal
    A[e] = v;
    V[e] = (r == c && r < n) ? make_double2(1.0, 0.0) : zero;
    const double m = norm2(v);
    tot += m;
    off += r != c ? m : 0.0;
  }
  off = wave_sum(off);
  tot = wave_sum(tot);
  wave_sync();
  bool converged = n <= 1 || off <= tol2 * tot;
  off = 0.0;
  tot = 0.0;
  const int max_sweeps = sweep_limit(status);
  for (int sweep = 0; sweep < max_sweeps && !converged; ++sweep) {
#pragma unroll 1
    for (int round = 0; round < N2 - 1; ++round) {
      if (lane < NP) {
        const int pq = L::kTable ? pqt[round * NP + lane] : pair_pq(lane, round, N2);
        const int p = pq & 0xff, q = pq >> 8;
        double c = 1.0;
        double2 sg = zero;
        if (q < n) {
          const double2 bpq = A[p * N2 + q];
          const double bm2 = norm2(bpq);
          if (bm2 > 0.0) {
            const double x = A[q * N2 + q].x - A[p * N2 + p].x;
            const double y2 = 4.0 * bm2;
            const double w = fabs(x) + sqrt(fma(x, x, y2));
            const double z = rsqrt(fma(w, w, y2));
            c = w * z;
            const double f = (x >= 0.0 ? 2.0 : -2.0) * z;  // sigma = sign(x) y z b/|b| = sign(x) 2 z b
            sg = make_double2(f * bpq.x, f * bpq.y);
          }
        }
        prm[2 * lane] = make_double2(c, 0.0);
        prm[2 * lane + 1] = sg;
      }
      wave_sync();
      const bool last = round == N2 - 2;
#pragma unroll
      for (int k = 0; k < L::TPL; ++k) {
        const int code = task[k];
        if (code < 0) continue;
        const bool is_v = code >= (1 << 16);
        const int i = (code >> 8) & 0xff, j = code & 0xff;
        const uint2 d = L::kTable ? ent[round * L::NT + lane + 64 * k] : task_entries<NP>(lane + 64 * k, round);
        const double cj = prm[2 * j].x;
        const double2 sj = prm[2 * j + 1];
        const double ci = is_v ? 1.0 : prm[2 * i].x;
        const double2 si = is_v ? zero : prm[2 * i + 1];
        // A holds its upper triangle only: an entry below the diagonal is the
        // conjugate of its transpose (flagged in its descriptor)
        double2 x00 = ld_entry(slice, d.x & 0xffff), x01 = ld_entry(slice, d.x >> 16);
        double2 x10 = ld_entry(slice, d.y & 0xffff), x11 = ld_entry(slice, d.y >> 16);
        rot_right(x00, x01, cj, sj);
        rot_right(x10, x11, cj, sj);
        rot_left(x00, x10, ci, si);
        rot_left(x01, x11, ci, si);
        const bool diag = !is_v && i == j;
        if (diag) {
          // a rotated Hermitian 2x2 block: real diagonal, the plane's pair
          // annihilated exactly (an unrotated one keeps its entries bit for bit)
          if (norm2(si) > 0.0) {
            x00.y = 0.0;
            x11.y = 0.0;
            x01 = zero;
            x10 = zero;
          }
        }
        st_entry(slice, d.x & 0xffff, x00);
        st_entry(slice, d.x >> 16, x01);
        st_entry(slice, d.y & 0xffff, x10);
        st_entry(slice, d.y >> 16, x11);
        if (last && !is_v) {
          const double d = norm2(x00) + norm2(x11), o = norm2(x01) + norm2(x10);
          tot += diag ? d + o : 2.0 * (d + o);
          off += diag ? o : 2.0 * (d + o);
        }
      }
      wave_sync();
    }
    off = wave_sum(off);
    tot = wave_sum(tot);
    converged = off <= tol2 * tot;
    off = 0.0;
    tot = 0.0;
  }
  if (!converged && lane == 0) atomicOr(status, kStatusNoConv);
  // ascending order (ties by index), then each column's largest entry made real positive
  if (lane < n) perm[ascending_place([&](int j) { return A[j * N2 + j].x; }, n, lane)] = lane;
  wave_sync();
  if (lane < n) {
    const int src = perm[lane];
    eps[b * n + lane] = A[src * N2 + src].x;
    double best = -1.0;
    double2 bv = make_double2(1.0, 0.0);
    for (int r = 0; r < n; ++r) {
      const double2 v = V[r * N2 + src];
      const double m = norm2(v);
      if (m > best) {
        best = m;
        bv = v;
      }
    }
    for (int r = 0; n > 16 && r < n; ++r) {
      const double2 v = V[r * N2 + src];
      if (norm2(v) >= kTied * best) {
        best = norm2(v);
        bv = v;
        break;
      }
    }
    const double mag = sqrt(best);
    fix[lane] = mag > 0.0 ? make_double2(bv.x / mag, -bv.y / mag) : make_double2(1.0, 0.0);
  }
  wave_sync();
  double2* out = reinterpret_cast<double2*>(Vout) + b * n * n;
  for (int e = lane; e < n * n; e += 64) {
    const int r = e / n, c = e % n;
    const double2 v = V[r * N2 + perm[c]], f = fix[c];
    out[e] = make_double2(v.x * f.x - v.y * f.y, v.x * f.y + v.y * f.x);
  }
}

// The solve for orders with one task per lane (n <= 12): A and V in position
// order, so every round loads and stores at the same per-lane offsets with
// no per-round descriptors (about a fifth fewer instructions per round).
// Larger orders keep the per-round descriptor tables: holding all of a
// lane's tasks in registers across the round would cost their occupancy.
//
// A wavefront runs several such solves: G lane groups of LPM lanes (the
// tasks of one solve, rounded up to a power of two) and S solves per group,
// whose blocks a lane updates one after the other with the same offsets.
// The plane parameters of the group's S solves come from S NP lanes at once,
// so the instructions of that step (about a third of a round's with one solve
// per wavefront) serve S solves.  The wavefront sweeps until all its solves have
// converged; a converged solve takes identity rotations (c = 1, sigma = 0,
// which leave every entry unchanged) and only moves its entries through the
// positions, so its results do not depend on the solves beside it.
template <int NP>
struct PosShape {
  static constexpr int NT = SmallLayout<NP>::NT;
  static constexpr int LPM = NT <= 2 ? 2 : NT <= 4 ? 4 : NT <= 8 ? 8 : NT <= 16 ? 16 : NT <= 32 ? 32 : 64;
  static constexpr int G = 64 / LPM;
  static constexpr int S = 2;
  static constexpr int M = G * S;  // solves per wavefront
  static_assert(S * NP <= LPM && 2 * NP <= LPM, "a group's lanes must cover its plane parameters and its order");
};

template <int NP>
constexpr int solves_per_wave() {
  if constexpr (SmallLayout<NP>::TPL == 1) return PosShape<NP>::M;
  else return 1;
}

// one solve of a wavefront: matrix b of H (n x n), its outputs; n = 0: none
struct PosJob {
  const double* H;
  double* eps;
  double* V;
  int64_t b;
  int n;
};

template <int LPM>
__device__ __forceinline__ double group_sum(double v) {
  for (int m = LPM / 2; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// job_at(s): the group's solve s (called before the sweeps and again for the
// outputs, so that no job is held in registers across them); slices: the
// group's S solve slices, one after the other; lg: lane in group
template <int NP, class JobAt>
__device__ __forceinline__ void jacobi_small_body_pos(JobAt job_at, uint32_t* status, double tol2, double2* slices,
                                                      int lg) {
  using L = SmallLayout<NP>;
  using P = PosShape<NP>;
  constexpr int N2 = L::N2, S = P::S, LPM = P::LPM;
  constexpr size_t SL = L::slice_elems, PO = L::data_elems;
  static_assert(L::kTaskMajor, "the one-task-per-lane solve keeps A and V task-major");
  // entry (r, c) of A (r <= c, no conjugate flag) or of V
  const auto at_a = [](int r, int c) { return entry_offset<NP>(false, r, c); };
  const auto at_v = [](int r, int c) { return entry_offset<NP>(true, r, c); };
  const double2 zero = make_double2(0.0, 0.0);

  // this lane's task: block (i, j) of A (i <= j) or of V, i.e. rows
  // {i, N2-1-i} x columns {j, N2-1-j} in position order (V: rows are the
  // basis, paired the same way), with the four entries' load offsets and the
  // offsets they are stored to (their positions in the next round); the
  // same in each of the group's solves
  int code = -1;
  uint2 ldo = make_uint2(0, 0), sto = make_uint2(0, 0);
  if (lg < L::NT) {
    bool is_v;
    int i, j;
    decode_task<NP>(lg, is_v, i, j);
    code = (is_v ? 1 << 16 : 0) | (i << 8) | j;
    const int rr[2] = {i, N2 - 1 - i}, cc[2] = {j, N2 - 1 - j};
    uint32_t l[4], w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = rr[e >> 1], c = cc[e & 1];
      l[e] = entry_offset<NP>(is_v, r, c);
      w[e] = entry_offset<NP>(is_v, is_v ? r : next_pos(r, N2), next_pos(c, N2));
    }
    ldo = make_uint2(l[0] | l[1] << 16, l[2] | l[3] << 16);
    sto = make_uint2(w[0] | w[1] << 16, w[2] | w[3] << 16);
  }
  const bool is_v = code >= (1 << 16);
  const int ti = (code >> 8) & 0xff, tj = code & 0xff;
  const bool diag = code >= 0 && !is_v && ti == tj;

  bool conv[S];
  double off[S], tot[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    double2* X = slices + s * SL;
    const PosJob job = job_at(s);
    const int n = job.n;
    const double2* h = reinterpret_cast<const double2*>(job.H) + job.b * n * n;
    double o = 0.0, t = 0.0;
    for (int e = lg; e < N2 * N2; e += LPM) {
      const int r = e / N2, c = e % N2;
      double2 v = (r < n && c < n) ? h[r * n + c] : zero;
      if (r == c) v.y = 0.0;  // Hermitian: a real diagonal
      if (r <= c) X[at_a(r, c)] = v;
      X[at_v(r, c)] = (r == c && r < n) ? make_double2(1.0, 0.0) : zero;
      const double m = norm2(v);
      t += m;
      o += r != c ? m : 0.0;
    }
    o = group_sum<LPM>(o);
    t = group_sum<LPM>(t);
    conv[s] = n <= 1 || o <= tol2 * t;
    off[s] = 0.0;
    tot[s] = 0.0;
  }
  wave_sync();
  const int max_sweeps = sweep_limit(status);
  for (int sweep = 0; sweep < max_sweeps; ++sweep) {
    bool all = true;
#pragma unroll
    for (int s = 0; s < S; ++s) all = all && conv[s];
    if (__all(all)) break;
#pragma unroll 1
    for (int round = 0; round < N2 - 1; ++round) {
      if (lg < S * NP) {
        // pair k of solve s: positions p = k, q = N2-1-k (a zero padding row
        // and column give b = 0, the identity)
        const int s = lg / NP, k = lg - s * NP;
        double2* A = slices + s * SL;
        double2* prm = A + PO;
        bool done = conv[0];
#pragma unroll
        for (int u = 1; u < S; ++u) done = s == u ? conv[u] : done;
        const int p = k, q = N2 - 1 - k;
        double c = 1.0;
        double2 sg = zero;
        const double2 bpq = A[at_a(p, q)];
        const double bm2 = norm2(bpq);
        if (!done && bm2 > 0.0) {
          const double x = A[at_a(q, q)].x - A[at_a(p, p)].x;
          const double y2 = 4.0 * bm2;
          const double w = fabs(x) + sqrt(fma(x, x, y2));
          const double z = rsqrt(fma(w, w, y2));
          c = w * z;
          const double f = (x >= 0.0 ? 2.0 : -2.0) * z;  // sigma = sign(x) y z b/|b| = sign(x) 2 z b
          sg = make_double2(f * bpq.x, f * bpq.y);
        }
        prm[k] = sg;
        reinterpret_cast<double*>(prm + NP)[k] = c;
      }
      wave_sync();
      const bool last = round == N2 - 2;
      // every entry is read before any is written (the stores go to the
      // moved positions, which other tasks read in this round)
      double2 x[S][4];
      if (code >= 0) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const double2* X = slices + s * SL;
          x[s][0] = ld_entry(X, ldo.x & 0xffff);
          x[s][1] = ld_entry(X, ldo.x >> 16);
          x[s][2] = ld_entry(X, ldo.y & 0xffff);
          x[s][3] = ld_entry(X, ldo.y >> 16);
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
          double2* X = slices + s * SL;
          // sigma of the NP planes, then their c: consecutive planes' parameters
          // in consecutive LDS banks
          const double2* prm = X + PO;
          const double* pc = reinterpret_cast<const double*>(prm + NP);
          const double cj = pc[tj];
          const double2 sj = prm[tj];
          const double ci = is_v ? 1.0 : pc[ti];
          const double2 si = is_v ? zero : prm[ti];
          double2 x00 = x[s][0], x01 = x[s][1], x10 = x[s][2], x11 = x[s][3];
          rot_right(x00, x01, cj, sj);
          rot_right(x10, x11, cj, sj);
          rot_left(x00, x10, ci, si);
          rot_left(x01, x11, ci, si);
          if (diag) {
            // a rotated Hermitian 2x2 block: real diagonal, the plane's pair
            // annihilated exactly (an unrotated one keeps its entries bit for bit)
            if (norm2(si) > 0.0) {
              x00.y = 0.0;
              x11.y = 0.0;
              x01 = zero;
              x10 = zero;
            }
          }
          st_entry(X, sto.x & 0xffff, x00);
          st_entry(X, sto.x >> 16, x01);
          st_entry(X, sto.y & 0xffff, x10);
          st_entry(X, sto.y >> 16, x11);
          if (last && !is_v) {
            const double d = norm2(x00) + norm2(x11), o = norm2(x01) + norm2(x10);
            tot[s] += diag ? d + o : 2.0 * (d + o);
            off[s] += diag ? o : 2.0 * (d + o);
          }
        }
      }
      wave_sync();
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const double o = group_sum<LPM>(off[s]), t = group_sum<LPM>(tot[s]);
      conv[s] = conv[s] || o <= tol2 * t;
      off[s] = 0.0;
      tot[s] = 0.0;
    }
  }
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (!conv[s] && lg == 0) atomicOr(status, kStatusNoConv);
  // ascending order (ties by index), then each column's largest entry made real positive
#pragma unroll
  for (int s = 0; s < S; ++s) {
    double2* A = slices + s * SL;
    int* perm = reinterpret_cast<int*>(A + PO + L::prm_elems + L::fix_elems);
    const int n = job_at(s).n;
    if (lg < n) perm[ascending_place([&](int j) { return A[at_a(j, j)].x; }, n, lg)] = lg;
  }
  wave_sync();
#pragma unroll
  for (int s = 0; s < S; ++s) {
    double2* A = slices + s * SL;
    double2* fix = A + PO + L::prm_elems;
    const int* perm = reinterpret_cast<const int*>(fix + L::fix_elems);
    const PosJob job = job_at(s);
    const int n = job.n;
    if (lg < n) {
      const int src = perm[lg];
      job.eps[job.b * n + lg] = A[at_a(src, src)].x;
      double best = -1.0;
      double2 bv = make_double2(1.0, 0.0);
      for (int r = 0; r < n; ++r) {
        const double2 v = A[at_v(r, src)];
        const double m = norm2(v);
        if (m > best) {
          best = m;
          bv = v;
        }
      }
      const double mag = sqrt(best);
      fix[lg] = mag > 0.0 ? make_double2(bv.x / mag, -bv.y / mag) : make_double2(1.0, 0.0);
    }
  }
  wave_sync();
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const double2* A = slices + s * SL;
    const double2* fix = A + PO + L::prm_elems;
    const int* perm = reinterpret_cast<const int*>(fix + L::fix_elems);
    const PosJob job = job_at(s);
    const int n = job.n;
    double2* out = reinterpret_cast<double2*>(job.V) + job.b * n * n;
    for (int e = lg; e < n * n; e += LPM) {
      const int r = e / n, c = e % n;
      const double2 v = A[at_v(r, perm[c])], f = fix[c];
      out[e] = make_double2(v.x * f.x - v.y * f.y, v.x * f.y + v.y * f.x);
    }
  }
}

// blockDim.x / 64 wavefronts per workgroup, each with solves_per_wave<NP>()
// solves: a CU's workgroup slots would otherwise cap it at one single-wave
// solve per slot
template <int NP>
__global__ void __launch_bounds__(64 * kSmallPerBlock)
    jacobi_small_kernel(const double* __restrict__ H, int64_t batch, int n, double* __restrict__ eps,
                        double* __restrict__ V, uint32_t* status, double tol2, bool some) {
  extern __shared__ double2 jlds[];
  using L = SmallLayout<NP>;
  constexpr int M = solves_per_wave<NP>();
  const int wave = threadIdx.x >> 6, per = blockDim.x >> 6;
  uint2* ent = reinterpret_cast<uint2*>(jlds + per * M * L::slice_elems);
  int* pqt = reinterpret_cast<int*>(ent + (L::N2 - 1) * L::NT);
  if (L::kTable) {
    build_tables<NP>(ent, pqt);
    __syncthreads();
  }
  const int64_t m0 = ((int64_t)blockIdx.x * per + wave) * M;
  if (m0 >= batch) return;
  const int lane = threadIdx.x & 63;
  if constexpr (L::TPL == 1) {
    using P = PosShape<NP>;
    const int g = lane / P::LPM;
    const int64_t mg = m0 + g * P::S;
    auto job_at = [=](int s) {
      const int64_t m = mg + s;
      return PosJob{H, eps, V, m < batch ? m : 0, m < batch ? n : 0};
    };
    jacobi_small_body_pos<NP>(job_at, status, tol2, jlds + (wave * M + g * P::S) * L::slice_elems, lane % P::LPM);
  } else {
    if (some && H[2 * m0 * n * n + 1] != 1.0) return;   // see jacobi_eigh_some
    jacobi_small_body<NP>(H, n, eps, V, status, tol2, m0, jlds + wave * L::slice_elems, lane, ent, pqt);
  }
}

__device__ __forceinline__ int find_job(const EighJob* __restrict__ jobs, int njobs, int64_t m) {
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].block_base <= m) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// NP covers the largest order among the jobs; smaller orders run padded
template <int NP>
__global__ void __launch_bounds__(64 * kSmallPerBlock)
    jacobi_grouped_kernel(const EighJob* __restrict__ jobs, int njobs, int64_t total, uint32_t* status) {
  extern __shared__ double2 jlds[];
  using L = SmallLayout<NP>;
  constexpr int M = solves_per_wave<NP>();
  const int wave = threadIdx.x >> 6, per = blockDim.x >> 6;
  uint2* ent = reinterpret_cast<uint2*>(jlds + per * M * L::slice_elems);
  int* pqt = reinterpret_cast<int*>(ent + (L::N2 - 1) * L::NT);
  if (L::kTable) {
    build_tables<NP>(ent, pqt);
    __syncthreads();
  }
  const int64_t m0 = ((int64_t)blockIdx.x * per + wave) * M;
  if (m0 >= total) return;
  const int lane = threadIdx.x & 63;
  if constexpr (L::TPL == 1) {
    using P = PosShape<NP>;
    const int g = lane / P::LPM;
    const int64_t mg = m0 + g * P::S;
    auto job_at = [=](int s) {
      const int64_t m = mg + s;
      if (m >= total) return PosJob{nullptr, nullptr, nullptr, 0, 0};
      const EighJob& j = jobs[find_job(jobs, njobs, m)];
      return PosJob{j.H, j.eps, j.V, m - j.block_base, j.n};
    };
    jacobi_small_body_pos<NP>(job_at, status, kOffTol2, jlds + (wave * M + g * P::S) * L::slice_elems,
                              lane % P::LPM);
  } else {
    const EighJob& j = jobs[find_job(jobs, njobs, m0)];
    jacobi_small_body<NP>(j.H, j.n, j.eps, j.V, status, kOffTol2, m0 - j.block_base, jlds + wave * L::slice_elems,
                          lane, ent, pqt);
  }
}

using SmallKernel = void (*)(const double*, int64_t, int, double*, double*, uint32_t*, double, bool);
using GroupedKernel = void (*)(const EighJob*, int, int64_t, uint32_t*);

template <int... NPs>
struct SmallTable {
  static SmallKernel small(int np) {
    SmallKernel k = nullptr;
    ((np == NPs ? (k = jacobi_small_kernel<NPs>, 0) : 0), ...);
    return k;
  }
  static GroupedKernel grouped(int np) {
    GroupedKernel k = nullptr;
    ((np == NPs ? (k = jacobi_grouped_kernel<NPs>, 0) : 0), ...);
    return k;
  }
  static int per_wave(int np) {
    int m = 1;
    ((np == NPs ? (m = solves_per_wave<NPs>(), 0) : 0), ...);
    return m;
  }
  // wavefronts per workgroup: up to kSmallPerBlock, their solves within the
  // 64 KB of dynamic LDS
  static int per_block(int np) {
    size_t v = 0, t = 0;
    ((np == NPs ? (v = SmallLayout<NPs>::slice_elems * 16 * solves_per_wave<NPs>(),
                   t = SmallLayout<NPs>::table_elems * 16, 0)
                : 0),
     ...);
    const size_t fit = v ? (65536 - t) / v : 1;
    return (int)(fit < (size_t)kSmallPerBlock ? (fit ? fit : 1) : kSmallPerBlock);
  }
  static size_t bytes(int np) {
    size_t v = 0, t = 0;
    ((np == NPs ? (v = SmallLayout<NPs>::slice_elems * 16 * solves_per_wave<NPs>(),
                   t = SmallLayout<NPs>::table_elems * 16, 0)
                : 0),
     ...);
    return v * per_block(np) + t;
  }
};
using Small = SmallTable<1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16>;

// ---------------------------------------------------------------------------
// Large solves (n > 32).  A stays in the caches, V does not travel with it:
// the rotations of a round depend on A alone, so one workgroup per matrix runs
// a sweep of rounds on A and logs their parameters, and the rows of V, each
// independent of the others, replay the log of the sweep before on as many
// wavefronts as there are rows to share out, in LDS, on the CUs the first
// workgroups leave idle.  One launch per sweep holds both (two logs in turn);
// after convergence the launches return at once.  Sweeps past kLargeSweeps (eight
// to twelve are usual) follow each other in one last launch.  The kernels read the
// limit: the launches of a call, which may be captured in a graph, are the same
// whatever it is.
//
// Per round J_i^H A J_j touches only the 2x2 block (pair i, pair j), so a
// thread loads a block's four elements, applies the column and then the row
// rotation, and stores them: one pass and one barrier where columns and rows
// of A would be two, and neighbouring lanes touch neighbouring elements (the
// players of consecutive pairs are consecutive).  A block is 4 + 4 accesses of
// 16 bytes, 720 KB a round at n = 150 through one CU's 64 bytes a cycle.
// n = 150, 8 matrices: 44.4 ms with one workgroup per matrix doing both
// passes on A and V (integer divisions per element, planes of re and im) ->
// 10 ms (7.2 us a round, 4.7 of it the traffic above).  Rows of A kept in LDS
// (4 in 10 at n = 150) and parameters picked up from LDS instead of A: 10.7.
// ---------------------------------------------------------------------------
constexpr int kLargeThreads = 1024;
constexpr int kReplayRows = 2;      // rows of V per wavefront
constexpr int kLargeSweeps = 16;    // launches of one sweep each

struct LargeRot {
  double c, s, er, ei;
};

// The rotation of two complex values in place, every rounding written out:
// complex64 results downstream (gradients) see the last bits of V, so both
// kernels, and any later form of them, round alike.
// columns: x' = c x - s conj(e) y ; y' = s e x + c y
__device__ __forceinline__ void rotate_columns(const LargeRot& r, double2& x, double2& y) {
  const double xr = x.x, xi = x.y, yr = y.x, yi = y.y;
  x.x = fma(r.c, xr, -(r.s * fma(r.er, yr, r.ei * yi)));
  x.y = fma(r.c, xi, -(r.s * fma(r.er, yi, -(r.ei * yr))));
  y.x = fma(r.c, yr, r.s * fma(r.er, xr, -(r.ei * xi)));
  y.y = fma(r.s, fma(r.ei, xr, r.er * xi), r.c * yi);
}
// rows: x' = c x - s e y ; y' = s conj(e) x + c y
__device__ __forceinline__ void rotate_rows(const LargeRot& r, double2& x, double2& y) {
  const double xr = x.x, xi = x.y, yr = y.x, yi = y.y;
  x.x = fma(r.c, xr, -(r.s * fma(r.er, yr, -(r.ei * yi))));
  x.y = fma(r.c, xi, -(r.s * fma(r.ei, yr, r.er * yi)));
  y.x = fma(r.c, yr, r.s * fma(r.er, xr, r.ei * xi));
  y.y = fma(r.s, fma(r.er, xi, -(r.ei * xr)), r.c * yi);
}

// number of pairs with two real players in a round, and the log's stride
__host__ __device__ inline int large_pairs(int n) { return n / 2; }

// Per matrix, state[0]: converged, or kLeaveOut; state[1 + parity]: rounds in the
// log that the sweep of that parity wrote.  Sweep number `sweep` of matrix b.
// some: state[0] is set before the first sweep, to kLeaveOut for the matrices
// whose eps and V are to stay as they are.
__device__ __forceinline__ void jacobi_sweep(double2* __restrict__ H, int n, LargeRot* __restrict__ log,
                                             int* __restrict__ state, const uint32_t* __restrict__ status, int sweep,
                                             int b, bool some) {
  __shared__ LargeRot prm[128];
  __shared__ int ip[128], iq[128];   // players of a pair, iq = -1 for the pair with the missing player
  __shared__ double red[kLargeThreads / 64];
  const int tid = threadIdx.x;
  int* st = state + 3 * b;
  if (sweep == 0 && some && st[0] == kLeaveOut) {
    if (tid == 0) st[1] = -1;
    return;
  }
  if ((sweep > 0 && st[0]) || sweep >= sweep_limit(status)) {
    if (tid == 0) {
      if (sweep == 0) st[0] = 0;
      st[1 + (sweep & 1)] = 0;
    }
    return;
  }
  double2* A = H + (int64_t)b * n * n;
  const int n2 = n + (n & 1), np = n2 / 2, full = large_pairs(n);
  LargeRot* lg = log + ((int64_t)b * 2 + (sweep & 1)) * (n2 - 1) * full;
  double off = 0.0, tot = 0.0;
  for (int e = tid; e < n * n; e += kLargeThreads) {
    const double2 a = A[e];
    const double v = a.x * a.x + a.y * a.y;
    tot += v;
    if (e / n != e % n) off += v;
  }
  off = block_sum<kLargeThreads>(off, red);
  tot = block_sum<kLargeThreads>(tot, red);
  const bool converged = off <= kOffTol2 * tot;
  if (!converged) {
    for (int round = 0; round < n2 - 1; ++round) {
      if (tid < np) {
        const int a = player_at(tid, round, n2), b = player_at(n2 - 1 - tid, round, n2);
        const int p = a < b ? a : b, q = a < b ? b : a;
        LargeRot r = {1.0, 0.0, 1.0, 0.0};
        if (q < n) {
          const double br = A[p * n + q].x, bi = A[p * n + q].y;
          const double bm = hypot(br, bi);
          if (bm > 0.0) {
            const double tau = (A[q * n + q].x - A[p * n + p].x) / (2.0 * bm);
            const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
            r.c = 1.0 / sqrt(1.0 + t * t);
            r.s = t * r.c;
            r.er = br / bm;
            r.ei = bi / bm;
          }
        }
        prm[tid] = r;
        ip[tid] = p;
        iq[tid] = q < n ? q : -1;
        // odd n: pair 0 is always player 0's, so the pair of the missing player
        // moves; its entry is left out (the pairs after it move up by one)
        const int miss = n & 1 ? missing_pair(round, n2) : np;
        if (tid != miss) lg[(int64_t)round * full + tid - (tid > miss ? 1 : 0)] = r;
      }
      __syncthreads();
      int i = tid / np, j = tid - i * np;
      const int di = kLargeThreads / np, dj = kLargeThreads - di * np;
      while (i < np) {
        const int pi = ip[i], qi = iq[i], pj = ip[j], qj = iq[j];
        const bool hi = qi >= 0, hj = qj >= 0;
        double2* rowp = A + pi * n;
        double2* rowq = A + (hi ? qi : pi) * n;
        const int cq = hj ? qj : pj;
        double2 x[2] = {rowp[pj], rowq[pj]}, y[2] = {rowp[cq], rowq[cq]};
        const LargeRot rj = prm[j], ri = prm[i];
        rotate_columns(rj, x[0], y[0]);
        rotate_columns(rj, x[1], y[1]);
        rotate_rows(ri, x[0], x[1]);
        rotate_rows(ri, y[0], y[1]);
        rowp[pj] = x[0];
        if (hj) rowp[qj] = y[0];
        if (hi) rowq[pj] = x[1];
        if (hi && hj) rowq[qj] = y[1];
        i += di;
        j += dj;
        if (j >= np) {
          j -= np;
          ++i;
        }
      }
      __syncthreads();
    }
  }
  if (tid == 0) {
    st[0] = converged;
    st[1 + (sweep & 1)] = converged ? 0 : n2 - 1;
  }
}

// V <- V J for the logged rounds: a wavefront owns kReplayRows rows of V in its
// own LDS slice, its lanes share the pairs of a round, so rounds are separated
// by wave-level waits only; the next round's parameters are loaded meanwhile.
__device__ __forceinline__ void jacobi_replay(double2* __restrict__ V, int n, const LargeRot* __restrict__ log,
                                              const int* __restrict__ state, int sweep, int b, int part,
                                              double2* replay_rows) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row0 = (part * (kLargeThreads / 64) + wave) * kReplayRows;
  const int rounds = state[3 * b + 1 + (sweep & 1)];
  if (row0 >= n || rounds < 0 || (rounds == 0 && sweep > 0)) return;
  const int n2 = n + (n & 1), full = large_pairs(n);
  const LargeRot* lg = log + ((int64_t)b * 2 + (sweep & 1)) * (n2 - 1) * full;
  double2* vb = V + (int64_t)b * n * n;
  double2* buf = replay_rows + wave * kReplayRows * n;
  const int rows = n - row0 < kReplayRows ? n - row0 : kReplayRows;
  for (int r = 0; r < kReplayRows; ++r)
    for (int c = lane; c < n; c += 64)
      buf[r * n + c] = sweep > 0 && r < rows ? vb[(row0 + r) * n + c] : make_double2(row0 + r == c ? 1.0 : 0.0, 0.0);
  wave_sync();
  const LargeRot idle = {1.0, 0.0, 1.0, 0.0};
  LargeRot next[2];
  auto fetch = [&](int t, int u) {
    const int k = lane + 64 * u;
    const int miss = n & 1 ? missing_pair(t, n2) : n2;
    return t < rounds && k < n2 / 2 && k != miss ? lg[(int64_t)t * full + k - (k > miss ? 1 : 0)] : idle;
  };
#pragma unroll
  for (int u = 0; u < 2; ++u) next[u] = fetch(0, u);
  for (int t = 0; t < rounds; ++t) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const LargeRot w = next[u];
      next[u] = fetch(t + 1, u);
      const int k = lane + 64 * u;
      if (k >= n2 / 2) continue;
      const int pa = player_at(k, t, n2), pb = player_at(n2 - 1 - k, t, n2);
      const int p = pa < pb ? pa : pb, q = pa < pb ? pb : pa;
      if (q >= n) continue;
#pragma unroll
      for (int r = 0; r < kReplayRows; ++r) {
        double2 x = buf[r * n + p], y = buf[r * n + q];
        rotate_columns(w, x, y);
        buf[r * n + p] = x;
        buf[r * n + q] = y;
      }
    }
    wave_sync();
  }
  for (int r = 0; r < rows; ++r)
    for (int c = lane; c < n; c += 64) vb[(row0 + r) * n + c] = buf[r * n + c];
}

// Workgroups 0 .. nb - 1 run sweep `sweep` on A, the others replay the sweep
// before it, `parts` of them per matrix.
__global__ void __launch_bounds__(kLargeThreads)
    jacobi_sweep_kernel(double2* __restrict__ H, double2* __restrict__ V, int n, int nb, int parts,
                        LargeRot* __restrict__ log, int* __restrict__ state, const uint32_t* __restrict__ status,
                        int sweep, bool some) {
  extern __shared__ double2 replay_rows[];
  const int b = blockIdx.x;
  if (b < nb)
    jacobi_sweep(H, n, log, state, status, sweep, b, some);
  else
    jacobi_replay(V, n, log, state, sweep - 1, (b - nb) / parts, (b - nb) % parts, replay_rows);
}

// Sweep number `last` is on A and in the log: its replay, then sweep after sweep
// until the matrix has converged or the limit is reached, a workgroup per matrix.
__global__ void __launch_bounds__(kLargeThreads)
    jacobi_tail_kernel(double2* H, double2* V, int n, int parts, LargeRot* log, int* state, const uint32_t* status,
                       int last) {
  extern __shared__ double2 replay_rows[];
  const int b = blockIdx.x, limit = sweep_limit(status);
  for (int sweep = last;; ++sweep) {
    for (int part = 0; part < parts; ++part) jacobi_replay(V, n, log, state, sweep, b, part, replay_rows);
    __syncthreads();
    if (state[3 * b] != 0 || sweep + 1 >= limit) return;   // the same for every thread
    jacobi_sweep(H, n, log, state, status, sweep + 1, b, false);
    __syncthreads();
  }
}

// Sort ascending, fix each column's phase: eps from the diagonal of A, the
// columns of V permuted and scaled in place, a row at a time.
__global__ void __launch_bounds__(kLargeThreads)
    jacobi_finish_kernel(const double2* __restrict__ H, int n, double* __restrict__ eps, double2* __restrict__ V,
                         const int* __restrict__ state, uint32_t* status, bool some) {
  if (some && state[3 * blockIdx.x] == kLeaveOut) return;
  __shared__ int perm[256];
  __shared__ double2 ph[256], row[kLargeThreads / 64][256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double2* A = H + (int64_t)blockIdx.x * n * n;
  double2* vb = V + (int64_t)blockIdx.x * n * n;
  double* eo = eps + (int64_t)blockIdx.x * n;
  if (tid == 0 && !state[3 * blockIdx.x]) atomicOr(status, kStatusNoConv);
  for (int i = tid; i < n; i += kLargeThreads) perm[ascending_place([&](int j) { return A[j * n + j].x; }, n, i)] = i;
  __syncthreads();
  for (int c = tid; c < n; c += kLargeThreads) {
    const int src = perm[c];
    eo[c] = A[src * n + src].x;
    double best = -1.0, br = 1.0, bi = 0.0;
    for (int r = 0; r < n; ++r) best = fmax(best, norm2(vb[r * n + src]));
    for (int r = 0; r < n; ++r) {
      const double2 v = vb[r * n + src];
      if (norm2(v) >= kTied * best) {
        best = norm2(v);
        br = v.x;
        bi = v.y;
        break;
      }
    }
    const double mag = sqrt(best);
    ph[c] = mag > 0 ? make_double2(br / mag, -bi / mag) : make_double2(1.0, 0.0);   // conj(v_max)/|v_max|
  }
  __syncthreads();
  for (int r = wave; r < n; r += kLargeThreads / 64) {
    for (int c = lane; c < n; c += 64) row[wave][c] = vb[r * n + c];
    wave_sync();
    for (int c = lane; c < n; c += 64) {
      const double vr = row[wave][perm[c]].x, vi = row[wave][perm[c]].y;
      const double fr = ph[c].x, fi = ph[c].y;
      vb[r * n + c] = make_double2(vr * fr - vi * fi, vr * fi + vi * fr);
    }
    wave_sync();
  }
}

constexpr int64_t kLargeChunk = 1024;  // matrices per large-n launch (bounds the workspace)

// doubles of one matrix's two logs: n2 - 1 rounds of n / 2 rotations each
inline int64_t log_doubles(int n) { return (int64_t)4 * 2 * (n + (n & 1) - 1) * large_pairs(n); }

ephw_status launch_small(const double* H, int64_t batch, int n, double* eps, double* V, uint32_t* status,
                         double off_tol2, bool some, hipStream_t s) {
  const int np = (n + 1) / 2, waves = Small::per_block(np), per = waves * Small::per_wave(np);
  const int64_t max_per_launch = (int64_t)0x7fffffff * per;
  for (int64_t b0 = 0; b0 < batch; b0 += max_per_launch) {
    const int64_t nb = (batch - b0) < max_per_launch ? (batch - b0) : max_per_launch;
    const int64_t grid = (nb + per - 1) / per;
    hipLaunchKernelGGL(Small::small(np), dim3((unsigned)grid), dim3(64 * waves), Small::bytes(np), s,
                       H + 2 * b0 * n * n, nb, n, eps + b0 * n, V + 2 * b0 * n * n, status, off_tol2, some);
    EPHW_CHECK_LAUNCH();
  }
  return EPHW_OK;
}

// nb <= kLargeChunk matrices
ephw_status launch_large(double2* h, int64_t nb, int n, double* eps, double2* v, double* work, uint32_t* status,
                         bool some, hipStream_t s) {
  const size_t lds = (size_t)(kLargeThreads / 64) * kReplayRows * n * sizeof(double2);
  const int parts = (int)ceil_div(n, (kLargeThreads / 64) * kReplayRows);
  EPHW_HIP(hipFuncSetAttribute((const void*)jacobi_sweep_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  EPHW_HIP(hipFuncSetAttribute((const void*)jacobi_tail_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  LargeRot* log = reinterpret_cast<LargeRot*>(work);
  int* state = jacobi_large_state(work, n, nb);
  for (int sweep = 0; sweep <= kLargeSweeps; ++sweep) {
    const int64_t grid = nb + (sweep > 0 ? nb * parts : 0);
    hipLaunchKernelGGL(jacobi_sweep_kernel, dim3((unsigned)grid), dim3(kLargeThreads), lds, s, h, v, n, (int)nb, parts,
                       log, state, status, sweep, some);
    EPHW_CHECK_LAUNCH();
  }
  hipLaunchKernelGGL(jacobi_tail_kernel, dim3((unsigned)nb), dim3(kLargeThreads), lds, s, h, v, n, parts, log, state,
                     status, kLargeSweeps);
  EPHW_CHECK_LAUNCH();
  hipLaunchKernelGGL(jacobi_finish_kernel, dim3((unsigned)nb), dim3(kLargeThreads), 0, s, h, n, eps, v, state, status,
                     some);
  EPHW_CHECK_LAUNCH();
  return EPHW_OK;
}

}  // namespace

ephw_status jacobi_eigh_some(double* H, int64_t nb, int n, double* eps, double* V, double* work, uint32_t* status,
                             hipStream_t s) {
  // (of the small solves, those with several matrices to a wavefront take them all)
  if (n <= 16 || n > 256 || nb < 1 || (n > kSmallN && (nb > kLargeChunk || !work))) {
    set_error("jacobi_eigh_some: matrices of order 17 to 256, above 32 a chunk of them and their workspace");
    return EPHW_EINVAL;
  }
  if (n <= kSmallN) return launch_small(H, nb, n, eps, V, status, kOffTol2, true, s);
  return launch_large(reinterpret_cast<double2*>(H), nb, n, eps, reinterpret_cast<double2*>(V), work, status, true, s);
}

int* jacobi_large_state(double* work, int n, int64_t nb) { return reinterpret_cast<int*>(work + log_doubles(n) * nb); }

int64_t jacobi_work_doubles(int n, int64_t batch) {
  if (n <= kSmallN) return 0;
  const int64_t chunk = batch < kLargeChunk ? batch : kLargeChunk;
  return log_doubles(n) * chunk + (3 * chunk + 1) / 2;
}

ephw_status jacobi_eigh_grouped(const EighJob* d_jobs, int njobs, int64_t total, int max_n, uint32_t* status,
                                hipStream_t s) {
  if (njobs <= 0 || total <= 0) return EPHW_OK;
  if (max_n < 1 || max_n > kSmallN) {
    set_error("jacobi_eigh_grouped: matrix orders must be in [1, 32]");
    return EPHW_EUNSUPPORTED;
  }
  const int np = (max_n + 1) / 2, waves = Small::per_block(np), per = waves * Small::per_wave(np);
  const int64_t grid = (total + per - 1) / per;
  if (grid > 0x7fffffff) {
    set_error("jacobi_eigh_grouped: too many matrices for one launch");
    return EPHW_EUNSUPPORTED;
  }
  hipLaunchKernelGGL(Small::grouped(np), dim3((unsigned)grid), dim3(64 * waves), Small::bytes(np), s, d_jobs, njobs,
                     total, status);
  EPHW_CHECK_LAUNCH();
  return EPHW_OK;
}

ephw_status jacobi_eigh(double* H, int64_t batch, int n, double* eps, double* V, double* work, uint32_t* status,
                        hipStream_t s, double off_tol2) {
  if (batch <= 0) return EPHW_OK;
  if (!(off_tol2 > 0.0) || off_tol2 < kOffTol2) off_tol2 = kOffTol2;
  if ((reinterpret_cast<uintptr_t>(H) | reinterpret_cast<uintptr_t>(V)) & 15) {
    set_error("jacobi_eigh: matrices and eigenvectors must be 16-byte aligned complex128 arrays");
    return EPHW_EINVAL;
  }
  if (n < 1 || n > 256) {
    set_error("jacobi_eigh: matrix order must be in [1, 256]");
    return EPHW_EUNSUPPORTED;
  }
  if (n <= kSmallN) return launch_small(H, batch, n, eps, V, status, off_tol2, false, s);
  if (!work) {
    set_error("jacobi_eigh: large matrices need a workspace");
    return EPHW_EINVAL;
  }
  for (int64_t b0 = 0; b0 < batch; b0 += kLargeChunk) {
    const int64_t nb = (batch - b0) < kLargeChunk ? (batch - b0) : kLargeChunk;
    EPHW_TRY(launch_large(reinterpret_cast<double2*>(H) + b0 * n * n, nb, n, eps + b0 * n,
                          reinterpret_cast<double2*>(V) + b0 * n * n, work, status, false, s));
  }
  return EPHW_OK;
}

}  // namespace ephw
