// Determinant and adjugate of batches of small matrices (QMCkl paper,
// Section 3.4: the inverse is adj(A) / det(A); returning det and adj(A)
// together serves the gradients of Slater determinants, and for n < 5 the
// explicit cofactor form beats an LU factorisation).
//
// n <= 4: one lane per matrix (staged through LDS for coalesced loads and
// stores); the n*n entries live in registers and every
// cofactor is an unrolled signed minor determinant (Laplace expansion along
// the first row, compile-time n), so the result is exact also for singular
// matrices.  5 <= n <= 32: two to eight matrices per wavefront, Gauss-Jordan
// elimination with partial pivoting and a row per lane in registers,
// det = sign * product of the pivots, adj = det * A^{-1}; a wavefront with a
// pivot or determinant outside the normal numbers takes a second pass over its
// matrices, which also knows singular ones.
#include <type_traits>

#include "qmk_internal.h"

namespace qmk {
namespace {

// Determinant of the m x m matrix made of rows r[0..m) and columns c[0..m)
// of the n x n row-major matrix a (Laplace expansion along the first row).
template <int N, int M>
struct Minor {
  static __device__ __forceinline__ double det(const double (&a)[N * N], const int (&r)[M],
                                               const int (&c)[M]) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < M; ++j) {
      int rr[M - 1], cc[M - 1];
#pragma unroll
      for (int k = 0; k < M - 1; ++k) {
        rr[k] = r[k + 1];
        cc[k] = c[k < j ? k : k + 1];
      }
      const double t = a[r[0] * N + c[j]] * Minor<N, M - 1>::det(a, rr, cc);
      s += (j & 1) ? -t : t;
    }
    return s;
  }
};
template <int N>
struct Minor<N, 1> {
  static __device__ __forceinline__ double det(const double (&a)[N * N], const int (&r)[1],
                                               const int (&c)[1]) {
    return a[r[0] * N + c[0]];
  }
};

// The 256 matrices of a workgroup pass through LDS (rows padded by one
// element against bank conflicts), so that the global loads and stores of the
// workgroup cover one contiguous range, coalesced across lanes.
template <int N>
__global__ __launch_bounds__(256) void det_adj_small_kernel(const double* __restrict__ A, int64_t batch,
                                                            double* __restrict__ det,
                                                            double* __restrict__ adj) {
  constexpr int E = N * N, LD = E + 1;
  __shared__ double s_m[256 * LD];
  const int64_t b0 = static_cast<int64_t>(blockIdx.x) * 256;
  const int64_t nb = min<int64_t>(256, batch - b0);
  const double* src = A + b0 * E;
  for (int64_t e = threadIdx.x; e < nb * E; e += 256) s_m[(e / E) * LD + e % E] = src[e];
  __syncthreads();
  const int t = threadIdx.x;
  double a[E];
  if (t < nb) {
#pragma unroll
    for (int i = 0; i < E; ++i) a[i] = s_m[t * LD + i];
  }
  __syncthreads();  // s_m is reused for the adjugates
  if (t < nb) {
    if constexpr (N == 1) {
      det[b0 + t] = a[0];
      s_m[t * LD] = 1.0;
    } else {
      double d = 0.0;
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) {
          // cofactor C_ij = (-1)^(i+j) det(A without row i, column j); adj = C^T
          int r[N - 1], c[N - 1];
#pragma unroll
          for (int k = 0; k < N - 1; ++k) {
            r[k] = k < i ? k : k + 1;
            c[k] = k < j ? k : k + 1;
          }
          const double m = Minor<N, N - 1>::det(a, r, c);
          const double cij = ((i + j) & 1) ? -m : m;
          s_m[t * LD + j * N + i] = cij;
          if (i == 0) d += a[j] * cij;
        }
      det[b0 + t] = d;
    }
  }
  __syncthreads();
  double* dst = adj + b0 * E;
  for (int64_t e = threadIdx.x; e < nb * E; e += 256) dst[e] = s_m[(e / E) * LD + e % E];
}

// Orders the LDS accesses of one wavefront's lanes (its part of the LDS is
// its own).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Largest v of each group of G consecutive lanes (8, 16 or 32), in every lane.
template <int G>
__device__ __forceinline__ double group_max(double v) {
  auto step = [&](auto ctl) {
    constexpr int c = decltype(ctl)::value;
    const int64_t b = __builtin_bit_cast(int64_t, v);
    const uint32_t lo = __builtin_amdgcn_mov_dpp(static_cast<int>(b), c, 0xF, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_mov_dpp(static_cast<int>(b >> 32), c, 0xF, 0xF, true);
    v = fmax(v, __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo));
  };
  step(std::integral_constant<int, 0xB1>{});   // quad_perm [1, 0, 3, 2]
  step(std::integral_constant<int, 0x4E>{});   // quad_perm [2, 3, 0, 1]
  step(std::integral_constant<int, 0x141>{});  // row_half_mirror
  if constexpr (G >= 16) step(std::integral_constant<int, 0x140>{});  // row_mirror
  if constexpr (G >= 32) v = fmax(v, __shfl_xor(v, 16, 64));
  return v;
}

// 5 <= N <= 32: a wavefront takes 64 / G matrices (G = 8, 16 or 32 lanes
// each), lane i of a group holding row i in registers; in-place Gauss-Jordan
// over the unused rows (no row is moved, and pivot rows stay unscaled until
// the end).  At step k the lane of the pivot row hands it to its group through
// LDS (16-byte accesses; ds_bpermute of every column measured 1.6x slower: the
// LDS unit is what bounds the kernel beside the traffic of 2 N^2 + 1 doubles
// per matrix) and every other lane subtracts its multiple; the columns rotate
// by one register, so that the step loop is not unrolled and the pivot column
// is always register 0.  One
// wavefront per matrix with the LU in LDS ran N serial steps with N of 64
// lanes busy and kept the solutions in scratch memory.
// 50,000 matrices of N = 16: 1082 us before, 76 us now (2.7 TB/s); N = 5, 8 and 24 166,
// 310 and 2552 us before, 13, 20 and 278 us now; 20,000 of N = 32 1991 and 214 us.
// Singular ones (a zero row) of N = 8, 16, 24 and 32: 233, 603, 1147 and 779 us before,
// 34, 151, 593 and 484 us now (the wavefront's LU one matrix after another took
// 312, 942, 1731 and 1485 us).
template <int N>
__global__ __launch_bounds__(256, N <= 14 ? 4 : (N <= 24 ? 3 : 2)) void det_adj_gj_kernel(const double* __restrict__ A,
                                                                          int64_t batch,
                                                                          double* __restrict__ det,
                                                                          double* __restrict__ adj) {
  constexpr int G = N <= 8 ? 8 : (N <= 16 ? 16 : 32), NM = 64 / G, E = N * N;
  constexpr int LD = N | 1;  // odd row pitch: rows of a group start on different banks
  constexpr int RP = (N + 1) / 2 + 1;  // pitch of the groups' pivot rows, in pairs of columns
  union alignas(16) Lds {
    double m[NM][N][LD];
    double2 row[NM][RP];
  };
  __shared__ Lds s_lds[4];
  __shared__ int s_piv[4][NM][N];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t b0 = (static_cast<int64_t>(blockIdx.x) * 4 + w) * NM;
  if (b0 >= batch) return;  // whole waves leave together; no workgroup barrier below
  const int nb = static_cast<int>(min<int64_t>(NM, batch - b0));
  double* const sm = &s_lds[w].m[0][0][0];
  const double* const src = A + b0 * E;
  double* const dst = adj + b0 * E;
  const int gi = lane / G, i = lane % G, base = lane - i;
  double a[N];
  constexpr int Q = (NM * E + 63) / 64;
  // the wavefront's matrices are contiguous: coalesced loads, all in flight
  // before the first is stored, rows padded in LDS (past the last matrix: its
  // last element again)
  {
    double in[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) in[q] = src[min(q * 64 + lane, nb * E - 1)];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = q * 64 + lane;
      if (NM * E % 64 == 0 || e < NM * E) sm[e / N * LD + e % N] = in[q];
    }
  }
  wave_lds_sync();
  auto take_rows = [&]() {
#pragma unroll
    for (int j = 0; j < N; ++j) a[j] = i < N ? sm[(gi * N + i) * LD + j] : 0.0;
    wave_lds_sync();  // the rows are read; the pivot rows take their place
  };
  double2* const row = &s_lds[w].row[0][0] + gi * RP;
  auto put_row = [&]() {  // two columns per access
#pragma unroll
    for (int j = 0; j < (N + 1) / 2; ++j) row[j] = double2{a[2 * j], 2 * j + 1 < N ? a[2 * j + 1] : 0.0};
  };
  double r[2 * ((N + 1) / 2)];
  auto get_row = [&]() {
#pragma unroll
    for (int j = 0; j < (N + 1) / 2; ++j) {
      const double2 v2 = row[j];
      r[2 * j] = v2.x;
      r[2 * j + 1] = v2.y;
    }
  };
  constexpr uint32_t kAll = N == 32 ? ~0u : (1u << (N & 31)) - 1u;

  take_rows();
  double d = 1.0, my_piv = 1.0;
  uint32_t unused = kAll;  // rows not yet a pivot row
  int my_k = 0, odd = 0;
  bool bad = false;
#pragma unroll(N % 2 == 0 ? 2 : 1)
  for (int k = 0; k < N; ++k) {
    // pivot: the unused row with the largest entry (ties to the lowest row)
    const bool cand = (unused >> i) & 1u;
    const double v = cand ? fabs(a[0]) : -1.0;
    const double vm = group_max<G>(v);
    const uint64_t hit = __ballot(cand && v == vm);
    const uint32_t mine = static_cast<uint32_t>(hit >> base) & (G == 32 ? ~0u : (1u << (G & 31)) - 1u);
    const int p = mine ? __builtin_ctz(mine) : 0;
    bad = bad || mine == 0;  // only NaNs are left in this column
    // sign of the permutation: unused rows before p
    odd ^= __builtin_popcount(unused & ((1u << p) - 1u)) & 1;
    unused &= ~(1u << p);
    const bool own = i == p;
    // the pivot row goes to its group through LDS
    if (own) put_row();
    wave_lds_sync();
    get_row();
    const double piv = r[0];
    d *= piv;
    if (own) {
      my_k = k;
      my_piv = piv;
    }
    if (i == 0) s_piv[w][gi][k] = p;
    // row i -= f * pivot row; the pivot row itself stays (f = 0).  Column k
    // of the result holds the coefficient of identity column p.
    const double f = own ? 0.0 : a[0] / piv;
#pragma unroll
    for (int j = 1; j < N; ++j) a[j - 1] = fma(-f, r[j], a[j]);
    a[N - 1] = own ? 1.0 : -f;
    wave_lds_sync();  // the row is read before the next one is written
  }
  if (odd) d = -d;
  // every lane looks at its own pivot
  const bool normal = fabs(my_piv) >= 0x1p-1022 && fabs(my_piv) <= 0x1p+1022;
  const uint64_t odd_pivots = __ballot(i < N && !normal) >> base;
  bad = bad || (odd_pivots & (G == 32 ? 0xffffffffu : (1u << (G & 31)) - 1u)) != 0 ||
        !(fabs(d) <= 1.7976931348623157e308);

  // A^{-1}[k of row i][p_k] = a[k] / pivot of row i
  wave_lds_sync();
  if (i < N) {
    const double inv = 1.0 / my_piv;
#pragma unroll
    for (int k = 0; k < N; ++k) sm[(gi * N + my_k) * LD + s_piv[w][gi][k]] = d * (a[k] * inv);
  }
  wave_lds_sync();
  const uint64_t again = __ballot(bad && gi < nb);
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = q * 64 + lane;
    if (e < nb * E && (again == 0 || !((again >> (e / E * G)) & 1u))) dst[e] = sm[e / N * LD + e % N];
  }
  if (i == 0 && gi < nb && !bad) det[b0 + gi] = d;
  if (again == 0) return;

  // Second pass for the wavefront's matrices that met a pivot that is zero,
  // NaN, or so small or large that its reciprocal is not a normal number, or
  // whose determinant is not finite: the same elimination, which multiplies a row by
  // the other rows' pivots instead of dividing det by its own, takes a row with a NaN where no other has an entry, and passes over a column
  // that is zero in every unused row.  One column k0 passed over (rank N - 1)
  // leaves one row p0 = t^T A of zeros, t its coefficients of the identity, and
  // the null vector x: x_k0 = 1, x_k = -(column k0 of the row of pivot k) / pivot k.
  // Then adj(A) = c x t^T with c the cofactor of (p0, k0), the signed product of
  // the pivots; with two or more adj(A) = 0.
  wave_lds_sync();
#pragma unroll 1
  for (int e = lane; e < NM * E; e += 64) sm[e / N * LD + e % N] = src[min(e, nb * E - 1)];
  wave_lds_sync();
  take_rows();
  d = 1.0;
  my_piv = 1.0;
  unused = kAll;
  my_k = odd = 0;
  double rest = 1.0;  // product of the pivots but this lane's
  int passed = 0, k0 = 0;
#pragma unroll 1
  for (int k = 0; k < N; ++k) {
    const bool cand = (unused >> i) & 1u;
    const double v = cand ? fabs(a[0]) : -1.0;
    const double vm = group_max<G>(v);
    const uint64_t hit = __ballot(cand && v == vm);
    const uint32_t mine = static_cast<uint32_t>(hit >> base) & (G == 32 ? ~0u : (1u << (G & 31)) - 1u);
    const uint64_t nan = __ballot(cand && v != v);
    const uint32_t nans = static_cast<uint32_t>(nan >> base) & (G == 32 ? ~0u : (1u << (G & 31)) - 1u);
    const bool none = vm == 0.0 && nans == 0;
    // (fewer rows than steps are used, so that one is left; NaNs beat zeros)
    const int p = __builtin_ctz(vm > 0.0 || nans == 0 ? mine : nans);
    const bool own = !none && i == p;
    if (none) {
      ++passed;
      k0 = k;
    } else {
      odd ^= __builtin_popcount(unused & ((1u << p) - 1u)) & 1;
      unused &= ~(1u << p);
    }
    if (own) put_row();
    wave_lds_sync();
    get_row();
    const double piv = none ? 1.0 : r[0];
    d *= piv;
    if (own) {
      my_k = k;
      my_piv = piv;
    } else {
      rest *= piv;
    }
    if (i == 0) s_piv[w][gi][k] = p;
    const double a0 = a[0], f = own || none ? 0.0 : a0 / piv;
#pragma unroll
    for (int j = 1; j < N; ++j) a[j - 1] = own || none ? a[j] : fma(-f, r[j], a[j]);
    a[N - 1] = none ? a0 : (own ? 1.0 : -f);
    wave_lds_sync();
  }
  const int p0 = unused ? __builtin_ctz(unused) : 0;
  // (the order of the pivot rows has p0 at k0, not after the rows of later steps)
  if ((odd + (passed ? N - 1 - k0 : 0)) & 1) {
    d = -d;
    rest = -rest;
  }
  if (d != d) rest = d;
  // x and t take the places of rows 0 and 1, and the results those of all rows
  // once they are read
  double* const x = sm + gi * N * LD;
  double* const t = x + LD;
  wave_lds_sync();
  if (passed == 1 && i < N) {
    if (i == p0) {
#pragma unroll
      for (int k = 0; k < N; ++k)
        if (k != k0) t[s_piv[w][gi][k]] = a[k];
      t[p0] = 1.0;
      x[k0] = 1.0;
    } else {
      double c = 0.0;
#pragma unroll
      for (int k = 0; k < N; ++k) c = k == k0 ? a[k] : c;
      x[my_k] = -c / my_piv;
    }
  }
  wave_lds_sync();
  if (passed == 1) {
    const double xi = i < N ? d * x[i] : 0.0;
#pragma unroll
    for (int j = 0; j < N; ++j) a[j] = xi * t[j];
  }
  wave_lds_sync();
  if (i < N) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
      if (passed == 0)
        sm[(gi * N + my_k) * LD + s_piv[w][gi][k]] = rest * a[k];
      else
        sm[(gi * N + i) * LD + k] = passed == 1 ? a[k] : 0.0;
    }
  }
  wave_lds_sync();
#pragma unroll 1
  for (int e = lane; e < nb * E; e += 64)
    if ((again >> (e / E * G)) & 1u) dst[e] = sm[e / N * LD + e % N];
  if (i == 0 && gi < nb && bad) det[b0 + gi] = passed ? d * 0.0 : d;
}

template <int N>
void run_det_adj_gj(int64_t batch, const double* A, double* det, double* adj, hipStream_t s) {
  constexpr int per_block = 4 * (64 / (N <= 8 ? 8 : (N <= 16 ? 16 : 32)));
  hipLaunchKernelGGL(det_adj_gj_kernel<N>, dim3(static_cast<unsigned>((batch + per_block - 1) / per_block)),
                     dim3(256), 0, s, A, batch, det, adj);
}

}  // namespace

hipError_t launch_det_adj(int n, int64_t batch, const double* A, double* det, double* adj, hipStream_t s) {
  if (batch <= 0) return hipSuccess;
  const dim3 blk(256);
  const dim3 g_small(static_cast<unsigned>((batch + 255) / 256));
  switch (n) {
    case 1: hipLaunchKernelGGL(det_adj_small_kernel<1>, g_small, blk, 0, s, A, batch, det, adj); break;
    case 2: hipLaunchKernelGGL(det_adj_small_kernel<2>, g_small, blk, 0, s, A, batch, det, adj); break;
    case 3: hipLaunchKernelGGL(det_adj_small_kernel<3>, g_small, blk, 0, s, A, batch, det, adj); break;
    case 4: hipLaunchKernelGGL(det_adj_small_kernel<4>, g_small, blk, 0, s, A, batch, det, adj); break;
#define QMK_DET(n) case n: run_det_adj_gj<n>(batch, A, det, adj, s); break;
    QMK_DET(5) QMK_DET(6) QMK_DET(7) QMK_DET(8) QMK_DET(9) QMK_DET(10) QMK_DET(11) QMK_DET(12) QMK_DET(13) QMK_DET(14)
    QMK_DET(15) QMK_DET(16) QMK_DET(17) QMK_DET(18) QMK_DET(19) QMK_DET(20) QMK_DET(21) QMK_DET(22) QMK_DET(23)
    QMK_DET(24) QMK_DET(25) QMK_DET(26) QMK_DET(27) QMK_DET(28) QMK_DET(29) QMK_DET(30) QMK_DET(31) QMK_DET(32)
#undef QMK_DET
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace qmk
