// Three-body (electron-electron-nucleus) Jastrow factor through the
// intermediate matrix P (QMCkl paper, Section 3.5):
//   P^{k,m}_{i a} = sum_{j != i} rt_ij^k Rt_ja^m,
//   J = sum_t sum_a c[t,a] sum_i Rt_ia^((p-k+l)/2) P^{k,(p-k-l)/2}_{i a},
// with rt_ij = exp(-kappa r_ij) and Rt_ia = exp(-kappa |r_i - R_a|).
//
// Grouping the terms by (k, m), J = sum_{k,m} sum_{i,a} w_{k,m,a}(Rt_ia)
// P^{k,m}_{ia} with w_{k,m,a} a polynomial in Rt_ia whose coefficients are
// the c[t,a] of the terms with that (k, m).  Terms with m >= 1 have
// k <= nord - 2 and m <= nord / 2; terms with m = 0 (k >= 1) need only
// P^{k,0}_i = sum_{j != i} rt_ij^k, which does not depend on the nucleus.
// Per walker:
//   een_en      Ra[w][j][(m-1) nnp + a] = Rt_ja^m, the left operand
//               of the product, and x[w][a][i] = Rt_ia;
//   een_g0      the nucleus sums of the m = 0 weights per electron;
//   een_ee      rt[w][j][i] (zero diagonal), the right operand, plus the
//               m = 0 part of J for electron i;
//   een_k0      the k = 0 terms (m >= 1), whose P^{0,m}_{ia} = sum_{j != i}
//               Rt_ja^m is a sum per nucleus and needs no product;
//   the product (jastrow_product.hip) forms P^{k,m} for k, m >= 1 on MFMA,
//               taking the powers of rt as it reads them, and folds the
//               weights into its epilogue, so neither rt^k nor P is stored;
//   een_finish  sums the partial sums of one walker in a fixed order
//               (deterministic).
// Both operands have their electrons j padded to a multiple of 16 with zero
// rows, so that the product has no partial step.
#include "qmk_internal.h"

namespace qmk {
namespace {

constexpr int kMaxOrd = 8;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Block = (walker, 16 electrons) x 64 nuclei.  Ra is written nucleus-fast
// and x electron-fast (through an LDS transpose), both in full lines.
__global__ __launch_bounds__(256) void een_en_kernel(PointArgs pts, int64_t ne, const double* __restrict__ nuc,
                                                     int64_t nn, double kappa, int mk, double* __restrict__ ra,
                                                     int64_t jp, int64_t lda, int64_t nnp,
                                                     double* __restrict__ xo) {
  __shared__ double xs[16][65];
  const int64_t nblk = jp / 16;
  const int64_t w = blockIdx.x / nblk, i0 = (blockIdx.x - w * nblk) * 16, a0 = static_cast<int64_t>(blockIdx.y) * 64;
  for (int idx = threadIdx.x; idx < 16 * 64; idx += 256) {
    const int il = idx >> 6, al = idx & 63;
    const int64_t i = i0 + il, a = a0 + al;
    if (a >= nn) continue;
    double* o = ra + (w * jp + i) * lda + a;
    if (i >= ne) {  // padding row
      for (int m = 1; m <= mk; ++m) o[(m - 1) * nnp] = 0.0;
      continue;
    }
    const int64_t p = w * ne + i;
    const double dx = pts.coord[p * pts.s_pt] - nuc[3 * a];
    const double dy = pts.coord[p * pts.s_pt + pts.s_ax] - nuc[3 * a + 1];
    const double dz = pts.coord[p * pts.s_pt + 2 * pts.s_ax] - nuc[3 * a + 2];
    const double x = exp(-kappa * sqrt(dx * dx + dy * dy + dz * dz));
    double v = x;
    for (int m = 1; m <= mk; ++m) {
      o[(m - 1) * nnp] = v;
      v *= x;
    }
    xs[il][al] = x;
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < 16 * 64; idx += 256) {
    const int al = idx >> 4, il = idx & 15;
    const int64_t i = i0 + il, a = a0 + al;
    if (i < ne && a < nn) xo[(w * nn + a) * ne + i] = xs[il][al];
  }
}

// One thread per point p = (walker w, electron i):
//   g0[p][k-1] = sum_a w_{k,0,a}(x[w][a][i]),  k = 1..NORD-1,
// with the polynomial coefficients q0[k-1][a][0..NORD] staged in LDS for 64
// nuclei at a time.
constexpr int kG0Chunk = 64;
template <int NORD>
__global__ __launch_bounds__(256) void een_g0_kernel(const double* __restrict__ x, int64_t P, int64_t ne, int64_t nn,
                                                     const double* __restrict__ q0, double* __restrict__ g0) {
  constexpr int NQ = (NORD - 1) * (NORD + 1);
  __shared__ double qs[kG0Chunk * NQ];
  const int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const bool valid = p < P;
  const int64_t w = valid ? p / ne : 0, i = valid ? p - w * ne : 0;
  double g[NORD - 1] = {};
  for (int64_t a0 = 0; a0 < nn; a0 += kG0Chunk) {
    const int an = static_cast<int>(min<int64_t>(kG0Chunk, nn - a0));
    __syncthreads();
    for (int t = threadIdx.x; t < an * NQ; t += blockDim.x) {
      const int al = t / NQ, r = t - al * NQ;  // r = (k-1) (NORD+1) + e
      const int k1 = r / (NORD + 1), e = r - k1 * (NORD + 1);
      qs[t] = q0[(k1 * nn + a0 + al) * (NORD + 1) + e];
    }
    __syncthreads();
    for (int al = 0; al < an; ++al) {
      const double xv = valid ? x[(w * nn + a0 + al) * ne + i] : 0.0;
      const double* q = qs + al * NQ;
#pragma unroll
      for (int k1 = 0; k1 < NORD - 1; ++k1) {
        double pw = q[k1 * (NORD + 1) + NORD];
#pragma unroll
        for (int e = NORD - 1; e >= 0; --e) pw = pw * xv + q[k1 * (NORD + 1) + e];
        g[k1] += pw;
      }
    }
  }
  if (!valid) return;
#pragma unroll
  for (int k1 = 0; k1 < kMaxOrd - 1; ++k1) g0[p * (kMaxOrd - 1) + k1] = k1 < NORD - 1 ? g[k1] : 0.0;
}

// Block = (walker w, 8 electrons i); each wave takes 2 of them and its
// lanes run over the electrons j, whose coordinates are staged in LDS in
// chunks.  Writes rt[w][i][j] = exp(-kappa r_ij), zero on the diagonal (and so
// in its powers) and in the padding rows, and
//   j0[w][i] = sum_{k=1}^{nord-1} (sum_{j != i} rt_ij^k) g0[w][i][k-1]
// (g0 from een_g0_kernel).
constexpr int kEeRows = 2, kEeChunk = 512;
template <int NORD>
__global__ __launch_bounds__(256) void een_ee_kernel(PointArgs pts, int64_t ne, double kappa,
                                                     const double* __restrict__ g0, double* __restrict__ rt,
                                                     int64_t jp, int64_t ldb, double* __restrict__ j0) {
  __shared__ double cs[3][kEeChunk];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t nblk = jp / (4 * kEeRows);
  const int64_t w = blockIdx.x / nblk, ib = (blockIdx.x - w * nblk) * 4 * kEeRows + wv * kEeRows;
  double xi[kEeRows], yi[kEeRows], zi[kEeRows];
#pragma unroll
  for (int r = 0; r < kEeRows; ++r) {
    const int64_t p = w * ne + min(ib + r, ne - 1);
    xi[r] = pts.coord[p * pts.s_pt];
    yi[r] = pts.coord[p * pts.s_pt + pts.s_ax];
    zi[r] = pts.coord[p * pts.s_pt + 2 * pts.s_ax];
  }
  double sk[kEeRows][NORD] = {};  // [row][k]: sum_j rt_ij^k, k = 1 .. NORD-1
  for (int64_t c0 = 0; c0 < ne; c0 += kEeChunk) {
    const int cn = static_cast<int>(min<int64_t>(kEeChunk, ne - c0));
    __syncthreads();
    for (int t = threadIdx.x; t < cn; t += blockDim.x) {
      const int64_t p = w * ne + c0 + t;
      cs[0][t] = pts.coord[p * pts.s_pt];
      cs[1][t] = pts.coord[p * pts.s_pt + pts.s_ax];
      cs[2][t] = pts.coord[p * pts.s_pt + 2 * pts.s_ax];
    }
    __syncthreads();
    for (int t = lane; t < cn; t += 64) {
      const int64_t j = c0 + t;
      const double xj = cs[0][t], yj = cs[1][t], zj = cs[2][t];
      // the rows are independent chains: no branch between them
      double x[kEeRows];
#pragma unroll
      for (int r = 0; r < kEeRows; ++r) {
        const double dx = xi[r] - xj, dy = yi[r] - yj, dz = zi[r] - zj;
        x[r] = exp(-kappa * sqrt(dx * dx + dy * dy + dz * dz));
      }
#pragma unroll
      for (int r = 0; r < kEeRows; ++r) {
        const int64_t i = ib + r;
        double v = j == i || i >= ne ? 0.0 : x[r];
        rt[(w * jp + i) * ldb + j] = v;
#pragma unroll
        for (int k = 1; k < NORD; ++k) {
          sk[r][k] += v;
          v *= x[r];
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < kEeRows; ++r) {
    const int64_t i = min(ib + r, ne - 1);
    const double* g = g0 + (w * ne + i) * (kMaxOrd - 1);
    double acc = 0.0;
#pragma unroll
    for (int k = 1; k < NORD; ++k) acc += wave_sum(sk[r][k]) * g[k - 1];
    if (lane == 0 && ib + r < ne) j0[w * ne + ib + r] = acc;
  }
}

// The k = 0 terms of one (walker, nucleus) per wave:
//   sum_m sum_i w_{0,m,a}(x_ia) sum_{j != i} x_ja^m.
// The inner sum is taken as the electrons before i plus those after it (no
// difference of nearly equal sums): each lane owns a contiguous run of
// electrons, starts from the other lanes' totals and walks its run forwards
// and backwards.
template <int NORD>
__global__ __launch_bounds__(256) void een_k0_kernel(const double* __restrict__ x, int64_t nw, int64_t ne, int64_t nn,
                                                     const double* __restrict__ q, double* __restrict__ part,
                                                     int64_t part_ld) {
  constexpr int MH = NORD / 2;
  const int lane = threadIdx.x & 63;
  const int64_t item =
      __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x * 4 + (threadIdx.x >> 6)));  // the same for a wave
  if (item >= nw * nn) return;
  const int64_t w = item / nn, a = item - w * nn;
  const double* const xr = x + item * ne;
  const int64_t run = (ne + 63) / 64, lo = min(ne, lane * run), hi = min(ne, lo + run);
  double c[MH][NORD];  // a term of k = 0 has e = p - m <= NORD - m
#pragma unroll
  for (int m = 0; m < MH; ++m)
#pragma unroll
    for (int d = 0; d < NORD; ++d) c[m][d] = q[(m * nn + a) * kJasCoef + d];
  auto weight = [&](int m, double v) {
    double p = c[m][NORD - 1];
#pragma unroll
    for (int d = NORD - 2; d >= 0; --d) p = p * v + c[m][d];
    return p;
  };
  double s[MH] = {};
  for (int64_t i = lo; i < hi; ++i) {
    const double v = xr[i];
    double p = v;
#pragma unroll
    for (int m = 0; m < MH; ++m, p *= v) s[m] += p;
  }
  double fwd[MH], bwd[MH];
#pragma unroll
  for (int m = 0; m < MH; ++m) {
    double before = s[m], after = s[m];  // inclusive scans over the lanes
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double b = __shfl_up(before, off, 64), f = __shfl_down(after, off, 64);
      if (lane >= off) before += b;
      if (lane + off < 64) after += f;
    }
    const double eb = __shfl_up(before, 1, 64), ea = __shfl_down(after, 1, 64);
    fwd[m] = lane > 0 ? eb : 0.0;
    bwd[m] = lane < 63 ? ea : 0.0;
  }
  double acc = 0.0;
  auto step = [&](double (&t)[MH], double v) {
    double p = v;
#pragma unroll
    for (int m = 0; m < MH; ++m, p *= v) {
      acc += weight(m, v) * t[m];
      t[m] += p;
    }
  };
  for (int64_t i = lo; i < hi; ++i) step(fwd, xr[i]);
  for (int64_t i = hi - 1; i >= lo; --i) step(bwd, xr[i]);
  acc = wave_sum(acc);
  if (lane == 0) part[w * part_ld + a] = acc;
}

// One wave per walker: J[w] = sum of the walker's `slots` partial sums and
// of its ne m = 0 parts (fixed lane assignment and tree: deterministic).
__global__ __launch_bounds__(256) void een_finish_kernel(const double* __restrict__ part, int64_t slots,
                                                         int64_t part_ld, const double* __restrict__ j0, int64_t nw, int64_t ne,
                                                         double* __restrict__ J) {
  const int lane = threadIdx.x & 63;
  const int64_t w = static_cast<int64_t>(blockIdx.x) * (blockDim.x / 64) + (threadIdx.x >> 6);
  if (w >= nw) return;
  double v = 0.0;
  for (int64_t t = lane; t < slots; t += 64) v += part[w * part_ld + t];
  for (int64_t i = lane; i < ne; i += 64) v += j0[w * ne + i];
  v = wave_sum(v);
  if (lane == 0) J[w] = v;
}

}  // namespace

hipError_t launch_een_en(const PointArgs& pts, int64_t ne, const double* nuc, int64_t nn, double kappa, int mk,
                         double* ra, int64_t jp, int64_t lda, int64_t nnp, double* x, hipStream_t s) {
  if (pts.P <= 0 || nn <= 0) return hipSuccess;
  if (jp % 16 != 0 || jp < ne || nnp < nn || lda < mk * nnp) return hipErrorInvalidValue;
  const int64_t nw = pts.P / ne, gx = nw * (jp / 16), gy = (nn + 63) / 64;
  if (gx > 0x7fffffff || gy > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(een_en_kernel, dim3(static_cast<unsigned>(gx), static_cast<unsigned>(gy)), dim3(256), 0, s, pts,
                     ne, nuc, nn, kappa, mk, ra, jp, lda, nnp, x);
  return hipGetLastError();
}

hipError_t launch_een_ee(const PointArgs& pts, int64_t ne, int64_t nn, double kappa, int nord, const double* x,
                         const double* q0, double* g0, double* rt, int64_t jp, int64_t ldb, double* j0,
                         const double* q, double* part, int64_t part_ld, hipStream_t s) {
  if (pts.P <= 0) return hipSuccess;
  if (nord < 2 || nord > kMaxOrd || jp % 16 != 0 || jp < ne || ldb < ne) return hipErrorInvalidValue;
  static_assert(16 % (4 * kEeRows) == 0, "whole blocks of padded rows");
  const dim3 gg(static_cast<unsigned>((pts.P + 255) / 256));
  const int64_t nw = pts.P / ne, g = nw * (jp / (4 * kEeRows));
  if (g > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 ge(static_cast<unsigned>(g));
  const int64_t k0 = (nw * nn + 3) / 4;
  if (k0 > 0x1fffffff) return hipErrorInvalidValue;
  const dim3 gk(static_cast<unsigned>(k0));
  switch (nord) {
#define QMK_EEN(n)                                                                                \
  case n:                                                                                         \
    hipLaunchKernelGGL(een_g0_kernel<n>, gg, dim3(256), 0, s, x, pts.P, ne, nn, q0, g0);          \
    if (hipPeekAtLastError() != hipSuccess) break;                                                \
    hipLaunchKernelGGL(een_ee_kernel<n>, ge, dim3(256), 0, s, pts, ne, kappa, g0, rt, jp, ldb, j0); \
    if (hipPeekAtLastError() != hipSuccess) break;                                                \
    hipLaunchKernelGGL(een_k0_kernel<n>, gk, dim3(256), 0, s, x, nw, ne, nn, q, part, part_ld);   \
    break;
    QMK_EEN(2) QMK_EEN(3) QMK_EEN(4) QMK_EEN(5) QMK_EEN(6) QMK_EEN(7) QMK_EEN(8)
#undef QMK_EEN
  }
  return hipGetLastError();
}

hipError_t launch_een_finish(const double* part, int64_t slots, int64_t part_ld, const double* j0, int64_t nw,
                             int64_t ne, double* J, hipStream_t s) {
  if (nw <= 0) return hipSuccess;
  hipLaunchKernelGGL(een_finish_kernel, dim3(static_cast<unsigned>((nw + 3) / 4)), dim3(256), 0, s, part, slots,
                     part_ld, j0, nw, ne, J);
  return hipGetLastError();
}

}  // namespace qmk
