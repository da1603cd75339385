// Conversions of the adjoint's weights W: FP64 -> FP32 in the FP32 mode, and
// the split into bf16 hi / lo planes in the BF16x3 mode.
//
// The FP32 products round each FP64 weight to FP32 as they load it; doing
// that once per call in a streaming pass (round to nearest, as the loaders
// do) gives the products the same values at half the bytes, and lets them
// run their FP32-operand instantiations.  The copy pads its rows to a
// multiple of four weights, so that both products can load it in 16-byte
// pieces; the same padded copy (without conversion) serves weights whose row
// length does not allow that.
//
// The copies of the MO coefficients that the products read (both layouts,
// padded, in the mode's types) are made here too.
#include <algorithm>
#include <type_traits>

#include "qmk_internal.h"

namespace qmk {
namespace {

// rows of n source values -> rows of ldd destination values (ldd a multiple
// of 4, zeros from n on; FP64 -> FP32 rounds to nearest); output quad q of
// the copy (four values of one row)
template <typename TS, typename TD>
__device__ __forceinline__ void pad_quad(const TS* __restrict__ src, TD* __restrict__ dst, int64_t n, int64_t ldd,
                                         int64_t q) {
  const int64_t qpr = ldd / 4, row = q / qpr, c0 = (q - row * qpr) * 4;
  const TS* sr = src + row * n;
  TD v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = c0 + e < n ? static_cast<TD>(sr[c0 + e]) : TD(0);
  TD* dr = dst + row * ldd + c0;
  if constexpr (sizeof(TD) == 4) {
    *reinterpret_cast<float4*>(dr) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
    reinterpret_cast<double2*>(dr)[0] = make_double2(v[0], v[1]);
    reinterpret_cast<double2*>(dr)[1] = make_double2(v[2], v[3]);
  }
}

template <typename TS, typename TD>
__global__ __launch_bounds__(256) void pad_rows_kernel(const TS* __restrict__ src, TD* __restrict__ dst,
                                                       int64_t rows, int64_t n, int64_t ldd) {
  const int64_t q = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (q >= rows * (ldd / 4)) return;
  pad_quad(src, dst, n, ldd, q);
}

template <typename T>
__global__ __launch_bounds__(256) void pad_rows_batch_kernel(const PadJob* __restrict__ jobs,
                                                             const int64_t* __restrict__ prefix, int n_jobs,
                                                             int64_t total) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int jb = find_job(prefix, n_jobs, wave_first(), e);
  const PadJob& j = jobs[jb];
  pad_quad(static_cast<const T*>(j.src), static_cast<T*>(j.dst), j.n, j.ldd, e - prefix[jb]);
}

// W[p][c][n] -> hi, lo planes [Pp][5][Nw]: hi = bf16(x), lo = bf16(x - hi) of
// the FP32-rounded weight x (round to nearest even); zeros beyond P and N.
// Bound by memory.  With eight loads of one weight where rows were not 16-byte
// aligned, and a search for the job by every thread, a batch of 48 molecules took
// 6.44 ms, 6.25 since.
// One thread per eight consecutive n of one (p, c) row: idx < Pp * 5 * Nw / 8,
// which the launchers keep below 2^32 (32-bit index arithmetic).
template <typename T>
__device__ __forceinline__ void split_w8(const T* __restrict__ w, int64_t P, int64_t N, int64_t Nw,
                                         const int32_t* __restrict__ perm, __bf16* __restrict__ hi,
                                         __bf16* __restrict__ lo, uint32_t idx) {
  typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
  const uint32_t cpr = static_cast<uint32_t>(Nw / 8);
  const uint32_t row32 = idx / cpr;
  const int64_t row = row32, n0 = static_cast<int64_t>(idx - row32 * cpr) * 8;
  // source row: point perm[p] (or p), same component
  const int64_t p = row32 / 5u;
  const int64_t srow = (perm && p < P) ? static_cast<int64_t>(perm[p]) * 5 + (row - p * 5) : row;
  float x[8];
  if (row < P * 5 && n0 + 8 <= N) {
    // 16 bytes a load at the alignment of one weight (rows of N weights start
    // anywhere)
    constexpr int E = 16 / sizeof(T);
    typedef T vec16 __attribute__((ext_vector_type(E), aligned(sizeof(T))));
    const T* src = w + srow * N + n0;
#pragma unroll
    for (int q = 0; q < 8 / E; ++q) {
      const vec16 v = *reinterpret_cast<const vec16*>(src + E * q);
#pragma unroll
      for (int e = 0; e < E; ++e) x[E * q + e] = static_cast<float>(v[e]);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      x[e] = (row < P * 5 && n0 + e < N) ? static_cast<float>(w[srow * N + n0 + e]) : 0.0f;
  }
  bf16x8 h, l;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    // hi is the bf16 rounding of the FP32 value: without this barrier the
    // two conversions of an FP64 weight would be merged into one rounding
    asm volatile("" : "+v"(x[e]));
    const __bf16 hh = static_cast<__bf16>(x[e]);
    h[e] = hh;
    l[e] = static_cast<__bf16>(x[e] - static_cast<float>(hh));
  }
  *reinterpret_cast<bf16x8*>(hi + row * Nw + n0) = h;
  *reinterpret_cast<bf16x8*>(lo + row * Nw + n0) = l;
}

template <typename T>
__global__ __launch_bounds__(256) void split_w_kernel(const T* __restrict__ w, int64_t P, int64_t N, int64_t Pp,
                                                      int64_t Nw, const int32_t* __restrict__ perm,
                                                      __bf16* __restrict__ hi, __bf16* __restrict__ lo) {
  const uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= static_cast<uint64_t>(Pp * 5 * (Nw / 8))) return;
  split_w8(w, P, N, Nw, perm, hi, lo, idx);
}

template <typename T>
__global__ __launch_bounds__(256) void split_w_batch_kernel(const SplitJob* __restrict__ jobs,
                                                            const int64_t* __restrict__ prefix, int n_jobs,
                                                            int64_t total) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int jb = find_job(prefix, n_jobs, wave_first(), e);
  const SplitJob& j = jobs[jb];
  split_w8(static_cast<const T*>(j.w), j.P, j.N, j.Nw, static_cast<const int32_t*>(nullptr),
           static_cast<__bf16*>(j.hi), static_cast<__bf16*>(j.lo), static_cast<uint32_t>(e - prefix[jb]));
}

// The products' copies of C [N][K] (FP64): C [Np][Kp] and C^T [Kp][Np] in FP64
// (MODE 0) or FP32 (1, 2), and in MODE 2 both split into bf16 hi / lo planes
// (hi = bf16(c), lo = bf16(c - hi), the residual in FP64); zeros beyond N
// and K; row k of the copies is the caller's AO ao_of[k], column n the caller's
// MO mo_of[n] (the density's occupied ones, which need C^T only).  Np and Kp are
// multiples of 32.  The planes are in slabs of 32 reduction indices, [Kp / 32]
// [Np][32] of C and [Np / 32][Kp][32] of C^T: a K step of a product's tile is
// one run of memory (with rows of Kp or Np, 64 bytes of every row: 7500-AO
// screened forward pass 2.53 ms, 2.43 in slabs; 800-AO gradient with a step of
// the parameters 3.23 and 3.16 ms).
// One 32 x 32 tile per workgroup, transposed through LDS, so that every copy is
// stored in full lines.  Bound by the latency of one pass: 800 AOs x 400 MOs
// 7 us, where the host loops and 4 to 6 blocking uploads that this replaces
// took 3 ms.
template <int MODE>
__global__ __launch_bounds__(256) void coef_layout_kernel(const double* __restrict__ src, int64_t N, int64_t K,
                                                          int64_t Np, int64_t Kp, const int32_t* __restrict__ ao_of,
                                                          const int32_t* __restrict__ mo_of, CoefCopies o) {
  typedef typename std::conditional<MODE == 0, double, float>::type T;
  __shared__ double tile[32][33];
  const uint32_t kb = static_cast<uint32_t>(Kp / 32), nb = blockIdx.x / kb;
  const int64_t k0 = static_cast<int64_t>(blockIdx.x - nb * kb) * 32, n0 = static_cast<int64_t>(nb) * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  auto put = [](const CoefCopies& c, bool transposed, int64_t at, int64_t slab_at, double v) {
    static_cast<T*>(transposed ? c.ct : c.c)[at] = static_cast<T>(v);
    if constexpr (MODE == 2) {
      float f = static_cast<float>(v);
      // hi is the bf16 rounding of the FP32 value (not one FP64 -> bf16 rounding)
      asm volatile("" : "+v"(f));
      const __bf16 h = static_cast<__bf16>(f);
      float r = static_cast<float>(v - static_cast<double>(static_cast<float>(h)));
      asm volatile("" : "+v"(r));
      static_cast<__bf16*>(transposed ? c.ct_hi : c.c_hi)[slab_at] = h;
      static_cast<__bf16*>(transposed ? c.ct_lo : c.c_lo)[slab_at] = static_cast<__bf16>(r);
    }
  };
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t n = n0 + ty + 8 * q, k = k0 + tx;
    const double v = n < N && k < K ? src[(mo_of ? mo_of[n] : n) * K + (ao_of ? ao_of[k] : k)] : 0.0;
    if (o.c) put(o, false, n * Kp + k, k0 * Np + n * 32 + tx, v);
    tile[ty + 8 * q][tx] = v;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t k = k0 + ty + 8 * q;
    put(o, true, k * Np + n0 + tx, n0 * Kp + k * 32 + tx, tile[tx][ty + 8 * q]);
  }
}

// dst = src, with *flag = 1 where a value is not finite; the first workgroup
// also copies the nuclei to `nucl_out` (host memory) and, where `nuc` is
// given, into the nucleus table.
__global__ __launch_bounds__(256) void take_params_kernel(const double* __restrict__ src, double* __restrict__ dst,
                                                          int64_t n, const double* __restrict__ nucl, int64_t n_nucl,
                                                          double* __restrict__ nucl_out, NucDev* __restrict__ nuc,
                                                          int32_t n_nuc, int32_t* __restrict__ flag) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  bool bad = false;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
    const double v = src[i];
    dst[i] = v;
    bad = bad || !isfinite(v);
  }
  if (bad) *flag = 1;
  if (blockIdx.x != 0) return;
  for (int64_t i = threadIdx.x; i < 3 * n_nucl; i += blockDim.x) nucl_out[i] = nucl[i];
  if (nuc)
    for (int32_t a = threadIdx.x; a < n_nuc; a += blockDim.x) {
      const double* r = nucl + 3 * static_cast<int64_t>(nuc[a].orig);
      nuc[a].x = r[0];
      nuc[a].y = r[1];
      nuc[a].z = r[2];
    }
}

}  // namespace

hipError_t launch_coef_layout(const double* src, int64_t N, int64_t K, int64_t Np, int64_t Kp, int mode,
                              const int32_t* ao_of, const int32_t* mo_of, const CoefCopies& o, hipStream_t s) {
  if (N <= 0 || K <= 0) return hipSuccess;
  if (Np % 32 != 0 || Kp % 32 != 0 || Np < N || Kp < K || (Np / 32) * (Kp / 32) > 0x7fffffff)
    return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>((Np / 32) * (Kp / 32)));
  if (mode == 0)
    hipLaunchKernelGGL(coef_layout_kernel<0>, grid, dim3(256), 0, s, src, N, K, Np, Kp, ao_of, mo_of, o);
  else if (mode == 1)
    hipLaunchKernelGGL(coef_layout_kernel<1>, grid, dim3(256), 0, s, src, N, K, Np, Kp, ao_of, mo_of, o);
  else
    hipLaunchKernelGGL(coef_layout_kernel<2>, grid, dim3(256), 0, s, src, N, K, Np, Kp, ao_of, mo_of, o);
  return hipGetLastError();
}

hipError_t launch_take_params(const double* coef, double* coef_out, int64_t n, const double* nucl, int64_t n_nucl,
                              double* nucl_out, NucDev* nuc, int32_t n_nuc, int32_t* flag, hipStream_t s) {
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 1024);
  hipLaunchKernelGGL(take_params_kernel, dim3(static_cast<unsigned>(std::max<int64_t>(blocks, 1))), dim3(256), 0, s,
                     coef, coef_out, n, nucl, n_nucl, nucl_out, nuc, n_nuc, flag);
  return hipGetLastError();
}

hipError_t launch_split_w(const void* w, int w_is_f32, int64_t P, int64_t N, int64_t Pp, int64_t Nw,
                          const int32_t* perm, void* hi, void* lo, hipStream_t s) {
  if (Pp <= 0 || Nw <= 0) return hipSuccess;
  if (Nw % 8 != 0 || Pp < P || Nw < N) return hipErrorInvalidValue;
  const int64_t n = Pp * 5 * (Nw / 8);
  if (n > 0xffffffffLL - 255) return hipErrorInvalidValue;
  const int64_t blocks = (n + 255) / 256;
  if (w_is_f32)
    hipLaunchKernelGGL(split_w_kernel<float>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s,
                       static_cast<const float*>(w), P, N, Pp, Nw, perm, static_cast<__bf16*>(hi),
                       static_cast<__bf16*>(lo));
  else
    hipLaunchKernelGGL(split_w_kernel<double>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s,
                       static_cast<const double*>(w), P, N, Pp, Nw, perm, static_cast<__bf16*>(hi),
                       static_cast<__bf16*>(lo));
  return hipGetLastError();
}

hipError_t launch_split_w_batch(const SplitJob* jobs, const int64_t* prefix, int n_jobs, int64_t total,
                                int w_is_f32, hipStream_t s) {
  if (total <= 0 || n_jobs <= 0) return hipSuccess;
  const int64_t blocks = (total + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  if (w_is_f32)
    hipLaunchKernelGGL(split_w_batch_kernel<float>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, jobs,
                       prefix, n_jobs, total);
  else
    hipLaunchKernelGGL(split_w_batch_kernel<double>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, jobs,
                       prefix, n_jobs, total);
  return hipGetLastError();
}

hipError_t launch_pad_rows_batch(const PadJob* jobs, const int64_t* prefix, int n_jobs, int64_t total, int f32,
                                 hipStream_t s) {
  if (total <= 0 || n_jobs <= 0) return hipSuccess;
  const int64_t blocks = (total + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  if (f32)
    hipLaunchKernelGGL(pad_rows_batch_kernel<float>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, jobs,
                       prefix, n_jobs, total);
  else
    hipLaunchKernelGGL(pad_rows_batch_kernel<double>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, jobs,
                       prefix, n_jobs, total);
  return hipGetLastError();
}

hipError_t launch_pad_rows(const void* src, int src_f32, void* dst, int dst_f32, int64_t rows, int64_t n,
                           int64_t ldd, hipStream_t s) {
  if (rows <= 0 || n <= 0) return hipSuccess;
  // the vector stores need 16-byte aligned rows; FP32 -> FP64 is not offered
  if (ldd < n || ldd % 4 != 0 || reinterpret_cast<uintptr_t>(dst) % 16 != 0 || (src_f32 && !dst_f32))
    return hipErrorInvalidValue;
  const int64_t blocks = (rows * (ldd / 4) + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(blocks));
  if (src_f32)
    hipLaunchKernelGGL((pad_rows_kernel<float, float>), grid, dim3(256), 0, s, static_cast<const float*>(src),
                       static_cast<float*>(dst), rows, n, ldd);
  else if (dst_f32)
    hipLaunchKernelGGL((pad_rows_kernel<double, float>), grid, dim3(256), 0, s, static_cast<const double*>(src),
                       static_cast<float*>(dst), rows, n, ldd);
  else
    hipLaunchKernelGGL((pad_rows_kernel<double, double>), grid, dim3(256), 0, s, static_cast<const double*>(src),
                       static_cast<double*>(dst), rows, n, ldd);
  return hipGetLastError();
}

}  // namespace qmk
