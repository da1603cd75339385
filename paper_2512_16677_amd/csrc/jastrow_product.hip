// The product of the three-body Jastrow factor with its fused weights (QMCkl
// paper, Section 3.5; the pieces around it are in jastrow_kernels.hip):
//   P^{k,m}_{ia} = sum_j rt_ij^k Rt_ja^m   (k >= 1, m >= 1; rt has a zero diagonal)
//   part[w][slot] = sum over the slot's (i, a, m) and powers k of
//                   w_{k,m,a}(Rt_ia) P^{k,m}_{ia}
// FP64 on v_mfma_f64_16x16x4.  Rows of the product are (m, a), columns the
// electrons i, the reduction runs over the electrons j.
//
// Only the (k, m) that some term uses are formed: p - k - l = 2 m with p <= N_ord
// leaves k <= N_ord - 2 m, in groups of one m and up to three consecutive k
// (EenGroups).  The k = 0 terms need no product (een_k0 in
// jastrow_kernels.hip).
//
// What bounds it is the FP64 matrix rate, so the layout keeps everything else
// out of the K loop: one tile forms the KP powers of its group (KP x TM x TN
// accumulator blocks per wavefront), so that both operands are read once for
// all of them, the powers are taken as the B fragments leave LDS (one
// multiplication per power, under the MFMAs), and both operand arrays are
// padded by their producers to whole 16-electron steps, so that every load is
// a direct global -> LDS transfer (two stages) and no step is partial.  The
// epilogue has the tile's x and coefficients in LDS.
//
// 80 nuclei, 280 electrons, 500 walkers, order 5: 1508 us with every (k, m) of k
// = 0 .. 3 and m = 1, 2, one tile per k, operands staged through registers;
// 520 to 540 us now (25.1 GF:
// 48 TF; whole call 1765 -> 847 us).
#include "gemm_impl.h"

namespace qmk {
namespace {

// Groups of order NORD, the longest first: m and the powers s0 .. s0 + kp - 1.
struct EenGroup {
  int m, kp, s0;
};
template <int NORD>
struct EenGroups;
template <>
struct EenGroups<3> {
  static constexpr EenGroup g[] = {{1, 1, 1}};
};
template <>
struct EenGroups<4> {
  static constexpr EenGroup g[] = {{1, 2, 1}};
};
template <>
struct EenGroups<5> {
  static constexpr EenGroup g[] = {{1, 3, 1}, {2, 1, 1}};
};
template <>
struct EenGroups<6> {
  static constexpr EenGroup g[] = {{1, 2, 1}, {1, 2, 3}, {2, 2, 1}};
};
template <>
struct EenGroups<7> {
  static constexpr EenGroup g[] = {{1, 3, 1}, {2, 3, 1}, {1, 2, 4}, {3, 1, 1}};
};
template <>
struct EenGroups<8> {
  static constexpr EenGroup g[] = {{1, 3, 1}, {1, 3, 4}, {2, 2, 1}, {2, 2, 3}, {3, 2, 1}};
};
template <int NORD>
constexpr int kNumGroups = sizeof(EenGroups<NORD>::g) / sizeof(EenGroup);

// Coefficients of a weight of a group: its degree is at most N_ord - k - m.
template <int NORD>
constexpr int kNumCoef = NORD - 1;

// LDS in doubles: two stages, then the epilogue's coefficients and x.
template <int NORD, int WGM, int WGN, int TM, int TN>
constexpr int een_lds() {
  constexpr int BM = 16 * WGM * TM, BN = 16 * WGN * TN, st = 2 * (BM + BN) * 16;
  constexpr int epi = BM * 3 * kNumCoef<NORD> + BM * (BN + 1);
  return st > epi ? st : epi;
}

template <int NORD, int KP, int S0, int WGM, int WGN, int TM, int TN>
__device__ __forceinline__ void een_tile_body(const JasArgs& g, int64_t w, int m, int mt, int nt, int nN, double* sm,
                                              double* __restrict__ part) {
  constexpr int BM = 16 * WGM * TM, BN = 16 * WGN * TN, NW = WGM * WGN, BK = 16;
  constexpr int NIA = BM * BK * 8 / 1024, NI = (BM + BN) * BK * 8 / 1024;  // 1 KB blocks per stage (A first)
  constexpr int IPW = (NI + NW - 1) / NW;
  constexpr int STAGE = (BM + BN) * BK;  // doubles
  constexpr int NC = kNumCoef<NORD>, QS = BM * KP * NC, XP = BN + 1;
  typedef Mfma<double>::v4 v4;
  const int64_t i0 = static_cast<int64_t>(mt) * BM, j0 = static_cast<int64_t>(nt) * BN;
  // rows: the nuclei; A holds Rt^m, nnp columns per m
  const double* const Aw = g.ra + w * g.jp * g.lda + (m - 1) * g.nnp;
  const double* const Bw = g.rt + w * g.jp * g.ldb;

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wm = wv / WGN, wn = wv % WGN;
  const int wu = __builtin_amdgcn_readfirstlane(wv);
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(dma_lds_address(sm));
  const char* gp[IPW];
  bool isa[IPW];
  uint32_t ldso[IPW];
#pragma unroll
  for (int q = 0; q < IPW; ++q) {
    int ig = wu + NW * q;
    if (NI % NW != 0 && ig >= NI) ig -= NI;  // (the same bytes written twice)
    ldso[q] = static_cast<uint32_t>(ig) * 1024u;
    isa[q] = ig < NIA;
    // columns past the padded rows of an operand read its last 16 bytes (their
    // outputs are masked)
    if (isa[q]) {
      const int sl = 64 * ig + lane, l = sl / (BM / 2);
      const int64_t i = i0 + ((2 * (sl % (BM / 2))) ^ dma_xr<double, BM>(l));
      gp[q] = reinterpret_cast<const char*>(Aw + min(i, g.nnp - 2) + l * g.lda);
    } else {
      const int sl = 64 * (ig - NIA) + lane, l = sl / (BN / 2);
      const int64_t j = j0 + ((2 * (sl % (BN / 2))) ^ dma_xr<double, BN>(l));
      gp[q] = reinterpret_cast<const char*>(Bw + min(j, g.ldb - 2) + l * g.ldb);
    }
  }
  const int64_t stepA = BK * 8 * g.lda, stepB = BK * 8 * g.ldb;
  auto issue = [&](int slot, int kt) {
    int64_t oa = kt * stepA, ob = kt * stepB;
    asm("" : "+s"(oa), "+s"(ob));
    const uint32_t sb = lds0 + static_cast<uint32_t>(slot * STAGE * 8);
#pragma unroll
    for (int q = 0; q < IPW; ++q) dma_b128(gp[q] + (isa[q] ? oa : ob), sb + ldso[q]);
  };

  v4 acc[KP][TM][TN];
#pragma unroll
  for (int k = 0; k < KP; ++k)
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int b = 0; b < TN; ++b) acc[k][a][b] = v4{0, 0, 0, 0};

  const int ci = lane & 15, kq = lane >> 4;
  auto compute = [&](const double* sa) {
    const double* sb = sa + BM * BK;
    double fa[2][TM], fb[2][TN];
    auto rd = [&](int kk, int u) {
      const int k = kk * 4 + kq;
#pragma unroll
      for (int a = 0; a < TM; ++a) fa[u][a] = sa[k * BM + (((wm * TM + a) * 16 + ci) ^ dma_xr<double, BM>(k))];
#pragma unroll
      for (int b = 0; b < TN; ++b) fb[u][b] = sb[k * BN + (((wn * TN + b) * 16 + ci) ^ dma_xr<double, BN>(k))];
    };
    rd(0, 0);
#pragma unroll
    for (int kk = 0; kk < BK / 4; ++kk) {
      const int u = kk & 1;
      if (kk + 1 < BK / 4) rd(kk + 1, u ^ 1);
      double pw[TN];
#pragma unroll
      for (int b = 0; b < TN; ++b) {
        pw[b] = fb[u][b];
#pragma unroll
        for (int e = 1; e < S0; ++e) pw[b] *= fb[u][b];
      }
#pragma unroll
      for (int k = 0; k < KP; ++k) {
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b) acc[k][a][b] = Mfma<double>::op(fa[u][a], pw[b], acc[k][a][b]);
        if (k + 1 < KP) {
#pragma unroll
          for (int b = 0; b < TN; ++b) pw[b] *= fb[u][b];
        }
      }
    }
  };
  const int nk = static_cast<int>(g.jp / BK);
  issue(0, 0);
  for (int kt = 0; kt < nk; ++kt) {
    dma_sync();
    if (kt + 1 < nk) issue((kt + 1) & 1, kt + 1);
    compute(sm + (kt & 1) * STAGE);
  }

  // weights: polynomials of the tile's rows in x[a][j], both staged in LDS
  __syncthreads();
  double* const qs = sm;
  double* const xs = sm + QS;
  for (int e = tid; e < QS; e += 64 * NW) {
    const int lr = e / (KP * NC), kd = e - lr * (KP * NC), k = kd / NC, d = kd - k * NC;
    const int64_t gi = i0 + lr;
    qs[e] = gi < g.nn ? g.q[((static_cast<int64_t>(S0 + k) * g.mh + m - 1) * g.nn + gi) * kJasCoef + d] : 0.0;
  }
  const double* const xw = g.x + w * g.nn * g.ne;
  for (int e = tid; e < BM * BN; e += 64 * NW) {
    const int lr = e / BN, lc = e - lr * BN;
    xs[lr * XP + lc] = xw[min(i0 + lr, g.nn - 1) * g.ne + min(j0 + lc, g.ne - 1)];
  }
  __syncthreads();
  double v = 0.0;
  bool col_in[TN];
#pragma unroll
  for (int b = 0; b < TN; ++b) col_in[b] = j0 + (wn * TN + b) * 16 + ci < g.ne;
#pragma unroll
  for (int a = 0; a < TM; ++a) {
    // a real loop over the four rows of a block: the weights of one row are in
    // registers at a time (unrolled, those of every row were formed ahead and
    // the accumulators spilled)
#pragma unroll 1
    for (int r4 = 0; r4 < 4; ++r4) {
      const int lr = (wm * TM + a) * 16 + Mfma<double>::row(lane, r4);
      const bool row_in = i0 + lr < g.nn;
      double xv[TN];
#pragma unroll
      for (int b = 0; b < TN; ++b) xv[b] = xs[lr * XP + (wn * TN + b) * 16 + ci];
#pragma unroll
      for (int k = 0; k < KP; ++k) {
        const double* const q = qs + (lr * KP + k) * NC;
        double p[TN];
        const double top = q[NC - 1];
#pragma unroll
        for (int b = 0; b < TN; ++b) p[b] = top;
#pragma unroll
        for (int d = NC - 2; d >= 0; --d) {
          const double c = q[d];
#pragma unroll
          for (int b = 0; b < TN; ++b) p[b] = p[b] * xv[b] + c;
        }
#pragma unroll
        for (int b = 0; b < TN; ++b) {
          const v4 t = acc[k][a][b];
          const double o = r4 < 2 ? (r4 == 0 ? t[0] : t[1]) : (r4 == 2 ? t[2] : t[3]);
          // (outputs past the last row or column hold anything)
          v += p[b] * (row_in & col_in[b] ? o : 0.0);
        }
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int64_t nNw = static_cast<int64_t>(nN) * WGN;
  if (lane == 0)
    part[(static_cast<int64_t>(mt) * WGM + wm) * nNw + static_cast<int64_t>(nt) * WGN + wn] = v;
}

template <int NORD, int WGM, int WGN, int TM, int TN>
__global__ __launch_bounds__(64 * WGM * WGN, 3) void een_product_kernel(JasArgs g, int nM, int nN, int64_t slots,
                                                                        int64_t full) {
  constexpr int NG = kNumGroups<NORD>, LDS = een_lds<NORD, WGM, WGN, TM, TN>();
  static_assert(LDS * 8 <= 160 * 1024, "LDS");
  __shared__ __align__(16) double sm[LDS];
  // The first `full` walkers go eight at a time to the eight XCDs, all tiles of one
  // walker to one XCD, because they share its operands; the tiles of the others
  // are dealt out over all XCDs (see run_een).
  const int tiles = NG * nM * nN;
  const int64_t rest = static_cast<int64_t>(blockIdx.x) - full * tiles;
  const int x = blockIdx.x & 7, r = rest < 0 ? static_cast<int>(blockIdx.x >> 3) : static_cast<int>(rest);
  const int64_t w = rest < 0 ? static_cast<int64_t>(r / tiles) * 8 + x : full + r / tiles;
  if (w >= g.nw) return;
  const int t = r - r / tiles * tiles, gr = t / (nM * nN), u = t - gr * (nM * nN), mt = u % nM, nt = u / nM;
  double* const part = g.part + w * g.part_ld + gr * slots;
  auto body = [&](auto idx) {
    constexpr EenGroup e = EenGroups<NORD>::g[decltype(idx)::value];
    een_tile_body<NORD, e.kp, e.s0, WGM, WGN, TM, TN>(g, w, e.m, mt, nt, nN, sm, part);
  };
  if (gr == 0) return body(std::integral_constant<int, 0>{});
  if constexpr (NG > 1)
    if (gr == 1) return body(std::integral_constant<int, 1>{});
  if constexpr (NG > 2)
    if (gr == 2) return body(std::integral_constant<int, 2>{});
  if constexpr (NG > 3)
    if (gr == 3) return body(std::integral_constant<int, 3>{});
  if constexpr (NG > 4) body(std::integral_constant<int, 4>{});
}

// Tiles {WGM, WGN, TM, TN}: rows are nuclei, columns electrons.  The small ones
// lead (80 nuclei x 280 electrons: 16 x 32 540 us, 80 x 32 600 us): two stages
// are in flight per workgroup, so it takes several workgroups per SIMD to
// cover the loads and the epilogues, and three or four stages cost more
// workgroups than they hide (80 x 32: 760 and 710 us).
#define QMK_JAS_TILES(X) \
  X(0, 1, 2, 1, 1)       \
  X(1, 1, 1, 1, 1)       \
  X(2, 2, 2, 1, 1)       \
  X(3, 1, 2, 1, 2)       \
  X(4, 1, 2, 5, 1)       \
  X(5, 1, 4, 5, 1)       \
  X(6, 1, 4, 2, 1)

constexpr TileCfg kJasTiles[] = {
#define QMK_JAS_ENTRY(id, wgm, wgn, tm, tn) {wgm, wgn, tm, tn, 16},
    QMK_JAS_TILES(QMK_JAS_ENTRY)
#undef QMK_JAS_ENTRY
};
constexpr int kNumJasTiles = sizeof(kJasTiles) / sizeof(kJasTiles[0]);

template <int NORD>
hipError_t run_een(int cfg, const JasArgs& g, hipStream_t s) {
  const TileCfg t = kJasTiles[cfg];
  const int64_t nM = (g.nn + t.bm() - 1) / t.bm(), nN = (g.ne + t.bn() - 1) / t.bn();
  const int64_t tiles = nM * nN * kNumGroups<NORD>;
  // Where few walkers are left over after whole rounds of eight, their tiles are
  // dealt out over all XCDs, some of which would idle: up to three of them, or
  // six of many tiles.  With more, sharing the operands in one L2 is worth more.
  // Whole call, order 5, one XCD per walker / dealt out: 300 nuclei x 1050 electrons,
  // 1 walker 549 / 248 us, 5 walkers 596 / 473, 7 walkers 609 / 628; 80 x 280, 3 walkers
  // 74 / 74, 5 walkers 77 / 81, 20 walkers (4 left) 110 / 103; 1000 x 3000, 1 walker
  // 9280 / 1721.
  const int64_t left = g.nw & 7;
  const bool deal = left <= 3 || (left <= 6 && tiles >= 1024);
  const int64_t full = deal ? g.nw - left : (g.nw + 7) / 8 * 8;
  const int64_t blocks = (deal ? g.nw : full) * tiles;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(blocks));
  switch (cfg) {
#define QMK_JAS_CASE(id, wgm, wgn, tm, tn)                                                                    \
  case id:                                                                                                    \
    hipLaunchKernelGGL((een_product_kernel<NORD, wgm, wgn, tm, tn>), grid, dim3(64 * wgm * wgn), 0, s, g,     \
                       static_cast<int>(nM), static_cast<int>(nN), een_slots(cfg, g.nn, g.ne), full);         \
    break;
    QMK_JAS_TILES(QMK_JAS_CASE)
#undef QMK_JAS_CASE
  }
  return hipGetLastError();
}

}  // namespace

int een_num_tiles() { return kNumJasTiles; }
TileCfg een_tile(int cfg) { return kJasTiles[cfg]; }

int64_t een_slots(int cfg, int64_t nn, int64_t ne) {
  const TileCfg t = kJasTiles[cfg];
  return (nn + t.bm() - 1) / t.bm() * t.wgm * ((ne + t.bn() - 1) / t.bn() * t.wgn);
}

int een_groups(int nord) {
  switch (nord) {
    case 3: return kNumGroups<3>;
    case 4: return kNumGroups<4>;
    case 5: return kNumGroups<5>;
    case 6: return kNumGroups<6>;
    case 7: return kNumGroups<7>;
    case 8: return kNumGroups<8>;
    default: return 0;  // order 2 has k = 0 terms only
  }
}

hipError_t launch_een_product(int cfg, int nord, const JasArgs& g, hipStream_t s) {
  if (cfg < 0 || cfg >= kNumJasTiles) return hipErrorInvalidValue;
  if (g.nw <= 0 || g.nn <= 0 || g.ne <= 0) return hipSuccess;
  // what the loaders assume of the operand arrays: 16-byte pieces, whole steps
  if (g.jp % 16 != 0 || g.jp < g.ne || g.nnp % 2 != 0 || g.nnp < g.nn || g.lda % 2 != 0 ||
      g.lda < (nord - 1) / 2 * g.nnp || g.ldb % 2 != 0 || g.ldb < g.ne)
    return hipErrorInvalidValue;
  switch (nord) {
    case 3: return run_een<3>(cfg, g, s);
    case 4: return run_een<4>(cfg, g, s);
    case 5: return run_een<5>(cfg, g, s);
    case 6: return run_een<6>(cfg, g, s);
    case 7: return run_een<7>(cfg, g, s);
    case 8: return run_een<8>(cfg, g, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qmk
