// Complex FP64 GEMM on v_mfma_f64_16x16x4_f64:
//   C = alpha * op(A) * diag(s) * op(B) + beta * C,   s_k = -1 for k >= kneg
// op(X) in {X, X^H}.  Used for the Gram matrices of CholeskyQR2 (X^H X), the
// Rayleigh quotient pieces of Alg. 2 (Q^H S T folds S through kneg = m,
// Q2^H Q2), the back-transforms Q Z and T Z, and the triangular products of
// the Cholesky / inverse kernels (batched).
// Tall-skinny inner products (K >> M, N) are split along K into a workspace
// and reduced in a fixed order (deterministic).  Real matrices held in c128
// (real_data) take only the real-by-real MFMA of each step.
//
// The FP64 MFMA takes 64 cycles, so a wave loads its fragments straight into
// registers (32 x 32 outputs: 8 16-byte loads per lane and slab of 8 k for 32
// MFMAs, 2048 cycles), one slab ahead, without LDS and barriers.  Large
// products: waves of 32 x 32, four a workgroup, K split over workgroups where
// the tiles leave CUs idle.  Small ones, bound by latency: the waves of a
// workgroup share K.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace chase {
namespace {

constexpr int NT = 256;
constexpr int RK = 8;   // K slab

typedef double doublex2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ doublex4 mfma64(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

struct ZgemmDev {
  int transA, transB;
  int64_t M, N, K;
  double ar, ai, br, bi;  // alpha, beta
  const c128* A;
  int64_t lda, strideA;
  const c128* B;
  int64_t ldb, strideB;
  c128* C;
  int64_t ldc, strideC;
  int64_t kneg;
  int lower_only, a_lower, b_upper;
  int real_data;
  int splits;
  int TM, TN;      // workgroup tiles of a large product (not lower_only)
  int tiles;
  int64_t kchunk;  // K range per split
  c128* ws;        // split-K partials: a workgroup's outputs per (split, batch, tile)
};

__device__ __forceinline__ int xcd_remap(int w, int T) {
  // workgroup w runs on XCD w % 8: give each XCD a contiguous range, so that
  // the tiles of a strip and of a K range stay in one L2
  const int xcd = w & 7, slot = w >> 3;
  const int q = T >> 3, r = T & 7;
  return xcd * q + (xcd < r ? xcd : r) + slot;
}

// First row and column of a wave's U x U outputs in workgroup tile t, false
// if it has none.  lower_only: the tiles of the lower triangle row by row, four
// neighbours a workgroup (no wave above the diagonal).  With a triangular
// operand the four waves have the same K range, 4 U rows of a column (b_upper)
// or 4 U columns of a row (a_lower), the longest ranges first.  Else 2 x 2.
// 8000 x 520 x 520 upper: 270 us strip by strip, 198 us longest first in 64 x 64 tiles, 183 so;
// 520 x 520 x 8000 lower: 200 us on 2 x 2, 171 so.
template <int U>
__device__ __forceinline__ bool wave_tile(const ZgemmDev& g, int t, int wave, int64_t* m0, int64_t* n0) {
  int i, j;
  if (g.lower_only) {
    const int u = 4 * t + wave;
    i = (int)((sqrt(8.0 * (double)u + 1.0) - 1.0) * 0.5);
    while (i * (i + 1) / 2 > u) --i;
    while ((i + 1) * (i + 2) / 2 <= u) ++i;
    j = u - i * (i + 1) / 2;
  } else if (g.b_upper) {
    j = t / g.TM;
    i = 4 * (t - j * g.TM) + wave;
    j = g.TN - 1 - j;
  } else if (g.a_lower) {
    i = t / g.TN;
    j = 4 * (t - i * g.TN) + wave;
    i = g.TM - 1 - i;
  } else {
    i = t / g.TN;
    j = 2 * (t - i * g.TN) + (wave & 1);
    i = 2 * i + (wave >> 1);
  }
  *m0 = U * (int64_t)i;
  *n0 = U * (int64_t)j;
  return *m0 < g.M && *n0 < g.N;
}

__device__ __forceinline__ double flip(double x, unsigned mask) {  // mask: 0 or 0x80000000
  return __hiloint2double(__double2hiint(x) ^ (int)mask, __double2loint(x));
}

// Output rows 4 (l / 16) + r of lane l (accumulator r) when the lane feeds the
// A row below; the f64 MFMA itself gives it rows l / 16 + 4 r.
__device__ __forceinline__ int feed_row(int l) { return 4 * (l & 3) + ((l & 15) >> 2); }

// C[gi .. gi + 3][gj] from alpha v + beta C
__device__ __forceinline__ void put4(const ZgemmDev& g, int bt, int64_t gi, int64_t gj, doublex4 vr, doublex4 vi) {
  if (gj >= g.N) return;
  c128* Cp = g.C + (int64_t)bt * g.strideC + gj * g.ldc + gi;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (gi + r >= g.M) break;
    double outr = vr[r], outi = vi[r];
    if (g.br != 0.0 || g.bi != 0.0) {
      const c128 c = Cp[r];
      outr += g.br * c.re - g.bi * c.im;
      outi += g.br * c.im + g.bi * c.re;
    }
    Cp[r] = c128{outr, outi};
  }
}

// cr + i ci = op(A) S op(B) over k in [kbeg, kend) for the 16 F x 16 F outputs
// at (m0, n0), a slab of 8 loaded ahead of its use.
// Lane l of a fragment of 16 rows of A or columns of B and 8 k holds row
// feed_row(l) of A, column l % 16 of B, at k = 2 (l / 16) + s, s = 0, 1: two loads of
// one c128, 128 contiguous bytes per row where k runs along memory, 256 per k
// where the rows do.
template <bool REAL, int TA, int TBT, int F>
__device__ __forceinline__ void accumulate(const ZgemmDev& g, int bt, int64_t m0, int64_t n0, int64_t kbeg, int64_t kend,
                                           doublex4 (&cr)[F][F], doublex4 (&ci)[F][F]) {
  const c128* A = g.A + (int64_t)bt * g.strideA;
  const c128* B = g.B + (int64_t)bt * g.strideB;
  const int lane = threadIdx.x & 63, lk = 2 * (lane >> 4);
  // addresses of the lane's first k of each fragment (rows past the end read
  // the last one: never stored)
  const doublex2 *pa[F], *pb[F];
#pragma unroll
  for (int i = 0; i < F; ++i) {
    const int64_t r = min(m0 + 16 * i + feed_row(lane), g.M - 1), c = min(n0 + 16 * i + (lane & 15), g.N - 1);
    pa[i] = reinterpret_cast<const doublex2*>(A) + (TA ? r * g.lda + lk : (int64_t)lk * g.lda + r);
    pb[i] = reinterpret_cast<const doublex2*>(B) + (TBT ? (int64_t)lk * g.ldb + c : c * g.ldb + lk);
  }
  const int64_t ka = TA ? 1 : g.lda, kb = TBT ? g.ldb : 1;  // step of one k
  using E = std::conditional_t<REAL, double, doublex2>;
  E fa[2][F][2], fb[2][F][2];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) cr[i][j] = ci[i][j] = doublex4{0, 0, 0, 0};

  auto load = [&](int64_t k, E (&xa)[F][2], E (&xb)[F][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        xa[i][s] = *reinterpret_cast<const E*>(pa[i] + (k + s) * ka);
        xb[i][s] = *reinterpret_cast<const E*>(pb[i] + (k + s) * kb);
      }
  };
  auto load_tail = [&](int64_t k, E (&xa)[F][2], E (&xb)[F][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const bool ok = k + lk + s < kend;
        const int64_t q = ok ? k + s : -lk;  // k = 0 of the operand where past the end
        const E va = *reinterpret_cast<const E*>(pa[i] + q * ka), vb = *reinterpret_cast<const E*>(pb[i] + q * kb);
        xa[i][s] = ok ? va : E{};
        xb[i][s] = ok ? vb : E{};
      }
  };
  auto mul = [&](int64_t k, const E (&xa)[F][2], const E (&xb)[F][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const unsigned neg = k + lk + s >= g.kneg ? 0x80000000u : 0u;
      double ar[F], ai[F], an[F], br[F], bi[F];
#pragma unroll
      for (int i = 0; i < F; ++i) {
        if constexpr (REAL) {
          ar[i] = xa[i][s];
          br[i] = flip(xb[i][s], neg);
        } else {
          ar[i] = xa[i][s][0];
          ai[i] = flip(xa[i][s][1], TA ? 0x80000000u : 0u);
          an[i] = flip(xa[i][s][1], TA ? 0u : 0x80000000u);
          br[i] = flip(xb[i][s][0], neg);
          bi[i] = flip(xb[i][s][1], TBT ? neg ^ 0x80000000u : neg);
        }
      }
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) {
          cr[i][j] = mfma64(ar[i], br[j], cr[i][j]);
          if constexpr (!REAL) ci[i][j] = mfma64(ar[i], bi[j], ci[i][j]);
        }
      if constexpr (!REAL) {
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
          for (int j = 0; j < F; ++j) {
            cr[i][j] = mfma64(an[i], bi[j], cr[i][j]);
            ci[i][j] = mfma64(ai[i], br[j], ci[i][j]);
          }
      }
    }
  };
  const int64_t kfull = kbeg + (max(kend - kbeg, (int64_t)0) / RK) * RK;
  if (kbeg < kfull) load(kbeg, fa[0], fb[0]);
#pragma unroll 1
  for (int64_t k = kbeg; k < kfull; k += RK) {
    load(min(k + RK, kfull - RK), fa[1], fb[1]);
    __builtin_amdgcn_sched_barrier(0);
    mul(k, fa[0], fb[0]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        fa[0][i][s] = fa[1][i][s];
        fb[0][i][s] = fb[1][i][s];
      }
  }
  if (kfull < kend) {
    load_tail(kfull, fa[0], fb[0]);
    mul(kfull, fa[0], fb[0]);
  }
}

// F: fragments per wave and operand.  Complex: 2.  Real data takes a quarter of
// the MFMAs on the same lines, which at F = 2 the L1 bounds (64 bytes a cycle);
// large real products run at F = 4 (24000 x 1920 x 1920 upper 3754 -> 1877 us,
// 1920 x 1920 x 24000 lower 5211 -> 2682).
template <bool REAL, int TA, int TBT, int F>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, F == 2 ? 3 : 2))) void zgemm_kernel(
    const ZgemmDev g) {
  constexpr int U = 16 * F, RT = 2 * U;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int id = g.b_upper || g.a_lower ? blockIdx.x : xcd_remap(blockIdx.x, gridDim.x);
  const int sp = id / g.tiles, bt = blockIdx.y, t = id - sp * g.tiles;
  int64_t m0, n0;
  if (!wave_tile<U>(g, t, wave, &m0, &n0)) return;
  int64_t klim = g.K;
  if (g.a_lower) klim = min(klim, m0 + U);
  if (g.b_upper) klim = min(klim, n0 + U);
  const int64_t kbeg = (int64_t)sp * g.kchunk;
  doublex4 cr[F][F], ci[F][F];
  accumulate<REAL, TA, TBT, F>(g, bt, m0, n0, kbeg, min(klim, kbeg + g.kchunk), cr, ci);

  double* w = g.splits > 1 ? reinterpret_cast<double*>(g.ws + (((int64_t)sp * gridDim.y + bt) * g.tiles + t) * RT * RT) +
                                 wave * (F * F * 512)
                           : nullptr;
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) {
      const doublex4 vr = g.ar * cr[i][j] - g.ai * ci[i][j], vi = g.ar * ci[i][j] + g.ai * cr[i][j];
      if (w) {
        doublex2* p = reinterpret_cast<doublex2*>(w + (i * F + j) * 512) + lane;
        p[0] = doublex2{vr[0], vr[1]};
        p[64] = doublex2{vr[2], vr[3]};
        p[128] = doublex2{vi[0], vi[1]};
        p[192] = doublex2{vi[2], vi[3]};
      } else {
        put4(g, bt, m0 + 16 * i + 4 * (lane >> 4), n0 + 16 * j + (lane & 15), vr, vi);
      }
    }
}

// Small products: a workgroup of NW waves takes 16 F x 16 F outputs, every wave
// a share of K, and adds the waves' sums in LDS in K order.  Bound by the
// latency of a slab's loads; one launch, no partial sums in memory.
template <bool REAL, int TA, int TBT, int F, int NW>
__global__ __launch_bounds__(64 * NW) void zgemm_short_kernel(const ZgemmDev g) {
  constexpr int PARTS = REAL ? 1 : 2;
  __shared__ double red[NW][F * F][PARTS][4][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bt = blockIdx.y, ti = blockIdx.x / g.TN;
  const int64_t m0 = (int64_t)ti * 16 * F, n0 = ((int64_t)blockIdx.x - (int64_t)ti * g.TN) * 16 * F;
  if (g.lower_only && m0 + 16 * F <= n0) return;  // strictly above the diagonal
  int64_t klim = g.K;
  if (g.a_lower) klim = min(klim, m0 + 16 * F);
  if (g.b_upper) klim = min(klim, n0 + 16 * F);
  const int64_t S = (klim + RK - 1) / RK;
  doublex4 cr[F][F], ci[F][F];
  accumulate<REAL, TA, TBT, F>(g, bt, m0, n0, S * wave / NW * RK, min(klim, S * (wave + 1) / NW * RK), cr, ci);
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        red[wave][i * F + j][0][r][lane] = cr[i][j][r];
        if constexpr (!REAL) red[wave][i * F + j][PARTS - 1][r][lane] = ci[i][j][r];
      }
  __syncthreads();
#pragma unroll 1
  for (int e = wave; e < F * F * 4; e += NW) {
    const int f = e >> 2, r = e & 3;
    double xr = 0, xi = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      xr += red[w][f][0][r][lane];
      if constexpr (!REAL) xi += red[w][f][PARTS - 1][r][lane];
    }
    const int64_t gi = m0 + 16 * (f / F) + 4 * (lane >> 4) + r, gj = n0 + 16 * (f % F) + (lane & 15);
    if (gi >= g.M || gj >= g.N) continue;
    c128* Cp = g.C + (int64_t)bt * g.strideC + gj * g.ldc + gi;
    double outr = g.ar * xr - g.ai * xi, outi = g.ar * xi + g.ai * xr;
    if (g.br != 0.0 || g.bi != 0.0) {
      const c128 c = *Cp;
      outr += g.br * c.re - g.bi * c.im;
      outi += g.br * c.im + g.bi * c.re;
    }
    *Cp = c128{outr, outi};
  }
}

// Sums the K splits of tile blockIdx.x in order; fragment blockIdx.z of each
// wave.
template <int F>
__global__ __launch_bounds__(NT) void zgemm_reduce_kernel(const ZgemmDev g) {
  constexpr int U = 16 * F, RT = 2 * U;
  const int t = blockIdx.x, bt = blockIdx.y, f = blockIdx.z;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int64_t m0, n0;
  if (!wave_tile<U>(g, t, wave, &m0, &n0)) return;
  const doublex2* p = reinterpret_cast<const doublex2*>(g.ws + ((int64_t)bt * g.tiles + t) * RT * RT) +
                      (wave * F * F + f) * 256 + lane;
  const int64_t step = (int64_t)gridDim.y * g.tiles * RT * RT;
  doublex2 v[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
  int s = 0;
  for (; s + 4 <= g.splits; s += 4) {
    doublex2 u[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) u[q][r] = p[(s + q) * step + 64 * r];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] += u[q][r];
  }
  for (; s < g.splits; ++s)
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] += p[s * step + 64 * r];
  put4(g, bt, m0 + 16 * (f / F) + 4 * (lane >> 4), n0 + 16 * (f % F) + (lane & 15),
       doublex4{v[0][0], v[0][1], v[1][0], v[1][1]}, doublex4{v[2][0], v[2][1], v[3][0], v[3][1]});
}

template <bool REAL, int F>
void launch_large(const ZgemmDev& g, dim3 grid, hipStream_t s) {
  if (g.transA) {
    if (g.transB) hipLaunchKernelGGL((zgemm_kernel<REAL, 1, 1, F>), grid, dim3(NT), 0, s, g);
    else hipLaunchKernelGGL((zgemm_kernel<REAL, 1, 0, F>), grid, dim3(NT), 0, s, g);
  } else {
    if (g.transB) hipLaunchKernelGGL((zgemm_kernel<REAL, 0, 1, F>), grid, dim3(NT), 0, s, g);
    else hipLaunchKernelGGL((zgemm_kernel<REAL, 0, 0, F>), grid, dim3(NT), 0, s, g);
  }
}

template <int F, int NW>
void launch_short(ZgemmDev g, int batch, hipStream_t s) {
  g.TN = (int)ceil_div(g.N, (int64_t)(16 * F));
  const dim3 grid((unsigned)(ceil_div(g.M, (int64_t)(16 * F)) * g.TN), (unsigned)batch), block(64 * NW);
  auto go = [&](auto REAL, auto TA, auto TB) {
    hipLaunchKernelGGL((zgemm_short_kernel<decltype(REAL)::value != 0, decltype(TA)::value, decltype(TB)::value,
                                           F, NW>),
                       grid, block, 0, s, g);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  auto tb = [&](auto REAL, auto TA) { g.transB ? go(REAL, TA, I1{}) : go(REAL, TA, I0{}); };
  auto ta = [&](auto REAL) { g.transA ? tb(REAL, I1{}) : tb(REAL, I0{}); };
  g.real_data ? ta(I1{}) : ta(I0{});
}

}  // namespace

Err zgemm(const ZgemmArgs& a, void* ws, size_t ws_bytes, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0 || a.batch <= 0) return ok();
  ZgemmDev g;
  g.transA = a.transA; g.transB = a.transB;
  g.M = a.M; g.N = a.N; g.K = a.K;
  g.ar = a.alpha.re; g.ai = a.alpha.im; g.br = a.beta.re; g.bi = a.beta.im;
  g.A = a.A; g.lda = a.lda; g.strideA = a.strideA;
  g.B = a.B; g.ldb = a.ldb; g.strideB = a.strideB;
  g.C = a.C; g.ldc = a.ldc; g.strideC = a.strideC;
  g.kneg = a.kneg;
  g.lower_only = a.lower_only; g.a_lower = a.a_lower; g.b_upper = a.b_upper;
  g.real_data = a.real_data;
  // Small products in one launch of workgroups whose waves share K.  us, here
  // against tiles of 64 x 64 with split K (or, before, of 32 x 32 through LDS):
  // 64^3 3.8 / 7.4, 192^3 5.8 / 17.5, 384^3 17.0 / 24.0, 512^3 23.2 / 38.2,
  // 4000 x 260 x 260 57 / 71, 200 x 200 x 640 11.9 / 19.1; past the line
  // 576^3 45.9 / 44.0, 8000 x 200 x 200 75 / 66, 140 x 140 x 4000 58 / 40 (few
  // workgroups, each waiting for its loads).  32 x 32 outputs on eight waves
  // instead of 16 x 16 on four halve the loads where K gives every wave enough to
  // do: 448^3 20.5 / 25.4, 384^3 17.7 / 17.0.
  const double mnk = (double)a.M * a.N * a.K * a.batch;
  if (a.K <= 640 && mnk <= (a.K <= 512 ? 2.8e8 : 1e8)) {
    if (a.K >= 384 && mnk >= 8e7) launch_short<2, 8>(g, a.batch, s);
    else launch_short<1, 4>(g, a.batch, s);
    CHASE_LAUNCH_CHECK();
    return ok();
  }
  // Real data on 64 x 64 outputs a wave where these fill the chip: 400 workgroups
  // of them, or enough for K splits to (us, 32 x 32 / 64 x 64: 12000 x 640 x 640
  // upper 190 / 156, 8000 x 520 x 520 upper 103 / 131; 376 x 376 x 8000 lower
  // 88 / 79, 260 x 260 x 8000 lower 61 / 71).
  const double outputs = (double)a.M * a.N * (a.lower_only ? 0.5 : 1.0);
  const bool wide = a.real_data && (outputs >= 400.0 * 128 * 128 || (outputs >= 65536 && a.K >= 4096));
  const int64_t U = wide ? 64 : 32, RT = 2 * U;
  const bool col = a.b_upper && !a.lower_only, row = a.a_lower && !a.lower_only && !a.b_upper;
  g.TM = (int)ceil_div(a.M, col ? 4 * U : row ? U : RT);
  g.TN = (int)ceil_div(a.N, col ? U : row ? 4 * U : RT);
  const int64_t tu = ceil_div(a.M, U);
  g.tiles = a.lower_only ? (int)ceil_div(tu * (tu + 1) / 2, (int64_t)4) : g.TM * g.TN;
  // K splits while the tiles leave workgroup slots empty, at least 8 slabs
  // each: to two workgroups per CU, and two splits where that leaves one tile
  // on most CUs (three fit: 8000 x 188 x 376, 375 tiles: 113 us whole, 89 + 17
  // in two splits; 45 tiles of 520 x 520 x 8000: 200 us with 11 splits as with
  // 17)
  int64_t splits = 1;
  if (a.K > 0 && ws) {
    const int64_t n = (int64_t)g.tiles * a.batch;
    splits = std::max<int64_t>(1, n <= 256 ? 512 / n : 768 / n);
    splits = std::min(splits, std::max<int64_t>(1, a.K / (8 * RK)));
    splits = std::min(splits, std::max<int64_t>(1, (int64_t)(ws_bytes / (n * RT * RT * sizeof(c128)))));
  }
  g.kchunk = ceil_div(ceil_div(std::max<int64_t>(a.K, 1), splits), (int64_t)RK) * RK;
  g.splits = (int)ceil_div(std::max<int64_t>(a.K, 1), g.kchunk);
  g.ws = (c128*)ws;
  const dim3 grid((unsigned)((int64_t)g.tiles * g.splits), (unsigned)a.batch);
  if (wide) launch_large<true, 4>(g, grid, s);
  else if (a.real_data) launch_large<true, 2>(g, grid, s);
  else launch_large<false, 2>(g, grid, s);
  CHASE_LAUNCH_CHECK();
  if (g.splits > 1) {
    const dim3 rgrid((unsigned)g.tiles, (unsigned)a.batch, wide ? 16 : 4);
    if (wide) hipLaunchKernelGGL(zgemm_reduce_kernel<4>, rgrid, dim3(NT), 0, s, g);
    else hipLaunchKernelGGL(zgemm_reduce_kernel<2>, rgrid, dim3(NT), 0, s, g);
    CHASE_LAUNCH_CHECK();
  }
  return ok();
}

}  // namespace chase
