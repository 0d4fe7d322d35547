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
// Two kernels.  Large products run without LDS and barriers: the FP64 MFMA
// takes 64 cycles, so a wave of 32 x 32 outputs loads its fragments straight
// into registers (8 16-byte loads per lane and slab of 8 k for 32 MFMAs,
// 2048 cycles), one slab ahead.  Small ones (few tiles, K <= 256) are bound
// by latency and run on 32 x 32 tiles of a workgroup, staged through LDS.
#include "common.h"

namespace chase {
namespace {

constexpr int BK = 16, NT = 256;  // small products: K slab
constexpr int RK = 8;             // large products: K slab
constexpr int RT = 64;            // and RT x RT outputs of a workgroup, 32 x 32 a wave

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
  c128* ws;        // split-K partials: one RT x RT tile per (split, batch, tile)
};

// Small products: 32 x 32 output tiles, a 16 x 16 MFMA tile per wave.
template <bool REAL>
__global__ __launch_bounds__(NT) void zgemm_small_kernel(const ZgemmDev g) {
  constexpr int TB = 32, BM = TB, BN = TB, FR = TB / 32;
  constexpr int LDS_A = BM + 2, LDS_B = BN + 2;
  __shared__ double As[2][2][BK][LDS_A];
  __shared__ double Bs[2][2][BK][LDS_B];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int TN = (int)((g.N + BN - 1) / BN);
  const int64_t m0 = (int64_t)(blockIdx.x / TN) * BM;
  const int64_t n0 = (int64_t)(blockIdx.x % TN) * BN;
  const int bt = blockIdx.y;
  if (g.lower_only && m0 + BM <= n0) return;  // strictly above the diagonal
  const c128* A = g.A + (int64_t)bt * g.strideA;
  const c128* B = g.B + (int64_t)bt * g.strideB;
  // triangular operands: products with k beyond the last row of this tile
  // (lower op(A)) or the last column (upper op(B)) vanish
  int64_t klim = g.K;
  if (g.a_lower) klim = min(klim, m0 + BM);
  if (g.b_upper) klim = min(klim, n0 + BN);
  const int64_t kbeg = 0, kend = klim;
  const int KT = (int)((kend - kbeg + BK - 1) / BK);
  const int wm0 = (wave >> 1) * (TB / 2), wn0 = (wave & 1) * (TB / 2);

  constexpr int PER = BM * BK / NT;  // elements of each operand per thread
  // raw loads (clamped addresses) plus validity bits; conj / sign are applied
  // when the tile is written to LDS, after the MFMAs of the previous slab
  doublex2 ra[PER], rb[PER];
  unsigned okA = 0, okB = 0, negB = 0;

  auto load = [&](int kt) {
    const int64_t k0 = kbeg + (int64_t)kt * BK;
    okA = okB = negB = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int el = tid + e * NT;
      int i, kk;
      if (g.transA == 0) { kk = el / BM; i = el % BM; } else { i = el / BK; kk = el % BK; }
      const int64_t gi = m0 + i, gk = k0 + kk;
      const bool ok = gi < g.M && gk < kend;
      const int64_t idx = ok ? (g.transA == 0 ? gk * g.lda + gi : gi * g.lda + gk) : 0;
      ra[e] = *reinterpret_cast<const doublex2*>(A + idx);
      if (ok) okA |= 1u << e;
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int el = tid + e * NT;
      int j, kk;
      if (g.transB == 0) { j = el / BK; kk = el % BK; } else { kk = el / BN; j = el % BN; }
      const int64_t gj = n0 + j, gk = k0 + kk;
      const bool ok = gj < g.N && gk < kend;
      const int64_t idx = ok ? (g.transB == 0 ? gj * g.ldb + gk : gk * g.ldb + gj) : 0;
      rb[e] = *reinterpret_cast<const doublex2*>(B + idx);
      if (ok) okB |= 1u << e;
      if (gk >= g.kneg) negB |= 1u << e;
    }
  };
  auto store = [&](int buf) {
    const double ca = g.transA ? -1.0 : 1.0, cb = g.transB ? -1.0 : 1.0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int el = tid + e * NT;
      int i, kk;
      if (g.transA == 0) { kk = el / BM; i = el % BM; } else { i = el / BK; kk = el % BK; }
      const bool ok = (okA >> e) & 1u;
      As[buf][0][kk][i] = ok ? ra[e][0] : 0.0;
      As[buf][1][kk][i] = ok ? ra[e][1] * ca : 0.0;
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int el = tid + e * NT;
      int j, kk;
      if (g.transB == 0) { j = el / BK; kk = el % BK; } else { kk = el / BN; j = el % BN; }
      const bool ok = (okB >> e) & 1u;
      const double sg = ((negB >> e) & 1u) ? -1.0 : 1.0;
      Bs[buf][0][kk][j] = ok ? rb[e][0] * sg : 0.0;
      Bs[buf][1][kk][j] = ok ? rb[e][1] * cb * sg : 0.0;
    }
  };

  doublex4 cr[FR][FR], ci[FR][FR];
#pragma unroll
  for (int i = 0; i < FR; ++i)
#pragma unroll
    for (int j = 0; j < FR; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) { cr[i][j][r] = 0; ci[i][j][r] = 0; }

  if (KT > 0) {
    load(0);
    store(0);
  }
  __syncthreads();
  const int lr = lane & 15, lk = lane >> 4;
  for (int kt = 0; kt < KT; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < KT) load(kt + 1);
#pragma unroll
    for (int ks = 0; ks < BK; ks += 4) {
      double fa_r[FR], fa_i[FR], fb_r[FR], fb_i[FR], fb_n[FR];
#pragma unroll
      for (int i = 0; i < FR; ++i) {
        fa_r[i] = As[buf][0][ks + lk][wm0 + 16 * i + lr];
        fa_i[i] = As[buf][1][ks + lk][wm0 + 16 * i + lr];
      }
#pragma unroll
      for (int j = 0; j < FR; ++j) {
        fb_r[j] = Bs[buf][0][ks + lk][wn0 + 16 * j + lr];
        fb_i[j] = Bs[buf][1][ks + lk][wn0 + 16 * j + lr];
        fb_n[j] = -fb_i[j];
      }
      if constexpr (REAL) {
#pragma unroll
        for (int i = 0; i < FR; ++i)
#pragma unroll
          for (int j = 0; j < FR; ++j) cr[i][j] = mfma64(fa_r[i], fb_r[j], cr[i][j]);
      } else {
#pragma unroll
        for (int i = 0; i < FR; ++i)
#pragma unroll
          for (int j = 0; j < FR; ++j) {
            cr[i][j] = mfma64(fa_r[i], fb_r[j], cr[i][j]);
            ci[i][j] = mfma64(fa_r[i], fb_i[j], ci[i][j]);
          }
#pragma unroll
        for (int i = 0; i < FR; ++i)
#pragma unroll
          for (int j = 0; j < FR; ++j) {
            cr[i][j] = mfma64(fa_i[i], fb_n[j], cr[i][j]);
            ci[i][j] = mfma64(fa_i[i], fb_r[j], ci[i][j]);
          }
      }
    }
    if (kt + 1 < KT) store(buf ^ 1);
    __syncthreads();
  }

#pragma unroll
  for (int i = 0; i < FR; ++i)
#pragma unroll
    for (int j = 0; j < FR; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gi = m0 + wm0 + 16 * i + (lane >> 4) + 4 * r;
        const int64_t gj = n0 + wn0 + 16 * j + (lane & 15);
        if (gi < g.M && gj < g.N) {
          const double xr = cr[i][j][r], xi = ci[i][j][r];
          const double yr = g.ar * xr - g.ai * xi, yi = g.ar * xi + g.ai * xr;
          c128* Cp = g.C + (int64_t)bt * g.strideC + gj * g.ldc + gi;
          double outr = yr, outi = yi;
          if (g.br != 0.0 || g.bi != 0.0) {
            c128 c = *Cp;
            outr += g.br * c.re - g.bi * c.im;
            outi += g.br * c.im + g.bi * c.re;
          }
          *Cp = c128{outr, outi};
        }
      }
}

// Large products.  Lane l of a fragment of 16 rows (columns) and 8 k holds row
// l % 16 at k = 2 (l / 16) + s, s = 0, 1: two loads of one c128, 128 contiguous
// bytes per row where k runs along memory, 256 per k where the rows do.
__device__ __forceinline__ int xcd_remap(int w, int T) {
  // workgroup w runs on XCD w % 8: give each XCD a contiguous range, so that
  // the tiles of a strip and of a K range stay in one L2
  const int xcd = w & 7, slot = w >> 3;
  const int q = T >> 3, r = T & 7;
  return xcd * q + (xcd < r ? xcd : r) + slot;
}

// First row and column of a wave's 32 x 32 outputs in workgroup tile t, false
// if it has none.  lower_only: the tiles of the lower triangle row by row, four
// neighbours a workgroup (no wave above the diagonal).  With a triangular
// operand the four waves have the same K range, 128 rows of a column (b_upper)
// or 128 columns of a row (a_lower), the longest ranges first.  Else 2 x 2.
// 8000 x 520 x 520 upper: 270 us strip by strip, 198 us longest first in 64 x 64 tiles, 183 so;
// 520 x 520 x 8000 lower: 200 us on 2 x 2, 171 so.
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
  *m0 = 32 * (int64_t)i;
  *n0 = 32 * (int64_t)j;
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

template <bool REAL, int TA, int TBT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 3))) void zgemm_kernel(const ZgemmDev g) {
  constexpr int F = 2;  // fragments per wave and operand
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int id = g.b_upper || g.a_lower ? blockIdx.x : xcd_remap(blockIdx.x, gridDim.x);
  const int sp = id / g.tiles, bt = blockIdx.y, t = id - sp * g.tiles;
  int64_t m0, n0;
  if (!wave_tile(g, t, wave, &m0, &n0)) return;
  const c128* A = g.A + (int64_t)bt * g.strideA;
  const c128* B = g.B + (int64_t)bt * g.strideB;
  int64_t klim = g.K;
  if (g.a_lower) klim = min(klim, m0 + 32);
  if (g.b_upper) klim = min(klim, n0 + 32);
  const int64_t kbeg = (int64_t)sp * g.kchunk;
  const int64_t kend = min(klim, kbeg + g.kchunk);
  const int lk = 2 * (lane >> 4);

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
  doublex2 fa[2][F][2], fb[2][F][2];
  doublex4 cr[F][F], ci[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) cr[i][j] = ci[i][j] = doublex4{0, 0, 0, 0};

  auto load = [&](int64_t k, doublex2 (&xa)[F][2], doublex2 (&xb)[F][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        xa[i][s] = pa[i][(k + s) * ka];
        xb[i][s] = pb[i][(k + s) * kb];
      }
  };
  auto load_tail = [&](int64_t k, doublex2 (&xa)[F][2], doublex2 (&xb)[F][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const bool ok = k + lk + s < kend;
        const int64_t q = ok ? k + s : -lk;  // k = 0 of the operand where past the end
        const doublex2 va = pa[i][q * ka], vb = pb[i][q * kb];
        xa[i][s] = ok ? va : doublex2{0, 0};
        xb[i][s] = ok ? vb : doublex2{0, 0};
      }
  };
  auto mul = [&](int64_t k, const doublex2 (&xa)[F][2], const doublex2 (&xb)[F][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const unsigned neg = k + lk + s >= g.kneg ? 0x80000000u : 0u;
      double ar[F], ai[F], an[F], br[F], bi[F];
#pragma unroll
      for (int i = 0; i < F; ++i) {
        ar[i] = xa[i][s][0];
        ai[i] = flip(xa[i][s][1], TA ? 0x80000000u : 0u);
        an[i] = flip(xa[i][s][1], TA ? 0u : 0x80000000u);
        br[i] = flip(xb[i][s][0], neg);
        bi[i] = flip(xb[i][s][1], TBT ? neg ^ 0x80000000u : neg);
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

// Sums the K splits of tile blockIdx.x in order; fragment blockIdx.z of each
// wave.
__global__ __launch_bounds__(NT) void zgemm_reduce_kernel(const ZgemmDev g) {
  const int t = blockIdx.x, bt = blockIdx.y, f = blockIdx.z;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int64_t m0, n0;
  if (!wave_tile(g, t, wave, &m0, &n0)) return;
  const doublex2* p = reinterpret_cast<const doublex2*>(g.ws + ((int64_t)bt * g.tiles + t) * RT * RT) +
                      (wave * 4 + f) * 256 + lane;
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
  put4(g, bt, m0 + 16 * (f >> 1) + 4 * (lane >> 4), n0 + 16 * (f & 1) + (lane & 15),
       doublex4{v[0][0], v[0][1], v[1][0], v[1][1]}, doublex4{v[2][0], v[2][1], v[3][0], v[3][1]});
}

template <bool REAL>
void launch_large(const ZgemmDev& g, dim3 grid, hipStream_t s) {
  if (g.transA) {
    if (g.transB) hipLaunchKernelGGL((zgemm_kernel<REAL, 1, 1>), grid, dim3(NT), 0, s, g);
    else hipLaunchKernelGGL((zgemm_kernel<REAL, 1, 0>), grid, dim3(NT), 0, s, g);
  } else {
    if (g.transB) hipLaunchKernelGGL((zgemm_kernel<REAL, 0, 1>), grid, dim3(NT), 0, s, g);
    else hipLaunchKernelGGL((zgemm_kernel<REAL, 0, 0>), grid, dim3(NT), 0, s, g);
  }
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
  // 32 x 32 tiles when 64 x 64 ones would leave most CUs idle and K is too
  // short for a split: a 64 x 64 x 64 complex tile is about 7 us of one CU's
  // FP64 MFMA, a 32 x 32 one a quarter of that
  const int64_t t64 = ceil_div(a.M, (int64_t)64) * ceil_div(a.N, (int64_t)64) * a.batch;
  if (t64 < 128 && a.K <= 256) {
    const dim3 grid((unsigned)(ceil_div(a.M, (int64_t)32) * ceil_div(a.N, (int64_t)32)), (unsigned)a.batch);
    if (a.real_data) hipLaunchKernelGGL((zgemm_small_kernel<true>), grid, dim3(NT), 0, s, g);
    else hipLaunchKernelGGL((zgemm_small_kernel<false>), grid, dim3(NT), 0, s, g);
    CHASE_LAUNCH_CHECK();
    return ok();
  }
  const bool col = a.b_upper && !a.lower_only, row = a.a_lower && !a.lower_only && !a.b_upper;
  g.TM = (int)ceil_div(a.M, (int64_t)(col ? 128 : row ? 32 : RT));
  g.TN = (int)ceil_div(a.N, (int64_t)(col ? 32 : row ? 128 : RT));
  const int64_t t32 = ceil_div(a.M, (int64_t)32);
  g.tiles = a.lower_only ? (int)ceil_div(t32 * (t32 + 1) / 2, (int64_t)4) : g.TM * g.TN;
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
  if (a.real_data) launch_large<true>(g, grid, s);
  else launch_large<false>(g, grid, s);
  CHASE_LAUNCH_CHECK();
  if (g.splits > 1) {
    hipLaunchKernelGGL(zgemm_reduce_kernel, dim3((unsigned)g.tiles, (unsigned)a.batch, 4), dim3(NT), 0, s, g);
    CHASE_LAUNCH_CHECK();
  }
  return ok();
}

}  // namespace chase
