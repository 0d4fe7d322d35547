// Cholesky factorisation M = L L^H of a padded kp x kp Hermitian matrix
// (kp a multiple of 64, leading dimension kp, lower triangle given) together
// with L^{-1}, 64 columns at a time (Section 2: Cholesky QR; Alg. 2: POTRF and
// the triangular solves, as products with L^{-1}).
//
// Right-looking on the augmented matrix [M | I]: after block column b,
//   A_ij -= L_ib L_jb^H  (i >= j > b),   R_ij -= L_ib X_bj  (i > b >= j),
// with X_b = L_bb^{-1} R_b the finished rows of L^{-1}; R starts at zero and
// lives where X goes.  Two launches per block column:
//   panel:  every workgroup factors the 64 x 64 diagonal block for itself and
//           takes 16 rows of L_ib = A_ib L_bb^{-H} or 16 columns of X_b;
//   update: one 16 x 16 tile of A or R per wave, K = 64.
// The chain of 64 dependent column steps bounds the whole.  It runs in four
// panels of 16 rows held in registers, a lane per column and the multipliers
// read from lanes, without LDS or barriers (4.3 us each); the 16 x 16 blocks
// below are updated on the MFMA, those the next panel does not need by other
// waves meanwhile.  A panel launch takes 28 us and an update 6 us; before, with
// a barrier and LDS broadcasts per column step, the block alone took 42 us,
// and copies, panel products, trailing updates and the inverse's block
// diagonals, in launches of their own, another 45 us per block column.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "dense.h"

namespace chase {
namespace {

constexpr int NB = 64;    // block column
constexpr int PB = 16;    // rows eliminated in registers at a time
constexpr int NT = 256;
constexpr int NTP = 512;  // panel kernel

// A non-positive or non-finite pivot is replaced by 1 so that the block stays
// finite (it is flagged, and the result discarded).
__device__ __forceinline__ double pivot(double d) { return d > 0.0 && isfinite(d) ? d : 1.0; }

// The value of lane l, uniform.
__device__ __forceinline__ double lane_value(double x, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(x), l);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ doublex4 mfma64(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

struct Shared {
  c128 S[NB][NB + 1];      // above and on the diagonal blocks: U = D L'^H; below: L'^{-1} (L' unit lower)
  c128 D[4][PB][PB + 1];   // diagonal blocks of L'^{-1}
  double d[NB], id[NB], rs[NB];  // pivots, 1 / d, 1 / sqrt(d)
};

// Elimination of rows 16 kb .. + 15 of [A | I] on one wave, lane = column: the
// diagonal block in lanes 0 .. 15 and, in the others, 48 (w = 0) or 16 (w = 1)
// of the 64 further columns: 16 (kb + 1) .. 63 of A, then 0 .. 16 kb + 15 of I.
// Row j is in x[j]; a step subtracts conj(U[j][i]) / d_j times row j from row
// i, the multiplier a uniform value read from lane i.
__device__ __forceinline__ void panel_rows(Shared& sh, int kb, int w) {
  const int lane = threadIdx.x & 63, p = PB * kb, na = 48 - p;
  const bool diag = lane < PB;
  const int o = 48 * w + lane - PB;
  const bool apart = !diag && o < na;
  // column of A, or of I (lanes past the last one repeat column 0 of the block
  // row and are not stored)
  const int col = diag ? p + lane : apart ? p + PB + o : o < NB ? o - na : 0;
  const bool own = !diag && !apart && o < NB && col >= p;  // identity column of this block
  c128 x[PB];
#pragma unroll
  for (int r = 0; r < PB; ++r) {
    // below the diagonal of the diagonal block: the conjugate of its mirror
    const bool mirror = diag && r > lane;
    c128 v = sh.S[p + (mirror ? lane : r)][mirror ? p + r : col];
    if (mirror) v.im = -v.im;
    if (own) v = c128{r == col - p ? 1.0 : 0.0, 0.0};
    x[r] = v;
  }
  __syncthreads();  // both waves have read the diagonal block
  double dv = 1.0;  // lane j: pivot j
#pragma unroll
  for (int j = 0; j < PB; ++j) {
    const double draw = lane_value(x[j].re, j);
    dv = lane == j ? draw : dv;
    const double inv = rcp_nr(pivot(draw));
    const double tr = x[j].re * inv, ti = x[j].im * inv;
#pragma unroll
    for (int i = j + 1; i < PB; ++i) {
      const double sr = lane_value(x[j].re, i), si = lane_value(x[j].im, i);  // U[j][i]; conj(s) t
      x[i].re = fma(-sr, tr, fma(-si, ti, x[i].re));
      x[i].im = fma(-sr, ti, fma(si, tr, x[i].im));
    }
  }
  if (diag ? w == 0 : o < NB) {
    c128* dst = own ? &sh.D[kb][0][col - p] : &sh.S[p][col];
    const int step = own ? PB + 1 : NB + 1;
#pragma unroll
    for (int r = 0; r < PB; ++r) dst[r * step] = x[r];
  }
  if (diag && w == 0) {
    const double d = pivot(dv);
    sh.d[p + lane] = dv;
    sh.id[p + lane] = rcp_nr(d);
    sh.rs[p + lane] = rsqrt_nr(d);
  }
}

// Block (ib, jb) of the rows below panel kb: minus conj(U)^T D^{-1} (rows of
// the panel), K = 16; jb > kb a block of A, else of I.
__device__ __forceinline__ void update_block(Shared& sh, int kb, int ib, int jb) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const int p = PB * kb;
  doublex4 cr, ci;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const c128 c = sh.S[PB * ib + lk + 4 * r][PB * jb + lr];
    cr[r] = c.re;
    ci[r] = c.im;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int k = 4 * q + lk;
    const c128 a = sh.S[p + k][PB * ib + lr];
    const c128 b = jb == kb ? sh.D[kb][k][lr] : sh.S[p + k][PB * jb + lr];
    const double s = -sh.id[p + k];
    const double ar = s * a.re, ai = s * a.im;
    cr = mfma64(ar, b.re, cr);
    ci = mfma64(ar, b.im, ci);
    cr = mfma64(ai, b.im, cr);
    ci = mfma64(-ai, b.re, ci);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) sh.S[PB * ib + lk + 4 * r][PB * jb + lr] = c128{cr[r], ci[r]};
}

// Factors the 64 x 64 block at column p of M: afterwards S holds, below and on
// the diagonal, L^{-1} and, above it, U.
__device__ __forceinline__ void factor64(Shared& sh, const c128* M, int64_t ld, int p) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int PER = NB * NB / NTP;
  c128 v[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int t = threadIdx.x + e * NTP;
    v[e] = M[(int64_t)(p + t / NB) * ld + p + t % NB];
  }
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int t = threadIdx.x + e * NTP, j = t / NB, i = t % NB;
    // A[j][i] = conj(A[i][j]); zero below the diagonal
    sh.S[j][i] = i >= j ? c128{v[e].re, -v[e].im} : c128{0.0, 0.0};
  }
  for (int t = threadIdx.x; t < NB * PB; t += NTP) sh.D[t / (PB * PB)][(t / PB) % PB][t % PB] = c128{0.0, 0.0};
  __syncthreads();
  for (int kb = 0; kb < 4; ++kb) {
    if (wave < 2) {
      panel_rows(sh, kb, wave);
    } else {
      __syncthreads();  // the one in panel_rows
      // meanwhile the rest of the previous panel's update: the blocks below row kb
      int n = 2;
      for (int ib = kb + 1; kb > 0 && ib < 4; ++ib) {
        for (int jb = 0; jb < kb; ++jb)
          if (n++ == wave) update_block(sh, kb - 1, ib, jb);
        for (int jb = ib; jb < 4; ++jb)
          if (n++ == wave) update_block(sh, kb - 1, ib, jb);
      }
    }
    __syncthreads();
    // the four blocks of the next panel's rows, one per wave
    if (kb < 3 && wave < 4) update_block(sh, kb, kb + 1, wave);
    __syncthreads();
  }
  // L^{-1} = diag(1 / sqrt(d)) L'^{-1} in place of L'^{-1}, diagonal blocks included
  for (int t = threadIdx.x; t < NB * NB; t += NTP) {
    const int i = t / NB, k = t % NB;
    if (k > i) continue;
    const c128 x = i / PB == k / PB ? sh.D[i / PB][i % PB][k % PB] : sh.S[i][k];
    sh.S[i][k] = c128{sh.rs[i] * x.re, sh.rs[i] * x.im};
  }
  __syncthreads();
}

// Workgroup 0: writes L_bb to Ldiag (64 x 64 blocks, ld 64) and L_bb^{-1} to X.
// Then 16 rows of the blocks of M below column block p each, L = A L_bb^{-H}
// (nrow workgroups), and 16 columns each of row block p of X left of it,
// X_b = L_bb^{-1} R_b.
__global__ __launch_bounds__(NTP) void chol_panel_kernel(c128* M, c128* X, int64_t ld, int p, int nrow, c128* Ldiag,
                                                         int* fail) {
  __shared__ Shared sh;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int wg = (int)blockIdx.x - 1;
  // one 16 x 16 tile on each of the first four waves, K = 64: the operand
  // from memory is loaded before the factorisation
  const bool rows = wg < nrow;
  const int64_t row = p + NB + PB * (int64_t)wg, col = PB * (int64_t)(wg - nrow) + lr;
  c128 a[16];
  if (wg >= 0 && wave < 4) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int k = 4 * q + lk;
      a[q] = rows ? M[(int64_t)(p + k) * ld + row + lr] : X[col * ld + p + k];
    }
  }
  factor64(sh, M, ld, p);
  if (wg >= 0) {
    if (wave >= 4) return;
    // Linv[16 wave + lr][k], zero above the diagonal
    doublex4 cr{0, 0, 0, 0}, ci{0, 0, 0, 0};
    const double sg = rows ? -1.0 : 1.0;  // rows: A conj(Linv), columns: Linv R
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int k = 4 * q + lk;
      if (q < 4 * wave + 4) {
        c128 b = sh.S[PB * wave + lr][k];
        if (k > PB * wave + lr) b = c128{0.0, 0.0};
        b.im *= sg;
        // rows: a b; columns: b a (the MFMA's output rows are the A operand's)
        const double xr = rows ? a[q].re : b.re, xi = rows ? a[q].im : b.im;
        const double yr = rows ? b.re : a[q].re, yi = rows ? b.im : a[q].im;
        cr = mfma64(xr, yr, cr);
        ci = mfma64(xr, yi, ci);
        cr = mfma64(-xi, yi, cr);
        ci = mfma64(xi, yr, ci);
      }
    }
    // (every wave has read its operand before the barriers of factor64)
    c128* dst = rows ? M + (int64_t)(p + PB * wave + lr) * ld + row + lk : X + col * ld + p + PB * wave + lk;
#pragma unroll
    for (int r = 0; r < 4; ++r) dst[4 * r] = c128{cr[r], ci[r]};
    return;
  }
  for (int t = threadIdx.x; t < NB * NB; t += NTP) {
    const int j = t / NB, i = t % NB;
    c128 l{0.0, 0.0}, x{0.0, 0.0};
    if (i > j) {
      const c128 u = sh.S[j][i];
      l = c128{sh.rs[j] * u.re, -sh.rs[j] * u.im};
    } else if (i == j) {
      const bool ok = sh.d[j] > 0.0 && isfinite(sh.d[j]);
      l.re = ok ? sqrt(sh.d[j]) : 1.0;
      if (!ok) atomicOr(fail, 1);
    }
    if (i >= j) x = sh.S[i][j];
    Ldiag[(int64_t)j * NB + i] = l;
    X[(int64_t)(p + j) * ld + p + i] = x;
  }
}

// One 16 x 16 tile per wave of the rows below block column p: A_ij -= L_ib
// L_jb^H for the tiles j <= i right of it, then R_ij -= L_ib X_bj for the
// columns up to and with it.  nt: 16-row tiles below.
__global__ __launch_bounds__(NT) void chol_update_kernel(c128* M, c128* X, int64_t ld, int p, int nt) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int ntri = nt * (nt + 1) / 2, nc = p / PB + 4;  // columns of R in tiles
  int t = blockIdx.x * 4 + wave;
  if (t >= ntri + nt * nc) return;
  const int64_t q0 = p + NB;
  int I, J;
  const bool tri = t < ntri;
  if (tri) {
    int i = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (i * (i + 1) / 2 > t) --i;
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    I = i;
    J = t - i * (i + 1) / 2;
  } else {
    t -= ntri;
    I = t / nc;
    J = t - I * nc;
  }
  const int64_t row = q0 + PB * (int64_t)I;
  const c128* a0 = M + (int64_t)p * ld + row + lr;
  c128* C = tri ? M + (q0 + PB * (int64_t)J + lr) * ld + row + lk : X + (PB * (int64_t)J + lr) * ld + row + lk;
  const c128* b0 = tri ? M + (int64_t)p * ld + q0 + PB * (int64_t)J + lr : X + (PB * (int64_t)J + lr) * ld + p;
  const int64_t bs = tri ? ld : 1;
  c128 a[16], b[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    a[q] = a0[(int64_t)(4 * q + lk) * ld];
    b[q] = b0[(int64_t)(4 * q + lk) * bs];
  }
  doublex4 cr, ci;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const c128 c = C[4 * r];
    cr[r] = c.re;
    ci[r] = c.im;
  }
  const double sg = tri ? -1.0 : 1.0;  // conj(L_jb)
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const double bi = sg * b[q].im;
    cr = mfma64(-a[q].re, b[q].re, cr);
    ci = mfma64(-a[q].re, bi, ci);
    cr = mfma64(a[q].im, bi, cr);
    ci = mfma64(-a[q].im, b[q].re, ci);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) C[4 * r] = c128{cr[r], ci[r]};
}

// The diagonal blocks of L from Ldiag, zeros above them.
__global__ __launch_bounds__(NT) void chol_finish_kernel(c128* M, int64_t ld, int kp, const c128* Ldiag) {
  const int64_t total = (int64_t)kp * kp;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int j = (int)(t / kp), i = (int)(t % kp);
    if (i / NB == j / NB)
      M[(int64_t)j * ld + i] = Ldiag[((int64_t)j) * NB + i % NB];
    else if (i < j)
      M[(int64_t)j * ld + i] = c128{0.0, 0.0};
  }
}

}  // namespace

Err cholesky_inverse(c128* M, c128* X, int kp, DenseWs& ws, hipStream_t s, int slot) {
  CHASE_TRY(fill_padded(X, kp, kp, 0.0, 0.0, true, s, ws.flag + slot));
  for (int p = 0; p < kp; p += NB) {
    const int rest = kp - p - NB;
    const int nrow = rest / PB, ncol = p / PB;
    hipLaunchKernelGGL(chol_panel_kernel, dim3((unsigned)(1 + nrow + ncol)), dim3(NTP), 0, s, M, X, (int64_t)kp, p,
                       nrow, ws.panel + (int64_t)p * NB, ws.flag + slot);
    CHASE_LAUNCH_CHECK();
    if (rest <= 0) break;
    const int tiles = nrow * (nrow + 1) / 2 + nrow * (ncol + 4);
    hipLaunchKernelGGL(chol_update_kernel, dim3((unsigned)ceil_div(tiles, 4)), dim3(NT), 0, s, M, X, (int64_t)kp, p,
                       nrow);
    CHASE_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(chol_finish_kernel, dim3((unsigned)std::min<int64_t>(ceil_div((int64_t)kp * kp, NT), 2048)),
                     dim3(NT), 0, s, M, (int64_t)kp, kp, (const c128*)ws.panel);
  CHASE_LAUNCH_CHECK();
  return ok();
}

}  // namespace chase
