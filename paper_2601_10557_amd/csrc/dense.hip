// Small dense FP64 kernels of the QR and Rayleigh-Ritz steps (Section 2:
// Cholesky QR; Alg. 2: POTRF, TRSM, HEEVD).  All operate on k x k Hermitian
// or triangular matrices stored in a padded kp x kp buffer (kp a multiple of
// 64, leading dimension kp) so that every blocked step has uniform sizes:
//  * triangular inverse L^{-1}, by block diagonals of batched GEMMs;
//  * Hermitian eigensolver: block Jacobi with 16-column blocks; each pair of
//    blocks (a 32 x 32 subproblem) gets one cyclic Jacobi sweep in LDS and
//    the block rotations are applied to the matrix and the eigenvectors with
//    32 x 32 complex products.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "common.h"
#include "dense.h"

namespace chase {
namespace {

constexpr int NB = 64;   // panel / padding granularity
constexpr int JB = 16;   // Jacobi block (subproblem is 2*JB)
constexpr int SP = 2 * JB;

__device__ __forceinline__ c128 cmul(c128 a, c128 b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ __forceinline__ c128 cconj(c128 a) { return {a.re, -a.im}; }
__device__ __forceinline__ c128 cadd(c128 a, c128 b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ c128 csub(c128 a, c128 b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ c128 cscale(double s, c128 a) { return {s * a.re, s * a.im}; }
// r - a b as four fused multiply-adds
__device__ __forceinline__ c128 cfms(c128 r, c128 a, c128 b) {
  return {fma(-a.re, b.re, fma(a.im, b.im, r.re)), fma(-a.re, b.im, fma(-a.im, b.re, r.im))};
}

// ---------------------------------------------------------------- fills
__global__ void fill_diag_kernel(c128* M, int64_t ld, int kp, int k, double inner, double pad, int zero_all,
                                 int* clear, int nclear) {
  const int64_t total = (int64_t)kp * kp;
  if (blockIdx.x == 0 && (int)threadIdx.x < nclear) clear[threadIdx.x] = 0;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int j = (int)(t / kp), i = (int)(t % kp);
    c128* p = M + (int64_t)j * ld + i;
    if (i == j) {
      *p = c128{i < k ? inner : pad, 0.0};
    } else if (zero_all || i >= k || j >= k) {
      *p = c128{0.0, 0.0};
    }
  }
}

// --------------------------------------------- triangular inverse blocks
// Inverse of 64 x 64 triangular blocks, 256 threads.  Lane c of every wave
// holds column c, and wave w the 16 rows w, w + 4, ..., w + 60 in registers:
// interleaved, so that the four waves share the shrinking trailing part
// evenly.  A step publishes one row through LDS, on rotating buffers, so it
// takes one barrier, and every other operand is a broadcast LDS read.
constexpr int CT = 256;     // threads of the block kernel
constexpr int CW = NB / 4;  // rows per wave

// Lane exchange inside a row of 16 lanes by DPP (no LDS round trip).
template <int CTRL>
__device__ __forceinline__ double dpp_swap(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Lane l of each row of 16 lanes takes the value of lane (l + 1) mod 16
// (DPP row_ror:15).
__device__ __forceinline__ double row_next(double x) { return dpp_swap<0x12F>(x); }

// f(std::integral_constant<int, B>), ..., f(std::integral_constant<int, E - 1>)
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// X = L^{-1} by forward substitution on the 64 unit right-hand sides at
// once: thread (w, c) holds X[4 t + w][c] in b[t]; step k finishes row k
// (x_k = b_k / L[k][k]) on wave k mod 4, which publishes it, and every
// wave updates its rows r > k by b_r -= L[r][k] x_k.  L (lower) is read
// from S, its reciprocal diagonal from rpiv.
__device__ __forceinline__ void trinv64(const c128 (*S)[NB + 1], const double* rpiv, c128 (*xb)[NB],
                                        c128 (&b)[CW]) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int t = 0; t < CW; ++t) b[t] = (4 * t + w == lane) ? c128{1.0, 0.0} : c128{0.0, 0.0};
#pragma unroll
  for (int tk = 0; tk < CW; ++tk) {
#pragma unroll 1
    for (int wk = 0; wk < 4; ++wk) {
      const int k = 4 * tk + wk;
      c128* xr = xb[k & 1];
      if (w == wk) {
        b[tk] = cscale(rpiv[k], b[tk]);
        xr[lane] = b[tk];
      }
      __syncthreads();
      const c128 x = xr[lane];
      c128 l[CW];
#pragma unroll
      for (int t = tk; t < CW; ++t) l[t] = S[4 * t + w][k];
#pragma unroll
      for (int t = tk; t < CW; ++t)
        if (t > tk || w > wk) b[t] = cfms(b[t], l[t], x);
    }
  }
}

// Invert each 64 x 64 diagonal block of a lower-triangular L (padded) and
// write it into the diagonal of Linv.
__global__ __launch_bounds__(CT) void trinv_diag_kernel(const c128* L, c128* X, int64_t ld) {
  __shared__ c128 S[NB][NB + 1];
  __shared__ c128 xb[2][NB];
  __shared__ double rpiv[NB];
  const int p = blockIdx.x * NB;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int t = threadIdx.x; t < NB * NB; t += CT) {
    const int j = t / NB, i = t % NB;
    S[i][j] = L[(int64_t)(p + j) * ld + p + i];
  }
  __syncthreads();
  if (threadIdx.x < NB) rpiv[threadIdx.x] = 1.0 / S[threadIdx.x][threadIdx.x].re;
  __syncthreads();
  c128 b[CW];
  trinv64(S, rpiv, xb, b);
  __syncthreads();
  static_for<0, CW>([&](auto U) {
    constexpr int t = decltype(U)::value;
    S[4 * t + w][lane] = b[t];
  });
  __syncthreads();
  for (int t = threadIdx.x; t < NB * NB; t += CT) {
    const int j = t / NB, i = t % NB;
    X[(int64_t)(p + j) * ld + p + i] = (i >= j) ? S[i][j] : c128{0.0, 0.0};
  }
}

// ------------------------------------------------------------- Jacobi

// Rotation annihilating b in [[a, b], [conj(b), d]] (a, d real).  With
// x = d - a and the classical t = sign(tau) / (|tau| + sqrt(1 + tau^2)),
// tau = x / (2|b|) (Golub & Van Loan, symmetric Schur 2x2, conjugated by
// diag(1, e^{-i arg b})), write t = tp |b| with
//   tp = 2 sign(x) / (|x| + sqrt(x^2 + 4|b|^2)),
// so that c = 1 / sqrt(1 + tp^2 |b|^2), s = tp c b and the diagonal shift
// t |b| = tp |b|^2 need no |b| itself.  The square roots and the division
// use refined hardware estimates; the rotation stays unitary to rounding.
__device__ __forceinline__ void jacobi_rot(double a, double d, c128 b, double thr, double& c, c128& s, double& t_out, int& did) {
  const double nb2 = b.re * b.re + b.im * b.im;
  if (!(nb2 > thr * thr)) {
    c = 1.0; s = c128{0.0, 0.0}; t_out = 0.0; did = 0;
    return;
  }
  const double x = d - a;
  const double y = x * x + 4.0 * nb2;
  const double tp = (x >= 0.0 ? 2.0 : -2.0) * rcp_nr(fabs(x) + y * rsqrt_nr(y));
  c = rsqrt_nr(1.0 + tp * tp * nb2);
  s = c128{tp * c * b.re, tp * c * b.im};
  t_out = tp * nb2;
  did = 1;
}

// Round-robin pairing of n players (n even), round r: position i plays
// position n-1-i; position 0 is fixed, positions 1..n-1 rotate.
__device__ __forceinline__ int rr_player(int pos, int r, int n) {
  if (pos == 0) return 0;
  return ((pos - 1 + r) % (n - 1)) + 1;
}

// One Jacobi sweep on the 32 x 32 subproblem S[0] = [[G_pp, G_pq], [G_qp, G_qq]]
// of a pair of blocks, in steps of 16 disjoint rotations.
// Round 0 of an outer sweep holds every block of G in exactly one pair, so
// there the subproblem gets a full cyclic sweep (31 steps, round-robin
// pairing) and every index pair inside a block is rotated once; the later
// rounds (CROSS) rotate only the 256 index pairs across the two blocks
// (16 steps; step r pairs row i of block p with row (i + r) mod 16 of block
// q).  The outer sweep thus meets every index pair of G once, as a cyclic
// Jacobi sweep does.  Thread (a, b) = (tid % 16, tid / 16) owns the 2 x 2
// block of rotation a's rows and rotation b's columns and rows b, b + 16 of
// rotation a's two columns of the accumulated unitary.  Every lane computes
// rotation a = lane % 16 from the step's input matrix and takes rotation b
// from lane b of its own wave by a lane shuffle; the matrix is
// double-buffered in LDS, so a step needs one barrier.  The unitary takes a
// step's rotation one step late, while the next step's operands are read
// (round 0), or holds it in registers (the cross rounds, below).
// Writes U (32 x 32, column-major) to Uo and sets *flag when it rotated.  A
// subproblem whose off-diagonal entries are all at or below thr (not needed) is
// left alone (U = I is implied by *flag = 0).  U: LDS, the identity, only used
// in round 0.
template <bool CROSS>
__device__ __forceinline__ void jacobi_block(c128 (*S)[SP][SP + 1], c128 (*U)[SP + 1], double thr, bool needed, c128* Uo,
                                             int* flag) {
  const int tid = threadIdx.x;
  const int a = tid % (SP / 2), b = tid / (SP / 2);
  constexpr int nsteps = CROSS ? JB : SP - 1;
  // U <- U J on the columns (up, uq) of a rotation (c, s), rows b and b + 16
  auto rotate_u = [&](int up_col, int uq_col, double c, c128 sr) {
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int i = b + (SP / 2) * v;
      const c128 up = U[i][up_col], uq = U[i][uq_col];
      U[i][up_col] = csub(cscale(c, up), cmul(cconj(sr), uq));
      U[i][uq_col] = cadd(cmul(sr, up), cscale(c, uq));
    }
  };
  // In the cross rounds U stays in registers: thread (a, b) holds U[b][a]
  // and U[b + 16][a] (its rotation's fixed column) and U[b][q], U[b + 16][q]
  // for the step's partner column q = 16 + (a + r) mod 16, which passes one
  // lane down the row of 16 lanes (DPP row rotation) after each step; after
  // the 16 steps q is 16 + a again.
  c128 up0{a == b ? 1.0 : 0.0, 0.0}, up1{0.0, 0.0}, uq0{0.0, 0.0}, uq1{a == b ? 1.0 : 0.0, 0.0};
  int did_any = 0;
  if (needed) {
    int lp = 0, lq = 0;  // the previous step's rotation a, not yet applied to U
    double lc = 1.0;
    c128 ls{0.0, 0.0};
    for (int r = 0; r < nsteps; ++r) {
      const c128 (*cur)[SP + 1] = S[r & 1];
      c128 (*nxt)[SP + 1] = S[(r + 1) & 1];
      int pa, qa, pb, qb;
      if constexpr (CROSS) {
        pa = a;
        qa = JB + ((a + r) & (JB - 1));
        pb = b;
        qb = JB + ((b + r) & (JB - 1));
      } else {
        const int pa0 = rr_player(a, r, SP), qa0 = rr_player(SP - 1 - a, r, SP);
        const int pb0 = rr_player(b, r, SP), qb0 = rr_player(SP - 1 - b, r, SP);
        pa = min(pa0, qa0);
        qa = max(pa0, qa0);
        pb = min(pb0, qb0);
        qb = max(pb0, qb0);
      }
      const double app = cur[pa][pa].re, aqq = cur[qa][qa].re;
      const c128 apq = cur[pa][qa];
      const c128 x00 = cur[pa][pb], x01 = cur[pa][qb], x10 = cur[qa][pb], x11 = cur[qa][qb];
      if (!CROSS && r > 0) rotate_u(lp, lq, lc, ls);
      double ca, ta;
      c128 sa;
      int da;
      jacobi_rot(app, aqq, apq, thr, ca, sa, ta, da);
      did_any |= da;
      // rotation b was computed by lane b of this wave (lane % 16 == b)
      const double cb = __shfl(ca, b);
      const c128 sb{__shfl(sa.re, b), __shfl(sa.im, b)};
      // rows: row_p' = c row_p - s row_q ; row_q' = conj(s) row_p + c row_q
      const c128 y00 = csub(cscale(ca, x00), cmul(sa, x10));
      const c128 y01 = csub(cscale(ca, x01), cmul(sa, x11));
      const c128 y10 = cadd(cmul(cconj(sa), x00), cscale(ca, x10));
      const c128 y11 = cadd(cmul(cconj(sa), x01), cscale(ca, x11));
      // cols: col_p' = c col_p - conj(s) col_q ; col_q' = s col_p + c col_q
      c128 z00 = csub(cscale(cb, y00), cmul(cconj(sb), y01));
      c128 z01 = cadd(cmul(sb, y00), cscale(cb, y01));
      c128 z10 = csub(cscale(cb, y10), cmul(cconj(sb), y11));
      c128 z11 = cadd(cmul(sb, y10), cscale(cb, y11));
      if (a == b) {
        if (ta != 0.0) {
          z00 = c128{x00.re - ta, 0.0};
          z11 = c128{x11.re + ta, 0.0};
          z01 = c128{0.0, 0.0};
          z10 = c128{0.0, 0.0};
        } else {
          z00.im = 0.0;
          z11.im = 0.0;
        }
      }
      nxt[pa][pb] = z00;
      nxt[pa][qb] = z01;
      nxt[qa][pb] = z10;
      nxt[qa][qb] = z11;
      if constexpr (CROSS) {
        // U <- U J on columns a and q: col_a' = c col_a - conj(s) col_q,
        // col_q' = s col_a + c col_q; then q moves on (lane a takes lane a + 1's)
        const c128 n0 = csub(cscale(ca, up0), cmul(cconj(sa), uq0));
        const c128 m0 = cadd(cmul(sa, up0), cscale(ca, uq0));
        const c128 n1 = csub(cscale(ca, up1), cmul(cconj(sa), uq1));
        const c128 m1 = cadd(cmul(sa, up1), cscale(ca, uq1));
        up0 = n0;
        up1 = n1;
        uq0 = c128{row_next(m0.re), row_next(m0.im)};
        uq1 = c128{row_next(m1.re), row_next(m1.im)};
      }
      lp = pa;
      lq = qa;
      lc = ca;
      ls = sa;
      __syncthreads();
    }
    if (!CROSS) rotate_u(lp, lq, lc, ls);
  }
  const bool rotated = __syncthreads_or(did_any);
  if (tid == 0) *flag = rotated;
  if (!rotated) return;
  if constexpr (CROSS) {
    Uo[a * SP + b] = up0;
    Uo[a * SP + b + JB] = up1;
    Uo[(JB + a) * SP + b] = uq0;
    Uo[(JB + a) * SP + b + JB] = uq1;
  } else {
    for (int t = tid; t < SP * SP; t += 256) Uo[t] = U[t % SP][t / SP];
  }
}

// The rotations of round `round` from G as it is, workgroup = pair: round 0 of a
// sweep (CROSS false) or a later one.
template <bool CROSS>
__global__ __launch_bounds__(256) void jacobi_pairs_kernel(const c128* G, int64_t ld, int nbj, int round, c128* Uw,
                                                           double thr, int* pflag) {
  __shared__ c128 S[2][SP][SP + 1];
  __shared__ c128 U[CROSS ? 1 : SP][SP + 1];
  const int pair = blockIdx.x;
  const int bp = rr_player(pair, round, nbj), bq = rr_player(nbj - 1 - pair, round, nbj);
  const int P = min(bp, bq) * JB, Q = max(bp, bq) * JB;
  int big = 0;
  for (int t = threadIdx.x; t < SP * SP; t += 256) {
    const int j = t / SP, i = t % SP;
    const int gi = i < JB ? P + i : Q + i - JB;
    const int gj = j < JB ? P + j : Q + j - JB;
    const c128 g = G[(int64_t)gj * ld + gi];
    S[0][i][j] = g;
    if constexpr (!CROSS) U[i][j] = (i == j) ? c128{1.0, 0.0} : c128{0.0, 0.0};
    if (i != j && g.re * g.re + g.im * g.im > thr * thr) big = 1;
  }
  const bool needed = __syncthreads_or(big);
  jacobi_block<CROSS>(S, U, thr, needed, Uw + (int64_t)pair * SP * SP, pflag + pair);
}

// Index of row/col i (0..2*JB-1) of the subproblem of pair `pair` in round `round`.
__device__ __forceinline__ int sub_index(int pair, int round, int nbj, int i) {
  const int bp = rr_player(pair, round, nbj), bq = rr_player(nbj - 1 - pair, round, nbj);
  const int P = min(bp, bq) * JB, Q = max(bp, bq) * JB;
  return i < JB ? P + i : Q + i - JB;
}

// 16 x 16 output tile of a 32 x 32 complex product on the FP64 MFMA
// (v_mfma_f64_16x16x4f64; lane l holds A[l % 16][k0 + l / 16] and
// B[k0 + l / 16][l % 16]; accumulator r of lane l is row l / 16 + 4 r,
// column l % 16).  a(i, k) and b(k, j) fetch the complex operands; two
// accumulators per tile take Re = Ar Br - Ai Bi and Im = Ar Bi + Ai Br.
template <typename FA, typename FB>
__device__ __forceinline__ void cgemm_tile32(int lane, FA a, FB b, doublex4& cr, doublex4& ci) {
  cr = doublex4{0, 0, 0, 0};
  ci = doublex4{0, 0, 0, 0};
  const int li = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int k0 = 0; k0 < SP; k0 += 4) {
    const c128 x = a(li, k0 + lk);
    const c128 y = b(k0 + lk, li);
    cr = __builtin_amdgcn_mfma_f64_16x16x4f64(x.re, y.re, cr, 0, 0, 0);
    ci = __builtin_amdgcn_mfma_f64_16x16x4f64(x.re, y.im, ci, 0, 0, 0);
    cr = __builtin_amdgcn_mfma_f64_16x16x4f64(x.im, -y.im, cr, 0, 0, 0);
    ci = __builtin_amdgcn_mfma_f64_16x16x4f64(x.im, y.re, ci, 0, 0, 0);
  }
}

// The same tile, operands given: v[q], z[q] at k = 4 q + lane / 16.
__device__ __forceinline__ void cgemm_k32(const c128 (&v)[8], const c128 (&z)[8], doublex4& cr, doublex4& ci) {
  cr = doublex4{0, 0, 0, 0};
  ci = doublex4{0, 0, 0, 0};
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    cr = __builtin_amdgcn_mfma_f64_16x16x4f64(v[q].re, z[q].re, cr, 0, 0, 0);
    ci = __builtin_amdgcn_mfma_f64_16x16x4f64(v[q].re, z[q].im, ci, 0, 0, 0);
    cr = __builtin_amdgcn_mfma_f64_16x16x4f64(v[q].im, -z[q].im, cr, 0, 0, 0);
    ci = __builtin_amdgcn_mfma_f64_16x16x4f64(v[q].im, z[q].re, ci, 0, 0, 0);
  }
}

// The pair that block p plays in round r, and whether p is its upper half.
__device__ __forceinline__ int pair_of(int p, int r, int n, int* half) {
  const int pos = p == 0 ? 0 : (p - 1 - r + (n - 1)) % (n - 1) + 1;
  *half = p > rr_player(n - 1 - pos, r, n);
  return min(pos, n - 1 - pos);
}

// The rotations of pair `pair` of round `round` + 1 from G as it is before the
// rotations Uw of round `round`: the three 16 x 16 blocks of the subproblem are
// taken through those first (T = X U, S = U^H T, on the MFMA).
__device__ __forceinline__ void next_rotations(c128* lds, const c128* G, int64_t ld, int nbj, int round, int pair,
                                               const c128* Uw, const int* pflag, c128* Uo, int* flag, double thr) {
  c128 (*S)[SP][SP + 1] = reinterpret_cast<c128 (*)[SP][SP + 1]>(lds);
  c128 (*T)[SP][JB + 1] = reinterpret_cast<c128 (*)[SP][JB + 1]>(lds + 2 * SP * (SP + 1));
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int x = rr_player(pair, round + 1, nbj), y = rr_player(nbj - 1 - pair, round + 1, nbj);
  int hp, hq;
  const int a = pair_of(min(x, y), round, nbj, &hp), b = pair_of(max(x, y), round, nbj, &hq);
  // column 16 h + li of the rotation of pair c, row k
  auto u = [&](int c, int h, int k) __attribute__((always_inline)) {
    return pflag[c] ? Uw[(int64_t)c * SP * SP + (JB * h + li) * SP + k] : c128{k == JB * h + li ? 1.0 : 0.0, 0.0};
  };
  // T[0] = X_aa U_a, T[1] = X_bb U_b, T[2] = X_ab U_b: 16 columns each
  for (int t = wave; t < 6; t += 4) {
    const int w = t >> 1, row = w == 1 ? b : a, col = w == 0 ? a : b, h = w == 0 ? hp : hq;
    const int gi = sub_index(row, round, nbj, JB * (t & 1) + li);
    c128 v[8], z[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      v[q] = G[(int64_t)sub_index(col, round, nbj, 4 * q + lk) * ld + gi];
      z[q] = u(col, h, 4 * q + lk);
    }
    doublex4 cr, ci;
    cgemm_k32(v, z, cr, ci);
#pragma unroll
    for (int r = 0; r < 4; ++r) T[w][JB * (t & 1) + lk + 4 * r][li] = c128{cr[r], ci[r]};
  }
  __syncthreads();
  int big = 0;
  if (wave < 3) {  // blocks pp, qq, pq
    const int c = wave == 1 ? b : a, h = wave == 1 ? hq : hp;
    c128 v[8], z[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      v[q] = cconj(u(c, h, 4 * q + lk));
      z[q] = T[wave][4 * q + lk][li];
    }
    doublex4 cr, ci;
    cgemm_k32(v, z, cr, ci);
    const int i0 = wave == 1 ? JB : 0, j0 = wave == 0 ? 0 : JB;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + lk + 4 * r, j = j0 + li;
      const c128 g{cr[r], i == j ? 0.0 : ci[r]};
      S[0][i][j] = g;
      if (wave == 2) S[0][j][i] = cconj(g);
      if (i != j && g.re * g.re + g.im * g.im > thr * thr) big = 1;
    }
  }
  const bool needed = __syncthreads_or(big);
  jacobi_block<true>(S, nullptr, thr, needed, Uo, flag);
}

// Round `round`: Gn = J^H G J with J block-diagonal (one 32 x 32 U per pair, in
// the pair's index set); block (a, b) of pairs is U_a^H G_ab U_b.  G stays
// Hermitian, so only the blocks a <= b are formed and each is also written,
// conjugate transposed, to (b, a) (a diagonal block from its upper triangle).
// Also V <- V J on row chunks of 32.  The first nspec = npair workgroups
// compute the next round's rotations meanwhile (none in the last round); then
// npair (npair + 1) / 2 G blocks; the rest: V blocks.  The data block and the
// rotation blocks are staged in LDS; each of the four waves computes one
// 16 x 16 quarter of each 32 x 32 product on MFMA.  Bound by the chain of a
// round's rotations; kp = 384: 20.8 us a round, of which the 16 rotation steps take
// 10.4 (0.65 each), the two products before them 6, and launch, loads and stores
// the rest.  In launches of their own the rotations take 14.8 and the update 10.0.
__global__ __launch_bounds__(256) void jacobi_round_kernel(const c128* G, c128* Gn, c128* V, int64_t ld, int kp, int nbj,
                                                           int round, const c128* Uw, const int* pflag, c128* Un,
                                                           int* pflagn, double thr, int nspec) {
  __shared__ c128 lds[4 * SP * (SP + 1)];
  if ((int)blockIdx.x < nspec) {
    next_rotations(lds, G, ld, nbj, round, blockIdx.x, Uw, pflag, Un + (int64_t)blockIdx.x * SP * SP,
                   pflagn + blockIdx.x, thr);
    return;
  }
  c128 (*X)[SP + 1] = reinterpret_cast<c128 (*)[SP + 1]>(lds);
  c128 (*Y)[SP + 1] = X + SP, (*UA)[SP + 1] = X + 2 * SP, (*UB)[SP + 1] = X + 3 * SP;
  const int npair = nbj / 2;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r0 = (wave >> 1) * 16, c0 = (wave & 1) * 16;  // this wave's quarter
  int blk = blockIdx.x - nspec;
  doublex4 cr, ci;
  const int ntri = npair * (npair + 1) / 2;
  if (blk < ntri) {
    // blk -> (a, b), a <= b, row by row of the upper triangle
    int a = 0, rest = blk;
    while (rest >= npair - a) {
      rest -= npair - a;
      ++a;
    }
    const int b = a + rest;
    const bool ua = pflag[a], ub = pflag[b];
    if (Gn == G && !ua && !ub) return;  // in place: both rotations are the identity
    const c128* Ua = Uw + (int64_t)a * SP * SP;
    const c128* Ub = Uw + (int64_t)b * SP * SP;
    for (int t = tid; t < SP * SP; t += 256) {
      const int j = t / SP, i = t % SP;
      X[i][j] = G[(int64_t)sub_index(b, round, nbj, j) * ld + sub_index(a, round, nbj, i)];
      if (ua) UA[i][j] = Ua[t];
      if (ub) UB[i][j] = Ub[t];
    }
    __syncthreads();
    // Y = X Ub
    if (ub) {
      cgemm_tile32(lane, [&](int i, int k) { return X[r0 + i][k]; }, [&](int k, int j) { return UB[k][c0 + j]; },
                   cr, ci);
#pragma unroll
      for (int r = 0; r < 4; ++r) Y[r0 + (lane >> 4) + 4 * r][c0 + (lane & 15)] = c128{cr[r], ci[r]};
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = r0 + (lane >> 4) + 4 * r, j = c0 + (lane & 15);
        Y[i][j] = X[i][j];
      }
    }
    __syncthreads();
    // out = Ua^H Y
    if (ua) {
      cgemm_tile32(lane, [&](int i, int k) { return cconj(UA[k][r0 + i]); },
                   [&](int k, int j) { return Y[k][c0 + j]; }, cr, ci);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const c128 y = Y[r0 + (lane >> 4) + 4 * r][c0 + (lane & 15)];
        cr[r] = y.re;
        ci[r] = y.im;
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = r0 + (lane >> 4) + 4 * r, j = c0 + (lane & 15);
      const int gi = sub_index(a, round, nbj, i), gj = sub_index(b, round, nbj, j);
      if (a != b) {
        Gn[(int64_t)gj * ld + gi] = c128{cr[r], ci[r]};
        Gn[(int64_t)gi * ld + gj] = c128{cr[r], -ci[r]};
      } else if (i < j) {
        Gn[(int64_t)gj * ld + gi] = c128{cr[r], ci[r]};
        Gn[(int64_t)gi * ld + gj] = c128{cr[r], -ci[r]};
      } else if (i == j) {
        Gn[(int64_t)gj * ld + gi] = c128{cr[r], 0.0};
      }
    }
  } else {
    blk -= ntri;
    const int a = blk % npair, rb = blk / npair;  // pair, row chunk
    if (!pflag[a]) return;
    const c128* Ua = Uw + (int64_t)a * SP * SP;
    const int v0 = rb * SP;
    for (int t = tid; t < SP * SP; t += 256) {
      const int j = t / SP, i = t % SP;
      X[i][j] = V[(int64_t)sub_index(a, round, nbj, j) * ld + v0 + i];
      UA[i][j] = Ua[t];
    }
    __syncthreads();
    cgemm_tile32(lane, [&](int i, int k) { return X[r0 + i][k]; }, [&](int k, int j) { return UA[k][c0 + j]; }, cr,
                 ci);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = r0 + (lane >> 4) + 4 * r, j = c0 + (lane & 15);
      V[(int64_t)sub_index(a, round, nbj, j) * ld + v0 + i] = c128{cr[r], ci[r]};
    }
  }
}

// Frobenius norm in two deterministic stages: one block per column writes the
// column's sum of squares, then one block adds the kp column sums in a fixed
// order.
__global__ __launch_bounds__(256) void frob_cols_kernel(const c128* G, int64_t ld, int kp, double* part) {
  __shared__ double red[256];
  const int64_t col = blockIdx.x;
  double s = 0;
  for (int i = threadIdx.x; i < kp; i += 256) {
    const c128 z = G[col * ld + i];
    s += z.re * z.re + z.im * z.im;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[col] = red[0];
}

__global__ __launch_bounds__(256) void frob_sum_kernel(const double* part, int kp, double* out) {
  __shared__ double red[256];
  double s = 0;
  for (int i = threadIdx.x; i < kp; i += 256) s += part[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sqrt(red[0]);
}

// Select eigenvalues theta > 0 of the first k diagonal entries, order them
// descending (ascending 1/theta), gather the matching eigenvector columns
// (first kp rows) into Ysel and write lambda = 1/theta.  Counts positives and
// negatives that are resolved away from zero.
__global__ void select_kernel(const c128* G, const c128* V, int64_t ld, int k, int kp, const double* fro,
                              c128* Ysel, double* lam, int* npos, int* nneg) {
  // 1e3 * u * max|theta| bounded by the Frobenius norm
  const double tiny = 1e3 * 1.1102230246251565e-16 * *fro;
  const int i = blockIdx.x;
  if (i >= k) return;
  const double ti = G[(int64_t)i * ld + i].re;
  if (threadIdx.x == 0) {
    if (ti > tiny) atomicAdd(npos, 1);
    if (ti < -tiny) atomicAdd(nneg, 1);
  }
  if (!(ti > tiny)) return;
  __shared__ int rank;
  if (threadIdx.x == 0) rank = 0;
  __syncthreads();
  int cnt = 0;
  for (int j = threadIdx.x; j < k; j += blockDim.x) {
    const double tj = G[(int64_t)j * ld + j].re;
    if (tj > ti || (tj == ti && j < i)) ++cnt;
  }
  atomicAdd(&rank, cnt);
  __syncthreads();
  const int r = rank;
  if (r >= k / 2) return;
  if (threadIdx.x == 0) lam[r] = 1.0 / ti;
  for (int row = threadIdx.x; row < kp; row += blockDim.x) Ysel[(int64_t)r * kp + row] = V[(int64_t)i * ld + row];
}

__global__ void copy_if_resolved_kernel(const c128* src, int64_t lds, c128* dst, int64_t ldd, int rows, int half,
                                        const int* counts) {
  if (counts[0] != half || counts[1] != half) return;
  for (int i = threadIdx.x; i < rows; i += blockDim.x) dst[blockIdx.x * ldd + i] = src[blockIdx.x * lds + i];
}

}  // namespace

// ---------------------------------------------------------------------------
// Words of two device buffers into pinned host memory.
__global__ __launch_bounds__(256) void to_host_kernel(const uint32_t* a, int na, const uint32_t* b, int nb,
                                                      uint32_t* out) {
  for (int i = threadIdx.x; i < na; i += 256) out[i] = a[i];
  for (int i = threadIdx.x; i < nb; i += 256) out[na + i] = b[i];
}

struct HostWords {
  uint32_t w[896];
};
__global__ __launch_bounds__(256) void from_host_kernel(uint32_t* dst, int n, const HostWords v) {
  for (int i = threadIdx.x; i < n; i += 256) dst[i] = v.w[i];
}

Err d2h_small(void* host, const void* dev, size_t bytes, const DenseWs& ws, hipStream_t s, void* host2,
              const void* dev2, size_t bytes2) {
  if (bytes + bytes2 == 0) return ok();
  if (ws.hpin && bytes + bytes2 <= ws.hpin_bytes && bytes % 4 == 0 && bytes2 % 4 == 0) {
    hipLaunchKernelGGL(to_host_kernel, dim3(1), dim3(256), 0, s, (const uint32_t*)dev, (int)(bytes / 4),
                       (const uint32_t*)dev2, (int)(bytes2 / 4), (uint32_t*)ws.hpin);
    CHASE_LAUNCH_CHECK();
    CHASE_HIP(hipStreamSynchronize(s));
    if (bytes) std::memcpy(host, ws.hpin, bytes);
    if (bytes2) std::memcpy(host2, (const char*)ws.hpin + bytes, bytes2);
    return ok();
  }
  if (bytes) CHASE_HIP(hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, s));
  if (bytes2) CHASE_HIP(hipMemcpyAsync(host2, dev2, bytes2, hipMemcpyDeviceToHost, s));
  CHASE_HIP(hipStreamSynchronize(s));
  return ok();
}

Err h2d_small(void* dev, const void* host, size_t bytes, hipStream_t s) {
  HostWords v;
  if (bytes % 4 || bytes > 4 * sizeof(v)) {
    CHASE_HIP(hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, s));
    CHASE_HIP(hipStreamSynchronize(s));
    return ok();
  }
  for (size_t o = 0; o < bytes; o += sizeof(v)) {
    const size_t n = std::min(bytes - o, sizeof(v));
    std::memcpy(v.w, (const char*)host + o, n);
    hipLaunchKernelGGL(from_host_kernel, dim3(1), dim3(256), 0, s, (uint32_t*)((char*)dev + o), (int)(n / 4), v);
    CHASE_LAUNCH_CHECK();
  }
  return ok();
}

static int grid_for(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(n, 256), 2048)); }

// dscalar[0] = ||G||_F
static Err frob_norm(const c128* G, int kp, DenseWs& ws, hipStream_t s) {
  double* part = reinterpret_cast<double*>(ws.panel);  // kp doubles (panel holds kp x 64 c128)
  hipLaunchKernelGGL(frob_cols_kernel, dim3(kp), dim3(256), 0, s, G, (int64_t)kp, kp, part);
  CHASE_LAUNCH_CHECK();
  hipLaunchKernelGGL(frob_sum_kernel, dim3(1), dim3(256), 0, s, (const double*)part, kp, ws.dscalar);
  CHASE_LAUNCH_CHECK();
  return ok();
}

Err fill_padded(c128* M, int kp, int k, double inner, double pad, bool zero_all, hipStream_t s, int* clear,
                int nclear) {
  hipLaunchKernelGGL(fill_diag_kernel, dim3(grid_for((int64_t)kp * kp)), dim3(256), 0, s, M, (int64_t)kp, kp, k,
                     inner, pad, zero_all ? 1 : 0, clear, clear ? nclear : 0);
  CHASE_LAUNCH_CHECK();
  return ok();
}

Err tri_inverse_lower(const c128* L, c128* X, int kp, DenseWs& ws, hipStream_t s) {
  const int nblk = kp / NB;
  CHASE_TRY(fill_padded(X, kp, kp, 0.0, 0.0, true, s));
  hipLaunchKernelGGL(trinv_diag_kernel, dim3(nblk), dim3(CT), 0, s, L, X, (int64_t)kp);
  CHASE_LAUNCH_CHECK();
  const int64_t stride = (int64_t)NB * (kp + 1);
  for (int d = 1; d < nblk; ++d) {
    const int batch = nblk - d;
    // T_j = L[j+d, j..j+d-1] * X[j..j+d-1, j]
    ZgemmArgs g{};
    g.transA = 0; g.transB = 0;
    g.M = NB; g.N = NB; g.K = (int64_t)d * NB;
    g.alpha = {1, 0}; g.beta = {0, 0};
    g.A = L + (int64_t)d * NB; g.lda = kp; g.strideA = stride;
    g.B = X; g.ldb = kp; g.strideB = stride;
    g.C = ws.tmp; g.ldc = NB; g.strideC = (int64_t)NB * NB;
    g.kneg = g.K; g.batch = batch;
    CHASE_TRY(zgemm(g, ws.gemm_ws, ws.gemm_ws_bytes, s));  // K = d * 64: split along K
    // X[j+d, j] = -X[j+d, j+d] * T_j
    ZgemmArgs h{};
    h.transA = 0; h.transB = 0;
    h.M = NB; h.N = NB; h.K = NB;
    h.alpha = {-1, 0}; h.beta = {0, 0};
    h.A = X + (int64_t)d * NB * (kp + 1); h.lda = kp; h.strideA = stride;
    h.B = ws.tmp; h.ldb = NB; h.strideB = (int64_t)NB * NB;
    h.C = X + (int64_t)d * NB; h.ldc = kp; h.strideC = stride;
    h.kneg = NB; h.batch = batch;
    CHASE_TRY(zgemm(h, nullptr, 0, s));
  }
  return ok();
}

// Per column j of the Hermitian G, over the off-diagonal entries o:
// part[j] = sum |o|^2, part[kp + j] = sum |e|^2 with e = o / (g_ii - g_jj) over
// those with |o| > thr, part[2 kp + j] = 1 if there is one; thr = thr_of(*fro).
__host__ __device__ inline double thr_of(double fro) { return 1e-16 * (fro < 1e-300 ? 1e-300 : fro); }
__global__ __launch_bounds__(256) void offdiag_cols_kernel(const c128* G, int kp, const double* fro, double* part) {
  __shared__ double r1[256], r2[256];
  const int j = blockIdx.x;
  const double dj = G[(int64_t)j * kp + j].re, thr2 = thr_of(*fro) * thr_of(*fro);
  double so = 0, se = 0;
  int big = 0;
  for (int i = threadIdx.x; i < kp; i += 256) {
    if (i == j) continue;
    const c128 g = G[(int64_t)j * kp + i];
    const double o2 = g.re * g.re + g.im * g.im;
    so += o2;
    if (o2 > thr2) {
      const double gap = G[(int64_t)i * kp + i].re - dj;
      se += o2 / (gap * gap);
      big = 1;
    }
  }
  r1[threadIdx.x] = so;
  r2[threadIdx.x] = se;
  const int any = __syncthreads_or(big);
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      r1[threadIdx.x] += r1[threadIdx.x + w];
      r2[threadIdx.x] += r2[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[j] = r1[0];
    part[kp + j] = r2[0];
    part[2 * kp + j] = any;
  }
}

// The same, and before the first sweep ||G||_F, in one workgroup for a small
// G; the numbers and *guard go to pinned host memory: out[0] = ||G||_F,
// out[1 .. 3] the sums, then the flag.  kp = 64: one launch for five, of about
// 3.5 us each.
__global__ __launch_bounds__(1024) void offdiag_small_kernel(const c128* G, int kp, int first, double* fro,
                                                             const int* guard, double* out) {
  __shared__ double red[2][1024];
  const int tid = threadIdx.x, total = kp * kp;
  auto sum = [&](double* r) {
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
      if (tid < w) r[tid] += r[tid + w];
      __syncthreads();
    }
    return r[0];
  };
  double norm;
  if (first) {
    double s = 0;
    for (int t = tid; t < total; t += 1024) s += G[t].re * G[t].re + G[t].im * G[t].im;
    red[0][tid] = s;
    norm = sqrt(sum(red[0]));
    __syncthreads();
    if (tid == 0) *fro = norm;
  } else {
    norm = *fro;
  }
  const double thr2 = thr_of(norm) * thr_of(norm);
  double so = 0, se = 0;
  int big = 0;
  for (int t = tid; t < total; t += 1024) {
    const int j = t / kp, i = t % kp;
    if (i == j) continue;
    const c128 g = G[t];
    const double o2 = g.re * g.re + g.im * g.im;
    so += o2;
    if (o2 > thr2) {
      const double gap = G[(int64_t)i * kp + i].re - G[(int64_t)j * kp + j].re;
      se += o2 / (gap * gap);
      big = 1;
    }
  }
  red[0][tid] = so;
  red[1][tid] = se;
  const int any = __syncthreads_or(big);
  so = sum(red[0]);
  se = sum(red[1]);
  if (tid == 0) {
    out[0] = norm;
    out[1] = so;
    out[2] = se;
    out[3] = any;
    *reinterpret_cast<int*>(out + 4) = guard ? *guard : 0;
  }
}
constexpr int OFFDIAG_SMALL = 128;  // largest kp of offdiag_small_kernel: 16 entries a thread

// out[b] = sum of part[b kp ... + kp - 1] in a fixed order, b = blockIdx.x.
__global__ __launch_bounds__(256) void offdiag_sum_kernel(const double* part, int kp, double* out) {
  __shared__ double red[256];
  const double* p = part + (int64_t)blockIdx.x * kp;
  double s = 0;
  for (int i = threadIdx.x; i < kp; i += 256) s += p[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

// The anti-Hermitian E of jacobi_eigh: e_ij = g_ij / (g_jj - g_ii) from the
// upper triangle, zero where |g_ij| <= thr.
__global__ void refine_e_kernel(const c128* G, c128* E, int kp, double thr2) {
  const int64_t total = (int64_t)kp * kp;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = t / kp, i = t % kp;
    c128 e{0.0, 0.0};
    if (i != j) {
      const int64_t a = i < j ? i : j, b = i < j ? j : i;
      const c128 g = G[b * kp + a];
      if (g.re * g.re + g.im * g.im > thr2) {
        const double q = 1.0 / (G[b * kp + b].re - G[a * kp + a].re);
        e = i < j ? c128{q * g.re, q * g.im} : c128{-q * g.re, q * g.im};
      }
    }
    E[t] = e;
  }
}

// With T = E^2 and T2 = T^2 (null: the terms past T are below rounding):
// E <- I + E + T / 2 - T2 / 8, T <- T / 16 - 5 T2 / 128 and, where given,
// Z = 7 T / 256 - 21 T2 / 1024.
__global__ void refine_w_kernel(c128* E, c128* T, const c128* T2, c128* Z, int kp) {
  const int64_t total = (int64_t)kp * kp;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const c128 f = T[t];
    c128 w = E[t];
    w.re += 0.5 * f.re + (t / kp == t % kp ? 1.0 : 0.0);
    w.im += 0.5 * f.im;
    if (T2) {
      const c128 h = T2[t];
      w.re -= 0.125 * h.re;
      w.im -= 0.125 * h.im;
      T[t] = c128{0.0625 * f.re - 0.0390625 * h.re, 0.0625 * f.im - 0.0390625 * h.im};
      if (Z) Z[t] = c128{0.02734375 * f.re - 0.0205078125 * h.re, 0.02734375 * f.im - 0.0205078125 * h.im};
    }
    E[t] = w;
  }
}

// C = op(A) B + beta C on kp x kp matrices
static Err gemm_kp(int ta, int kp, const c128* A, const c128* B, double beta, c128* C, DenseWs& ws,
                   hipStream_t s) {
  ZgemmArgs g{};
  g.transA = ta;
  g.M = g.N = g.K = kp;
  g.alpha = {1, 0};
  g.beta = {beta, 0};
  g.A = A; g.lda = kp;
  g.B = B; g.ldb = kp;
  g.C = C; g.ldc = kp;
  g.kneg = kp;
  g.batch = 1;
  return zgemm(g, ws.gemm_ws, ws.gemm_ws_bytes, s);
}

// Largest ||E||_F at which a sweep is replaced by a refinement step, up to which
// the form with E^8 is enough, and that of I + E + E^2 / 2: there the first term
// left out, 33/2048 ||E||^14, 7/256 ||E||^10 and ||E||^4 / 8, is below the unit
// roundoff (in the spectral norm, at most the Frobenius one: 7.9e-17, 7.5e-17 and
// 1.3e-17).
// From 0.05 on, a sweep (500 us at kp = 384) and two steps are left, or four
// steps of 60 to 180 us: Rayleigh-Ritz m = 4000, k = 376 4.19 -> 3.80 ms against a
// limit of 0.04.
constexpr double REFINE_MAX = 0.095, REFINE_MID = 0.035, REFINE_SHORT = 1e-4;
// From REFINE_KP on, a step of 6 or 7 products takes as long as a sweep and does
// less, so only the short form replaces one (k = 2600, solve of 5 iterations:
// Rayleigh-Ritz 525 -> 502 ms).
constexpr int REFINE_KP = 1536;
// From IN_PLACE_KP on, a round is bound by reading and writing G and V: there
// the rotations are found in a launch of their own and applied in place, so that
// blocks whose pairs did not rotate, most of them in late sweeps, stay untouched.
// That launch reads its blocks of G as they are (taken through identity blocks, as
// next_rotations would: Rayleigh-Ritz m = 5000, k = 4800 2000 ms against 1959, k = 3072
// 542 / 518).
constexpr int IN_PLACE_KP = 3072;

// Eigenvectors V and (on the diagonal) eigenvalues of the Hermitian G: block
// Jacobi sweeps until the off-diagonal entries are small against the gaps of
// the diagonal, then GEMMs.  With D the diagonal, O the rest and
// e_ij = o_ij / (d_j - d_i), the unitary W = E + sqrt(I + E^2) =
// E + I + T / 2 - T^2 / 8 + T^3 / 16 - 5 T^4 / 128 + 7 T^5 / 256 - 21 T^6 / 1024
// + ... (T = E^2) takes G to
// W^H G W with off-diagonal part [O, E] / 2 to second order, ||O||_F ||E||_F
// at most: quadratic like a sweep, which is kp / 16 - 1 dependent
// launches.  At kp = 384 a sweep takes 500 us (21 a round), a step 150,
// the last one, which leaves G alone, 60; a Rayleigh-Ritz step at m = 4000 and
// k = 376 went from 5.06 ms to 4.41, one of the converging iterations at k = 500
// (m = 4000) from 3 sweeps to 1 or 2.
Err jacobi_eigh(c128* G, c128* V, int kp, DenseWs& ws, hipStream_t s, int max_sweeps, int* sweeps_out, int guard,
                bool* tripped) {
  const int nbj = kp / JB;  // even since kp % 64 == 0
  const int npair = nbj / 2;
  CHASE_TRY(fill_padded(V, kp, kp, 1.0, 1.0, true, s, ws.flag + DenseWs::COUNTS, 2));
  const bool in_place = kp >= IN_PLACE_KP;
  const bool small = kp <= OFFDIAG_SMALL && ws.hpin && ws.hpin_bytes >= 5 * sizeof(double);
  if (!small) CHASE_TRY(frob_norm(G, kp, ws, s));
  // G is in cur; every round writes it to o[0] and the two change places.
  // V is in vec, which a refinement step exchanges with o[1].
  c128 *cur = G, *vec = V, *o[3] = {ws.k1, ws.k2, ws.k3};
  int first = 1;
  double* part = reinterpret_cast<double*>(ws.panel);  // 3 kp doubles
  int sweep = 0;
  double ef_last = 1e300;  // ||E||_F of the step before, where there was one
  bool converged = false;
  for (;;) {
    double st[4] = {0, 0, 0, 0};
    int bad = 0;
    if (small) {
      hipLaunchKernelGGL(offdiag_small_kernel, dim3(1), dim3(1024), 0, s, (const c128*)cur, kp, first, ws.dscalar,
                         guard < 0 ? (const int*)nullptr : (const int*)ws.flag + guard, (double*)ws.hpin);
      CHASE_LAUNCH_CHECK();
      CHASE_HIP(hipStreamSynchronize(s));
      std::memcpy(st, ws.hpin, sizeof(st));
      std::memcpy(&bad, (const char*)ws.hpin + sizeof(st), sizeof(int));
      first = 0;
    } else {
      hipLaunchKernelGGL(offdiag_cols_kernel, dim3(kp), dim3(256), 0, s, (const c128*)cur, kp,
                         (const double*)ws.dscalar, part);
      CHASE_LAUNCH_CHECK();
      hipLaunchKernelGGL(offdiag_sum_kernel, dim3(3), dim3(256), 0, s, (const double*)part, kp, ws.dscalar + 1);
      CHASE_LAUNCH_CHECK();
      CHASE_TRY(d2h_small(st, ws.dscalar, sizeof(st), ws, s, &bad, ws.flag + guard, guard < 0 ? 0 : sizeof(int)));
    }
    if (bad) {
      *tripped = true;
      return ok();
    }
    const double thr = thr_of(st[0]), of = std::sqrt(st[1]), ef = std::sqrt(st[2]);
    if (st[3] == 0.0) {  // no off-diagonal entry above thr
      converged = true;
      break;
    }
    // steps do not count as sweeps: where one at least halves ||E||_F there are
    // fewer than 30 in a row, where it does not a sweep is next
    if (ef <= std::min(kp < REFINE_KP ? REFINE_MAX : REFINE_SHORT, 0.5 * ef_last)) {
      ef_last = ef;
      const int blocks = grid_for((int64_t)kp * kp);
      c128 *W = o[0], *T = o[1], *T2 = ef > REFINE_SHORT ? o[2] : nullptr, *Z = ef > REFINE_MID ? ws.k4 : nullptr;
      hipLaunchKernelGGL(refine_e_kernel, dim3(blocks), dim3(256), 0, s, (const c128*)cur, W, kp, thr * thr);
      CHASE_LAUNCH_CHECK();
      CHASE_TRY(gemm_kp(0, kp, W, W, 0.0, T, ws, s));
      if (T2) CHASE_TRY(gemm_kp(0, kp, T, T, 0.0, T2, ws, s));
      hipLaunchKernelGGL(refine_w_kernel, dim3(blocks), dim3(256), 0, s, W, T, (const c128*)T2, Z, kp);
      CHASE_LAUNCH_CHECK();
      if (Z) CHASE_TRY(gemm_kp(0, kp, T2, Z, 1.0, T, ws, s));
      if (T2) CHASE_TRY(gemm_kp(0, kp, T2, T, 1.0, W, ws, s));
      CHASE_TRY(gemm_kp(0, kp, vec, W, 0.0, T, ws, s));
      std::swap(vec, o[1]);
      T = o[1];
      if (of * ef <= 0.5 * thr) {  // what is left off the diagonal, and its shift, is below thr
        converged = true;
        break;
      }
      CHASE_TRY(gemm_kp(0, kp, cur, W, 0.0, T, ws, s));
      CHASE_TRY(gemm_kp(1, kp, W, T, 0.0, cur, ws, s));
      continue;
    }
    if (sweep == max_sweeps) break;
    ++sweep;
    ef_last = 1e300;
    // U and flags of a round and of the next
    c128* U[2] = {ws.U, ws.U + (int64_t)npair * SP * SP};
    int* fl[2] = {ws.pflag, ws.pflag + npair};
    hipLaunchKernelGGL(jacobi_pairs_kernel<false>, dim3(npair), dim3(256), 0, s, (const c128*)cur, (int64_t)kp, nbj, 0,
                       U[0], thr, fl[0]);
    CHASE_LAUNCH_CHECK();
    const int apply = npair * (npair + 1) / 2 + npair * (kp / SP);
    for (int r = 0; r < nbj - 1; ++r) {
      const int nspec = r < nbj - 2 && !in_place ? npair : 0;
      c128* Gn = in_place ? cur : o[0];
      hipLaunchKernelGGL(jacobi_round_kernel, dim3(nspec + apply), dim3(256), 0, s, (const c128*)cur, Gn, vec,
                         (int64_t)kp, kp, nbj, r, (const c128*)U[r & 1], (const int*)fl[r & 1], U[(r + 1) & 1],
                         fl[(r + 1) & 1], thr, nspec);
      CHASE_LAUNCH_CHECK();
      if (!in_place) {
        std::swap(cur, o[0]);
      } else if (r < nbj - 2) {
        hipLaunchKernelGGL(jacobi_pairs_kernel<true>, dim3(npair), dim3(256), 0, s, (const c128*)cur, (int64_t)kp, nbj,
                           r + 1, U[(r + 1) & 1], thr, fl[(r + 1) & 1]);
        CHASE_LAUNCH_CHECK();
      }
    }
  }
  if (vec != V) CHASE_HIP(hipMemcpyAsync(V, vec, (size_t)kp * kp * sizeof(c128), hipMemcpyDeviceToDevice, s));
  if (cur != G) CHASE_HIP(hipMemcpyAsync(G, cur, (size_t)kp * kp * sizeof(c128), hipMemcpyDeviceToDevice, s));
  if (sweeps_out) *sweeps_out = sweep;
  if (!converged)
    return fail(CHASE_PH_ERR_EIG, "Jacobi eigensolver: off-diagonal entries above 1e-16 ||G||_F after " +
                                      std::to_string(max_sweeps) + " sweeps");
  return ok();
}

Err select_positive(const c128* G, const c128* V, int k, int kp, c128* Ysel, double* dlam, DenseWs& ws,
                    hipStream_t s) {
  int* counts = ws.flag + DenseWs::COUNTS;
  hipLaunchKernelGGL(select_kernel, dim3(k), dim3(256), 0, s, G, V, (int64_t)kp, k, kp, (const double*)ws.dscalar, Ysel,
                     dlam, counts, counts + 1);
  CHASE_LAUNCH_CHECK();
  return ok();
}

Err copy_if_resolved(const c128* src, int64_t lds, c128* dst, int64_t ldd, int rows, int half, DenseWs& ws,
                     hipStream_t s) {
  hipLaunchKernelGGL(copy_if_resolved_kernel, dim3(half), dim3(256), 0, s, src, lds, dst, ldd, rows, half,
                     (const int*)ws.flag + DenseWs::COUNTS);
  CHASE_LAUNCH_CHECK();
  return ok();
}

int pad64(int k) { return (int)ceil_div(std::max(k, 1), NB) * NB; }

}  // namespace chase
