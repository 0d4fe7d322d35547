// Block-structured product H X, H = [[A, B], [-conj(B), -conj(A)]]
// (Section 1, eq. 1.1), in FP64, as one real GEMM over the real structure of H.
//
// H is real-linear on K-real vectors (Thm 3.1: H K conj = -K conj H): for
// u = [a; conj(a)],
//   H u = [t; -conj(t)],   t = A a + B conj(a) = (A + B) Re(a) + i (A - B) Im(a).
// Every column x = [x1; x2] splits into K-real parts, x = u + i v, with
//   a_u = (x1 + conj(x2)) / 2,   a_v = (x1 - conj(x2)) / (2 i),
// so that  H x = [t_u + i t_v; -conj(t_u) - i conj(t_v)], whose own K-real
// parts are a_u' = i t_v and a_v' = -i t_u.  With M the real 2m x 2m matrix of
// hx.h, the real coordinates of t are M y for y those of a, and two products
// in a row act on every real column alike: H^2 = -J M J M, J the
// multiplication by i (a swap of the two reals of an entry, one negated).
// So the recurrences on H^2 stay in real coordinates from the first product
// to the last: one GEMM of 2m x 2m by 2m x 2k per product (16 m^2 k = 4 n^2 k
// real flops, half of the complex GEMM [A B] [X, K conj(X)]), its epilogue
// writes the next product's operand, and nothing is packed in between.
//
// The GEMM has no LDS and no barriers.  The FP64 MFMA is slow against the
// caches (a 16 x 16 x 4 takes 64 cycles for one 16-byte load per lane every
// two of them and operand), so each wave loads its fragments straight into
// registers, ahead of their use, in the order the MFMA lanes take them: M is
// stored fragment by fragment (hx_make_operand), the X4 layout gives a lane 2
// consecutive k of its column with one 16-byte load, and the four
// accumulators of a lane are exactly one quad of an X4 column, so the result
// is stored with 16-byte accesses too.  The four waves of a workgroup work on
// 32 rows each of one 128-row strip and the same columns, which they share
// through the L1.
//
// Work split: the columns are cut into TN tiles of nearly equal width (at most
// 8 fragments), one workgroup each, which form a team; the (strip, K) range of
// the matrix is cut into equal parts, one per team, so that M passes the L2 of
// the team's XCD once.  Two workgroups per CU in all.  A part may start or end
// inside a strip; the partial sums of such a strip go to a workspace and a
// second kernel adds them in K order and applies the epilogue, so results do
// not depend on timing.  Short products (hx_plan.h) run in one launch of
// hx_short_kernel instead, where the waves of a workgroup share K.
//
// Bound by the FP64 MFMA for N >= 100 or so at m >= 4000 (below that by the
// read of M), by latency at m <= 500.  Measured per product of the filter
// (us; before: a kernel on LDS rings with barriers, packing before every
// product): m = 500, k = 30: 6.5 (32.8 before); m = 2000, k = 70: 85 (114);
// m = 4000, k = 256: 965 = 67.9 TF/s (1116); k = 376: 1418 (1765);
// m = 10000, k = 512: 11463 = 71.5 TF/s, as much as MFMAs on registers alone.
// M read by a team's workgroups in step, rather than by workgroups with parts
// of their own of (strip, tile, K): 2 - 7% at m = 4000.
#include "hx.h"
#include "hx_plan.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

namespace chase {
namespace {

typedef double doublex2 __attribute__((ext_vector_type(2)));

// v_mfma_f64_16x16x4f64: lane l holds A row l % 16 and B column l % 16 at
// k = l / 16 of the four, and rows l / 16 + 4 r of output column l % 16.  A
// fragment load of 16 bytes covers two MFMAs: a slab of 8 reals of K, lane l
// holding k = 2 (l / 16) + s for MFMA s.
constexpr int V = 2, BK = HX_BK;
constexpr int FM = HX_FM;
constexpr int WROWS = 16 * FM;   // rows per wave
constexpr int BM = HX_BM;        // rows per workgroup
static_assert(BM == 4 * WROWS && HX_RPAD % BM == 0, "row padding");
constexpr int MAX_WG = HX_MAX_WG, MAX_NL = HX_MAX_NL;
static_assert(HX_KPAD % (4 * BK) == 0, "column padding");

// Real row (of 16) whose M entries lane l holds: fed from row
// 4 (rho % 4) + rho / 4, output row rho lands so that a lane's accumulators
// are rows 4 (l / 16) .. + 3.
__device__ __forceinline__ int a_row(int l) { return 4 * (l & 3) + ((l & 15) >> 2); }

struct HxDev : HxPlan {
  const double* M;
  const double* y;
  int64_t ldc4;   // reals per quad row
  int64_t wstep;  // reals of M per 32-row group
  int rows2, N, m;
  double* ws;  // partial sums
  // epilogue: X4 output (out != null) or complex Y of one product
  double* out;
  const double *P, *Q;
  double alpha, beta, gamma;
  int rot, kind;
  c128* Yc;
  int64_t ldy;
};

struct Pos {
  int strip, kb;
};

__device__ __forceinline__ int tile_width(const HxDev& a, int ct) { return a.wq + (ct < a.wr ? 1 : 0); }
__device__ __forceinline__ int tile_first(const HxDev& a, int ct) { return ct * a.wq + min(ct, a.wr); }

// x / d and x % d for 0 <= x < 2^52 from the reciprocal of d (a 64-bit integer
// division costs the workgroup more than a microsecond before its first load).
__device__ __forceinline__ int64_t quot(int64_t x, int64_t d, double inv, int64_t* rem) {
  int64_t q = (int64_t)((double)x * inv), r = x - q * d;
  if (r < 0) {
    --q;
    r += d;
  } else if (r >= d) {
    ++q;
    r -= d;
  }
  *rem = r;
  return q;
}
// Start of the part of team t.
__device__ __forceinline__ Pos part_start(const HxDev& a, int t) {
  int64_t kb;
  const int64_t x = (t * a.lq + quot((int64_t)t * a.lr, a.teams, a.i_teams, &kb)) * a.unit;
  const int strip = (int)quot(x, a.KB, a.i_KB, &kb);
  return Pos{strip, (int)kb};
}

__device__ __forceinline__ bool before(const Pos& p, const Pos& q) {  // p < q
  return p.strip != q.strip ? p.strip < q.strip : p.kb < q.kb;
}

__device__ __forceinline__ int xcd_remap(int w, int T) {
  // Workgroup w runs on XCD w % 8.  Give each XCD a contiguous range of
  // parts, so that neighbouring tiles stay in one L2.
  const int xcd = w & 7, slot = w >> 3;
  const int q = T >> 3, r = T & 7;
  return xcd * q + (xcd < r ? xcd : r) + slot;
}

__device__ __forceinline__ doublex4 load4(const double* p) {
  const doublex2 a = *reinterpret_cast<const doublex2*>(p), b = *reinterpret_cast<const doublex2*>(p + 2);
  return doublex4{a[0], a[1], b[0], b[1]};
}
__device__ __forceinline__ void store4(double* p, doublex4 v) {
  *reinterpret_cast<doublex2*>(p) = doublex2{v[0], v[1]};
  *reinterpret_cast<doublex2*>(p + 2) = doublex2{v[2], v[3]};
}

__device__ __forceinline__ doublex4 times_i(doublex4 t) { return doublex4{-t[1], t[0], -t[3], t[2]}; }

// Rows row .. row + 3 (row a multiple of 4) of column c of M y; every lane of
// the wave calls it, lanes l and l ^ 1 with the two columns of a pair.
__device__ __forceinline__ void finish(const HxDev& a, int row, int c, doublex4 t) {
  const bool live = row < a.rows2 && c < a.N;
  if (a.out) {
    if (!live) return;
    if (a.rot == HX_I) t = times_i(t);
    if (a.rot == HX_MINUS_I) t = -times_i(t);
    const int64_t off = (int64_t)(row >> 2) * a.ldc4 + 4 * c;
    doublex4 v = a.alpha * t;
    if (a.P) v += a.beta * load4(a.P + off);
    if (a.Q) v += a.gamma * load4(a.Q + off);
    store4(a.out + off, v);
    return;
  }
  doublex4 o;
#pragma unroll
  for (int r = 0; r < 4; ++r) o[r] = __shfl_xor(t[r], 1);
  if (!live) return;
  const int ci = row >> 1;
  const bool two = ci + 1 < a.m;
  if (a.kind != HX_GENERAL) {
    c128* y = a.Yc + (int64_t)c * a.ldy + ci;
    y[0] = c128{t[0], t[1]};
    if (two) y[1] = c128{t[2], t[3]};
    if (a.kind == HX_KREAL) {  // -conj(t)
      y += a.m;
      y[0] = c128{-t[0], t[1]};
      if (two) y[1] = c128{-t[2], t[3]};
    }
  } else if (!(c & 1)) {  // t = t_u, o = t_v: t_u + i t_v
    c128* y = a.Yc + (int64_t)(c >> 1) * a.ldy + ci;
    y[0] = c128{t[0] - o[1], t[1] + o[0]};
    if (two) y[1] = c128{t[2] - o[3], t[3] + o[2]};
  } else {                // t = t_v, o = t_u: -conj(t_u) - i conj(t_v)
    c128* y = a.Yc + (int64_t)(c >> 1) * a.ldy + a.m + ci;
    y[0] = c128{-o[0] - t[1], o[1] - t[0]};
    if (two) y[1] = c128{-o[2] - t[3], o[3] - t[2]};
  }
}

// Stages kb0 .. kb1 of a tile of NL column fragments starting at fragment cb:
// KS slabs of K per stage.  The fragments of y are loaded one stage ahead;
// those of M, which come from HBM or the Infinity Cache, two to three ahead
// where a stage is one slab (wide tiles), else one.
template <int NL, int KS>
__device__ __forceinline__ void run_tile(const HxDev& a, int strip, int cb, int kb0, int kb1, double* slot) {
  constexpr int AS = KS == 1 ? 2 : 1;  // stages of M loaded together
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, lc = lane & 15;
  const int row0 = strip * BM + wave * WROWS;
  const doublex2* mp = reinterpret_cast<const doublex2*>(a.M + (int64_t)(row0 / WROWS) * a.wstep) + lane;
  const double* yp = a.y + 64 * cb + (g >> 1) * a.ldc4 + 4 * lc + 2 * (g & 1);
  const int64_t ystep = (BK / 4) * a.ldc4;

  doublex2 fa[2][AS][KS][FM], fb[2][KS][NL];
  doublex4 acc[FM][NL];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < NL; ++j) acc[i][j] = doublex4{0, 0, 0, 0};
  auto load_m = [&](int kb, doublex2 (&x)[KS][FM]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < KS; ++q)
#pragma unroll
      for (int i = 0; i < FM; ++i) x[q][i] = mp[((int64_t)kb * KS + q) * (FM * 64) + i * 64];
  };
  auto load_y = [&](int kb, doublex2 (&x)[KS][NL]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < KS; ++q)
#pragma unroll
      for (int j = 0; j < NL; ++j)
        x[q][j] = *reinterpret_cast<const doublex2*>(yp + ((int64_t)kb * KS + q) * ystep + 64 * j);
  };
  auto mul = [&](const doublex2 (&xa)[KS][FM], const doublex2 (&xb)[KS][NL]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < KS; ++q)
#pragma unroll
      for (int s = 0; s < V; ++s)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < NL; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[q][i][s], xb[q][j][s], acc[i][j], 0, 0, 0);
  };
  const int kl = kb1 - 1;
#pragma unroll
  for (int h = 0; h < AS; ++h) load_m(min(kb0 + h, kl), fa[0][h]);
  load_y(kb0, fb[0]);
  // a fixed place in the 64-byte lines of the instruction cache: where the loops of
  // two tile widths lie decides up to 2% (m = 5607, k = 411, tiles of 6 and 5: 3245 us
  // here, 3242 to 3315 at other places, as code before them comes and goes)
  __asm__ volatile(".p2align 6");
#pragma unroll 1
  for (int kb = kb0; kb < kb1; kb += AS) {
#pragma unroll
    for (int h = 0; h < AS; ++h) load_m(min(kb + AS + h, kl), fa[1][h]);
    load_y(min(kb + 1, kl), fb[1]);
    __builtin_amdgcn_sched_barrier(0);
    mul(fa[0][0], fb[0]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (AS == 2) {
      load_y(min(kb + 2, kl), fb[0]);
      __builtin_amdgcn_sched_barrier(0);
      if (kb < kl) mul(fa[0][1], fb[1]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < KS; ++q) {
#pragma unroll
      for (int h = 0; h < AS; ++h)
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[0][h][q][i] = fa[1][h][q][i];
      if constexpr (AS == 1) {
#pragma unroll
        for (int j = 0; j < NL; ++j) fb[0][q][j] = fb[1][q][j];
      }
    }
  }
  // the lane number anew, so that the compiler does not keep the epilogue's
  // addresses in registers through the loop
  int el = lane;
  __asm__ volatile("" : "+v"(el));
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      __builtin_amdgcn_sched_barrier(0);
      if (slot)
        store4(slot + ((int64_t)((wave * FM + i) * a.wmax + j) * 64 + el) * 4, acc[i][j]);
      else
        finish(a, row0 + 16 * i + 4 * (el >> 4), 16 * (cb + j) + (el & 15), acc[i][j]);
    }
}

// The parts of one team's range [b, e) for column tile ct of NL fragments.
template <int NL, int KS>
__device__ __forceinline__ void run_part(const HxDev& a, int id, int ct, Pos b, const Pos& e) {
#pragma unroll 1
  for (; before(b, e); b = Pos{b.strip + 1, 0}) {
    const int kb1 = b.strip == e.strip ? e.kb : a.KB;
    double* slot = b.kb == 0 && kb1 == a.KB ? nullptr : a.ws + (2 * (int64_t)id + (b.kb == 0 ? 1 : 0)) * a.slot;
    run_tile<NL, KS>(a, b.strip, tile_first(a, ct), b.kb, kb1, slot);
  }
}

// Tiles of W and W - 1 fragments.
template <int W, int KS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void hx_kernel(const HxDev a) {
  const int id = xcd_remap(blockIdx.x, a.teams * a.TN);
  const int team = id / a.TN, ct = id - team * a.TN;
  const Pos b = part_start(a, team), e = part_start(a, team + 1);
  if (tile_width(a, ct) == W) {
    run_part<W, KS>(a, id, ct, b, e);
  } else {
    if constexpr (W > 1) run_part<W - 1, KS>(a, id, ct, b, e);
  }
}

// Sums the parts of strip blockIdx.x and applies the epilogue; column fragment
// blockIdx.y, FM row fragments per wave.  The lanes look up the starts of 64
// neighbouring parts at once, so that every load's address is known before the
// first one is waited for.
__global__ __launch_bounds__(256) void hx_reduce_kernel(const HxDev a) {
  const int strip = blockIdx.x, cf = blockIdx.y;
  const int cut = a.wr * (a.wq + 1);
  const int ct = cf < cut ? cf / (a.wq + 1) : a.wr + (cf - cut) / a.wq;
  const int j = cf - tile_first(a, ct);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Pos start{strip, 0}, next{strip + 1, 0};
  // the last part starting at or before the strip: floor(strip * KB * teams /
  // (TM * KB)) or a neighbour
  int t0 = max(0, (int)((double)strip * a.teams / a.TM) - 1);
  {
    const int t = t0 + lane;
    const uint64_t at = __ballot(t < a.teams && !before(start, part_start(a, t)));
    t0 += 63 - __builtin_clzll(at | 1);
  }
  int cnt = 1;  // parts of the strip: t0 .. t0 + cnt - 1
  for (int o = 1;; o += 64) {
    const int t = t0 + o + lane;
    const uint64_t in = __ballot(t < a.teams && before(part_start(a, t), next));
    cnt += __builtin_popcountll(in);
    if (~in) break;
  }
  if (cnt == 1) return;  // whole in one part: finished there
  const int64_t off = ((int64_t)(wave * FM * a.wmax + j) * 64 + lane) * 4, istep = (int64_t)a.wmax * 256;
  const int64_t tstep = 2 * a.TN * a.slot;
  const double* w = a.ws + t0 * tstep + 2 * ct * a.slot + off;
  doublex4 v[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) v[i] = load4(w + a.slot + i * istep);  // the part starting with the strip
  int n = 1;
  for (; n + 4 <= cnt; n += 4) {
    doublex4 u[4][FM];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < FM; ++i) u[q][i] = load4(w + (n + q) * tstep + i * istep);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < FM; ++i) v[i] += u[q][i];
  }
  for (; n < cnt; ++n)
#pragma unroll
    for (int i = 0; i < FM; ++i) v[i] += load4(w + n * tstep + i * istep);
  const int row0 = strip * BM + wave * WROWS;
#pragma unroll
  for (int i = 0; i < FM; ++i) finish(a, row0 + 16 * i + 4 * (lane >> 4), 16 * cf + (lane & 15), v[i]);
}

// Short products in one launch, without partial sums in memory: a workgroup of
// NW waves takes 16 FMS rows x 16 NL columns, each wave a share of K, KS slabs
// a stage, loaded one stage ahead; the waves' sums are added in LDS in K order.
// Bound by launch and load latency below m = 500 or so, above it by the MFMA
// and the L1 in turn, at k <= 16 and m >= 3000 by the read of M (5.9 TB/s).
// Few slabs a stage and many workgroups per CU hide the loads better than
// long stages (KS = 4 for 2 where two fragments are shared: 3 - 10% slower).
template <int FMS, int NL, int NW, int KS>
__global__ __launch_bounds__(64 * NW) void hx_short_kernel(const HxDev a) {
  __shared__ double red[NW][FMS * NL][2][64][2];
  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int strip = id / a.TN, ct = id - strip * a.TN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, lc = lane & 15;
  const int row0 = strip * 16 * FMS, cb = ct * NL;
  const doublex2* mp = reinterpret_cast<const doublex2*>(a.M + (int64_t)(row0 / WROWS) * a.wstep) +
                       (row0 / 16 % FM) * 64 + lane;
  const double* yp = a.y + (g >> 1) * a.ldc4 + 4 * lc + 2 * (g & 1);
  const int64_t ystep = (BK / 4) * a.ldc4;
  int yo[NL];  // the last tile's fragments past column N repeat its last one
#pragma unroll
  for (int j = 0; j < NL; ++j) yo[j] = 64 * min(cb + j, (a.N - 1) / 16);
  const int k0 = a.KB * wave / NW, k1 = a.KB * (wave + 1) / NW;  // slabs
  doublex4 acc[FMS][NL];
#pragma unroll
  for (int i = 0; i < FMS; ++i)
#pragma unroll
    for (int j = 0; j < NL; ++j) acc[i][j] = doublex4{0, 0, 0, 0};
  doublex2 fa[2][KS][FMS], fb[2][KS][NL];
  auto load = [&](int k, doublex2 (&x)[KS][FMS], doublex2 (&y)[KS][NL]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      const int64_t kk = min(k + q, k1 - 1);
#pragma unroll
      for (int i = 0; i < FMS; ++i) x[q][i] = mp[kk * (FM * 64) + i * 64];
#pragma unroll
      for (int j = 0; j < NL; ++j) y[q][j] = *reinterpret_cast<const doublex2*>(yp + kk * ystep + yo[j]);
    }
  };
  auto mul = [&](int k, const doublex2 (&x)[KS][FMS], const doublex2 (&y)[KS][NL]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < KS; ++q)
      if (k + q < k1) {
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
          for (int i = 0; i < FMS; ++i)
#pragma unroll
            for (int j = 0; j < NL; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[q][i][v], y[q][j][v], acc[i][j], 0, 0, 0);
      }
  };
  if (k0 < k1) {
    load(k0, fa[0], fb[0]);
#pragma unroll 1
    for (int k = k0; k < k1; k += 2 * KS) {
      load(k + KS, fa[1], fb[1]);
      __builtin_amdgcn_sched_barrier(0);
      mul(k, fa[0], fb[0]);
      __builtin_amdgcn_sched_barrier(0);
      load(k + 2 * KS, fa[0], fb[0]);
      __builtin_amdgcn_sched_barrier(0);
      mul(k + KS, fa[1], fb[1]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int i = 0; i < FMS; ++i)
#pragma unroll
    for (int j = 0; j < NL; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *reinterpret_cast<doublex2*>(red[wave][i * NL + j][h][lane]) = doublex2{acc[i][j][2 * h], acc[i][j][2 * h + 1]};
  __syncthreads();
#pragma unroll 1
  for (int f = wave; f < FMS * NL; f += NW) {
    doublex4 v{0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const doublex2 x = *reinterpret_cast<const doublex2*>(red[w][f][0][lane]),
                     y = *reinterpret_cast<const doublex2*>(red[w][f][1][lane]);
      v += doublex4{x[0], x[1], y[0], y[1]};
    }
    finish(a, row0 + 16 * (f / NL) + 4 * g, 16 * (cb + f % NL) + lc, v);
  }
}

// ---------------------------------------------------------------- plan
// CHASE_PH_APPLY_PLAN="w,splits" forces tiles of at most 8 >> w column
// fragments and about `splits` parts per tile, w = 4 .. 9 the short product's
// shape w - 4, so that every tile width, split and shape can be checked for
// parity on one problem.
bool plan_override(int* w, int* splits) {
  const char* e = std::getenv("CHASE_PH_APPLY_PLAN");
  return e && std::sscanf(e, "%d,%d", w, splits) == 2 && *w >= 0 && *w <= 9 && *splits >= 1;
}

// The plan of a's product into a.
void make_plan(HxDev& a, size_t ws_bytes) {
  HxPlan& p = a;
  int w = 0, splits = 0;
  if (!plan_override(&w, &splits)) {
    p = hx_plan(a.rows2, a.N, ws_bytes);
  } else if (w >= 4) {
    hx_set_short(p, a.rows2, a.N, w - 4);
  } else {
    const int NB = (int)ceil_div(a.N, (int64_t)16), TN = (int)ceil_div(NB, (int64_t)(MAX_NL >> w));
    const int64_t strips = ceil_div(a.rows2, (int64_t)BM);
    hx_cut(p, a.rows2, NB, TN, std::min<int64_t>(strips * splits, std::max(1, MAX_WG / TN)), ws_bytes);
  }
}

Err launch(HxDev& a, void* ws, size_t ws_bytes, hipStream_t s) {
  a.ws = (double*)ws;
  make_plan(a, ws ? ws_bytes : 0);
  if (a.shape >= 0) {
    auto go = [&](auto F, auto NL, auto NW, auto KS) {
      constexpr int f = decltype(F)::value, nl = decltype(NL)::value, nw = decltype(NW)::value;
      const unsigned blocks = (unsigned)(ceil_div(a.rows2, (int64_t)(16 * f)) * a.TN);
      hipLaunchKernelGGL((hx_short_kernel<f, nl, nw, decltype(KS)::value>), dim3(blocks), dim3(64 * nw), 0, s, a);
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    using I4 = std::integral_constant<int, 4>;
    using I8 = std::integral_constant<int, 8>;
    switch (a.shape) {
      case 0: go(I1{}, I1{}, I4{}, I4{}); break;
      case 1: go(I1{}, I2{}, I4{}, I2{}); break;
      case 2: go(I2{}, I1{}, I4{}, I2{}); break;
      case 3: go(I2{}, I2{}, I4{}, I2{}); break;
      case 4: go(I2{}, I3{}, I4{}, I2{}); break;
      default: go(I2{}, I4{}, I8{}, I1{}); break;
    }
    CHASE_LAUNCH_CHECK();
    return ok();
  }
  const dim3 grid((unsigned)(a.teams * a.TN)), block(256);
  auto go = [&](auto W) {
    constexpr int w = decltype(W)::value;
    hipLaunchKernelGGL((hx_kernel<w, hx_stage_slabs(w)>), grid, block, 0, s, a);
  };
  switch (a.wmax) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    case 5: go(std::integral_constant<int, 5>{}); break;
    case 6: go(std::integral_constant<int, 6>{}); break;
    case 7: go(std::integral_constant<int, 7>{}); break;
    default: go(std::integral_constant<int, 8>{}); break;
  }
  CHASE_LAUNCH_CHECK();
  if (hx_plan_bytes(a) == 0) return ok();  // every strip whole in one part
  hipLaunchKernelGGL(hx_reduce_kernel, dim3((unsigned)a.TM, (unsigned)ceil_div(a.N, (int64_t)16)), block, 0, s, a);
  CHASE_LAUNCH_CHECK();
  return ok();
}

HxDev operand(const double* M, int64_t m, const double* y, int64_t ldc, int N) {
  HxDev a{};
  a.M = M;
  a.y = y;
  a.ldc4 = 4 * ldc;
  a.wstep = hx_group_reals(m);
  a.rows2 = (int)(2 * m);
  a.m = (int)m;
  a.N = N;
  return a;
}

// ---------------------------------------------------------------- layouts
// M entry (row, k) sits in 32-row group row / 32, slab k / 8, fragment
// (row / 16) % 2, lane, place s of 2: one thread writes the two entries of one
// lane.  Reads run along 8 complex rows of a column.
__global__ void make_operand_kernel(const c128* A, const c128* B, int64_t ld, int a_conj, doublex2* M, int64_t m,
                                    int64_t rows, int64_t cols, int64_t group) {
  const int64_t total = rows * cols / V;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int lane = (int)(t & 63), i = (int)((t >> 6) % FM);
    const int64_t q = t / (64 * FM), kb = q % (cols / BK), grp = q / (cols / BK);
    const int64_t row = grp * WROWS + 16 * i + a_row(lane), k = kb * BK + V * (lane >> 4);
    const int64_t ci = row >> 1, p = k >> 1;
    doublex2 f{0, 0};
    if (ci < m && p < m) {
      const c128 x = A[p * ld + ci];
      const c128 b = B ? B[p * ld + ci] : c128{0.0, 0.0};
      const double ai = a_conj ? -x.im : x.im;
      if (row & 1)
        f = doublex2{ai + b.im, x.re - b.re};     // Im (A + B), Im i (A - B)
      else
        f = doublex2{x.re + b.re, -(ai - b.im)};  // Re (A + B), Re i (A - B)
    }
    M[(grp * group + kb * (WROWS * BK)) / V + i * 64 + lane] = f;
  }
}

// Complex rows 2q, 2q + 1 of column j (both: of both halves), zero past m.
struct Rows2 {
  c128 a0, a1, b0, b1;
};
__device__ __forceinline__ Rows2 load_rows(const c128* X, int64_t ldx, int64_t m, int64_t q, int j, bool both) {
  Rows2 v{};
  const c128* x = X + (int64_t)j * ldx + 2 * q;
  const bool one = 2 * q < m, two = 2 * q + 1 < m;
  if (one) v.a0 = x[0];
  if (two) v.a1 = x[1];
  if (both && one) v.b0 = x[m];
  if (both && two) v.b1 = x[m + 1];
  return v;
}

// A wave takes 8 quads x 8 columns: 8 lanes along the rows of a column of X,
// and 8 along the columns of a quad row of X4.
__device__ __forceinline__ void pack_place(int64_t* q, int* j) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  *q = (int64_t)blockIdx.x * 32 + wave * 8 + (lane & 7);
  *j = blockIdx.y * 8 + (lane >> 3);
}

__global__ __launch_bounds__(256) void hx_pack_kernel(const c128* X, int64_t ldx, int64_t m, int k, int general,
                                                      double* Y, int64_t ldc4, int64_t k4, double* Z) {
  int64_t q;
  int j;
  pack_place(&q, &j);
  if (q >= k4 || j >= k) return;
  const Rows2 v = load_rows(X, ldx, m, q, j, general != 0);
  if (Z && 2 * q >= m) {  // zeros past row 2m of another block
    const int64_t at = q * ldc4 + (general ? 8 : 4) * j;
    store4(Z + at, doublex4{0, 0, 0, 0});
    if (general) store4(Z + at + 4, doublex4{0, 0, 0, 0});
  }
  if (!general) {
    store4(Y + q * ldc4 + 4 * j, doublex4{v.a0.re, v.a0.im, v.a1.re, v.a1.im});
    return;
  }
  double* y = Y + q * ldc4 + 8 * j;
  // a_u = (x1 + conj(x2)) / 2, a_v = (x1 - conj(x2)) / (2 i)
  store4(y, doublex4{0.5 * (v.a0.re + v.b0.re), 0.5 * (v.a0.im - v.b0.im), 0.5 * (v.a1.re + v.b1.re),
                     0.5 * (v.a1.im - v.b1.im)});
  store4(y + 4, doublex4{0.5 * (v.a0.im + v.b0.im), 0.5 * (v.b0.re - v.a0.re), 0.5 * (v.a1.im + v.b1.im),
                         0.5 * (v.b1.re - v.a1.re)});
}

// x1 = a_u + i a_v, x2 = conj(a_u) + i conj(a_v)
__global__ __launch_bounds__(256) void hx_unpack_kernel(const double* Y, int64_t ldc4, int64_t m, int k, int general,
                                                        c128* X, int64_t ldx) {
  int64_t q;
  int j;
  pack_place(&q, &j);
  if (2 * q >= m || j >= k) return;
  const bool two = 2 * q + 1 < m;
  c128* x = X + (int64_t)j * ldx + 2 * q;
  if (!general) {
    const doublex4 u = load4(Y + q * ldc4 + 4 * j);
    x[0] = c128{u[0], u[1]};
    if (two) x[1] = c128{u[2], u[3]};
    return;
  }
  const doublex4 u = load4(Y + q * ldc4 + 8 * j), v = load4(Y + q * ldc4 + 8 * j + 4);
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    if (r == 1 && !two) break;
    const double ur = u[2 * r], ui = u[2 * r + 1], vr = v[2 * r], vi = v[2 * r + 1];
    x[r] = c128{ur - vi, ui + vr};
    x[m + r] = c128{ur + vi, vr - ui};
  }
}

inline dim3 pack_grid(int64_t quads, int k) {
  return dim3((unsigned)ceil_div(quads, (int64_t)32), (unsigned)ceil_div(k, (int64_t)8));
}

}  // namespace

Err hx_make_operand(const c128* A, const c128* B, int64_t ld, int a_conj, double* M, int64_t m, hipStream_t s) {
  const int64_t total = hx_operand_reals(m) / V;
  const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(total, 256), 16384));
  hipLaunchKernelGGL(make_operand_kernel, dim3(blocks), dim3(256), 0, s, A, B, ld, a_conj, (doublex2*)M, m,
                     hx_rows(m), hx_cols(m), hx_group_reals(m));
  CHASE_LAUNCH_CHECK();
  return ok();
}

Err hx_step(const HxStep& a, void* ws, size_t ws_bytes, hipStream_t s) {
  if (a.N <= 0 || a.m <= 0) return ok();
  if (!a.M || !a.y || !a.out || a.ldc < ceil_div(a.N, (int64_t)16) * 16)
    return fail(CHASE_PH_ERR_ARG, "hx_step: operand or output missing");
  const int group = (int)std::min<int64_t>(a.N, hx_group(2 * a.m));
  for (int c0 = 0; c0 < a.N; c0 += group) {
    const int64_t off = 4 * (int64_t)c0;
    HxDev d = operand(a.M, a.m, a.y + off, a.ldc, std::min(group, a.N - c0));
    d.out = a.out + off;
    d.P = a.P ? a.P + off : nullptr;
    d.Q = a.Q ? a.Q + off : nullptr;
    d.alpha = a.alpha;
    d.beta = a.beta;
    d.gamma = a.gamma;
    d.rot = a.rot;
    CHASE_TRY(launch(d, ws, ws_bytes, s));
  }
  return ok();
}

Err hx_apply(const HxApply& a, void* ws, size_t ws_bytes, hipStream_t s) {
  if (a.k <= 0 || a.m <= 0) return ok();
  if (!a.M || !a.yr || a.kcap <= 0) return fail(CHASE_PH_ERR_ARG, "apply_h: operand or packed buffer missing");
  const int64_t ldc = hx_ldc(2 * (int64_t)a.kcap);
  const int per = a.kind == HX_GENERAL ? 2 : 1;  // real columns of one of X
  const int cap = (int)std::min<int64_t>(a.kcap, hx_group(2 * a.m) / per);
  for (int c0 = 0; c0 < a.k; c0 += cap) {
    const int k = std::min(cap, a.k - c0);
    CHASE_TRY(hx_pack(a.X + (int64_t)c0 * a.ldx, a.ldx, a.m, k, a.kind, a.yr, ldc, s));
    HxDev d = operand(a.M, a.m, a.yr, ldc, per * k);
    d.kind = a.kind;
    d.Yc = a.Y + (int64_t)c0 * a.ldy;
    d.ldy = a.ldy;
    CHASE_TRY(launch(d, ws, ws_bytes, s));
  }
  return ok();
}

Err hx_pack(const c128* X, int64_t ldx, int64_t m, int k, int kind, double* Y, int64_t ldc, hipStream_t s, double* Z) {
  if (k <= 0) return ok();
  const int64_t k4 = hx_k4(m);
  hipLaunchKernelGGL(hx_pack_kernel, pack_grid(k4, k), dim3(256), 0, s, X, ldx, m, k, kind == HX_GENERAL ? 1 : 0, Y,
                     4 * ldc, k4, Z);
  CHASE_LAUNCH_CHECK();
  return ok();
}

Err hx_unpack(const double* Y, int64_t ldc, int64_t m, int k, int kind, c128* X, int64_t ldx, hipStream_t s) {
  if (k <= 0) return ok();
  hipLaunchKernelGGL(hx_unpack_kernel, pack_grid(ceil_div(m, (int64_t)2), k), dim3(256), 0, s, Y, 4 * ldc, m, k,
                     kind == HX_GENERAL ? 1 : 0, X, ldx);
  CHASE_LAUNCH_CHECK();
  return ok();
}

}  // namespace chase
