// How a c128 product of hx.hip is cut into workgroups.  Plain host code, so that
// the rules can be checked without a GPU.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace chase {

constexpr int HX_BK = 8;           // reals of K per slab
constexpr int HX_FM = 2;           // 16-row fragments per wave
constexpr int HX_BM = 64 * HX_FM;  // rows per workgroup: four waves
constexpr int HX_MAX_WG = 512;     // two workgroups per CU
constexpr int HX_MAX_NL = 8;       // column fragments of the widest tile
// partial sums of the widest long product: two slots a workgroup
constexpr size_t HX_WS_MAX = (size_t)2 * HX_MAX_WG * HX_BM * 16 * HX_MAX_NL * sizeof(double);
// K slabs per stage: about as many loads in flight at every width
constexpr int hx_stage_slabs(int w) { return w <= 2 ? 4 : w <= 4 ? 2 : 1; }

// Shapes (16-row fragments, 16-column fragments) of the short products.
constexpr int HX_SHORT_SHAPES = 6;
constexpr int hx_short_f[HX_SHORT_SHAPES] = {1, 1, 2, 2, 2, 2}, hx_short_n[HX_SHORT_SHAPES] = {1, 2, 1, 2, 3, 4};

// Long product: TM strips x TN tiles of wq or wq + 1 (the first wr) fragments, KB
// stages of K per strip; team t of `teams` starts at stage
// unit * floor(t len / teams) of the TM * KB, with len = lq * teams + lr.
// Short product (shape >= 0): TN tiles, KB slabs.
struct HxPlan {
  int shape;
  int TM, TN, wq, wr, wmax, KB, teams, lr;
  int64_t lq, unit;
  double i_KB, i_teams;  // reciprocals
  int64_t slot;          // reals per partial-sum slot (two per workgroup)
};

inline int64_t hx_ceil(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Bytes of partial sums of a long plan: none where every part is whole strips.
inline size_t hx_plan_bytes(const HxPlan& p) {
  if (p.shape >= 0 || p.unit != 1 || p.TM % p.teams == 0) return 0;
  return 2 * (size_t)p.teams * p.TN * p.slot * sizeof(double);
}

// NB column fragments in TN tiles, the strips' (strip, K) range in equal parts for
// at most `most` teams (HX_MAX_WG / TN): at least two stages a part, so that none
// is empty, and as many as the workspace takes the partial sums of.  Whole strips
// where that leaves fewer teams than there are strips, and where these are exactly
// one workgroup of the widest tiles per CU (m = 2000, k = 512: 520 us, split in two
// 531; with tiles of 4 fragments split parts are the faster: k = 256 300 us
// against 315).
inline void hx_cut(HxPlan& p, int64_t rows2, int NB, int TN, int64_t most, size_t ws_bytes) {
  p.shape = -1;
  p.TM = (int)hx_ceil(rows2, HX_BM);
  p.TN = TN;
  p.wq = NB / TN;
  p.wr = NB % TN;
  p.wmax = p.wq + (p.wr ? 1 : 0);
  p.KB = (int)hx_ceil(rows2, (int64_t)hx_stage_slabs(p.wmax) * HX_BK);
  p.slot = (int64_t)HX_BM * 16 * p.wmax;
  int64_t teams = std::min(most, std::max<int64_t>(p.TM, (int64_t)p.TM * p.KB / 2));
  const int64_t fit = (int64_t)(ws_bytes / (2 * (size_t)TN * p.slot * sizeof(double)));
  const int64_t strips = std::min<int64_t>(p.TM, most);
  const bool one_per_cu = p.wq == HX_MAX_NL && (int64_t)p.TM * TN == HX_MAX_WG / 2;
  p.unit = 1;
  int64_t len = (int64_t)p.TM * p.KB;
  if (one_per_cu || (teams > fit && fit * hx_ceil(p.TM, strips) <= p.TM)) {
    p.unit = p.KB;
    len = p.TM;
    teams = strips;
  } else {
    teams = std::min(teams, fit);
  }
  p.teams = (int)teams;
  p.lq = len / teams;
  p.lr = (int)(len % teams);
  p.i_KB = 1.0 / p.KB;
  p.i_teams = 1.0 / p.teams;
}

// Estimate of a long plan's time: a team's widest tile, where the padding of
// unequal tiles shows, plus the partial sums (at 12 TB/s, mostly from the
// Infinity Cache).  Tiles of fewer than 5 fragments read more per MFMA.
// m = 4000: k = 130 (17 fragments) 549 us on 3 tiles, 573 on 5, 597 on 4; k = 260
// (33) 1037 on 5, 1071 on 6.
inline double hx_long_us(const HxPlan& p, int64_t rows2) {
  const double frag_us = HX_FM * 2 * 64 / 2400.0;  // MFMA time of one slab and column fragment
  static const double narrow[5] = {0, 1.2, 1.12, 1.06, 1.05};
  double w = p.wmax * (p.wmax < 5 ? narrow[p.wmax] : 1.0);
  // From m = 16000 on near ties go to the widest tiles: N = 384 in 4 tiles of 6
  // fragments or 3 of 8: m = 16000 11.9 / 11.5 ms, 20000 18.8 / 18.2, 30000 47 / 42
  // (N = 320, 4 of 5 or 3 of 7, is no tie: 35 / 43).
  if (rows2 >= 32000 && p.wmax < HX_MAX_NL) w *= 1.02;
  // slabs of a team's part; alone on its CU a workgroup takes half the time
  double part = (double)p.TM / p.teams;
  if (p.unit != 1) part = hx_ceil(p.TM, p.teams) * (p.teams * p.TN <= HX_MAX_WG / 2 ? 0.5 : 1.0);
  const double slabs = hx_ceil(rows2, HX_BK) * part;
  const double sums = p.unit != 1 ? 0 : 2.0 * HX_BM * 16 * p.wmax * p.TN * p.teams * sizeof(double);
  return slabs * frag_us * w + sums / 12e6;
}

inline double hx_long_plan(HxPlan& best, int64_t rows2, int64_t N, size_t ws_bytes) {
  const int NB = (int)hx_ceil(N, 16), t0 = (int)hx_ceil(NB, HX_MAX_NL);
  double us = 1e300;
  for (int t = t0; t <= std::min(NB, 3 * t0); ++t) {
    HxPlan p;
    hx_cut(p, rows2, NB, t, std::max(1, HX_MAX_WG / t), ws_bytes);
    const double e = hx_long_us(p, rows2);
    if (e < us) {
      us = e;
      best = p;
    }
  }
  return us;
}

inline void hx_set_short(HxPlan& p, int64_t rows2, int64_t N, int shape) {
  p = HxPlan{};
  p.shape = shape;
  p.TN = (int)hx_ceil(N, 16 * hx_short_n[shape]);
  p.KB = (int)hx_ceil(rows2, HX_BK);
}

// The shape that computes a short product soonest, or teams on long parts.  A
// CU's workgroups each cost 10.6 ns per slab and fragment pair (MFMA) and 5.8 per
// fragment loaded (L1), on top of 3.6 us; M comes from the caches at 10 TB/s or
// so, from HBM at 6 (4.5 where a workgroup reads only half of a 32-row group).
// Whole workgroups per CU count: that is what the teams' equal parts avoid, at
// the price of a second launch and of partial sums (5 us and 2.3 times the
// estimate of hx_long_us, M at 4.8 TB/s).  Measured (us a product; teams / this):
// m = 100, k = 30 11.9 / 4.0; m = 500, k = 30 15.1 / 6.5; m = 1000, k = 120
// 46.2 / 35.4; m = 2000, k = 35 61.0 / 53.2, k = 70 85.2 / 91; m = 3000, k = 35
// 111 / 128; m = 4000, k = 4 107 / 91, k = 32 158 / 136.
inline HxPlan hx_plan(int64_t rows2, int64_t N, size_t ws_bytes) {
  HxPlan p{};
  const double slabs = (double)hx_ceil(rows2, HX_BK);
  const double bytes = 8.0 * rows2 * rows2 * 1e-6;
  const bool cached = bytes < 256;
  auto overlap = [](double x, double y) { return std::max(x, y) + 0.2 * std::min(x, y); };
  double best = overlap(5.0 + 2.3 * hx_long_plan(p, rows2, N, ws_bytes), bytes / 4.8);
  for (int c = 0; c < HX_SHORT_SHAPES; ++c) {
    const int f = hx_short_f[c], n = hx_short_n[c];
    const int64_t rounds = hx_ceil(hx_ceil(rows2, 16 * f) * hx_ceil(N, 16 * n), HX_MAX_WG / 2);
    if (rounds > 4) continue;
    const double comp = 3.6 + slabs * rounds * (f * n * 0.0106 + (f + n) * 0.0058);
    const double mem = bytes / (cached ? 10.0 : f == 1 ? 4.5 : 6.0);
    const double us = overlap(comp, mem);
    if (us < best) {
      best = us;
      hx_set_short(p, rows2, N, c);
    }
  }
  return p;
}

// Real columns of one launch: as many as stay in the Infinity Cache (256 MB),
// whole tiles of 128.  Every strip of 128 rows reads all of them again, and the
// one slab that a fragment of y is loaded ahead does not cover HBM: m = 30000,
// N = 4800 (2.3 GB) 737 ms in one launch, 522 in launches of 512 columns (66 TF/s);
// N = 1536 216 / 168; m = 16000, N = 2400 75.3 / 73.5 (1024 columns).
inline int64_t hx_group(int64_t rows2) {
  return std::max<int64_t>(128, ((int64_t)256 << 20) / (8 * rows2) / 128 * 128);
}

// Workspace with which every product of up to N real columns runs as planned with
// unlimited room: none up to m = 850 or so (short products), 84 to 128 MiB above.
// With less, parts are fewer: m = 1050, 2 k = 544 in 70 MB ran 17 teams of 73 and took
// 195 us instead of 119, m = 1450, 2 k = 576 304 instead of 193.
inline size_t hx_workspace(int64_t rows2, int64_t N) {
  size_t most = 0;
  N = std::min(N, hx_group(rows2));
  for (int64_t c = 16; c < N + 16; c += 16)
    most = std::max(most, hx_plan_bytes(hx_plan(rows2, std::min(c, N), (size_t)1 << 40)));
  return most;
}

}  // namespace chase
