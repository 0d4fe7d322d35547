// Block-structured operator H X in FP64 from the blocks A, B (hx.hip).
//
// Everything runs on real coordinates.  A K-real vector [a; conj(a)] is held
// by the reals [Re a_0, Im a_0, Re a_1, ...] of a; a general column x = u + i v
// by the two K-real parts u, v (real columns 2j, 2j + 1), an m-row column of
// the Hermitian problem (TDA) by its own reals.  A block of N real columns in
// this form ("X4") is stored as X[k4][c][4]: four consecutive reals (two
// complex rows) of column c together, k4 = 0 .. hx_k4(m) - 1, column pitch
// hx_ldc(N).  Reals past 2m are zero.
#pragma once
#include "common.h"

namespace chase {

// The real operand M (2m x 2m): columns 2p, 2p + 1 are the reals of A[:, p] +
// B[:, p] and i (A[:, p] - B[:, p]), so that M maps the coordinates of a to
// those of t = A a + B conj(a).  Stored fragment by fragment in the order the
// MFMA lanes read it, rows padded to HX_RPAD and columns to HX_KPAD with zeros.
constexpr int HX_RPAD = 128, HX_KPAD = 64;

inline int64_t hx_rows(int64_t m) { return ceil_div(2 * m, (int64_t)HX_RPAD) * HX_RPAD; }
inline int64_t hx_cols(int64_t m) { return ceil_div(2 * m, (int64_t)HX_KPAD) * HX_KPAD; }
// reals of one 32-row group of M: a slab of 8 columns more than it holds, so
// that groups read in step do not start at a common multiple of the memory
// channels' period
inline int64_t hx_group_reals(int64_t m) { return 32 * (hx_cols(m) + 8); }
inline int64_t hx_operand_reals(int64_t m) { return hx_rows(m) / 32 * hx_group_reals(m); }
// quads of reals of one column, and the column pitch of a block of N columns
// (a 16-column fragment may start at any column)
inline int64_t hx_k4(int64_t m) { return hx_cols(m) / 4; }
inline int64_t hx_ldc(int64_t ncols) { return ceil_div(ncols, (int64_t)16) * 16 + 16; }
inline int64_t hx_block_reals(int64_t m, int64_t ncols) { return hx_k4(m) * hx_ldc(ncols) * 4; }

// M from the c128 blocks (column-major, ld); A is conj of its buffer when
// a_conj; B may be null (B = 0: the real form of A).
Err hx_make_operand(const c128* A, const c128* B, int64_t ld, int a_conj, double* M, int64_t m, hipStream_t s);

// Factor applied to M y: the recurrences on H^2 use H^2 = -J M J M on every
// real column (J = multiplication by i).
enum HxRot { HX_NONE = 0, HX_I = 1, HX_MINUS_I = 2 };

// One product on N real columns, X4 to X4 (pitch ldc for every block):
//   out = alpha rot(M y) + beta P + gamma Q
// P, Q optional; out may alias P or Q.
struct HxStep {
  const double* M = nullptr;
  int64_t m = 0, ldc = 0;
  int N = 0;
  const double* y = nullptr;
  double* out = nullptr;
  const double *P = nullptr, *Q = nullptr;
  double alpha = 1, beta = 0, gamma = 0;
  int rot = HX_NONE;
};
// ws: device workspace for the partial sums of tiles whose K range is shared
// by several workgroups (ws_bytes may be 0: then none is).
Err hx_step(const HxStep& a, void* ws, size_t ws_bytes, hipStream_t s);

// Column kinds of the complex blocks that hx_apply, hx_pack and hx_unpack take.
enum HxKind {
  HX_GENERAL = 0,  // n x k, two real columns each
  HX_KREAL = 1,    // n x k, every column [a; conj(a)]: one real column each
  HX_TDA = 2       // m x k: one real column each
};

// Y = H X (HX_TDA: A X) on k columns of complex X; yr holds the packed X
// (hx_block_reals(m, 2 kcap) reals); calls with more columns than that, or than
// the cache holds packed (hx_group), run in chunks.
struct HxApply {
  const double* M = nullptr;
  int64_t m = 0;
  int k = 0, kind = HX_GENERAL;
  const c128* X = nullptr;
  int64_t ldx = 0;
  c128* Y = nullptr;
  int64_t ldy = 0;
  double* yr = nullptr;
  int kcap = 0;
};
Err hx_apply(const HxApply& a, void* ws, size_t ws_bytes, hipStream_t s);

// Complex block -> X4 (pads written as zero, also those of the block Z, which
// products will be written to, if given) and back.
Err hx_pack(const c128* X, int64_t ldx, int64_t m, int k, int kind, double* Y, int64_t ldc, hipStream_t s,
            double* Z = nullptr);
Err hx_unpack(const double* Y, int64_t ldc, int64_t m, int k, int kind, c128* X, int64_t ldx, hipStream_t s);

}  // namespace chase
