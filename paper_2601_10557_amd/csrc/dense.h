// Small dense FP64 kernels on padded kp x kp matrices (dense.hip).
#pragma once
#include "common.h"

namespace chase {

struct DenseWs {
  c128* panel = nullptr;   // kp_max x 64
  c128* tmp = nullptr;     // kp_max x 64 (batched 64 x 64 blocks)
  c128* U = nullptr;       // kp_max x 64 (a rotation block per Jacobi pair, of two rounds)
  c128 *k1 = nullptr, *k2 = nullptr, *k3 = nullptr, *k4 = nullptr;  // kp_max x kp_max each (jacobi_eigh)
  int* flag = nullptr;     // 4 ints: positives, negatives (select_positive), two Cholesky breakdowns
  int* pflag = nullptr;    // kp_max / 16 ints (Jacobi pair rotated?, of two rounds)
  double* dscalar = nullptr;  // 4 doubles
  void* gemm_ws = nullptr;     // split-K partials of the batched GEMMs (may be null)
  size_t gemm_ws_bytes = 0;
  void* hpin = nullptr;        // pinned host staging for small device-to-host reads (may be null)
  size_t hpin_bytes = 0;
  enum { COUNTS = 0, CHOL = 2, CHOL2 = 3 };  // places in flag
};

// Copy bytes (and bytes2) from device memory to host memory and wait for it:
// a kernel stores them in the pinned staging buffer of ws when they fit there
// (a runtime copy costs several times its launch), else by runtime copies.
Err d2h_small(void* host, const void* dev, size_t bytes, const DenseWs& ws, hipStream_t s, void* host2 = nullptr,
              const void* dev2 = nullptr, size_t bytes2 = 0);
// Copy bytes of host memory to device memory; the host buffer is free on
// return.  Up to 14 kB travel as kernel arguments, which needs no wait.
Err h2d_small(void* dev, const void* host, size_t bytes, hipStream_t s);

int pad64(int k);
// M = diag(inner) on the first k, pad on the rest; off-diagonals zeroed
// everywhere when zero_all, else only in the padded rows/columns.
Err fill_padded(c128* M, int kp, int k, double inner, double pad, bool zero_all, hipStream_t s,
                int* clear = nullptr, int nclear = 1);  // clear[0 .. nclear - 1] = 0 too
// In place lower Cholesky of a Hermitian padded matrix (lower triangle given)
// and X = L^{-1} (chol.hip; both ld kp); ws.flag[slot] != 0 on breakdown, both
// then unspecified.
Err cholesky_inverse(c128* M, c128* X, int kp, DenseWs& ws, hipStream_t s, int slot);
// X = L^{-1} for lower-triangular L (both kp x kp, ld kp); X must not alias L.
Err tri_inverse_lower(const c128* L, c128* X, int kp, DenseWs& ws, hipStream_t s);
// G (Hermitian, in place) -> eigenvalues theta on the diagonal, V ->
// eigenvectors, by at most max_sweeps block Jacobi sweeps and by GEMM refinement
// steps, which are not counted.  guard >= 0: if ws.flag[guard] is set, *tripped
// and nothing else.
Err jacobi_eigh(c128* G, c128* V, int kp, DenseWs& ws, hipStream_t s, int max_sweeps, int* sweeps_out,
                int guard = -1, bool* tripped = nullptr);
// Positive eigenvalues theta of the first k: Ysel (kp x k/2, ld kp) and
// dlam[r] = 1/theta for rank r by descending theta; the numbers of positive
// and negative ones in ws.flag[COUNTS] and the next (columns of Ysel past the
// first are unspecified).  Follows jacobi_eigh, which leaves ||G||_F in dscalar
// and the counters at zero.
Err select_positive(const c128* G, const c128* V, int k, int kp, c128* Ysel, double* dlam, DenseWs& ws,
                    hipStream_t s);
// dst (rows x half) <- src if select_positive found half positive and half
// negative eigenvalues, else nothing.
Err copy_if_resolved(const c128* src, int64_t lds, c128* dst, int64_t ldd, int rows, int half, DenseWs& ws,
                     hipStream_t s);

// Householder QR (householder.hip): panels of HH_PANEL columns, row-parallel
// launches of HH_PARTS one-wave workgroups.
constexpr int HH_PANEL = 32;
constexpr int HH_PARTS = 512;
struct HouseholderWs {
  c128* Q = nullptr;        // n x kmax (ld n): the accumulated basis
  c128* Vb = nullptr;       // n x HH_PANEL (ld n): explicit reflectors of one panel
  c128* Tb = nullptr;       // HH_PANEL x kmax: compact WY factor of every panel
  c128* W1 = nullptr;       // HH_PANEL x kmax
  c128* W2 = nullptr;       // HH_PANEL x kmax
  c128* taus = nullptr;     // kmax
  double* part = nullptr;   // HH_PARTS
  c128* dpart = nullptr;    // HH_PARTS x HH_PANEL
  double* dsign = nullptr;  // kmax
  int kmax = 0;
  void* gemm_ws = nullptr;  // split-K partials of the GEMMs (may be null)
  size_t gemm_ws_bytes = 0;
};
// In place: X (n x k, ld ldx) -> Q with Q^H Q = I and, if R is non-null,
// R (k x k, ld ldr) upper triangular with a real non-negative diagonal and
// X = Q R (any rank; k <= n, k <= w.kmax).
Err householder_qr(c128* X, int64_t ldx, int64_t n, int k, c128* R, int64_t ldr, const HouseholderWs& w,
                   hipStream_t s);

}  // namespace chase
