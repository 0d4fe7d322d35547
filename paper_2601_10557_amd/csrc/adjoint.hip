// Eigenvalue adjoint as one contraction over the eigenvector pairs.
//
// For unit right eigenvectors v_j = [x_j; y_j] and weights
// gt_j = g_j / (x_j^H x_j - y_j^H y_j) (first-order perturbation with the
// left eigenvector u = S v, Thm 3.2 and eq. 3.5):
//   G_A = sum_j gt_j (x_j x_j^H + conj(y_j) y_j^T)     (Hermitian)
//   G_B = sum_j gt_j (x_j y_j^H + conj(y_j) x_j^T)     (complex symmetric)
// Both outputs share the left factor [gt x_j, gt conj(y_j)], so one kernel
// computes the tile (I, J) of both from one pass over the rows I and J of
// V, and, by the symmetry of both outputs, only tiles with I >= J are
// computed: the tile (J, I) is written from the same registers
// (conjugate transpose for G_A, transpose for G_B).
#include <mutex>

#include "common.h"
#include "vec.h"

// Fixed device memory of the allocation-free adjoint entry point
// (chase_ph_eigval_backward_noalloc): the host weights g (first
// CHASE_PH_NOALLOC_MAX_NEV doubles) and the scaled weights gt (the next
// CHASE_PH_NOALLOC_MAX_NEV).  Each device holds its own copy at its own
// address, resolved once per device with hipGetSymbolAddress; host code
// never passes the array's name itself to a kernel or a copy.
static __device__ __align__(256) double scratch[2 * CHASE_PH_NOALLOC_MAX_NEV];

namespace chase {
namespace {

constexpr int TB = 64;        // output tile (rows and columns)
constexpr int NT = 256;       // 4 waves, each a 32 x 32 quadrant of the tile

__device__ __forceinline__ doublex4 mfma64(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__global__ __launch_bounds__(256) void adjoint_weights_kernel(const c128* V, int64_t ldv, int64_t m, const double* g,
                                                              double* gt) {
  __shared__ double red[256];
  const int j = blockIdx.x;
  const c128* v = V + (int64_t)j * ldv;
  double s = 0;
  for (int64_t i = threadIdx.x; i < 2 * m; i += 256) {
    const double p = v[i].re * v[i].re + v[i].im * v[i].im;
    s += i < m ? p : -p;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) gt[j] = g[j] / red[0];
}

// Lower tile index t -> (I, J) with I >= J, t = I (I + 1) / 2 + J.
__device__ __forceinline__ void lower_tile(int64_t t, int64_t* I, int64_t* J) {
  int64_t i = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  while (i * (i + 1) / 2 > t) --i;
  while ((i + 1) * (i + 2) / 2 <= t) ++i;
  *I = i;
  *J = t - i * (i + 1) / 2;
}

// One 64 x 64 tile of both outputs, each wave a 32 x 32 quadrant.  Bound by the
// FP64 MFMA: 64 of them (4096 cycles) per four eigenpairs on eight 16-byte
// loads, so the fragments come straight from V one step ahead (lane l holds
// row l % 16, eigenpair l / 16) and no wave waits for another.  m = 4000,
// nev = 200: 800 us (64 TF/s, 512 MB written), 915 on LDS slabs with a barrier
// every two steps.
template <bool NT_STORES>
__global__ __launch_bounds__(NT, 2) void adjoint_kernel(const c128* __restrict__ V, int64_t ldv, int64_t m, int nev,
                                                        const double* __restrict__ gt, c128* GA, c128* GB,
                                                        int64_t ldg) {
  int64_t I, J;
  lower_tile(blockIdx.x, &I, &J);
  const int64_t r0 = I * TB, c0 = J * TB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  const int lr = lane & 15, lk = lane >> 4;
  // rows past m - 1 repeat it (their sums are not written), eigenpairs past
  // nev - 1 repeat it with weight 0
  int64_t rr[2], rc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    rr[i] = min(r0 + wr + 16 * i + lr, m - 1);
    rc[i] = min(c0 + wc + 16 * i + lr, m - 1);
  }
  struct Step {
    c128 p[2], q[2], x[2], y[2];
    double w;
  };
  auto load = [&](int k, Step& f) __attribute__((always_inline)) {
    const int j = min(k + lk, nev - 1);
    const c128* v = V + (int64_t)j * ldv;
    f.w = gt[j];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      f.p[i] = v[rr[i]];
      f.q[i] = v[m + rr[i]];
      f.x[i] = v[rc[i]];
      f.y[i] = v[m + rc[i]];
    }
  };

  doublex4 ar[2][2], ai[2][2], br[2][2], bi[2][2];   // G_A, G_B accumulators
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) ar[i][j][r] = ai[i][j][r] = br[i][j][r] = bi[i][j][r] = 0.0;

  Step cur, nxt;
  load(0, cur);
#pragma unroll 1
  for (int k = 0; k < nev; k += 4) {
    load(min(k + 4, nev - 1), nxt);
    __builtin_amdgcn_sched_barrier(0);
    const double w = k + lk < nev ? cur.w : 0.0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const double pr = w * cur.p[i].re, pi = w * cur.p[i].im;   // p = gt x_r
      const double qr = w * cur.q[i].re, qi = -w * cur.q[i].im;  // q = gt conj(y_r)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const double xr = cur.x[j].re, xi = cur.x[j].im, yr = cur.y[j].re, yi = cur.y[j].im;
        // G_A += p conj(x_c) + q y_c
        ar[i][j] = mfma64(pr, xr, ar[i][j]);
        ai[i][j] = mfma64(pi, xr, ai[i][j]);
        br[i][j] = mfma64(pr, yr, br[i][j]);
        bi[i][j] = mfma64(pi, yr, bi[i][j]);
        ar[i][j] = mfma64(pi, xi, ar[i][j]);
        ai[i][j] = mfma64(-pr, xi, ai[i][j]);
        // G_B += p conj(y_c) + q x_c
        br[i][j] = mfma64(pi, yi, br[i][j]);
        bi[i][j] = mfma64(-pr, yi, bi[i][j]);
        ar[i][j] = mfma64(qr, yr, ar[i][j]);
        ai[i][j] = mfma64(qr, yi, ai[i][j]);
        br[i][j] = mfma64(qr, xr, br[i][j]);
        bi[i][j] = mfma64(qr, xi, bi[i][j]);
        ar[i][j] = mfma64(-qi, yi, ar[i][j]);
        ai[i][j] = mfma64(qi, yr, ai[i][j]);
        br[i][j] = mfma64(-qi, xi, br[i][j]);
        bi[i][j] = mfma64(qi, xr, bi[i][j]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    cur = nxt;
  }

  // D = 16 x 16 block: lane holds rows (lane >> 4) + 4 r, column lane & 15
  typedef double doublex2 __attribute__((ext_vector_type(2)));
  auto put = [&](c128* p, double re, double im) __attribute__((always_inline)) {
    if constexpr (NT_STORES)
      __builtin_nontemporal_store(doublex2{re, im}, reinterpret_cast<doublex2*>(p));
    else
      *reinterpret_cast<doublex2*>(p) = doublex2{re, im};
  };
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gi = r0 + wr + 16 * i + (lane >> 4) + 4 * r;
        const int64_t gj = c0 + wc + 16 * j + (lane & 15);
        if (gi < m && gj < m) {
          put(GA + gj * ldg + gi, ar[i][j][r], ai[i][j][r]);
          put(GB + gj * ldg + gi, br[i][j][r], bi[i][j][r]);
          if (I != J) {
            put(GA + gi * ldg + gj, ar[i][j][r], -ai[i][j][r]);
            put(GB + gi * ldg + gj, br[i][j][r], bi[i][j][r]);
          }
        }
      }
}

}  // namespace

Err adjoint_contract(const c128* V, int64_t ldv, int64_t m, int nev, const double* dg, double* dgt, c128* GA,
                     c128* GB, int64_t ldg, hipStream_t s) {
  if (m <= 0 || nev <= 0) return ok();
  hipLaunchKernelGGL(adjoint_weights_kernel, dim3(nev), dim3(256), 0, s, V, ldv, m, dg, dgt);
  CHASE_LAUNCH_CHECK();
  const int64_t T = ceil_div(m, TB);
  const int64_t tiles = T * (T + 1) / 2;
  if (tiles > 0x7fffffffLL) return fail(CHASE_PH_ERR_ARG, "eigval_backward: m too large");
  // Stores past the L2 where columns start on 64 bytes, the four rows of one store,
  // while both outputs are at most 32 MiB or behind enough MFMAs (us, through the L2 /
  // past it: m = 800, nev = 20 43.6 / 41.4, m = 1000 45.3 / 43.9, 1300 47.5 / 49.0, 4000
  // 163 / 178, 8000 483 / 585; m = 4000, nev = 100 429 / 433, 200 816 / 804 on the handle).
  // Other columns write parts of lines, which only the L2 merges: m = 1777 61 / 109.
  const bool past = (m <= 1024 || nev >= 160) && ldg % 4 == 0 && ((uintptr_t)GA | (uintptr_t)GB) % 64 == 0;
  if (past)
    hipLaunchKernelGGL(adjoint_kernel<true>, dim3((unsigned)tiles), dim3(NT), 0, s, V, ldv, m, nev, dgt, GA, GB, ldg);
  else
    hipLaunchKernelGGL(adjoint_kernel<false>, dim3((unsigned)tiles), dim3(NT), 0, s, V, ldv, m, nev, dgt, GA, GB, ldg);
  CHASE_LAUNCH_CHECK();
  return ok();
}

namespace {

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
double* scratch_ptr[kMaxDevices] = {};
thread_local std::string noalloc_err;

// Device address of this device's copy of the scratch array (resolved on the
// first call on each device, with that device current).
Err scratch_on_current_device(double** out) {
  int dev = 0;
  CHASE_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(CHASE_PH_ERR_ARG, "eigval_backward_noalloc: device index out of range");
  std::lock_guard<std::mutex> lk(scratch_mu);
  if (!scratch_ptr[dev]) {
    void* p = nullptr;
    CHASE_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(CHASE_PH_ERR_HIP, "eigval_backward_noalloc: no device address for the scratch array");
    scratch_ptr[dev] = static_cast<double*>(p);
  }
  *out = scratch_ptr[dev];
  return ok();
}

Err backward_noalloc(int64_t m, int nev, const c128* V, int64_t ldv, const double* hG, c128* GA, c128* GB,
                     int64_t ldg, hipStream_t s) {
  double* ws = nullptr;
  CHASE_TRY(scratch_on_current_device(&ws));
  double* dg = ws;
  double* dgt = ws + CHASE_PH_NOALLOC_MAX_NEV;
  CHASE_HIP(hipMemcpyAsync(dg, hG, (size_t)nev * sizeof(double), hipMemcpyHostToDevice, s));
  CHASE_TRY(adjoint_contract(V, ldv, m, nev, dg, dgt, GA, GB, ldg, s));
  CHASE_HIP(hipStreamSynchronize(s));
  return ok();
}

}  // namespace

const char* noalloc_last_error() { return noalloc_err.c_str(); }

}  // namespace chase

extern "C" chase_ph_status chase_ph_eigval_backward_noalloc(int64_t m, int32_t nev, const void* dV, int64_t ldv,
                                                            const double* hG, void* dGA, void* dGB, int64_t ldg,
                                                            void* hip_stream) {
  using namespace chase;
  Err e;
  if (m <= 0 || nev <= 0 || !dV || !hG || !dGA || !dGB || ldv < 2 * m || ldg < m)
    e = fail(CHASE_PH_ERR_ARG, "eigval_backward_noalloc: bad arguments");
  else if (nev > CHASE_PH_NOALLOC_MAX_NEV)
    e = fail(CHASE_PH_ERR_ARG, "eigval_backward_noalloc: nev = " + std::to_string(nev) +
                                   " exceeds the fixed scratch of " + std::to_string(CHASE_PH_NOALLOC_MAX_NEV) +
                                   " pairs");
  else
    e = backward_noalloc(m, nev, (const c128*)dV, ldv, hG, (c128*)dGA, (c128*)dGB, ldg, (hipStream_t)hip_stream);
  if (e) {
    noalloc_err = e.msg;
    return e.st;
  }
  return CHASE_PH_OK;
}
