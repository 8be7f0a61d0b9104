// FP64 ratio-tap construction on the device (Sec. V.A) and the fitted
// template norms (Sec. VI.B).
//
// Weighted ridge least squares: minimise sum_i u_i |R_i - A_i|^2 + lam |a|^2
// with u_i = w_i |h_ref,i|^2, R = h/h_ref, A_i = sum_k a_k exp(-2 pi i i
// (k0+k)/N).  Setting the gradient to zero gives the normal equations
//     (M + lam I) a = b,  M[l,k] = g[l-k],  g[m] = sum_i u_i exp(+2 pi i i m/N),
//     b[l] = sum_i w_i h_i conj(h_ref,i) exp(+2 pi i i (k0+l)/N),
// a Hermitian Toeplitz system shared by the whole sub-bank: g and every b
// come from FP64 FFTs (fft.hip), M + lam I is factored once per sub-bank
// (L L^H, by the Schur recursion that its Toeplitz structure allows), and each
// template costs two triangular solves.
// Norm of the fitted template h_fit = h_ref A (Parseval form of Sec. VI.B):
//     sigma_fit^2 = sum_i w_i |h_ref A|^2 = a^H M a.
// The FIR applies c = conj(a) sigma_ref / sigma_fit to zhat = z_ref/sigma_ref,
// so its output is directly the normalised SNR of h_fit.
#include <algorithm>
#include <chrono>
#include <thread>

#include "dev_common.h"
#include "rfd_internal.h"

namespace rfd {

__device__ __forceinline__ double2 gval(const double2* g, int m) {
  return m >= 0 ? g[m] : cconj(g[-m]);
}

// Cholesky factor L (column-major, zeros above the diagonal) of the ridge
// normal matrix M + lam I, lam = eps g[0].  M[l][k] = g[l - k] is Hermitian
// Toeplitz, so its factor follows from the Schur recursion on M's
// displacement generators in O(T^2) work instead of the O(T^3) of a general
// Cholesky.  With Z the down-shift and r = (g[0] + lam, g[1], ..., g[T-1]) the
// first column, M + lam I - Z (M + lam I) Z^H = u u^H - v v^H for
// u = r / sqrt(r[0]) and v = u with v[0] = 0.  Column k of L is the current
// u; the next Schur complement has generators (Z u, v), which a hyperbolic
// rotation with rho = v[k+1] / u[k] returns to the form v[k+1] = 0:
//   v <- (v - rho Z u) / s,   u <- s Z u - conj(rho) v,   s = sqrt(1 - |rho|^2),
// the "mixed" order of the two updates, which keeps the recursion backward
// stable for positive-definite matrices.  |rho| >= 1 means M + lam I is not
// positive definite: info = step + 1.  One workgroup, T dependent steps.
constexpr int kSchurPer = (RFD_MAX_TAPS + 1023) / 1024;   // elements per thread
__global__ __launch_bounds__(1024) void k_schur_chol(const double2* __restrict__ g, int T, double eps,
                                                     double2* __restrict__ L, int* __restrict__ info) {
  __shared__ double2 u[RFD_MAX_TAPS], v[RFD_MAX_TAPS];
  const double r0 = g[0].x + eps * g[0].x;
  if (!(r0 > 0.0)) {                      // uniform
    if (threadIdx.x == 0) *info = 1;
    return;
  }
  const double inv = 1.0 / sqrt(r0);
  for (int i = threadIdx.x; i < T; i += 1024) {
    const double2 r = i == 0 ? make_double2(r0, 0.0) : g[i];
    const double2 x = make_double2(r.x * inv, r.y * inv);
    u[i] = x;
    v[i] = i == 0 ? make_double2(0.0, 0.0) : x;
    L[i] = x;                             // column 0
  }
  __syncthreads();
  for (int k = 0; k + 1 < T; ++k) {
    const double a = u[k].x;              // L[k][k]: real and positive
    const double2 b = v[k + 1];
    const double2 rho = make_double2(b.x / a, b.y / a);
    const double q = 1.0 - (rho.x * rho.x + rho.y * rho.y);
    double2 zu[kSchurPer], vi[kSchurPer];
#pragma unroll
    for (int e = 0; e < kSchurPer; ++e) {
      const int i = threadIdx.x + 1024 * e;
      if (i > k && i < T) {
        zu[e] = u[i - 1];
        vi[e] = v[i];
      }
    }
    __syncthreads();                      // every read of step k is done
    if (!(q > 0.0)) {                     // uniform: the same q in every thread
      if (threadIdx.x == 0) *info = k + 2;
      return;
    }
    const double s = sqrt(q), is = 1.0 / s;
    double2* col = L + (int64_t)(k + 1) * T;
#pragma unroll
    for (int e = 0; e < kSchurPer; ++e) {
      const int i = threadIdx.x + 1024 * e;
      if (i >= T) continue;
      if (i <= k) {
        col[i] = make_double2(0.0, 0.0);
        continue;
      }
      double2 un, vn;
      if (i == k + 1) {                   // the rotated pair: v exactly 0, u = s a
        vn = make_double2(0.0, 0.0);
        un = make_double2(s * a, 0.0);
      } else {
        vn = make_double2((vi[e].x - (rho.x * zu[e].x - rho.y * zu[e].y)) * is,
                          (vi[e].y - (rho.x * zu[e].y + rho.y * zu[e].x)) * is);
        un = make_double2(s * zu[e].x - (rho.x * vn.x + rho.y * vn.y),
                          s * zu[e].y - (rho.x * vn.y - rho.y * vn.x));
      }
      u[i] = un;
      v[i] = vn;
      col[i] = un;
    }
    __syncthreads();
  }
}

// U = L^H (column-major upper triangle)
__global__ void k_upper(const double2* __restrict__ L, int T, double2* __restrict__ U) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < (int64_t)T * T;
       e += (int64_t)gridDim.x * blockDim.x) {
    int col = (int)(e / T), row = (int)(e % T);
    U[e] = row <= col ? cconj(L[(int64_t)row * T + col]) : make_double2(0.0, 0.0);
  }
}

// Inverses of the 64 x 64 diagonal blocks of L, column-major, the last one padded with the identity: one workgroup
// per block, in LDS.  Its four 16 x 16 diagonal tiles by substitution, a column per lane; then, a row of tiles at a time,
// X = -L_ii^-1 (L_i0 .. L_i,i-1) X above.  Bound by the latency of the substitutions and sums; a substitution over all 64
// rows took 86 us, half of the first call for a sub-bank of short filters, now 24.
constexpr int kTrsmBlock = 64;
__global__ __launch_bounds__(256) void k_diag_inv(const double2* __restrict__ L, int T, double2* __restrict__ inv) {
  constexpr int N = kTrsmBlock, S = N + 1, B = 16;
  extern __shared__ double2 sh[];
  double2* blk = sh;               // [row][col]
  double2* x = sh + N * S;         // [row][col], the inverse
  const int o = blockIdx.x * N;
  for (int e = threadIdx.x; e < N * N; e += 256) {
    const int r = e % N, c = e / N;
    double2 v = make_double2(c == r ? 1.0 : 0.0, 0.0);
    if (o + r < T && o + c < T && r >= c) v = L[(int64_t)(o + c) * T + o + r];
    blk[r * S + c] = v;
    x[r * S + c] = make_double2(0.0, 0.0);
  }
  __syncthreads();
  if (threadIdx.x < N) {
    const int c = threadIdx.x, t0 = c / B * B;
    const double2* tile = blk + t0 * S + t0;
    double2 y[B];                          // (zero above the diagonal)
#pragma unroll
    for (int r = 0; r < B; ++r) {
      double2 s = make_double2(t0 + r == c ? 1.0 : 0.0, 0.0);
#pragma unroll
      for (int k = 0; k < r; ++k) s = csub(s, cmul(tile[r * S + k], y[k]));
      const double d = 1.0 / tile[r * S + r].x;
      y[r] = make_double2(s.x * d, s.y * d);
      x[(t0 + r) * S + c] = y[r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = B; i < N; i += B) {         // rows i .. i + B - 1 of the columns before i
    if (o + i >= T) break;                 // (those of the identity)
    for (int e = threadIdx.x; e < B * i; e += 256) {
      const int r = i + e / i, c = e % i;
      double2 s = make_double2(0.0, 0.0);
      for (int k0 = c / B * B; k0 < i; k0 += B)
#pragma unroll
        for (int k = k0; k < k0 + B; ++k) s = csub(s, cmul(blk[r * S + k], x[k * S + c]));
      x[r * S + c] = s;
    }
    __syncthreads();
    double2 y[B * (N - B) / 256];
#pragma unroll
    for (int u = 0; u < B * i / 256; ++u) {
      const int e = threadIdx.x + 256 * u, r = i + e / i, c = e % i;
      y[u] = make_double2(0.0, 0.0);
#pragma unroll
      for (int k = i; k < i + B; ++k) y[u] = cadd(y[u], cmul(x[r * S + k], x[k * S + c]));
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < B * i / 256; ++u) {
      const int e = threadIdx.x + 256 * u;
      x[(i + e / i) * S + e % i] = y[u];
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < N * N; e += 256) inv[(int64_t)blockIdx.x * N * N + e] = x[(e % N) * S + e / N];
}

// (L L^H) a = b for TPW templates per workgroup on the FP64 matrix cores: their right-hand sides stay
// in LDS as 2 TPW real columns, X = [Re | Im], through a forward sweep with L and a backward
// sweep with U = L^H in block rows of 64.  Off the diagonal a block row is a complex GEMM,
// L X = Re L [Re | Im] + Im L [-Im | Re], one v_mfma_f64_16x16x4 for either part of four columns of L;
// wave w takes 16 of the 64 rows, its operands come straight from L2 eight steps ahead.  The
// diagonal block is a product with its inverse, D, refined once: x = D r, x += D (r - L_ii x).  Without,
// the residual of the solve carries the block's condition where a substitution's carries none (T = 64: 3e-16 of
// |M| |a| against 2e-17 at a ridge of 1e-4, 2e-13 against 1e-17 at 1e-10), and the taps are 2 to 30 times further
// from the exact solution.  Bound by the matrix cores where count fills the chip: 2 T^2 / 4 / 16 / 4
// pairs of 64-cycle instructions per wave, 0.4 ms at T = 1024 however few the templates, and three more
// block products per block row.  256 templates at T = 1024: 2836 us with one wave per template
// sweeping the factor's columns -> 520 us (424 unrefined); 500 at T = 256: 178 -> 70 us (47 unrefined).
typedef __attribute__((ext_vector_type(4))) double f64x4;
// N: rows of a block; 16, one wave, for T <= 16 (calls of 8 templates at T = 8: 39.7 -> 32.4 us each).
template <int TPW, int N = kTrsmBlock>
__global__ __launch_bounds__(4 * N) void k_trsm(const double2* __restrict__ L, const double2* __restrict__ U,
                                              const double2* __restrict__ inv, int T, const double2* __restrict__ b,
                                              int64_t bstride, double2* __restrict__ a, int64_t astride,
                                              int64_t count) {
  constexpr int NC = 2 * TPW;
  extern __shared__ __align__(16) double X[];       // [nb N][NC]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nb = (T + N - 1) / N;
  const int64_t t0 = (int64_t)blockIdx.x * TPW;
  for (int e = threadIdx.x; e < nb * N * TPW; e += 4 * N) {
    const int tt = e / (nb * N), row = e % (nb * N);
    const double2 v = row < T && t0 + tt < count ? b[(t0 + tt) * bstride + row] : make_double2(0.0, 0.0);
    X[row * NC + tt] = v.x;
    X[row * NC + TPW + tt] = v.y;
  }
  __syncthreads();
  // matrix operands: lane holds row lane % 16 (A) or column lane % 16 (B) at k = lane / 16; results: row
  // 4 v + lane / 16 and column lane % 16 in register v
  const int kq = lane >> 4, col = (lane & 15) % NC, mate = col ^ TPW;
  const double sgn = col < TPW ? -1.0 : 1.0;
  // p + q += M X over columns [c0, c1) of the factor (c0, c1 multiples of 64, columns past T read T - 1
  // and meet zero rows of X)
  auto gemm = [&](const double2* M, int row, int c0, int c1, f64x4& p, f64x4& q) {
    auto fetch = [&](double2 (&m)[8], int c) {
#pragma unroll
      for (int u = 0; u < 8; ++u) m[u] = M[(int64_t)min(c + 4 * u + kq, T - 1) * T + row];
    };
    auto products = [&](const double2 (&m)[8], int c) {
      __builtin_amdgcn_sched_barrier(0);       // the next loads leave before this step's products
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double* x = X + (c + 4 * u + kq) * NC;
        p = __builtin_amdgcn_mfma_f64_16x16x4f64(m[u].x, x[col], p, 0, 0, 0);
        q = __builtin_amdgcn_mfma_f64_16x16x4f64(m[u].y, x[mate], q, 0, 0, 0);
      }
    };
    double2 m[8], n[8];
    if (c0 < c1) fetch(m, c0);
    for (int c = c0; c < c1; c += 64) {        // two sets in turn: moving one to the other would wait for it
      fetch(n, c + 32);
      products(m, c);
      fetch(m, min(c + 64, c1 - 32));
      products(n, c + 32);
    }
  };
  const bool mine = (lane & 15) < NC;
  for (int sweep = 0; sweep < 2; ++sweep) {
    for (int s = 0; s < nb; ++s) {
      const int i = sweep ? nb - 1 - s : s;
      const int r0 = i * N + 16 * wave;                       // this wave's rows
      // the diagonal block's operands (inv(L_ii) or its conjugate transpose, L_ii or U_ii), loaded ahead of the GEMM
      const double2 *D = inv + (int64_t)i * kTrsmBlock * kTrsmBlock, *F = sweep ? U : L;
      const int row = min(r0 + (lane & 15), T - 1);
      double2 dm[N / 4], fm[N / 4];
#pragma unroll
      for (int u = 0; u < N / 4; ++u) {
        const int k = 4 * u + kq, r = 16 * wave + (lane & 15);
        dm[u] = sweep ? D[r * kTrsmBlock + k] : D[k * kTrsmBlock + r];
        if (sweep) dm[u].y = -dm[u].y;
        fm[u] = F[(int64_t)min(i * N + k, T - 1) * T + row];
      }
      f64x4 p = {0.0, 0.0, 0.0, 0.0}, q = {0.0, 0.0, 0.0, 0.0};
      if (sweep) gemm(F, row, (i + 1) * N, nb * N, p, q);
      else gemm(F, row, 0, i * N, p, q);
      auto product = [&](const double2 (&m)[N / 4]) {         // with the block's rows of X; all of them are read on return
        p = q = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < N / 4; ++u) {
          const double* x = X + (i * N + 4 * u + kq) * NC;
          p = __builtin_amdgcn_mfma_f64_16x16x4f64(m[u].x, x[col], p, 0, 0, 0);
          q = __builtin_amdgcn_mfma_f64_16x16x4f64(m[u].y, x[mate], q, 0, 0, 0);
        }
        __syncthreads();
      };
      auto put = [&](const double (&x)[4]) {                  // rows from T on stay zero
        if (mine) {
#pragma unroll
          for (int v = 0; v < 4; ++v) X[(r0 + 4 * v + kq) * NC + col] = r0 + 4 * v + kq < T ? x[v] : 0.0;
        }
        __syncthreads();
      };
      double res[4], sol[4], x[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) res[v] = X[(r0 + 4 * v + kq) * NC + col] - (p[v] + sgn * q[v]);
      put(res);
      product(dm);
#pragma unroll
      for (int v = 0; v < 4; ++v) sol[v] = p[v] + sgn * q[v];
      put(sol);
      product(fm);
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = res[v] - (p[v] + sgn * q[v]);
      put(x);
      product(dm);
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = sol[v] + (p[v] + sgn * q[v]);
      put(x);
    }
  }
  for (int e = threadIdx.x; e < T * TPW; e += 4 * N) {
    const int tt = e / T, row = e % T;
    if (t0 + tt < count) a[(t0 + tt) * astride + row] = make_double2(X[row * NC + tt], X[row * NC + TPW + tt]);
  }
}

// Windowed variant: a = tukey(0.25) * (truncated inverse transform of R).
__device__ double tukey(int l, int T) {
  const double alpha = 0.25;
  if (T == 1) return 1.0;
  const double x = (double)l / (double)(T - 1);
  const double pi = 3.141592653589793238462643;
  if (x < alpha / 2) return 0.5 * (1.0 + cos(pi * (2.0 * x / alpha - 1.0)));
  if (x > 1.0 - alpha / 2) return 0.5 * (1.0 + cos(pi * (2.0 * x / alpha - 2.0 / alpha + 1.0)));
  return 1.0;
}

// The same sweeps in launches, one per block row, for banks too small to fill the chip with a workgroup per
// eight templates.  Launch j has the solution of block j: a workgroup takes 64 rows of eight templates and
// subtracts that block's share from their residual, X_i -= M_ij X_j, and the one whose rows come next
// solves them as well (j = -1 before the first block: that alone).  Solutions go to `x`, other residuals to r; src is
// r, or the right-hand sides until r holds them.  Bound by the latency of each launch, 8 us with one
// template at T = 1024 and 11 with 256 (364 us for the solve in place of 520).  With the block solved
// again in every workgroup of the next launch the refinement took 4.3 us per launch, here 2.2.
template <bool BACK>
__global__ __launch_bounds__(256) void k_trsm_step(const double2* __restrict__ M, const double2* __restrict__ inv, int T,
                                                 int j, const double2* src, int64_t src_stride, double2* r,
                                                 double2* x, int64_t xstride, int64_t count) {
  constexpr int TPW = 8, NC = 16, N = kTrsmBlock;
  __shared__ double X[2][N * NC];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kq = lane >> 4, col = lane & 15, mate = col ^ TPW;
  const double sgn = col < TPW ? -1.0 : 1.0;
  const int64_t t0 = (int64_t)blockIdx.x * TPW;
  const int i = BACK ? (j < 0 ? (T - 1) / N : j - 1 - (int)blockIdx.y) : j + 1 + (int)blockIdx.y;
  const bool solve = blockIdx.y == 0;
  const int row = 16 * wave + col;                            // of the block: the one whose operands this lane holds
  const int own = (16 * wave + kq) * NC + col;                // this lane's values of X: own + 4 v NC, real or
  const bool re = col < TPW;                                  // imaginary part of template col % 8 ...
  const int64_t tmpl = t0 + col % TPW;
  const int g0 = i * N + 16 * wave + kq;                      // ... at rows g0 + 4 v
  double2 m[N / 4], dm[N / 4], fm[N / 4];
  if (j >= 0) {
    for (int e = threadIdx.x; e < N * TPW; e += 256) {
      const int tt = e / N, k = e % N;
      const double2 v = j * N + k < T && t0 + tt < count ? x[(t0 + tt) * xstride + j * N + k] : make_double2(0.0, 0.0);
      X[0][k * NC + tt] = v.x;
      X[0][k * NC + TPW + tt] = v.y;
    }
#pragma unroll
    for (int u = 0; u < N / 4; ++u)
      m[u] = M[(int64_t)min(j * N + 4 * u + kq, T - 1) * T + min(i * N + row, T - 1)];
  }
  double res[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    res[v] = 0.0;
    if (g0 + 4 * v < T && tmpl < count) {
      const double2 y = src[tmpl * src_stride + g0 + 4 * v];
      res[v] = re ? y.x : y.y;
    }
  }
  if (solve) {
    const double2* D = inv + (int64_t)i * N * N;
#pragma unroll
    for (int u = 0; u < N / 4; ++u) {
      dm[u] = BACK ? D[row * N + 4 * u + kq] : D[(4 * u + kq) * N + row];
      if (BACK) dm[u].y = -dm[u].y;
      fm[u] = M[(int64_t)min(i * N + 4 * u + kq, T - 1) * T + min(i * N + row, T - 1)];
    }
  }
  f64x4 p, q;
  auto product = [&](const double2 (&a)[N / 4], const double* y) {
    p = q = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < N / 4; ++u) {
      p = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].x, y[(4 * u + kq) * NC + col], p, 0, 0, 0);
      q = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].y, y[(4 * u + kq) * NC + mate], q, 0, 0, 0);
    }
  };
  auto put = [&](double* y, const double (&v)[4]) {           // rows from T on stay zero
#pragma unroll
    for (int e = 0; e < 4; ++e) y[own + 4 * e * NC] = g0 + 4 * e < T ? v[e] : 0.0;
    __syncthreads();
  };
  auto store = [&](double2* to, int64_t stride, const double (&v)[4]) {
    double* o = reinterpret_cast<double*>(to);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (g0 + 4 * e < T && tmpl < count) o[2 * (tmpl * stride + g0 + 4 * e) + (re ? 0 : 1)] = v[e];
  };
  if (j >= 0) {
    __syncthreads();
    product(m, X[0]);
#pragma unroll
    for (int v = 0; v < 4; ++v) res[v] -= p[v] + sgn * q[v];
  }
  if (!solve) {
    store(r, T, res);
    return;
  }
  double sol[4], z[4];                                        // as in k_trsm, X[0] and X[1] in turn
  put(X[1], res);
  product(dm, X[1]);
#pragma unroll
  for (int v = 0; v < 4; ++v) sol[v] = p[v] + sgn * q[v];
  put(X[0], sol);
  product(fm, X[0]);
#pragma unroll
  for (int v = 0; v < 4; ++v) z[v] = res[v] - (p[v] + sgn * q[v]);
  put(X[1], z);
  product(dm, X[1]);
#pragma unroll
  for (int v = 0; v < 4; ++v) sol[v] += p[v] + sgn * q[v];
  store(x, xstride, sol);
}

__global__ void k_window(const double2* __restrict__ b, int64_t bstride, int T, int64_t count,
                         double2* __restrict__ a, int64_t astride) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count * T;
       e += (int64_t)gridDim.x * blockDim.x) {
    int64_t t = e / T;
    int l = (int)(e % T);
    double2 v = b[t * bstride + l];
    double wv = tukey(l, T);
    a[t * astride + l] = make_double2(v.x * wv, v.y * wv);
  }
}

// sigma_fit^2 = a^H M a, M[l,k] = g[l-k], for eight templates per workgroup on the FP64 matrix cores: as in k_trsm their
// taps are X = [Re | Im], M a is Re M [Re | Im] + Im M [-Im | Re], and the norm is the sum of its product with X.
// M is Hermitian: what lies left of the 16 x 16 tiles on its diagonal counts twice, what lies right of them not at all.
// A wave takes a row of tiles and its mirror (of the same work together, whichever the row); the taps pass through LDS in
// panels, in runs along each template (as operands from L2 eight templates met one channel of it at a time, a power of two
// apart).  Up to T = 128 a group's rows are one workgroup's of four waves, up to 256 of eight; beyond, they are spread
// over workgroups, whose parts k_sigma_sum adds.  Bound by the matrix cores and, at small T, by the latency of its panels:
// 256 templates at T = 1024 in 27 us and 5 for the parts (345 by products of one row at a time, 41 from L2), 500
// at T = 256 in 13 (10 + 5 in parts).
// The sum over the normal equations, Re(a^H b) - lam |a|^2, has T products per template and not T^2, but its
// error is the solve's residual at small ridges and a difference of large numbers at large ones: 3e-14
// of the norm against 1e-15 at T = 200 and a ridge of 1e-4, 2e-10 against 2e-11 at 1e-8, 3e-9 against 1e-16 at 1e8.
constexpr int kSigmaParts = RFD_MAX_TAPS / 16 / 2 / 4;
constexpr int64_t kSigmaBatch = 4096;
constexpr int kSigmaPanel = 128, kSigmaStride = 17;      // columns of a panel; values from one to the next (odd: banks)
static int sigma_parts(int T) { return T <= 256 ? 1 : ((T + 15) / 16 + 7) / 8; }
size_t sigma_part_values(int T, int64_t count) {
  static_assert(kSigmaParts * 128 == RFD_MAX_TAPS, "a wave has a row of tiles and its mirror");
  const int parts = sigma_parts(T);
  return parts > 1 ? (size_t)(parts * std::min(count, kSigmaBatch)) : 0;
}
// part: [gridDim.y][count], or with one workgroup per group NULL and the norms to sigma
template <int W>
__global__ __launch_bounds__(64 * W) void k_sigma_fit(const double2* __restrict__ a, int64_t astride, int T,
                                                 const double2* __restrict__ g, int64_t count,
                                                 double* __restrict__ part, double* __restrict__ sigma) {
  constexpr int TPW = 8, PW = kSigmaPanel, ST = kSigmaStride, NT = 64 * W;
  extern __shared__ double2 gs[];                     // g, then two panels [PW][ST]
  double* panels = reinterpret_cast<double*>(gs + T);
  __shared__ double red[W][TPW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kq = lane >> 4, col = lane & 15;
  const int64_t t0 = (int64_t)blockIdx.x * TPW;
  double2 next[PW * TPW / NT];
  auto fetch = [&](int c) {
#pragma unroll
    for (int i = 0; i < PW * TPW / NT; ++i) {
      const int e = threadIdx.x + NT * i, tt = e / PW, k = c + e % PW;
      next[i] = k < T && t0 + tt < count ? a[(t0 + tt) * astride + k] : make_double2(0.0, 0.0);
    }
  };
  auto store = [&](double* x) {
#pragma unroll
    for (int i = 0; i < PW * TPW / NT; ++i) {
      const int e = threadIdx.x + NT * i, tt = e / PW, k = e % PW;
      x[k * ST + tt] = next[i].x;
      x[k * ST + TPW + tt] = next[i].y;
    }
  };
  fetch(0);
  for (int i = threadIdx.x; i < T; i += NT) gs[i] = g[i];
  store(panels);
  __syncthreads();
  const int nt = (T + 15) / 16, unit = blockIdx.y * W + wave;
  // first rows of the two tiles, T where the wave has none; the lane holds M operands of row r0 + col (of row T - 1
  // past the end, where they meet zeros)
  const int rows[2] = {2 * unit < nt ? 16 * unit : T, nt - 1 - unit > unit ? 16 * (nt - 1 - unit) : T};
  f64x4 p[2], q[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) p[h] = q[h] = f64x4{0.0, 0.0, 0.0, 0.0};
  const double sgn = col < TPW ? -1.0 : 1.0;
  double acc = 0.0;
  for (int c0 = 0, b = 0; c0 < T; c0 += PW, b ^= 1) {
    const double* x = panels + b * PW * ST;
    if (c0 + PW < T) fetch(c0 + PW);
    auto product = [&](int h, double2 m, int k) {      // column c0 + k
      p[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(m.x, x[k * ST + col], p[h], 0, 0, 0);
      q[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(m.y, x[k * ST + (col ^ TPW)], q[h], 0, 0, 0);
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r0 = rows[h];
      if (r0 >= T) continue;
      const double2* m = gs + min(r0 + col, T - 1) - c0;
      const int left = min(r0 - c0, PW);                // columns of the panel left of the diagonal tile
      for (int k = 0; k < left; k += 16) {
#pragma unroll
        for (int u = 0; u < 4; ++u) product(h, m[-(k + kq + 4 * u)], k + kq + 4 * u);
      }
      if (r0 < c0 || r0 >= c0 + PW) continue;
      p[h] *= 2.0;
      q[h] *= 2.0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int d = col - kq - 4 * u;
        double2 v = gs[min(abs(d), T - 1)];
        if (d < 0) v.y = -v.y;
        product(h, v, r0 - c0 + kq + 4 * u);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) acc += x[(r0 - c0 + 4 * v + kq) * ST + col] * (p[h][v] + sgn * q[h][v]);
    }
    if (c0 + PW < T) store(panels + (b ^ 1) * PW * ST);
    __syncthreads();
  }
  acc += __shfl_xor(acc, TPW);
  acc += __shfl_xor(acc, 16);
  acc += __shfl_xor(acc, 32);
  if (lane < TPW) red[wave][lane] = acc;
  __syncthreads();
  if (threadIdx.x < TPW && t0 + lane < count) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W; w += 4) s += (red[w][lane] + red[w + 1][lane]) + (red[w + 2][lane] + red[w + 3][lane]);
    if (part) part[blockIdx.y * count + t0 + lane] = s;
    else sigma[t0 + lane] = sqrt(s);
  }
}
__global__ void k_sigma_sum(const double* __restrict__ part, int parts, int64_t count, double* __restrict__ sigma) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= count) return;
  double s = part[t];
  for (int k = 1; k < parts; ++k) s += part[k * count + t];
  sigma[t] = sqrt(s);
}
static int launch_sigma_fit(Plan& p, Taps& tp, const double2* a, int64_t astride, int T, const double2* g, int64_t count,
                            double* sigma) {
  const int parts = sigma_parts(T);
  const int64_t batch = parts > 1 ? kSigmaBatch : count;
  for (int64_t t0 = 0; t0 < count; t0 += batch) {
    const int64_t cn = std::min(batch, count - t0);
    const bool wide = T > 128 && parts == 1;
    hipLaunchKernelGGL(wide ? k_sigma_fit<8> : k_sigma_fit<4>, dim3((unsigned)((cn + 7) / 8), (unsigned)parts),
                       dim3(wide ? 512 : 256),
                       (size_t)T * sizeof(double2) + (size_t)2 * kSigmaPanel * kSigmaStride * sizeof(double), p.stream,
                       a + t0 * astride, astride, T, g, cn, parts > 1 ? tp.sig_part : nullptr, sigma + t0);
    RFD_CHECK_LAUNCH();
    if (parts == 1) continue;
    hipLaunchKernelGGL(k_sigma_sum, dim3((unsigned)((cn + 255) / 256)), dim3(256), 0, p.stream,
                       (const double*)tp.sig_part, parts, cn, sigma + t0);
    RFD_CHECK_LAUNCH();
  }
  return RFD_OK;
}

// Normalised taps c = conj(a) sigma_ref / sigma_fit, and their MFMA A-operand
// packings.  Row 2t holds (Re c, -Im c) per tap, row 2t+1 holds (Im c, Re c).
//  16-bit: element e = 2 (k%4) + comp of lane (row + 16 ((k%16)/4)) in K block k/16,
//          uint4 index ((tb*KB + kb)*2 + plane)*64 + lane.
//  FP32:   K step kb2 = k/2, lane row + 16 (2 (k%2) + comp), float4 (tb*(Tp/8) + kq)*64 + lane
//          with kq = kb2/4, component kb2 % 4.
// A workgroup takes a tile of 8 templates (tb) x 16 taps (kb): the 128
// normalised taps are staged in LDS, then each wave writes one packing of the
// tile as 64 consecutive 16-byte lanes: wave 0 the BF16 hi and lo planes,
// wave 1 the FP16 planes, waves 2 and 3 the two FP32 K quads.  Lanes of
// templates outside [t_first, t_first + count) store nothing.
__device__ __forceinline__ double pack_val(double2 c, int o, int comp) {
  return o == 0 ? (comp == 0 ? c.x : -c.y) : (comp == 0 ? c.y : c.x);
}

__global__ __launch_bounds__(256) void k_pack(const double2* __restrict__ a, int64_t astride,
                                            const double* __restrict__ sigma_fit, const double2* __restrict__ g,
                                            int T, int Tp, int64_t t_first, int64_t count, float2* __restrict__ c32,
                                            uint4* __restrict__ pbf, uint4* __restrict__ pfh,
                                            float4* __restrict__ p32) {
  __shared__ double2 cs[8][16];
  const double sig_ref = sqrt(g[0].x);
  const int KB = Tp / 16;
  const int64_t tb0 = t_first / 8, tb1 = (t_first + count - 1) / 8;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int64_t tb = tb0 + blockIdx.y; tb <= tb1; tb += gridDim.y) {
    for (int kb = blockIdx.x; kb < KB; kb += gridDim.x) {
      if (threadIdx.x < 128) {
        const int trow = threadIdx.x >> 4, kk = threadIdx.x & 15;
        const int k = kb * 16 + kk;
        const int64_t t = tb * 8 + trow;
        const int64_t tl = t - t_first;
        double2 c = make_double2(0.0, 0.0);
        if (tl >= 0 && tl < count) {
          if (k < T) {
            const double2 av = a[tl * astride + k];
            const double sc = sig_ref / sigma_fit[tl];
            c = make_double2(av.x * sc, -av.y * sc);
          }
          c32[t * Tp + k] = make_float2((float)c.x, (float)c.y);
        }
        cs[trow][kk] = c;
      }
      __syncthreads();
      if (w < 2) {
        // 16-bit planes: lane = row + 16 gq, taps 4 gq .. 4 gq + 3 of the tile
        const int row = lane & 15, gq = lane >> 4, trow = row >> 1, o = row & 1;
        const int64_t tl = tb * 8 + trow - t_first;
        if (tl >= 0 && tl < count) {
          uint32_t hw[4], lw[4];
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const double2 c = cs[trow][gq * 4 + jj];
            uint32_t h0, l0, h1, l1;
            if (w == 0) {
              split_bf16(pack_val(c, o, 0), h0, l0);
              split_bf16(pack_val(c, o, 1), h1, l1);
            } else {
              split_f16(pack_val(c, o, 0), h0, l0);
              split_f16(pack_val(c, o, 1), h1, l1);
            }
            hw[jj] = (h0 & 0xffffu) | (h1 << 16);
            lw[jj] = (l0 & 0xffffu) | (l1 << 16);
          }
          uint4* dst = (w == 0 ? pbf : pfh) + ((tb * KB + kb) * 2) * 64 + lane;
          dst[0] = make_uint4(hw[0], hw[1], hw[2], hw[3]);
          dst[64] = make_uint4(lw[0], lw[1], lw[2], lw[3]);
        }
      } else {
        // FP32: lane = row + 16 (2 par + comp); component sub holds tap 8 q + 2 sub + par
        const int q = w - 2;
        const int row = lane & 15, par = lane >> 5, comp = (lane >> 4) & 1, trow = row >> 1, o = row & 1;
        const int64_t tl = tb * 8 + trow - t_first;
        if (tl >= 0 && tl < count) {
          float v[4];
#pragma unroll
          for (int sub = 0; sub < 4; ++sub) v[sub] = (float)pack_val(cs[trow][8 * q + 2 * sub + par], o, comp);
          p32[(tb * (Tp / 8) + 2 * kb + q) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
        }
      }
      __syncthreads();
    }
  }
}

// ------------------------------------------------------------ launchers
int taps_factor(Plan& p, Taps& tp, int b, double eps) {
  SubBankTaps& s = tp.sb[b];
  const int T = s.T;
  if (T > RFD_MAX_TAPS) return fail(RFD_E_INVALID, "taps out of range");
  int64_t el = (int64_t)T * T;
  int blocks = (int)((el + 255) / 256 < 4096 ? (el + 255) / 256 : 4096);
  int* info = reinterpret_cast<int*>(p.dscratch + 8);
  s.factored = false;
  RFD_HIP(hipMemsetAsync(info, 0, sizeof(int), p.stream));
  hipLaunchKernelGGL(k_schur_chol, dim3(1), dim3(1024), 0, p.stream, s.g, T, eps, s.L, info);
  RFD_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_upper, dim3(blocks), dim3(256), 0, p.stream, s.L, T, s.U);
  RFD_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_diag_inv, dim3((unsigned)((T + kTrsmBlock - 1) / kTrsmBlock)), dim3(256),
                     (size_t)2 * kTrsmBlock * (kTrsmBlock + 1) * sizeof(double2), p.stream, s.L, T, s.Dinv);
  RFD_CHECK_LAUNCH();
  int hinfo = 0;
  RFD_HIP(hipMemcpyAsync(&hinfo, info, sizeof(int), hipMemcpyDeviceToHost, p.stream));
  RFD_HIP(hipStreamSynchronize(p.stream));
  if (hinfo != 0) return fail(RFD_E_INVALID, "ridge-regularised Gram matrix is not positive definite");
  RFD_HIP(hipMemcpyAsync(s.gf, s.g, T * sizeof(double2), hipMemcpyDeviceToDevice, p.stream));
  s.eps = eps;
  s.factored = true;
  return RFD_OK;
}

// The factor is a function of g and the ridge alone, and g of the plan's weights and the caller's reference: where
// either has changed since, g has, and the factor with it.  The sums that make g have a fixed
// order, so that unchanged inputs give the same bits.
// answer: pinned, call << 1 | differs.
__global__ __launch_bounds__(256) void k_g_differs(const double2* __restrict__ g, const double2* __restrict__ gf, int T,
                                                 unsigned int call, unsigned int* __restrict__ answer) {
  int d = 0;
  for (int i = threadIdx.x; i < T; i += 256)
    d |= __double_as_longlong(g[i].x) != __double_as_longlong(gf[i].x) ||
         __double_as_longlong(g[i].y) != __double_as_longlong(gf[i].y);
  d = __syncthreads_or(d);
  if (threadIdx.x == 0)
    __hip_atomic_store(answer, call << 1 | (d ? 1u : 0u), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
int taps_factor_compare(Plan& p, Taps& tp, int b) {
  const SubBankTaps& s = tp.sb[b];
  tp.compares = (tp.compares + 1) & 0x7FFFFFFFu;
  hipLaunchKernelGGL(k_g_differs, dim3(1), dim3(256), 0, p.stream, (const double2*)s.g, (const double2*)s.gf, s.T,
                     tp.compares, tp.factor_answer);
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}
// Read as it comes, for a while: it is mostly there when the correlations are queued.  (An event for it took 4 us of
// a call's 43 at T = 8, 8 templates.)
int taps_factor_current(Plan& p, Taps& tp, bool* current) {
  const auto answered = [&] { return __atomic_load_n(tp.factor_answer, __ATOMIC_ACQUIRE) >> 1 == tp.compares; };
  const auto end = std::chrono::steady_clock::now() + std::chrono::milliseconds(1);
  while (!answered() && std::chrono::steady_clock::now() < end) {}
  // (earlier work on the stream: not its wait, which would take in the correlations too)
  while (!answered()) {
    const hipError_t e = hipStreamQuery(p.stream);
    if (e == hipErrorNotReady) {
      (void)hipGetLastError();             // (not one that a later launch check is to find)
      std::this_thread::sleep_for(std::chrono::microseconds(50));
      continue;
    }
    RFD_HIP(e);
    if (!answered()) return fail(RFD_E_DEVICE, "taps: the factor was not compared");
  }
  *current = (*tp.factor_answer & 1u) == 0;
  return RFD_OK;
}

int taps_norm_and_pack(Plan& p, Taps& tp, int b, int64_t first, int64_t count);
int taps_pack(Plan& p, Taps& tp, int b, int64_t first, int64_t count);

// A launch per block row (k_trsm_step) or all rows in one (k_trsm); by the call's sizes alone, so that equal calls give
// equal bits.  make_taps of a 2^15-sample segment, one launch and steps: T = 512 210 -> 180 us (1 template), 315 -> 302 (256),
// 425 -> 422 (512), 704 -> 731 (1000); T = 1024 543 -> 339 (1), 712 -> 558 (256), 888 -> 775 (512), 1343 -> 1423 (1000);
// T = 2048 1747 -> 663 (1), 2360 -> 1830 (512), 3024 -> 3212 (1000); T = 384 147 -> 142 (1), 210 -> 213 (256), 458 -> 479
// (1000); T = 256 99 -> 103 (1), 151 -> 162 (256).
static bool trsm_in_steps(int T, int64_t count) { return T >= 512 && count <= 512; }
// (the steps' residuals and forward solutions)
size_t taps_solve_work(int T, int64_t count) { return trsm_in_steps(T, count) ? (size_t)(2 * count * T) : 0; }

int taps_solve_and_pack(Plan& p, Taps& tp, int b, int64_t first, int64_t count, int method) {
  SubBankTaps& s = tp.sb[b];
  const int T = s.T;
  double2* abase = tp.a64 + s.a_base + first * s.Tp;
  if (method == RFD_TAPS_LS) {
    const int Tn = (int)round_up(T, kTrsmBlock), nb = Tn / kTrsmBlock;
    if (trsm_in_steps(T, count)) {
      if (tp.work64_cap < taps_solve_work(T, count)) return fail(RFD_E_INVALID, "taps: work buffer too small");
      // forward residuals and solutions in the (now idle) transform buffer; the latter are the backward sweep's residuals
      double2 *r = tp.work64, *y = tp.work64 + count * T;
      const unsigned groups = (unsigned)((count + 7) / 8);
      for (int j = -1; j < nb - 1; ++j) {
        hipLaunchKernelGGL(k_trsm_step<false>, dim3(groups, j < 0 ? 1u : (unsigned)(nb - 1 - j)), dim3(256), 0, p.stream,
                           (const double2*)s.L, (const double2*)s.Dinv, T, j, (const double2*)(j > 0 ? r : tp.bvec),
                           (int64_t)T, r, y, (int64_t)T, count);
        RFD_CHECK_LAUNCH();
      }
      for (int j = nb; j > 0; --j) {
        hipLaunchKernelGGL(k_trsm_step<true>, dim3(groups, j == nb ? 1u : (unsigned)j), dim3(256), 0, p.stream,
                           (const double2*)s.U, (const double2*)s.Dinv, T, j == nb ? -1 : j, (const double2*)y, (int64_t)T, y,
                           abase, (int64_t)s.Tp, count);
        RFD_CHECK_LAUNCH();
      }
    } else if (T <= 16)
      hipLaunchKernelGGL((k_trsm<8, 16>), dim3((unsigned)((count + 7) / 8)), dim3(64), (size_t)16 * 16 * sizeof(double),
                         p.stream, s.L, s.U, s.Dinv, T, tp.bvec, (int64_t)T, abase, (int64_t)s.Tp, count);
    else if (T <= 1024)       // eight templates per workgroup while their columns fit LDS (128 KiB at T = 1024), else four
      hipLaunchKernelGGL(k_trsm<8>, dim3((unsigned)((count + 7) / 8)), dim3(256), (size_t)Tn * 16 * sizeof(double),
                         p.stream, s.L, s.U, s.Dinv, T, tp.bvec, (int64_t)T, abase, (int64_t)s.Tp, count);
    else
      hipLaunchKernelGGL(k_trsm<4>, dim3((unsigned)((count + 3) / 4)), dim3(256), (size_t)Tn * 8 * sizeof(double),
                         p.stream, s.L, s.U, s.Dinv, T, tp.bvec, (int64_t)T, abase, (int64_t)s.Tp, count);
  } else {
    int64_t el = count * T;
    int blocks = (int)((el + 255) / 256 < 4096 ? (el + 255) / 256 : 4096);
    hipLaunchKernelGGL(k_window, dim3(blocks), dim3(256), 0, p.stream, tp.bvec, (int64_t)T, T, count, abase,
                       (int64_t)s.Tp);
  }
  RFD_CHECK_LAUNCH();
  return taps_norm_and_pack(p, tp, b, first, count);
}

// sigma_fit of taps already in a64, then the normalised taps and MFMA packings.
int taps_norm_and_pack(Plan& p, Taps& tp, int b, int64_t first, int64_t count) {
  SubBankTaps& s = tp.sb[b];
  int rc = launch_sigma_fit(p, tp, tp.a64 + s.a_base + first * s.Tp, s.Tp, s.T, s.g, count,
                            tp.sigma_fit + s.first + first);
  if (rc) return rc;
  return taps_pack(p, tp, b, first, count);
}

// normalised taps and MFMA packings from a64 and sigma_fit already in place
int taps_pack(Plan& p, Taps& tp, int b, int64_t first, int64_t count) {
  SubBankTaps& s = tp.sb[b];
  s.ols_valid = false;   // the overlap-save tap spectra follow the packed taps
  if (count <= 0) return RFD_OK;
  const int T = s.T;
  double2* abase = tp.a64 + s.a_base + first * s.Tp;
  double* sig = tp.sigma_fit + s.first + first;
  const int64_t ntb = (first + count - 1) / 8 - first / 8 + 1;
  const int KB = s.Tp / 16;
  dim3 grid((unsigned)std::min(KB, 8), (unsigned)std::min<int64_t>(ntb, 8192));
  hipLaunchKernelGGL(k_pack, grid, dim3(256), 0, p.stream, abase, (int64_t)s.Tp, sig, s.g, T, s.Tp, first, count,
                     tp.c32 + s.a_base, tp.pbf + s.p16_base, tp.pfh + s.p16_base, tp.p32 + s.p32_base);
  RFD_CHECK_LAUNCH();
  return RFD_OK;
}

}  // namespace rfd
