// One majorise-minimise step on a caller's K without K's own factorisation.
//
// The step needs (2 lambda I + K/(n kappa))^{-1} applied to two vectors of each
// column. The band reduction of K and its Q serve every column, but are chains
// of N/16 dependent panels; a blocked Cholesky factorisation per column is a
// chain of N/64 and runs all columns at once, with the two right-hand sides as
// further rows of the matrix, so that the forward substitution comes with it.
// The tiles are solved by inverted 64 x 64 triangles, which costs digits where
// lambda is small; one refinement with the residual brings the error below that
// of the factorisation of K (n = 1403, 20 columns, alpha: 2.2e-13 without it,
// 6.8e-14 with it, 1.0e-13 by the factorisation of K) for 0.5 of the 2.9 ms.
#include "kmp_common.h"
#include "kmp_kernels.h"

#include <algorithm>

namespace kmp {

namespace {
constexpr int ST = 512;                 // threads of a column's workgroup
constexpr int SB = 1024;                // the same for the back substitution
constexpr int SBG = SB / 64;

// out = K u for `cols` columns: two rows of K and four columns per wavefront,
// each sum by lanes and then across them, so that its rounding error grows with
// the square root of n/64 terms: what enters w here is divided by 2 lambda later
// (with one sequence of matrix-core sums, n = 1403, the refined alpha was off by
// 1.3e-12, so by 7e-14).
__global__ __launch_bounds__(256) void step_product_kernel(int n, int cols,
                                                           const double* __restrict__ K,
                                                           const double* __restrict__ u, int64_t ldu,
                                                           double* __restrict__ out) {
  const int lane = threadIdx.x & 63, i0 = 2 * (4 * (int)blockIdx.x + (int)(threadIdx.x >> 6));
  if (i0 >= n) return;
  const int i1 = min(i0 + 1, n - 1), c0 = 4 * (int)blockIdx.y;
  const double *k0 = K + (int64_t)i0 * n, *k1 = K + (int64_t)i1 * n;
  const double* uc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) uc[q] = u + (int64_t)min(c0 + q, cols - 1) * ldu;
  double s[2][4] = {};
#pragma unroll 2
  for (int j = lane; j < n; j += 64) {
    const double a = k0[j], b = k1[j];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double x = uc[q][j];
      s[0][q] = fma(a, x, s[0][q]);
      s[1][q] = fma(b, x, s[1][q]);
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double t0 = wave_sum(s[0][q]), t1 = wave_sum(s[1][q]);
    if (lane == 0 && c0 + q < cols) {
      out[(int64_t)(c0 + q) * n + i0] = t0;
      if (i0 + 1 < n) out[(int64_t)(c0 + q) * n + i0 + 1] = t1;
    }
  }
}

int product(hipStream_t s, const StepArrays& a, int cols, const double* u, int64_t ldu, double* out) {
  hipLaunchKernelGGL(step_product_kernel, dim3((unsigned)ceil_div(a.n, 8), (unsigned)ceil_div(cols, 4)),
                     dim3(256), 0, s, a.n, cols, a.K, u, ldu, out);
  KMP_LAUNCH_CHECK();
  return 0;
}

// z = psi(y, f + beta)/n, w = z + 2 lambda alpha and the KKT measure of a column.
__global__ __launch_bounds__(ST) void step_loss_kernel(const StepArrays a) {
  __shared__ double red[2][ST / 64];
  const int c = blockIdx.x, n = a.n;
  const double* al = a.alpha_in + (int64_t)c * n;
  const double* f = a.f + (int64_t)c * n;
  double* w = a.w + (int64_t)c * a.N;
  const double lam2 = 2.0 * a.lam[c], b = a.beta_in[c], tau = a.tau[c], inv = 1.0 / (double)n;
  double zs = 0.0, n2 = 0.0;
  for (int i = threadIdx.x; i < a.N; i += ST) {
    double u = 0.0;
    if (i < n) {
      const double z = loss_psi(a.loss, a.y[i], f[i] + b, a.delta, tau) * inv;
      u = fma(lam2, al[i], z);
      zs += z;
      n2 = fma(u, u, n2);
    }
    w[i] = u;
  }
  zs = block_sum<ST / 64>(zs, red[0]);
  n2 = block_sum<ST / 64>(n2, red[1]);
  if (threadIdx.x == 0) {
    // (fmax drops a NaN, so both terms are tested)
    const double kkt = (double)n * fmax(sqrt(n2), fabs(zs));
    a.kkt[c] = kkt;
    a.stay[c] = !(n2 == n2) || !(zs == zs) || !(kkt <= 1e300) ? 1.0 : 0.0;
  }
}

// The two solutions of a column from its factor, a workgroup per column. The
// right-hand sides came forward with the factorisation (rows N and N + 1 of P);
// with REFINE they are the residuals r0, r1, solved forward first, from the
// first block of 64 rows to the last (a row of G per wavefront step, lanes
// along it), and the result is added to x and v. Back substitution goes from
// the last block to the first: the columns of the block over all rows below
// it (lanes along a row of G), then G_JJ^{-T}. Bound by reading the factor
// through one compute unit (N = 1408: 331 us, with REFINE 445).
template <bool REFINE>
__global__ __launch_bounds__(SB) void step_solve_kernel(const StepArrays a, int c0) {
  extern __shared__ double sol[];                 // 2 N: the solutions
  __shared__ double part[2][SBG][64], rhs[2][64];
  const int b = blockIdx.x, c = c0 + b, N = a.N;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double* P = a.P + (int64_t)b * (N + 64) * N;
  double *x = a.x + (int64_t)c * N, *v = a.v + (int64_t)c * N;
  if constexpr (REFINE) {
    const double *r0 = a.r0 + (int64_t)c * N, *r1 = a.r1 + (int64_t)c * N;
    for (int J = 0; J < N / 64; ++J) {
      double s[2][4] = {};
      const double* g = P + (int64_t)(64 * J + 4 * w) * N + lane;
#pragma unroll 4
      for (int k = 0; k < 64 * J; k += 64) {
        const double y0 = sol[k + lane], y1 = sol[N + k + lane];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double gq = g[(int64_t)q * N + k];
          s[0][q] = fma(gq, y0, s[0][q]);
          s[1][q] = fma(gq, y1, s[1][q]);
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double t0 = wave_sum(s[0][q]), t1 = wave_sum(s[1][q]);
        const int i = 4 * w + q;
        if (lane == 0) {
          rhs[0][i] = r0[64 * J + i] - t0;
          rhs[1][i] = r1[64 * J + i] - t1;
        }
      }
      __syncthreads();
      const double* d = a.dinv + ((int64_t)b * N + 64 * J) * 64;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = 4 * w + q;
        const double e = d[64 * i + lane];
        const double t0 = wave_sum(e * rhs[0][lane]), t1 = wave_sum(e * rhs[1][lane]);
        if (lane == 0) {
          sol[64 * J + i] = t0;
          sol[N + 64 * J + i] = t1;
        }
      }
      __syncthreads();
    }
  }
  for (int J = N / 64 - 1; J >= 0; --J) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll 8
    for (int i = 64 * (J + 1) + w; i < N; i += SBG) {
      const double g = P[(int64_t)i * N + 64 * J + lane];
      s0 = fma(g, sol[i], s0);
      s1 = fma(g, sol[N + i], s1);
    }
    part[0][w][lane] = s0;
    part[1][w][lane] = s1;
    __syncthreads();
    if (w < 2) {
      double r = REFINE ? sol[w * N + 64 * J + lane] : P[(int64_t)(N + w) * N + 64 * J + lane];
      for (int k = 0; k < SBG; ++k) r -= part[w][k][lane];
      rhs[w][lane] = r;
    }
    __syncthreads();
    {                                             // four rows of G_JJ^{-1} per wavefront
      const double* d = a.dinv + ((int64_t)b * N + 64 * J) * 64;
      s0 = s1 = 0.0;
#pragma unroll
      for (int k = 4 * w; k < 4 * w + 4; ++k) {
        const double g = d[64 * k + lane];
        s0 = fma(g, rhs[0][k], s0);
        s1 = fma(g, rhs[1][k], s1);
      }
      part[0][w][lane] = s0;
      part[1][w][lane] = s1;
    }
    __syncthreads();
    if (w < 2) {
      double r = 0.0;
      for (int k = 0; k < SBG; ++k) r += part[w][k][lane];
      sol[w * N + 64 * J + lane] = r;
      double* o = (w == 0 ? x : v) + 64 * J + lane;
      *o = REFINE ? *o + r : r;
    }
    __syncthreads();
  }
}

// Residuals of the two systems, from K x and K v (in f and kv).
__global__ __launch_bounds__(256) void step_residual_kernel(const StepArrays a, int c0) {
  const int c = c0 + (int)blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
  if (i >= a.N) return;
  const int64_t to = (int64_t)c * a.N + i, at = (int64_t)c * a.n + i;
  const double sc = 1.0 / ((double)a.n * a.kappa), lam2 = 2.0 * a.lam[c];
  a.r0[to] = i < a.n ? fma(-sc, a.f[at], fma(-lam2, a.x[to], a.w[to])) : 0.0;
  a.r1[to] = i < a.n ? fma(-sc, a.kv[at], fma(-lam2, a.v[to], sc)) : 0.0;
}

// alpha - x - g (t - d0) v and beta - g (d0 - t) with g = 1/(2 lambda 1'v) and
// t = v'K w = 1'w - 2 lambda 1'x (d0 = 1'z), so that g (t - d0) = (1'alpha -
// 1'x)/1'v: no product with K. 1'x is taken as n kappa v'w (M v = 1/(n kappa)),
// whose terms are of the size of w and not of w/(2 lambda).
__global__ __launch_bounds__(ST) void step_finish_kernel(const StepArrays a, double* alpha_out,
                                                         double* beta_out, double* kkt_out) {
  __shared__ double red[2][ST / 64];
  if (*a.bad != 0) return;
  const int c = blockIdx.x, n = a.n;
  const double *x = a.x + (int64_t)c * a.N, *v = a.v + (int64_t)c * a.N;
  const double *al = a.alpha_in + (int64_t)c * n, *wv = a.w + (int64_t)c * a.N;
  const double nk = (double)n * a.kappa;
  double vs = 0.0, t = 0.0;
  for (int i = threadIdx.x; i < n; i += ST) {
    vs += v[i];
    t += fma(-nk * v[i], wv[i], al[i]);
  }
  vs = block_sum<ST / 64>(vs, red[0]);
  t = block_sum<ST / 64>(t, red[1]);
  const bool stay = a.stay[c] != 0.0;             // no step from a state that is not finite
  const double q = stay ? 0.0 : t / vs;
  for (int i = threadIdx.x; i < n; i += ST)
    alpha_out[(int64_t)c * n + i] = stay ? al[i] : fma(-q, v[i], al[i] - x[i]);
  if (threadIdx.x == 0) {
    beta_out[c] = a.beta_in[c] + q;
    if (kkt_out) kkt_out[c] = a.kkt[c];
  }
}
}  // namespace

// Times in us, both ways, n by columns: 60 by 1 129 and 397, by 450 276 and 507, by
// 800 635 and 478; 128 by 300 657 and 755, by 600 785 and 751; 190 by 300 843 and
// 972, by 600 1153 and 967; 256 by 300 784 and 1210; 700 by 20 1064 and 3168, by 300
// 3221 and 3450; 1403 by 20 2995 and 7329, by 60 4086 and 7351, by 200 10.6 and 7.4
// ms; 2000 by 60 8.5 and 12.5 ms, by 120 17.3 and 12.5; 3000 by 20 11.8 and 32.1. A
// column costs n^3/3 operations at 16 TFLOP/s and the 1.5 us of its workgroups beyond
// the common chain of 0.9 n + 0.00075 n^2; the factorisation of K takes 1.5 n + 0.0031
// n^2 and next to nothing a column.
bool step_pays(int64_t n, int C) {
  const double m = (double)n;
  return n <= kStepMaxOrder && C * (m * m / 47e6 + 1.5e-3) <= 0.6 + 0.0023 * m;
}

size_t step_doubles(int N, int C, int cap) {
  const size_t n = (size_t)N, c = (size_t)C, k = (size_t)cap;
  return 7 * c * n + 4 * c + k * ((n + 64) * n + 64 * n) + 2;
}

void step_carve(StepArrays* a, double* q) {
  const size_t n = (size_t)a->N, c = (size_t)a->C, k = (size_t)a->cap;
  a->P = q; q += k * (n + 64) * n;
  a->dinv = q; q += k * 64 * n;
  a->f = q; q += c * (size_t)a->n;
  a->kv = q; q += c * (size_t)a->n;
  a->w = q; q += c * n;
  a->x = q; q += c * n;
  a->v = q; q += c * n;
  a->r0 = q; q += c * n;
  a->r1 = q; q += c * n;
  a->kkt = q; q += c;
  a->stay = q; q += c;
  a->lam = q; q += c;
  a->tau = q; q += c;
  a->bad = reinterpret_cast<int*>(q);
}

int step_columns(hipStream_t s, const StepArrays& a, double* alpha_out, double* beta_out,
                 double* kkt_out) {
  int rc;
  KMP_HIP_TRY(hipMemsetAsync(a.bad, 0, sizeof(int), s));
  if ((rc = product(s, a, a.C, a.alpha_in, a.n, a.f)) != 0) return rc;
  hipLaunchKernelGGL(step_loss_kernel, dim3((unsigned)a.C), dim3(ST), 0, s, a);
  KMP_LAUNCH_CHECK();
  const size_t lds = 2 * sizeof(double) * a.N;
  // (the largest at every call: the attribute is the process's, and calls of other
  // threads may have other sizes)
  for (const void* k : {(const void*)step_solve_kernel<false>, (const void*)step_solve_kernel<true>})
    KMP_HIP_TRY(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)(2 * sizeof(double) * kStepMaxOrder)));
  for (int c0 = 0; c0 < a.C; c0 += a.cap) {
    const int cols = std::min(a.cap, a.C - c0);
    for (int J = 0; J < a.N / 64; ++J)
      if ((rc = step_panel(s, a, c0, cols, J)) != 0) return rc;
    hipLaunchKernelGGL((step_solve_kernel<false>), dim3((unsigned)cols), dim3(SB), lds, s, a, c0);
    KMP_LAUNCH_CHECK();
    // K x and K v
    if ((rc = product(s, a, cols, a.x + (int64_t)c0 * a.N, a.N, a.f + (int64_t)c0 * a.n)) != 0 ||
        (rc = product(s, a, cols, a.v + (int64_t)c0 * a.N, a.N, a.kv + (int64_t)c0 * a.n)) != 0)
      return rc;
    hipLaunchKernelGGL(step_residual_kernel, dim3((unsigned)ceil_div(a.N, 256), (unsigned)cols),
                       dim3(256), 0, s, a, c0);
    KMP_LAUNCH_CHECK();
    hipLaunchKernelGGL((step_solve_kernel<true>), dim3((unsigned)cols), dim3(SB), lds, s, a, c0);
    KMP_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(step_finish_kernel, dim3((unsigned)a.C), dim3(ST), 0, s, a, alpha_out, beta_out,
                     kkt_out);
  KMP_LAUNCH_CHECK();
  return 0;
}

}  // namespace kmp
