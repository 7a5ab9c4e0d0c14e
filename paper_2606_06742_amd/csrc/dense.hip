// The last columns of a stage in observation space, by their dense resolvents.
//
// The batched iteration (path.hip) pays for two passes over every group's
// factor, the loss pass and the banded solve's serial chain, whatever the
// number of columns still active. Once few are, each of them takes its own
// dense N x N resolvent
//   R = (2 lambda I + K/(n_v kappa))^{-1} = Q (2 lambda I + B/(n_v kappa))^{-1} Q'
// and iterates on (alpha, f = K alpha) directly: the step x = R w is one
// symmetric matrix-vector product, and since K R = n_v kappa (I - 2 lambda R),
//   K x   = n_v kappa (w - 2 lambda x),
//   K Da  = g (t - d0) K v + n_v kappa (w - 2 lambda x),
// so f follows alpha without a product with K. The iterates are those of
// the batched form up to rounding (the inner products of its restart and KKT
// tests do not change under the orthogonal Q). The carried f drifts as lambda
// shrinks: it is formed again from alpha through the factor at intervals and when
// the columns have stopped, and a column stops as converged by that f only
// (dense_check).
//
// An iteration is two launches: the products of all dense columns spread over
// the chip, then one workgroup per column for everything elementwise. An
// iteration of some columns in 4 groups, batched and dense: order 320, 48
// columns 36 and 13 us, 832, 16 columns 58 and 22 us, 1536, 4 columns 81 and
// 22 us. It is bound by the two launches and then by reading R (8 TB/s from
// the last-level cache). (Up to order kSmallOrder see small.hip.)
#include "kmp_common.h"
#include "kmp_kernels.h"

namespace kmp {

typedef double ddbl4 __attribute__((ext_vector_type(4)));

namespace {
constexpr int DT = 512;                 // threads of a column's workgroup
constexpr int DW = DT / 64;
constexpr int BND = kBand;

// vectors of the dense columns (DenseArrays::vec)
enum { VA = 0, VAB, VF, VFB, VV, VKV, VW, VX, VT };

__device__ __forceinline__ double* dvec(const DenseArrays& a, int N, int which, int t) {
  return a.vec + ((int64_t)which * a.cap + t) * N;
}

// Sums of three values over the workgroup, in a fixed order, to every thread.
__device__ __forceinline__ void block_sum3(double& x, double& y, double& z, double (*red)[3]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  x = wave_sum(x);
  y = wave_sum(y);
  z = wave_sum(z);
  __syncthreads();
  if (lane == 0) {
    red[w][0] = x;
    red[w][1] = y;
    red[w][2] = z;
  }
  __syncthreads();
  x = y = z = 0.0;
#pragma unroll
  for (int i = 0; i < DW; ++i) {
    x += red[i][0];
    y += red[i][1];
    z += red[i][2];
  }
}

// The dense columns: every active column, group by group in the order of the
// active lists (one wavefront).
__global__ __launch_bounds__(64) void dense_list_kernel(int G, int C, int cap,
                                                        const int* __restrict__ cmap,
                                                        const int* __restrict__ nact,
                                                        int* __restrict__ list,
                                                        int* __restrict__ sure,
                                                        int* __restrict__ count) {
  int base = 0;
  for (int g = 0; g < G; ++g) {
    const int n = nact[g];
    for (int k = threadIdx.x; k < n; k += 64)
      if (base + k < cap) list[base + k] = g * C + cmap[(int64_t)g * C + k];
    base += n;
  }
  for (int k = threadIdx.x; k < cap; k += 64) sure[k] = 0;
  if (threadIdx.x == 0) count[0] = min(base, cap);
}

// Y = Q M^{-1} by rows (M = 2 lambda I + B/(n_v kappa) of a column, from its
// block LDL' factors): row j of Y is M^{-1} q for row q of Q. One wavefront
// takes 16 rows as the 16 columns of an MFMA operand, so that a block step
// of the solve, whose chain bounds the one-vector form, serves 16 of them:
// with A = -C_I (or L_I^{-1}) the accumulator of one 16x16x4 product is
// laid out as the B operand of the next. A workgroup takes the 64-row block
// e0 + blockIdx.x (block e: column e / (N/64) of the list, rows 64 (e mod
// N/64) ..), stored at Y + blockIdx.x * 64 N. Operands are loaded DPF blocks
// ahead.
constexpr int DPF = 4;                  // N/16 is a multiple of it
__global__ __launch_bounds__(256) void dense_rows_kernel(
    int N, int C, int e0, const DenseArrays a, const double* __restrict__ Q,
    const double* __restrict__ Vfac, const double* __restrict__ Dfac, double* Y) {
  const int e = e0 + (int)blockIdx.x, nb = N / 64;
  const int t = e / nb;
  if (t >= *a.count) return;
  const int64_t gc = a.list[t];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int g = (int)(gc / C);
  const double* Vc = Vfac + gc * (int64_t)BND * N;
  const double* Dc = Dfac + gc * (int64_t)N;
  const double* q = Q + (int64_t)g * N * N + (int64_t)(64 * (e % nb) + 16 * w + li) * N;
  double* y = Y + ((int64_t)blockIdx.x * 64 + 16 * w + li) * N;
  const int NB = N / BND;
  double vt[DPF][4], wr[DPF][4], dr[DPF][4];
#pragma unroll
  for (int p = 0; p < DPF; ++p)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      vt[p][s] = Vc[(int64_t)(4 * s + lk) * N + BND * p + li];
      wr[p][s] = q[BND * p + 4 * s + lk];
    }
  ddbl4 prev = {0.0, 0.0, 0.0, 0.0};
  for (int I0 = 0; I0 < NB; I0 += DPF) {
#pragma unroll
    for (int p = 0; p < DPF; ++p) {
      const int I = I0 + p, In = min(I + DPF, NB - 1);
      ddbl4 r = {wr[p][0], wr[p][1], wr[p][2], wr[p][3]};
      double cm[4], lm[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = 4 * s + lk;
        cm[s] = (k >= li && I > 0) ? -vt[p][s] : 0.0;            // -C_I
        lm[s] = k < li ? vt[p][s] : (k == li ? 1.0 : 0.0);       // L_I^{-1}
        vt[p][s] = Vc[(int64_t)k * N + BND * In + li];
        wr[p][s] = q[BND * In + k];
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
        r = __builtin_amdgcn_mfma_f64_16x16x4f64(cm[s], prev[s], r, 0, 0, 0);
      ddbl4 o = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s)
        o = __builtin_amdgcn_mfma_f64_16x16x4f64(lm[s], r[s], o, 0, 0, 0);
#pragma unroll
      for (int s = 0; s < 4; ++s) y[BND * I + 4 * s + lk] = o[s];
      prev = o;
    }
  }
  // backward: x_I = L_I^{-T} (D_I^{-1} y_I - C_{I+1}' x_{I+1}); a lane reads
  // back the entries of y that it stored
#pragma unroll
  for (int p = 0; p < DPF; ++p)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int I = NB - 1 - p, k = 4 * s + lk;
      vt[p][s] = Vc[(int64_t)li * N + BND * I + k];
      wr[p][s] = y[BND * I + k];
      dr[p][s] = Dc[BND * I + k];
    }
  double vn[4] = {0.0, 0.0, 0.0, 0.0};           // the tile entries of block I + 1
  prev = ddbl4{0.0, 0.0, 0.0, 0.0};
  for (int T0 = 0; T0 < NB; T0 += DPF) {
#pragma unroll
    for (int p = 0; p < DPF; ++p) {
      const int I = NB - 1 - (T0 + p), In = max(I - DPF, 0);
      ddbl4 r = {wr[p][0] * dr[p][0], wr[p][1] * dr[p][1], wr[p][2] * dr[p][2], wr[p][3] * dr[p][3]};
      double cm[4], lm[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = 4 * s + lk;
        cm[s] = li >= k ? -vn[s] : 0.0;                          // -C_{I+1}'
        lm[s] = k > li ? vt[p][s] : (k == li ? 1.0 : 0.0);       // L_I^{-T}
        vn[s] = vt[p][s];
        vt[p][s] = Vc[(int64_t)li * N + BND * In + k];
        wr[p][s] = y[BND * In + k];
        dr[p][s] = Dc[BND * In + k];
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
        r = __builtin_amdgcn_mfma_f64_16x16x4f64(cm[s], prev[s], r, 0, 0, 0);
      ddbl4 o = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s)
        o = __builtin_amdgcn_mfma_f64_16x16x4f64(lm[s], r[s], o, 0, 0, 0);
#pragma unroll
      for (int s = 0; s < 4; ++s) y[BND * I + 4 * s + lk] = o[s];
      prev = o;
    }
  }
}

// Vectors of the dense columns in observation space from those in the factor
// basis: alpha = Q ahat, abar = Q abar^, f = Q B ahat, fbar = Q B abar^,
// v = Q vhat, K v = Q B vhat; with REFRESH f and fbar only, into the vectors
// VX and VT. One wavefront per row; rows past the group's valid ones are zero.
template <bool REFRESH>
__global__ __launch_bounds__(256) void dense_vectors_kernel(
    int N, int C, const DenseArrays a, const double* __restrict__ Q, const double* __restrict__ QB,
    const int* __restrict__ nv, const double* __restrict__ ahat, const double* __restrict__ abar,
    const double* __restrict__ vhat, const double* __restrict__ uvec) {
  const int t = blockIdx.y;
  if (t >= *a.count || (REFRESH && a.sure[t] == 1)) return;
  const int64_t gc = a.list[t];
  const int g = (int)(gc / C);
  const int i = 4 * (int)blockIdx.x + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const double* q = Q + (int64_t)g * N * N + (int64_t)i * N;
  const double* b = QB + (int64_t)g * N * N + (int64_t)i * N;
  const double *xa = ahat + gc * N, *xb = abar + gc * N, *xv = vhat + gc * N, *xu = uvec + gc * N;
  double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (i < nv[g]) {
#pragma unroll 4
    for (int k = lane; k < N; k += 64) {
      const double bk = b[k], ak = xa[k], abk = xb[k];
      s[2] = fma(bk, ak, s[2]);
      s[3] = fma(bk, abk, s[3]);
      if constexpr (!REFRESH) {
        const double qk = q[k];
        s[0] = fma(qk, ak, s[0]);
        s[1] = fma(qk, abk, s[1]);
        s[4] = fma(qk, xv[k], s[4]);
        s[5] = fma(qk, xu[k], s[5]);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    if (REFRESH && j != 2 && j != 3) continue;
    const double v = wave_sum(s[j]);
    const int to = !REFRESH ? j : (j == 2 ? VX : VT);
    if (lane == 0) dvec(a, N, to, t)[i] = v;
  }
}

// ahat = Q'alpha and abar^ = Q'abar of the dense columns (lanes over 64
// columns of Q, 16 row groups added in a fixed order).
constexpr int DPC = 64, DPR = 16;
__global__ __launch_bounds__(DPC * DPR) void dense_project_kernel(
    int N, int C, const DenseArrays a, const double* __restrict__ Q, const int* __restrict__ nv,
    double* __restrict__ ahat, double* __restrict__ abar) {
  __shared__ double pa[DPR][DPC], pb[DPR][DPC];
  const int t = blockIdx.y, j = blockIdx.x * DPC + threadIdx.x, ry = threadIdx.y;
  if (t == 0 && j == 0 && ry == 0) a.count[1] = 0;
  if (t >= a.count[0] || a.sure[t] == 1) return;
  const int64_t gc = a.list[t];
  const int g = (int)(gc / C), m = nv[g];
  const double* q = Q + (int64_t)g * N * N + j;
  const double *xa = dvec(a, N, VA, t), *xb = dvec(a, N, VAB, t);
  double s0 = 0.0, s1 = 0.0;
#pragma unroll 4
  for (int i = ry; i < m; i += DPR) {
    const double qi = q[(int64_t)i * N];
    s0 = fma(qi, xa[i], s0);
    s1 = fma(qi, xb[i], s1);
  }
  pa[ry][threadIdx.x] = s0;
  pb[ry][threadIdx.x] = s1;
  __syncthreads();
  if (ry == 0) {
    s0 = s1 = 0.0;
    for (int r = 0; r < DPR; ++r) {
      s0 += pa[r][threadIdx.x];
      s1 += pb[r][threadIdx.x];
    }
    ahat[gc * N + j] = s0;
    abar[gc * N + j] = s1;
  }
}

// x = R w of every dense column: two rows per wavefront.
__global__ __launch_bounds__(DT) void dense_product_kernel(int N, const DenseArrays a,
                                                           const int* __restrict__ flag) {
  const int t = blockIdx.y;
  if (t >= *a.count || flag[a.list[t]] != 0) return;
  const int lane = threadIdx.x & 63;
  const int i = 2 * (DW * (int)blockIdx.x + (int)(threadIdx.x >> 6));
  if (i >= N) return;
  const double* r0 = a.R + (int64_t)t * N * N + (int64_t)i * N;
  const double* r1 = r0 + N;
  const double* w = dvec(a, N, VW, t);
  double s0 = 0.0, s1 = 0.0, u0 = 0.0, u1 = 0.0;
#pragma unroll 4
  for (int k = 2 * lane; k < N; k += 128) {
    const double2 wk = *reinterpret_cast<const double2*>(w + k);
    const double2 a0 = *reinterpret_cast<const double2*>(r0 + k);
    const double2 a1 = *reinterpret_cast<const double2*>(r1 + k);
    s0 = fma(a0.x, wk.x, s0);
    u0 = fma(a0.y, wk.y, u0);
    s1 = fma(a1.x, wk.x, s1);
    u1 = fma(a1.y, wk.y, u1);
  }
  s0 = wave_sum(s0 + u0);
  s1 = wave_sum(s1 + u1);
  if (lane == 0) {
    double* x = dvec(a, N, VX, t);
    x[i] = s0;
    x[i + 1] = s1;
  }
}

// One column per workgroup, RPT rows per thread in registers. The step from
// x = R w (not with START, which begins at the current point):
//   Da = g (t - d0) v + x, a+ = abar - Da, f+ likewise, Db = g (d0 - t),
//   the restart test and the momentum to the next extrapolated point;
// there z = psi(y, fbar + bbar)/n_v, w = z + 2 lambda abar, d0 = 1'z,
// t = (K v)'w and the KKT test, with which the column stops as in the
// batched update. scal keeps d0 and t for the next step.
template <int RPT, bool START>
__global__ __launch_bounds__(DT) void dense_update_kernel(const DenseArrays a, const PathArrays p,
                                                          double delta, double kappa, double tol,
                                                          int max_iter, int restart) {
  __shared__ double red[DW][3];
  __shared__ double red1[DW];
  const int t = blockIdx.x;
  if (t >= *a.count) return;
  const int64_t gc = a.list[t];
  if (p.flag[gc] != 0) return;                    // uniform over the block
  const bool may = !START || a.sure[t] == 2;      // stop here: with START in a check only
  const int N = p.N, g = (int)(gc / p.C), nv = p.nv[g];
  const double lam2 = 2.0 * p.lam[gc], nvd = (double)p.cnv[gc], tau = p.tau[gc];
  const int32_t hf = p.cfold ? p.cfold[gc] : -1;
  const int32_t* rf = p.rfold ? p.rfold + (int64_t)g * N : nullptr;
  const double* y = p.ylab + (int64_t)g * N;
  double *pa = dvec(a, N, VA, t), *pab = dvec(a, N, VAB, t);
  double *pf = dvec(a, N, VF, t), *pfb = dvec(a, N, VFB, t);
  const double *pv = dvec(a, N, VV, t), *pkv = dvec(a, N, VKV, t);
  double *pw = dvec(a, N, VW, t), *px = dvec(a, N, VX, t);
  double ab[RPT], fb[RPT], kv[RPT], yv[RPT];
  bool live[RPT];
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int i = threadIdx.x + DT * q, ii = i < N ? i : 0;
    ab[q] = pab[ii];
    fb[q] = pfb[ii];
    kv[q] = pkv[ii];
    yv[q] = y[ii];
    live[q] = i < nv && !(rf && rf[ii] == hf);
  }
  double bb = p.bbar[gc];
  int it = 0;
  if constexpr (!START) {
    double ea[RPT], ef[RPT];
    const double gco = p.gcoef[gc], d0 = a.scal[2 * t], tv = a.scal[2 * t + 1];
    const double sa = gco * (tv - d0), db = gco * (d0 - tv);
    const double bn = bb - db, bold = p.beta[gc], rm = p.rmom[gc];
    const double nk = nvd * kappa;
    double rd = 0.0;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const int i = threadIdx.x + DT * q;
      ea[q] = ef[q] = 0.0;
      if (i < nv) {
        const double x = px[i];
        const double da = fma(sa, pv[i], x);
        ab[q] -= da;                                            // a+
        fb[q] -= fma(sa, kv[q], nk * fma(-lam2, x, pw[i]));     // f+
        ea[q] = ab[q] - pa[i];
        ef[q] = fb[q] - pf[i];
        rd = fma(da, ea[q], rd);
      }
    }
    rd = block_sum<DW>(rd, red1) + db * (bn - bold);
    const double rn = (restart && rd > 0.0) ? 1.0 : 0.5 * (1.0 + sqrt(1.0 + 4.0 * rm * rm));
    const double coef = (rn - 1.0) / (0.5 * (1.0 + sqrt(1.0 + 4.0 * rn * rn)));
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const int i = threadIdx.x + DT * q;
      if (i < nv) {
        pa[i] = ab[q];
        pf[i] = fb[q];
        ab[q] = fma(coef, ea[q], ab[q]);
        fb[q] = fma(coef, ef[q], fb[q]);
        pab[i] = ab[q];
        pfb[i] = fb[q];
      }
    }
    bb = fma(coef, bn - bold, bn);
    it = p.iters[gc] + 1;
    __syncthreads();                              // the scalars read by all
    if (threadIdx.x == 0) {
      p.beta[gc] = bn;
      p.bbar[gc] = bb;
      p.rmom[gc] = rn;
      p.iters[gc] = it;
      p.iters_total[gc] += 1;
      if (it >= max_iter) p.flag[gc] = 2;
    }
    if (it >= max_iter) return;
  }
  double zs = 0.0, n2 = 0.0, tv = 0.0;
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int i = threadIdx.x + DT * q;
    if (i < nv) {
      const double z = live[q] ? loss_psi(p.loss, yv[q], fb[q] + bb, delta, tau) / nvd : 0.0;
      const double w = fma(lam2, ab[q], z);
      zs += z;
      n2 = fma(w, w, n2);
      tv = fma(kv[q], w, tv);
      pw[i] = w;
    } else if (START && i < N) {
      pw[i] = 0.0;                                // padding rows stay zero
    }
  }
  block_sum3(zs, n2, tv, red);
  const double kkt = nvd * fmax(sqrt(n2), fabs(zs));
  const bool bad = !(n2 == n2) || !(zs == zs) || !(kkt <= 1e300);
  const bool done = !bad && kkt <= tol && may;
  if (done) {
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const int i = threadIdx.x + DT * q;
      if (i < nv) pa[i] = ab[q];                  // certified at the extrapolated point
    }
  }
  if (threadIdx.x == 0) {
    p.kkt[gc] = kkt;
    a.scal[2 * t] = zs;
    a.scal[2 * t + 1] = tv;
    if (bad) p.flag[gc] = 3;
    else if (done) {
      p.flag[gc] = 1;
      p.beta[gc] = bb;
    }
    if (START) a.sure[t] = done ? 1 : 0;
  }
}

// A column takes the f that was formed again from its alpha (VX, VT). One that has
// converged is active again until its residual there is known (the update with
// START, which follows; sure: 2, then 1 if it stays converged, with nothing left to
// check). One at max_iter must not stop there (count[1]) if the new f moves its
// residual n_v ||z + 2 lambda alpha|| by more than tol and 3/10 of itself.
__global__ __launch_bounds__(DT) void dense_check_kernel(const DenseArrays a, const PathArrays p,
                                                         double delta, double tol) {
  __shared__ double red[DW];
  const int t = blockIdx.x;
  if (t >= a.count[0] || a.sure[t] == 1) return;
  const int64_t gc = a.list[t];
  const int fl = p.flag[gc];
  if (fl > 2) return;                             // uniform over the block
  const int N = p.N, g = (int)(gc / p.C), nv = p.nv[g];
  const double *pn = dvec(a, N, VX, t), *pnb = dvec(a, N, VT, t);
  double *pf = dvec(a, N, VF, t), *pfb = dvec(a, N, VFB, t);
  if (fl < 2) {
    for (int i = threadIdx.x; i < nv; i += DT) {
      pf[i] = pn[i];
      pfb[i] = pnb[i];
    }
    if (threadIdx.x == 0) {
      p.flag[gc] = 0;
      a.sure[t] = 2 * fl;
    }
    return;
  }
  const double tau = p.tau[gc], kkt = p.kkt[gc], b = p.beta[gc];
  const int32_t hf = p.cfold ? p.cfold[gc] : -1;
  const int32_t* rf = p.rfold ? p.rfold + (int64_t)g * N : nullptr;
  const double* y = p.ylab + (int64_t)g * N;
  double e = 0.0;
  for (int i = threadIdx.x; i < nv; i += DT) {
    const double dz = loss_psi(p.loss, y[i], pn[i] + b, delta, tau) -
                      loss_psi(p.loss, y[i], pf[i] + b, delta, tau);
    if (!(rf && rf[i] == hf)) e = fma(dz, dz, e);
  }
  e = sqrt(block_sum<DW>(e, red));
  if (threadIdx.x == 0 && !(e <= fmax(tol, 0.3 * kkt))) atomicAdd(a.count + 1, 1);
}

// count[1]: also the columns that are not finite. count[2]: the least number of
// iterations of an active one.
__global__ __launch_bounds__(64) void dense_report_kernel(const DenseArrays a, const PathArrays p) {
  int least = INT32_MAX;
  for (int t = threadIdx.x; t < a.count[0]; t += 64) {
    const int64_t gc = a.list[t];
    const int fl = p.flag[gc];
    if (fl == 0) least = min(least, p.iters[gc]);
    if (fl > 2) atomicAdd(a.count + 1, 1);
  }
  for (int off = 32; off >= 1; off >>= 1) least = min(least, __shfl_xor(least, off, 64));
  if (threadIdx.x == 0) a.count[2] = least;
}

template <bool START>
int launch_update(hipStream_t s, const PathArrays& p, const DenseArrays& a, int cols, double delta,
                  double kappa, double tol, int max_iter, int restart) {
  const int rpt = (int)ceil_div(p.N, DT);
#define KMP_DENSE_CASE(R)                                                                        \
  if (rpt <= R) {                                                                                \
    hipLaunchKernelGGL((dense_update_kernel<R, START>), dim3((unsigned)cols), dim3(DT), 0, s, a, p, \
                       delta, kappa, tol, max_iter, restart);                                    \
    KMP_LAUNCH_CHECK();                                                                          \
    return 0;                                                                                    \
  }
  KMP_DENSE_CASE(1)
  KMP_DENSE_CASE(2)
  KMP_DENSE_CASE(4)
  KMP_DENSE_CASE(6)
#undef KMP_DENSE_CASE
  set_error("dense columns: order above " + std::to_string(kDenseMaxOrder));
  return KMP_EINVAL;
}
}  // namespace

int dense_begin(hipStream_t s, const PathArrays& p, const DenseArrays& a, int cols, double delta,
                double kappa, double tol) {
  int rc;
  const int N = p.N, nb = N / 64;
  hipLaunchKernelGGL(dense_list_kernel, dim3(1), dim3(64), 0, s, p.G, p.C, cols, p.cmap, p.nact,
                     a.list, a.sure, a.count);
  KMP_LAUNCH_CHECK();
  const int64_t blocks = (int64_t)cols * nb;
  for (int64_t e0 = 0; e0 < blocks; e0 += a.yblocks) {
    const int nblk = (int)std::min<int64_t>(a.yblocks, blocks - e0);
    hipLaunchKernelGGL(dense_rows_kernel, dim3((unsigned)nblk), dim3(256), 0, s, N, p.C, (int)e0, a,
                       p.Q, p.ldl_l, p.ldl_d, a.Y);
    KMP_LAUNCH_CHECK();
    if ((rc = resolvent_gemm(s, N, p.C, (int)e0, nblk, p.Q, a)) != 0) return rc;
  }
  hipLaunchKernelGGL((dense_vectors_kernel<false>), dim3((unsigned)(N / 4), (unsigned)cols), dim3(256),
                     0, s, N, p.C, a, p.Q, p.QB, p.nv, p.ahat, p.abar, p.vhat, p.uvec);
  KMP_LAUNCH_CHECK();
  return launch_update<true>(s, p, a, cols, delta, kappa, tol, 1 << 30, 0);
}

int dense_iterations(hipStream_t s, const PathArrays& p, const DenseArrays& a, int cols, double delta,
                     double kappa, double tol, int max_iter, int restart, int count) {
  int rc = 0;
  // the resolvent and 14 vectors of each column
  const double n = (double)p.N, flops = cols * (2.0 * n * n + 24.0 * n);
  for (int k = 0; k < count && rc == 0; ++k) {
    kc_begin(KMP_KC_UPDATE, s);
    hipLaunchKernelGGL(dense_product_kernel, dim3((unsigned)ceil_div(p.N, 2 * DW), (unsigned)cols),
                       dim3(DT), 0, s, p.N, a, p.flag);
    KMP_LAUNCH_CHECK();
    rc = launch_update<false>(s, p, a, cols, delta, kappa, tol, max_iter, restart);
    kc_end(KMP_KC_UPDATE, s, 8.0 * cols * (n * n + 14.0 * n), flops);
  }
  return rc;
}

int dense_check(hipStream_t s, const PathArrays& p, const DenseArrays& a, int cols, double delta,
                double kappa, double tol) {
  const int N = p.N;
  hipLaunchKernelGGL(dense_project_kernel, dim3((unsigned)(N / DPC), (unsigned)cols), dim3(DPC, DPR),
                     0, s, N, p.C, a, p.Q, p.nv, p.ahat, p.abar);
  KMP_LAUNCH_CHECK();
  hipLaunchKernelGGL((dense_vectors_kernel<true>), dim3((unsigned)(N / 4), (unsigned)cols), dim3(256),
                     0, s, N, p.C, a, p.Q, p.QB, p.nv, p.ahat, p.abar, p.vhat, p.uvec);
  KMP_LAUNCH_CHECK();
  hipLaunchKernelGGL(dense_check_kernel, dim3((unsigned)cols), dim3(DT), 0, s, a, p, delta, tol);
  KMP_LAUNCH_CHECK();
  const int rc = launch_update<true>(s, p, a, cols, delta, kappa, tol, 1 << 30, 0);
  if (rc != 0) return rc;
  hipLaunchKernelGGL(dense_report_kernel, dim3(1), dim3(64), 0, s, a, p);
  KMP_LAUNCH_CHECK();
  return 0;
}

}  // namespace kmp
