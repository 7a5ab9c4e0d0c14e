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
// tests do not change under the orthogonal Q). f is compared with K alpha
// through the factor when the columns have stopped (dense_check).
//
// Up to order kDenseSmall a column's whole stage runs in one workgroup with R
// in its registers; above, an iteration is two launches: the products of all
// dense columns spread over the chip, then one workgroup per column for
// everything elementwise. An iteration of 48 columns in 4 groups, batched and
// dense: order 64 27 and 1.1 us, 192 31 and 1.6 us, 256 33 and 3.4 us, 320
// 36 and 13 us, 832 (16 columns) 58 and 22 us, 1536 (4 columns) 81 and 22 us.
// Up to order 256 it is bound by the three barriers and the sums between
// them, above by the two launches and then by reading R (8 TB/s from the
// last-level cache). n = 200, 5 folds x 10 penalties, hinge: 77.9 -> 5.8 ms
// per call.
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

// The dense columns: the active columns first .. first + cap - 1, counted
// group by group in the order of the active lists (one wavefront).
__global__ __launch_bounds__(64) void dense_list_kernel(int G, int C, int first, int cap,
                                                        const int* __restrict__ cmap,
                                                        const int* __restrict__ nact,
                                                        int* __restrict__ list,
                                                        int* __restrict__ count) {
  int base = -first;
  for (int g = 0; g < G; ++g) {
    const int n = nact[g];
    for (int k = threadIdx.x; k < n; k += 64)
      if (base + k >= 0 && base + k < cap) list[base + k] = g * C + cmap[(int64_t)g * C + k];
    base += n;
  }
  if (threadIdx.x == 0) *count = max(0, min(base, cap));
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
  if (t >= *a.count) return;
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
  const int t = blockIdx.y;
  if (t >= *a.count) return;
  const int64_t gc = a.list[t];
  const int g = (int)(gc / C), m = nv[g];
  const int j = blockIdx.x * DPC + threadIdx.x, ry = threadIdx.y;
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
  const bool done = !bad && kkt <= tol;
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
  }
}

// A column's f against f formed again from alpha (VX, VT). Evaluating K alpha
// through the factor carries an error of the order of eps ||K|| ||alpha|| <=
// eps n ||alpha||_2, so a difference of at most 16 of these keeps f; beyond
// it the column takes the new f and, when it had converged, goes on.
__global__ __launch_bounds__(DT) void dense_check_kernel(const DenseArrays a, const PathArrays p) {
  __shared__ double red[DW];
  const int t = blockIdx.x;
  if (t >= *a.count) return;
  const int64_t gc = a.list[t];
  const int fl = p.flag[gc];
  if (fl > 1) return;                             // uniform over the block
  const int N = p.N, nv = p.nv[(int)(gc / p.C)];
  const double *pab = dvec(a, N, VAB, t), *pn = dvec(a, N, VX, t), *pnb = dvec(a, N, VT, t);
  double *pf = dvec(a, N, VF, t), *pfb = dvec(a, N, VFB, t);
  double n2 = 0.0, far = 0.0;
  for (int i = threadIdx.x; i < nv; i += DT) n2 = fma(pab[i], pab[i], n2);
  n2 = block_sum<DW>(n2, red);
  const double bound = 16.0 * 2.220446049250313e-16 * nv * sqrt(n2);
  for (int i = threadIdx.x; i < nv; i += DT) far += fabs(pnb[i] - pfb[i]) <= bound ? 0.0 : 1.0;
  far = block_sum<DW>(far, red);
  if (far == 0.0) return;
  for (int i = threadIdx.x; i < nv; i += DT) {
    pf[i] = pn[i];
    pfb[i] = pnb[i];
  }
  if (threadIdx.x == 0) p.flag[gc] = 0;
}

// Orders up to kDenseSmall. R = Y Q' in place: a wavefront multiplies its own
// 16 rows of Y, read whole before they are overwritten. Both operands are
// rows along k: lane group lk takes k = 16 c + 4 lk + s in MFMA step s, 32
// contiguous bytes of each row.
template <int NT>
__global__ __launch_bounds__(256) void dense_small_gemm_kernel(int C, const DenseArrays a,
                                                               const double* __restrict__ Q) {
  constexpr int N = 16 * NT, nb = N / 64;
  const int t = (int)blockIdx.x / nb;
  if (t >= *a.count) return;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const double* q = Q + (int64_t)(a.list[t] / C) * N * N + (int64_t)li * N + 4 * lk;
  double* y = a.R + ((int64_t)blockIdx.x * 64 + 16 * w) * N;
  ddbl4 acc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[j] = ddbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int k = 0; k < N; k += 16) {
    const double2* yr = reinterpret_cast<const double2*>(y + (int64_t)li * N + 4 * lk + k);
    const double2 a01 = yr[0], a23 = yr[1];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const double2* qr = reinterpret_cast<const double2*>(q + (int64_t)16 * j * N + k);
      const double2 b01 = qr[0], b23 = qr[1];
      acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a01.x, b01.x, acc[j], 0, 0, 0);
      acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a01.y, b01.y, acc[j], 0, 0, 0);
      acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a23.x, b23.x, acc[j], 0, 0, 0);
      acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a23.y, b23.y, acc[j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) y[(int64_t)(4 * r + lk) * N + 16 * j + li] = acc[j][r];
}

// Sum over the wavefront in every lane: rotations within the rows of 16
// lanes, then the permlane swaps.
template <int R>
__device__ __forceinline__ double row_ror(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x120 + R, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x120 + R, 0xf, 0xf, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ double fast_wave_sum(double v) {
  v += row_ror<8>(v);
  v += row_ror<4>(v);
  v += row_ror<2>(v);
  v += row_ror<1>(v);
  {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    v = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
        __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
  }
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}

// Up to `count` iterations of one column per workgroup (order N = 64 NR), the
// same steps as dense_product_kernel and dense_update_kernel with nothing
// leaving the compute unit: wavefront w keeps columns CW w .. of R, lane l the
// rows l, l + 64, .., in registers (the last CL of them in LDS at NR = 4,
// where the registers hold no more); w is read from LDS as a broadcast and
// the wavefronts' partial products are added through LDS by thread i < N,
// which owns row i. Three barriers per iteration: w and its sums, the
// partial products, the restart test. LOSS is the loss code: fixed, so that
// the registers hold nothing for the other losses.
template <int NR, int LOSS>
__global__ __launch_bounds__(DT) void dense_small_kernel(const DenseArrays a, const PathArrays p,
                                                         double delta, double kappa, double tol,
                                                         int max_iter, int restart, int count) {
  constexpr int N = 64 * NR, CW = N / DW, CL = NR == 4 ? 8 : 0, CR = CW - CL;
  __shared__ double ws[N];
  __shared__ double xp[DW][N];
  __shared__ double red[NR][3], red1[NR];
  __shared__ double rl[CL > 0 ? DW * CL : 1][CL > 0 ? N : 1];
  __shared__ double own_lds[5][CL > 0 ? N : 1];   // the owner's v, K v, y, alpha, f at NR = 4
  const int t = blockIdx.x;
  if (t >= *a.count) return;
  const int64_t gc = a.list[t];
  if (p.flag[gc] != 0) return;                    // uniform over the block
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  const int g = (int)(gc / p.C), nv = p.nv[g];
  const double lam2 = 2.0 * p.lam[gc], nvd = (double)p.cnv[gc], tau = p.tau[gc];
  const double nk = nvd * kappa, gco = p.gcoef[gc];
  // R is symmetric: its row c holds column c contiguously
  double rr[NR][CR];
  const double* R = a.R + (int64_t)t * N * N + (int64_t)(CW * wv) * N + lane;
#pragma unroll
  for (int c = 0; c < CR; ++c)
#pragma unroll
    for (int q = 0; q < NR; ++q) rr[q][c] = R[c * N + 64 * q];
#pragma unroll
  for (int c = 0; c < CL; ++c)
#pragma unroll
    for (int q = 0; q < NR; ++q) rl[CL * wv + c][64 * q + lane] = R[(CR + c) * N + 64 * q];
  const bool own = tid < N, valid = tid < nv;
  const int i = own ? tid : 0;
  double reg[5];
  const auto mine = [&](int k) -> double& {
    if constexpr (CL > 0) return own_lds[k][i];
    else return reg[k];
  };
  if (own) {
    mine(0) = dvec(a, N, VV, t)[i];
    mine(1) = dvec(a, N, VKV, t)[i];
    mine(2) = p.ylab[(int64_t)g * N + i];
    mine(3) = dvec(a, N, VA, t)[i];
    mine(4) = dvec(a, N, VF, t)[i];
  }
  double ab = dvec(a, N, VAB, t)[i], fb = dvec(a, N, VFB, t)[i], w = dvec(a, N, VW, t)[i];
  const bool live = valid && !(p.rfold && p.rfold[(int64_t)g * N + i] == p.cfold[gc]);
  double d0 = a.scal[2 * t], tv = a.scal[2 * t + 1];
  double beta = p.beta[gc], bb = p.bbar[gc], rm = p.rmom[gc], kkt = p.kkt[gc];
  const int it0 = p.iters[gc];
  int it = it0, fl = 0;
  if (own) ws[tid] = w;
  __syncthreads();
  for (int n = 0; n < count; ++n) {
    // x = R w: the wavefront's columns
    double s[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) s[q] = 0.0;
#pragma unroll
    for (int c = 0; c < CR; c += 2) {
      const double2 wc = *reinterpret_cast<const double2*>(&ws[CW * wv + c]);
#pragma unroll
      for (int q = 0; q < NR; ++q) s[q] = fma(rr[q][c + 1], wc.y, fma(rr[q][c], wc.x, s[q]));
      // at NR = 4 no registers are left to read w far ahead
      if constexpr (CL > 0) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int c = 0; c < CL; ++c) {
#pragma unroll
      for (int q = 0; q < NR; ++q)
        s[q] = fma(rl[CL * wv + c][64 * q + lane], ws[CW * wv + CR + c], s[q]);
      if constexpr (CL > 0) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) xp[wv][64 * q + lane] = s[q];
    // the momentum without a restart needs nothing of this step
    const double rn1 = 0.5 * (1.0 + sqrt(1.0 + 4.0 * rm * rm));
    const double co1 = (rn1 - 1.0) / (0.5 * (1.0 + sqrt(1.0 + 4.0 * rn1 * rn1)));
    const double sa = gco * (tv - d0), db = gco * (d0 - tv);
    const double bn = bb - db;
    __syncthreads();
    double ea = 0.0, ef = 0.0, rd = 0.0;
    if (wv < NR) {
      double x = 0.0;
#pragma unroll
      for (int j = 0; j < DW; ++j) x += xp[j][tid];
      if (valid) {
        const double da = fma(sa, mine(0), x);
        ab -= da;
        fb -= fma(sa, mine(1), nk * fma(-lam2, x, w));
        ea = ab - mine(3);
        ef = fb - mine(4);
        rd = da * ea;
      }
      rd = fast_wave_sum(rd);
      if (lane == 0) red1[wv] = rd;
    }
    __syncthreads();
    rd = db * (bn - beta);
#pragma unroll
    for (int j = 0; j < NR; ++j) rd += red1[j];
    const bool turn = restart && rd > 0.0;
    const double coef = turn ? 0.0 : co1;
    rm = turn ? 1.0 : rn1;
    if (valid) {
      mine(3) = ab;
      mine(4) = fb;
    }
    ab = fma(coef, ea, ab);
    fb = fma(coef, ef, fb);
    bb = fma(coef, bn - beta, bn);
    beta = bn;
    if (++it >= max_iter) {
      fl = 2;
      break;
    }
    double zs = 0.0, n2 = 0.0, tw = 0.0;
    if (wv < NR) {
      if (valid) {
        zs = live ? loss_psi(LOSS, mine(2), fb + bb, delta, tau) / nvd : 0.0;
        w = fma(lam2, ab, zs);
        n2 = w * w;
        tw = mine(1) * w;
        ws[tid] = w;
      }
      zs = fast_wave_sum(zs);
      n2 = fast_wave_sum(n2);
      tw = fast_wave_sum(tw);
      if (lane == 0) {
        red[wv][0] = zs;
        red[wv][1] = n2;
        red[wv][2] = tw;
      }
    }
    __syncthreads();
    d0 = tv = n2 = 0.0;
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      d0 += red[j][0];
      n2 += red[j][1];
      tv += red[j][2];
    }
    kkt = nvd * fmax(sqrt(n2), fabs(d0));
    if (!(n2 == n2) || !(d0 == d0) || !(kkt <= 1e300)) {
      fl = 3;
      break;
    }
    if (kkt <= tol) {                             // certified at the extrapolated point
      fl = 1;
      if (valid) mine(3) = ab;
      beta = bb;
      break;
    }
  }
  if (own) {
    dvec(a, N, VA, t)[i] = mine(3);
    dvec(a, N, VAB, t)[i] = ab;
    dvec(a, N, VF, t)[i] = mine(4);
    dvec(a, N, VFB, t)[i] = fb;
    dvec(a, N, VW, t)[i] = w;
  }
  if (tid == 0) {
    a.scal[2 * t] = d0;
    a.scal[2 * t + 1] = tv;
    p.beta[gc] = beta;
    p.bbar[gc] = bb;
    p.rmom[gc] = rm;
    p.kkt[gc] = kkt;
    p.iters[gc] = it;
    p.iters_total[gc] += it - it0;
    if (fl != 0) p.flag[gc] = fl;
  }
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

int dense_begin(hipStream_t s, const PathArrays& p, const DenseArrays& a, int first, int cols,
                double delta, double kappa, double tol) {
  int rc;
  const int N = p.N, nb = N / 64;
  hipLaunchKernelGGL(dense_list_kernel, dim3(1), dim3(64), 0, s, p.G, p.C, first, cols, p.cmap,
                     p.nact, a.list, a.count);
  KMP_LAUNCH_CHECK();
  const int64_t blocks = (int64_t)cols * nb;
  if (N <= kDenseSmall) {
    hipLaunchKernelGGL(dense_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, s, N, p.C, 0, a, p.Q,
                       p.ldl_l, p.ldl_d, a.R);
    KMP_LAUNCH_CHECK();
#define KMP_SMALL_CASE(NR)                                                                       \
  if (N == 64 * NR)                                                                              \
    hipLaunchKernelGGL((dense_small_gemm_kernel<4 * NR>), dim3((unsigned)blocks), dim3(256), 0, s, \
                       p.C, a, p.Q);
    KMP_SMALL_CASE(1)
    KMP_SMALL_CASE(2)
    KMP_SMALL_CASE(3)
    KMP_SMALL_CASE(4)
#undef KMP_SMALL_CASE
    KMP_LAUNCH_CHECK();
  } else {
    for (int64_t e0 = 0; e0 < blocks; e0 += a.yblocks) {
      const int nblk = (int)std::min<int64_t>(a.yblocks, blocks - e0);
      hipLaunchKernelGGL(dense_rows_kernel, dim3((unsigned)nblk), dim3(256), 0, s, N, p.C, (int)e0, a,
                         p.Q, p.ldl_l, p.ldl_d, a.Y);
      KMP_LAUNCH_CHECK();
      if ((rc = resolvent_gemm(s, N, p.C, (int)e0, nblk, p.Q, a)) != 0) return rc;
    }
  }
  hipLaunchKernelGGL((dense_vectors_kernel<false>), dim3((unsigned)(N / 4), (unsigned)cols), dim3(256),
                     0, s, N, p.C, a, p.Q, p.QB, p.nv, p.ahat, p.abar, p.vhat, p.uvec);
  KMP_LAUNCH_CHECK();
  return launch_update<true>(s, p, a, cols, delta, kappa, tol, 1 << 30, 0);
}

int dense_iterations(hipStream_t s, const PathArrays& p, const DenseArrays& a, int cols, double delta,
                     double kappa, double tol, int max_iter, int restart, int count) {
  int rc = 0;
  // the resolvent and 14 vectors of each column and iteration (the register
  // form reads them once)
  const double n = (double)p.N, flops = cols * (2.0 * n * n + 24.0 * n);
  if (p.N <= kDenseSmall) {
    kc_begin(KMP_KC_UPDATE, s);
#define KMP_SMALL_CASE(NR, LS)                                                                   \
  if (p.N == 64 * NR && p.loss == LS)                                                            \
    hipLaunchKernelGGL((dense_small_kernel<NR, LS>), dim3((unsigned)cols), dim3(DT), 0, s, a, p, \
                       delta, kappa, tol, max_iter, restart, count);
#define KMP_SMALL_CASES(LS) \
  KMP_SMALL_CASE(1, LS)     \
  KMP_SMALL_CASE(2, LS)     \
  KMP_SMALL_CASE(3, LS)     \
  KMP_SMALL_CASE(4, LS)
    KMP_SMALL_CASES(0)
    KMP_SMALL_CASES(1)
    KMP_SMALL_CASES(2)
#undef KMP_SMALL_CASES
#undef KMP_SMALL_CASE
    KMP_LAUNCH_CHECK();
    kc_end(KMP_KC_UPDATE, s, 8.0 * cols * (n * n + 14.0 * n), flops);
    return 0;
  }
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
  hipLaunchKernelGGL(dense_check_kernel, dim3((unsigned)cols), dim3(DT), 0, s, a, p);
  KMP_LAUNCH_CHECK();
  return launch_update<true>(s, p, a, cols, delta, kappa, tol, 1 << 30, 0);
}

}  // namespace kmp
