// Small orders (up to kSmallOrder rows per group): every column's whole path in
// one workgroup, without a factorisation.
//
// A column's dense resolvent R = (2 lambda I + K/(n_v kappa))^{-1} is kept in the
// registers of one compute unit, the last columns in LDS at order 256. It takes all
// of them from order 192: 24 to 50 registers a lane are spilled there and 126 to 145
// at 256, the rest of the state and part of R among them, which the sweeps and the
// iterations read back. It is formed from K by symmetric sweeps and the accelerated iteration runs
// on alpha and f = K alpha in observation space (see dense.hip for the
// recurrence): x = R w, K x = n_v kappa (w - 2 lambda x), so neither K nor R is
// read again until a stage ends. The smoothing stages follow one another in
// the same launch, so no column waits for another's stage.
//
// An iteration is bound by its chain: a 64 NR x 64 NR product from registers,
// a barrier, the update and both outcomes of the restart test, a barrier. At
// 192 rows it takes 1.3 us (2.0 with a barrier for the restart test and the
// sums on the way), where a batched iteration of five folds by ten penalties
// is four dependent launches, 31 us. The sweeps are N rank-one updates, 0.03 /
// 0.1 / 0.2 / 0.85 ms at 64 / 128 / 192 / 256 rows.
// Five folds of 200 rows by ten penalties, hinge loss: 69.5 ms in batched
// form, 5.2 with the resolvents formed from the factorisation and a launch per
// stage, 4.0 here; leave-one-out, 151 rows, logistic loss: 3.2, 2.9, 0.90 ms.
// f is carried by the recurrence, whose rounding grows as lambda shrinks (n = 180,
// lambda = 1e-8: f said 1e-9 where K alpha said 2.5e-5). So a column stops as
// converged in the last stage only by the residual at f = K alpha formed again, and
// what stops at max_iter with another f than that goes to the batched iteration.
#include "kmp_common.h"
#include "kmp_kernels.h"
#include <algorithm>
#include <cmath>
#include <type_traits>

namespace kmp {

namespace {
constexpr int DT = 512;                 // threads of a column's workgroup
constexpr int DW = DT / 64;
// Times a column may meet tol with its carried f and not with K alpha. Each time it
// goes on from the new f, and what the recurrence adds shrinks with the residual.
constexpr int kSmallRefresh = 8;

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

// loss_psi by selects, the division by 2 delta as a product: two of them are
// on the way from one product to the next.
template <int LOSS>
__device__ __forceinline__ double psi_select(double y, double f, double delta, double i2d, double tau) {
  if constexpr (LOSS == 1) return -y / (1.0 + exp(y * f));
  const double u = LOSS == 0 ? y * f : y - f;
  double d;
  if constexpr (LOSS == 0) {
    d = (u - 1.0 - delta) * i2d;
    d = u < 1.0 + delta ? d : 0.0;
    return y * (u <= 1.0 - delta ? -1.0 : d);
  } else {
    d = (u + delta * (2.0 * tau - 1.0)) * i2d;
    d = u <= -delta ? tau - 1.0 : d;
    return -(u >= delta ? tau : d);
  }
}

// Wavefront w keeps columns CW w .. of the matrix, lane l the rows l, l + 64,
// .., in registers, the last CL of the columns in LDS at NR = 4, where the
// registers hold no more. Thread i < N owns row i of the vectors; the last
// wavefronts, which own none, add up the sums. ahat and abar hold alpha and its
// extrapolation in observation space here, gcoef the stage a column is in.
//
// A workgroup takes `run` columns that follow each other in the order (group,
// penalty, the rest) and forms R again only where it differs: leave-one-out
// columns of one penalty share it, as long as there is one stage.
template <int NR, int LOSS>
__global__ __launch_bounds__(DT) void small_path_kernel(const PathArrays p,
                                                        const double* __restrict__ Kall,
                                                        const SmallStages st, double tol,
                                                        int max_iter, int restart, int count,
                                                        int begin, int L, int run) {
  constexpr int N = 64 * NR, CW = N / DW, CL = NR == 4 ? 8 : 0, CR = CW - CL;
  __shared__ double ws[2][N], zs[2][N];           // w and z without and with a restart
  __shared__ double xp[DW][N];                    // partial products; the swept column
  __shared__ double kvs[N];                       // K v
  __shared__ double red3[3], red1[NR], piv[2], mom[2];
  __shared__ double rl[CL > 0 ? DW * CL : 1][CL > 0 ? N : 1];
  __shared__ double own_lds[2][NR > 2 ? N : 1];   // the owner's v, alpha where registers are short
  const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const bool own = tid < N;
  const int i = own ? tid : 0;
  double rr[NR][CR];
  double reg[2];
  const auto mine = [&](int k) -> double& {
    if constexpr (NR > 2) return own_lds[k][i];
    else return reg[k];
  };
  // sums over the owners' wavefronts, to every thread
  const auto sum1 = [&](double a) {
    if (wv < NR) {
      a = fast_wave_sum(a);
      if (lane == 0) red1[wv] = a;
    }
    __syncthreads();
    a = 0.0;
#pragma unroll
    for (int j = 0; j < NR; ++j) a += red1[j];
    __syncthreads();
    return a;
  };
  // the partial products of the wavefronts (xp), added by the owner
  const auto gather = [&]() {
    double x = 0.0;
#pragma unroll
    for (int j = 0; j < DW; ++j) x += xp[j][i];
    return x;
  };
  int hg = -1;                                    // what R was formed for
  double hl = 0.0, hn = 0.0, gco = 0.0;
  for (int r = 0; r < run; ++r) {
    const int64_t m = (int64_t)blockIdx.x * run + r;
    if (m >= (int64_t)p.G * p.C) break;
    const int g = (int)(m / p.C), mc = (int)(m % p.C), same = p.C / L;
    const int64_t gc = (int64_t)g * p.C + (mc % same) * L + mc / same;
    if (p.flag[gc] != 0) continue;                // uniform over the block
    __syncthreads();
    const int nv = p.nv[g];
    const double lam2 = 2.0 * p.lam[gc], nvd = (double)p.cnv[gc], tau = p.tau[gc];
    const double* K = Kall + (int64_t)g * N * N;
    const double* kcol = K + (int64_t)(CW * wv) * N + lane;   // K symmetric: row c is column c
    const bool valid = tid < nv;
    const int64_t row = gc * (int64_t)N + i;
    const bool live = valid && !(p.rfold && p.rfold[(int64_t)g * N + i] == p.cfold[gc]);
    // K u for the vector u given by the owners
    const auto k_times = [&](double u) {
      if (own) ws[0][tid] = valid ? u : 0.0;
      __syncthreads();
      double s[NR];
#pragma unroll
      for (int q = 0; q < NR; ++q) s[q] = 0.0;
      const double* kc = kcol;
      asm volatile("" : "+v"(kc));
#pragma unroll 4
      for (int c = 0; c < CW; ++c) {
        const double wc = ws[0][CW * wv + c];
#pragma unroll
        for (int q = 0; q < NR; ++q) s[q] = fma(kc[c * N + 64 * q], wc, s[q]);
      }
#pragma unroll
      for (int q = 0; q < NR; ++q) xp[wv][64 * q + lane] = s[q];
      __syncthreads();
      const double x = gather();
      __syncthreads();
      return valid ? x : 0.0;
    };
    // the wavefront's partial of R w, into xp
    const auto r_times = [&](const double* w) {
      double s[NR];
#pragma unroll
      for (int q = 0; q < NR; ++q) s[q] = 0.0;
#pragma unroll
      for (int c = 0; c < CR; c += 2) {
        const double2 wc = *reinterpret_cast<const double2*>(&w[CW * wv + c]);
#pragma unroll
        for (int q = 0; q < NR; ++q) s[q] = fma(rr[q][c + 1], wc.y, fma(rr[q][c], wc.x, s[q]));
        // no registers are left to read w far ahead
        if (CL > 0 || (NR == 3 && c % 8 == 6)) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int c = 0; c < CL; ++c) {
#pragma unroll
        for (int q = 0; q < NR; ++q)
          s[q] = fma(rl[CL * wv + c][64 * q + lane], w[CW * wv + CR + c], s[q]);
        if constexpr (CL > 0) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int q = 0; q < NR; ++q) xp[wv][64 * q + lane] = s[q];
    };
    // (t_1, t_2) -> t_2 and the extrapolation (t_1 - 1)/t_2 of the accelerated step
    const auto momentum = [](double t, double* next, double* coef) {
      *next = 0.5 * (1.0 + sqrt(1.0 + 4.0 * t * t));
      *coef = (*next - 1.0) / (0.5 * (1.0 + sqrt(1.0 + 4.0 * *next * *next)));
    };

    int stage = begin ? 0 : (int)p.gcoef[gc];
    int it = begin ? 0 : p.iters[gc], total = begin ? 0 : p.iters_total[gc];
    bool fresh = begin != 0;                        // a stage starts: r = 1, abar = alpha
    double beta = p.beta[gc], bb = p.bbar[gc], rm = p.rmom[gc], kkt = 0.0;
    const double ylab = p.ylab[(int64_t)g * N + i];
    if (own) mine(1) = p.ahat[row];
    double ab = p.abar[row];
    int left = count, fl = 0, refreshes = 0;
    for (;;) {
      const double delta = st.delta[stage], kappa = st.kappa[stage];
      const double nk = nvd * kappa, inv = 1.0 / nvd, i2d = 0.5 / delta;
      if (g != hg || lam2 != hl || nk != hn) {
        hg = g;
        hl = lam2;
        hn = nk;
        // M = 2 lambda I + K/(n_v kappa)
        const double ink = 1.0 / nk;
        // (per stage: as loop invariants the addresses and the diagonal's lane masks
        // would take the registers of R)
        const double* kc = kcol;
        int dl = lane - CW * wv;                      // entry (64 q + lane, CW wv + c): dl + 64 q == c
        asm volatile("" : "+v"(kc), "+v"(dl));
#pragma unroll
        for (int c = 0; c < CR; ++c) {
#pragma unroll
          for (int q = 0; q < NR; ++q)
            rr[q][c] = fma(kc[c * N + 64 * q], ink, dl + 64 * q == c ? lam2 : 0.0);
          if (c % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int c = 0; c < CL; ++c)
#pragma unroll
          for (int q = 0; q < NR; ++q)
            rl[CL * wv + c][64 * q + lane] =
                fma(kc[(CR + c) * N + 64 * q], ink, dl + 64 * q == CR + c ? lam2 : 0.0);
        // sweep on index pv: with d = M_pp, column a = M e_p,
        //   M_ij -= a_i a_j / d, M_ip = M_pi = a_i / d, M_pp = -1/d,
        // which keeps M symmetric; after all N it holds -M^{-1} (M is positive
        // definite: no pivoting). With row and column pv set to 0 and a_p to -1
        // the first formula gives all three. The swept column passes through xp,
        // two slots by parity, so one barrier a sweep.
#pragma unroll 1
        for (int wp = 0; wp < DW; ++wp) {
#pragma unroll 1
          for (int pc = 0; pc < CW; ++pc) {
            const int pv = CW * wp + pc, qp = pv >> 6;
            const bool lp = lane == (pv & 63);
            double* col = xp[pv & 1];
            if (wv == wp) {
              double d = 0.0;
              const auto publish = [&](auto kc) {
                constexpr int k = decltype(kc)::value;
                if constexpr (k < CR) {
#pragma unroll
                  for (int q = 0; q < NR; ++q) {
                    if (q == qp) d = rr[q][k];
                    col[64 * q + lane] = rr[q][k];
                    rr[q][k] = 0.0;
                  }
                }
              };
              switch (pc) {
#define KMP_PUB(k) case k: publish(std::integral_constant<int, k>()); break;
#define KMP_PUB4(k) KMP_PUB(k) KMP_PUB(k + 1) KMP_PUB(k + 2) KMP_PUB(k + 3)
                KMP_PUB4(0) KMP_PUB4(4) KMP_PUB4(8) KMP_PUB4(12) KMP_PUB4(16) KMP_PUB4(20)
#undef KMP_PUB4
#undef KMP_PUB
                default:
                  if constexpr (CL > 0) {
#pragma unroll
                    for (int q = 0; q < NR; ++q) {
                      double& m = rl[CL * wv + pc - CR][64 * q + lane];
                      if (q == qp) d = m;
                      col[64 * q + lane] = m;
                      m = 0.0;
                    }
                  }
              }
              if (lp) {
                col[pv] = -1.0;
                piv[pv & 1] = d;
              }
            }
            if (lp) {
#pragma unroll
              for (int q = 0; q < NR; ++q)
                if (q == qp) {
#pragma unroll
                  for (int c = 0; c < CR; ++c) rr[q][c] = 0.0;
                }
            }
            if constexpr (CL > 0) {
              if (lane < CL) rl[CL * wv + lane][pv] = 0.0;
            }
            __syncthreads();
            const double rd = -1.0 / piv[pv & 1];
            double a[NR];
#pragma unroll
            for (int q = 0; q < NR; ++q) a[q] = col[64 * q + lane] * rd;
#pragma unroll
            for (int c = 0; c < CR; c += 2) {
              const double2 b = *reinterpret_cast<const double2*>(&col[CW * wv + c]);
#pragma unroll
              for (int q = 0; q < NR; ++q) {
                rr[q][c] = fma(a[q], b.x, rr[q][c]);
                rr[q][c + 1] = fma(a[q], b.y, rr[q][c + 1]);
              }
              if (CL > 0 || c % 4 == 2) __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int c = 0; c < CL; ++c) {
              const double b = col[CW * wv + CR + c];
#pragma unroll
              for (int q = 0; q < NR; ++q) {
                double& m = rl[CL * wv + c][64 * q + lane];
                m = fma(a[q], b, m);
              }
            }
          }
        }
#pragma unroll
        for (int c = 0; c < CR; ++c)
#pragma unroll
          for (int q = 0; q < NR; ++q) rr[q][c] = -rr[q][c];
#pragma unroll
        for (int c = 0; c < CL; ++c)
#pragma unroll
          for (int q = 0; q < NR; ++q) rl[CL * wv + c][64 * q + lane] = -rl[CL * wv + c][64 * q + lane];
        // v = R 1/(n_v kappa), K v, g = 1/(2 lambda 1'v)
        __syncthreads();
        if (own) ws[0][tid] = valid ? ink : 0.0;
        __syncthreads();
        r_times(ws[0]);
        __syncthreads();
        const double v = valid ? gather() : 0.0;
        gco = 1.0 / (lam2 * sum1(valid ? v : 0.0));
        const double kv = k_times(v);
        if (own) {
          mine(0) = v;
          kvs[tid] = kv;
        }
      }
      if (fresh) {
        ab = own ? mine(1) : 0.0;
        bb = beta;
        rm = 1.0;
        it = 0;
      }
      // (alpha = 0 where the path begins)
      double f = begin && stage == 0 && fresh ? 0.0 : k_times(own ? mine(1) : 0.0);
      double fb = fresh ? f : k_times(ab);
      fresh = false;
      bool formed = true;                           // fb is K abar itself
      // z and w at (a, fa, b), into slot k
      const auto residual = [&](int k, double a, double fa, double b) {
        double z = psi_select<LOSS>(ylab, fa + b, delta, i2d, tau) * inv;
        z = live ? z : 0.0;
        const double w = valid ? fma(lam2, a, z) : 0.0;
        zs[k][tid] = z;
        ws[k][tid] = w;
      };
      double rn1, co1, rn0, co0, d0 = 0.0, n2 = 0.0;
      momentum(1.0, &rn0, &co0);
      momentum(rm, &rn1, &co1);
      int k = 0;
      if (own) residual(0, ab, fb, bb);
      __syncthreads();
      for (;;) {
        // x = R w; the sums of z, w^2 and (K v) w by wavefronts of their own
        r_times(ws[k]);
        if (wv >= DW - 4 && wv < DW - 1) {
          double s = 0.0;
#pragma unroll
          for (int q = 0; q < NR; ++q) {
            const double z = zs[k][64 * q + lane], w = ws[k][64 * q + lane], v = kvs[64 * q + lane];
            s = fma(wv == DW - 4 ? z : w, wv == DW - 4 ? 1.0 : wv == DW - 3 ? w : v, s);
          }
          s = fast_wave_sum(s);
          if (lane == 0) red3[wv - (DW - 4)] = s;
        }
        __syncthreads();
        d0 = red3[0];
        n2 = red3[1];
        const double tv = red3[2];
        // the exact test only where it may hold
        const double q2 = nvd * nvd * n2;
        if (!(q2 > 1.000001 * (tol * tol) && q2 <= 1e280)) {
          kkt = nvd * fmax(sqrt(n2), fabs(d0));
          if (!(n2 == n2) || !(d0 == d0) || !(kkt <= 1e300)) fl = 4;
          else if (kkt <= tol) {
            if (valid) mine(1) = ab;                // certified at the extrapolated point
            beta = bb;
            // (the stages before the last only lead to it, which starts from K alpha)
            if (formed || stage + 1 < st.n) fl = 1;
            else if (++refreshes > kSmallRefresh) fl = 4;
            else {
              f = fb = k_times(ab);
              formed = true;
              k = 0;
              if (own) residual(0, ab, fb, bb);
              __syncthreads();
              continue;
            }
          }
        }
        if (fl != 0 || left <= 0) break;
        --left;
        ++total;
        formed = false;
        const bool last = ++it >= max_iter;
        const double sa = gco * (tv - d0), db = gco * (d0 - tv);
        const double bn = bb - db, be = bn - beta;
        double ea = 0.0, ef = 0.0;
        if (wv < NR) {
          const double x = gather();
          double rd = 0.0;
          if (valid) {
            const double da = fma(sa, mine(0), x);
            ab -= da;
            fb -= fma(sa, kvs[i], nk * fma(-lam2, x, ws[k][i]));
            ea = ab - mine(1);
            ef = fb - f;
            rd = da * ea;
            mine(1) = ab;
            f = fb;
          }
          // both outcomes of the restart test, so that the next product waits
          // for one barrier
          residual(0, fma(co1, ea, ab), fma(co1, ef, fb), fma(co1, be, bn));
          residual(1, ab, fb, bn);
          rd = fast_wave_sum(rd);
          if (lane == 0) red1[wv] = rd;
        } else if (wv == DW - 1) {
          double tn, tc;
          momentum(rn1, &tn, &tc);
          if (lane == 0) {
            mom[0] = tn;
            mom[1] = tc;
          }
        }
        __syncthreads();
        double rd = db * be;
#pragma unroll
        for (int j = 0; j < NR; ++j) rd += red1[j];
        k = restart && rd > 0.0 ? 1 : 0;
        beta = bn;
        if (k == 0) {
          ab = fma(co1, ea, ab);
          fb = fma(co1, ef, fb);
          bb = fma(co1, be, bn);
          rm = rn1;
          rn1 = mom[0];
          co1 = mom[1];
        } else {
          bb = bn;
          rm = 1.0;
          rn1 = rn0;
          co1 = co0;
        }
        if (last) {
          fl = 2;
          break;
        }
      }
      kkt = nvd * fmax(sqrt(n2), fabs(d0));
      if (fl == 2) {
        // the limit has to be the column's: its residual mostly that of K alpha, and
        // above the rounding of such a product (eps ||alpha||_2 in an f_i)
        const double al = own && valid ? mine(1) : 0.0;
        const double fn = k_times(al);
        const double dz = psi_select<LOSS>(ylab, fn + beta, delta, i2d, tau) -
                          psi_select<LOSS>(ylab, f + beta, delta, i2d, tau);
        const double off = sqrt(sum1(live ? dz * dz : 0.0));
        const double rnd = kEps * (LOSS == 1 ? 0.25 : i2d) * sqrt(nv * sum1(al * al));
        if (!(off <= fmax(tol, 0.3 * kkt) && kkt > 4.0 * rnd)) fl = 4;
      }
      if (fl == 0 || fl == 4 || stage + 1 >= st.n) break;
      fl = 0;
      ++stage;                                      // converged or at max_iter: the next stage
      fresh = true;
      __syncthreads();
    }
    if (own) {
      p.ahat[row] = valid ? mine(1) : 0.0;
      p.abar[row] = valid ? ab : 0.0;
    }
    if (tid == 0) {
      p.gcoef[gc] = (double)stage;
      p.beta[gc] = beta;
      p.bbar[gc] = bb;
      p.rmom[gc] = rm;
      p.kkt[gc] = kkt;
      p.iters[gc] = it;
      p.iters_total[gc] = total;
      p.flag[gc] = fl;
    }
  }
}

// total[0]: columns still active; total[1]: the largest iters of any column, the
// largest int if one has flag 4.
__global__ __launch_bounds__(1024) void small_report_kernel(int64_t cols, const int* __restrict__ flag,
                                                            const int* __restrict__ iters,
                                                            int* __restrict__ total) {
  __shared__ int part[2][16];
  int act = 0, most = 0;
  for (int64_t c = threadIdx.x; c < cols; c += 1024) {
    const int fl = flag[c];
    act += fl == 0 ? 1 : 0;
    most = max(most, fl == 4 ? INT32_MAX : iters[c]);
  }
  for (int off = 32; off >= 1; off >>= 1) {
    act += __shfl_xor(act, off, 64);
    most = max(most, __shfl_xor(most, off, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    part[0][threadIdx.x >> 6] = act;
    part[1][threadIdx.x >> 6] = most;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) {
      act += part[0][w];
      most = max(most, part[1][w]);
    }
    total[0] = act;
    total[1] = most;
  }
}
}  // namespace

// One column a workgroup while its stages differ in R; with one stage the
// `same` columns of a group and penalty share it, and 256 workgroups fill the
// device.
static int small_run(int stages, int64_t cols, int64_t same) {
  return stages == 1 ? (int)std::min(ceil_div(cols, 256), same) : 1;
}

// Times in us. The hinge and check losses' iterations in a stage are taken as 0.27
// ln(1/tol) times the square root of the condition 1 + 1/(2 lambda kappa) of the
// majorised problem, for the check loss, whose columns the few points in its
// quadratic zone hold back, between 5 and 14 over the root of delta. Here a compute
// unit forms a resolvent after the other (12, 110, 215 and 850 by order) and takes
// 0.8, 1.1, 1.6 and 3.6 an iteration; in batched form the factorisation, then every
// column's iteration at its share of the products and the slowest column's launches.
// Fitted to 640 fits of 60 to 310 rows, 50 to 20000 columns in 1 to 30 groups,
// penalties 1e-4 to 100, tol 1e-2 to 1e-9, one or three stages, max_iter 20 to
// 100000, both ways: the worse form is taken by more than 10 % in 12 of them (5000
// columns of order 256 at tol = 1e-2: 16 ms batched, 67 here; by default 115 and 34).
// The logistic loss takes tens of iterations, so the resolvents decide (order 256:
// 2.08 ms against 2.62 batched at 2 each, 3.73 and 2.93 at 4; order 192: 3.98 and
// 4.75 at 16, growing by 0.23 and 0.17 each).
bool small_pays(const SmallFit& f, int stages, const double* delta, const double* kappa) {
  if (f.N > kSmallOrder || stages > kSmallStages) return false;
  const int run = small_run(stages, f.cols, f.same);
  const int64_t rounds = ceil_div(ceil_div(f.cols, run), 256) * (run > 1 ? 2 : 1);
  if (f.loss == KMP_LOGISTIC) return f.N <= 128 || rounds <= (f.N <= 192 ? 24 : 2);
  double sum = 0.0, most = 0.0;                   // iterations of a column
  const int step = f.L / 64 + 1;
  int count = 0;
  for (int l = 0; l < f.L; l += step, ++count) {
    double its = 0.0;
    for (int st = 0; st < stages; ++st) {
      const double zone = 1.0 / std::sqrt(delta[st]);
      double c = std::sqrt(1.0 + 1.0 / (2.0 * f.lambdas[l] * kappa[st]));
      if (f.loss == KMP_CHECK) c = std::min(std::max(c, 5.0 * zone), 14.0 * zone);
      its += std::min((double)f.max_iter, 0.27 * std::max(1.0, -std::log(f.tol)) * c);
    }
    sum += its;
    most = std::max(most, its);
  }
  sum *= (double)f.cols / count;
  const int nr = f.N / 64 - 1;
  const double form[] = {12.0, 110.0, 215.0, 850.0}, iter[] = {0.8, 1.1, 1.6, 3.6};
  const double here = rounds * stages * form[nr] + std::max(0.6 * most, sum / 256.0) * iter[nr];
  const double more = f.groups - 1;
  const double batched = (160.0 + 13.5 * f.N) * (1.0 + 0.01 * more) +
                         22.0 * (1.0 + 0.02 * more) * most + 0.039 * std::sqrt(f.N / 256.0) * sum;
  return here <= batched;
}

int small_path(hipStream_t s, const PathArrays& p, const double* K, const SmallStages& st, double tol,
               int max_iter, int restart, int count, int64_t active, bool begin, int L) {
  const int64_t cols = (int64_t)p.G * p.C;
  const int run = small_run(st.n, cols, p.C / L);
  const unsigned blocks = (unsigned)ceil_div(cols, run);
#define KMP_SMALL_CASE(NR, LS)                                                                   \
  if (p.N == 64 * NR && p.loss == LS)                                                            \
    hipLaunchKernelGGL((small_path_kernel<NR, LS>), dim3(blocks), dim3(DT), 0, s, p, K, st, tol, \
                       max_iter, restart, count, begin ? 1 : 0, L, run);
#define KMP_SMALL_CASES(LS) \
  KMP_SMALL_CASE(1, LS)     \
  KMP_SMALL_CASE(2, LS)     \
  KMP_SMALL_CASE(3, LS)     \
  KMP_SMALL_CASE(4, LS)
  kc_begin(KMP_KC_UPDATE, s);
  KMP_SMALL_CASES(0)
  KMP_SMALL_CASES(1)
  KMP_SMALL_CASES(2)
#undef KMP_SMALL_CASES
#undef KMP_SMALL_CASE
  KMP_LAUNCH_CHECK();
  // K read once and the sweeps for each resolvent formed (two at most in a run, one
  // a column and stage otherwise), and the columns' vectors; the products of the
  // iterations, whose number is not known here, are not counted
  const double n = (double)p.N;
  const double formed = run > 1 ? (double)std::min<int64_t>(active, 2 * (int64_t)blocks)
                                : (double)active * (begin ? st.n : 1);
  kc_end(KMP_KC_UPDATE, s, 8.0 * (formed * n * n + 6.0 * active * n), 2.0 * formed * n * n * n);
  hipLaunchKernelGGL(small_report_kernel, dim3(1), dim3(1024), 0, s, cols, p.flag, p.iters_total,
                     p.active_count);
  KMP_LAUNCH_CHECK();
  return 0;
}

}  // namespace kmp
