// Gram + fold gather: RBF kernel blocks written straight into per-fold
// matrices. The inner products x_r . x_c are an fp64 MFMA contraction over
// the feature dimension; the epilogue forms the squared distance by the norm
// expansion |x_r|^2 + |x_c|^2 - 2 x_r.x_c (clamped at 0), the norms added up
// from the same loads, and applies exp(-dist^2 / (2 sigma^2)) for every
// requested bandwidth, so one distance tile feeds all bandwidths. Diagonal
// entries (same point) are exactly 1, padding entries (negative index)
// exactly 0.
#include "kmp_common.h"
#include "kmp_kernels.h"

namespace kmp {

typedef double dbl4 __attribute__((ext_vector_type(4)));

// out[0] = number of non-finite entries of X (n x d, ldx), out[1] = of y;
// one workgroup (16 wavefronts: rows over waves, columns over lanes), fixed
// order, no atomics.
__global__ __launch_bounds__(1024) void count_nonfinite_kernel(const double* __restrict__ X,
                                                                int64_t n, int64_t d, int64_t ldx,
                                                                const double* __restrict__ y,
                                                                int* __restrict__ out) {
  __shared__ double red[2][16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double cx = 0.0, cy = 0.0;
  for (int64_t i = w; i < n; i += 16) {
    const double* xr = X + i * ldx;
    for (int64_t k = lane; k < d; k += 64) cx += isfinite(xr[k]) ? 0.0 : 1.0;
  }
  for (int64_t i = threadIdx.x; i < n; i += 1024) cy += isfinite(y[i]) ? 0.0 : 1.0;
  cx = wave_sum(cx);
  cy = wave_sum(cy);
  if (lane == 0) {
    red[0][w] = cx;
    red[1][w] = cy;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double c = 0.0;
    for (int q = 0; q < 16; ++q) c += red[threadIdx.x][q];
    out[threadIdx.x] = (int)c;
  }
}

int count_nonfinite(hipStream_t s, const double* X, int64_t n, int64_t d, int64_t ldx,
                    const double* y, int* out) {
  hipLaunchKernelGGL(count_nonfinite_kernel, dim3(1), dim3(1024), 0, s, X, n, d, ldx, y, out);
  KMP_LAUNCH_CHECK();
  return 0;
}

// exp(x) for x <= 0: x = k ln 2 + r with |r| <= ln(2)/2 (ln 2 in two parts, the
// first with 25 trailing zero bits, so k times it is exact), exp(r) by its
// Taylor polynomial to degree 13 (remainder below 5e-18), scaled by 2^k. The
// kernel below takes one per entry and bandwidth: with the library's exp they
// took as long as the products at d = 100.
__device__ __forceinline__ double exp_neg(double x) {
  const double k = rint(fmax(x, -800.0) * 1.4426950408889634074);
  double r = fma(k, -0x1.62e42fep-1, x);
  r = fma(k, -0x1.f473de6af278fp-30, r);
  double p = 1.0 / 6227020800.0;
  p = fma(p, r, 1.0 / 479001600.0);
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  const double e = ldexp(fma(r, fma(p, r, 1.0), 1.0), (int)k);
  return x < -746.0 ? 0.0 : e;                    // (-inf too; NaN stays)
}

constexpr int GT = 64, GK = 16, GPAD = 4, MAXS = 8;

// LDS column of element (k, c) of a staged slice (a thread stages four
// consecutive k of one row): the lanes of one store land in distinct banks.
__device__ __forceinline__ int gcol(int k, int c) { return c ^ (((k >> 2) & 3) << 2); }

// Features gk .. gk + 3 of one point; those past d repeat others (zeroed when
// they are staged).
template <bool PAIRS>
__device__ __forceinline__ void gram_fetch(const double* __restrict__ x, int64_t gk, int64_t d,
                                           double (&r)[4]) {
  if constexpr (PAIRS) {
#pragma unroll
    for (int u = 0; u < 4; u += 2) {               // d even: a pair is in or out
      const double2 a = *reinterpret_cast<const double2*>(x + min(gk + u, d - 2));
      r[u] = a.x;
      r[u + 1] = a.y;
    }
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u) r[u] = x[min(gk + u, d - 1)];
  }
}

// One 64 x 64 tile per workgroup, wave w the 32 x 32 quadrant (32 (w&1),
// 32 (w>>1)); X in slices of 16 features through two LDS stages, the next
// slice's loads in flight during the products of the current one (no branch
// around a load and no arithmetic on it before it is staged: rows and features
// past the end read valid ones and are zeroed there). PAIRS: d and ldx even and X
// 16-byte aligned, so a row's features load as pairs. SYM: rows and columns are one
// list, so the matrix is symmetric: the tiles on and below the diagonal are computed and stored
// on both sides, through LDS in whole row pieces (straight from the
// accumulators an odd leading dimension took 900 us where it now takes 590).
// A tile's phases (index and row loads, slices, exp, stores) are short chains
// that only other workgroups hide: four of them share a compute unit (at most
// 128 registers); 128 x 128 and 128 x 64 tiles, which leave one to two, were
// slower by a fifth to a half, six and eight (fewer registers) too. Three
// bandwidths of one matrix at d = 100: order 8191 980 -> 590 us, order 8192
// 500 us (1.6 GB written: 240 us at the rate of a plain fill); one, 8192 at
// d = 16: 136 us.
template <bool PAIRS, bool SYM>
__global__ __launch_bounds__(256, 4) void rbf_blocks_kernel(
    const double* __restrict__ X, int64_t d, int64_t ldx, const int32_t* __restrict__ idx_r, int64_t sr,
    int64_t m, const int32_t* __restrict__ idx_c, int64_t sc, int64_t p, Small8 f2, int S,
    double* __restrict__ out, int64_t sout_s, int64_t sout_q, int64_t ld) {
  if (SYM && blockIdx.y > blockIdx.x) return;
  __shared__ double sh[4 * GK * (GT + GPAD)];      // two stages of A and B, then the entries
  double (*As)[GK][GT + GPAD] = reinterpret_cast<double (*)[GK][GT + GPAD]>(sh);
  double (*Bs)[GK][GT + GPAD] = reinterpret_cast<double (*)[GK][GT + GPAD]>(sh + 2 * GK * (GT + GPAD));
  __shared__ double nr[GT], nc[GT];
  __shared__ int32_t ri[GT], ci[GT];
  const int q = blockIdx.z;
  const int64_t i0 = (int64_t)blockIdx.x * GT, j0 = (int64_t)blockIdx.y * GT;
  const int t = threadIdx.x;
  const int lane = t & 63, w = t >> 6;
  const int wi = (w & 1) * 32, wj = (w >> 1) * 32;
  const int li = lane & 15, lk = lane >> 4;
  // thread t stages features 4 (t%4) .. +3 of row t/4 of both sides
  const int row = t >> 2, kb = (t & 3) * 4;
  const int32_t xr = i0 + row < m ? idx_r[q * sr + i0 + row] : -1;
  const int32_t xc = j0 + row < p ? idx_c[q * sc + j0 + row] : -1;
  if ((t & 3) == 0) {
    ri[row] = xr;
    ci[row] = xc;
  }
  const double* pr = X + (int64_t)(xr >= 0 ? xr : 0) * ldx;
  const double* pc = X + (int64_t)(xc >= 0 ? xc : 0) * ldx;
  double ra[4], rb[4], sr2 = 0.0, sc2 = 0.0;
  const auto fetch = [&](int64_t k0) {
    gram_fetch<PAIRS>(pr, k0 + kb, d, ra);
    gram_fetch<PAIRS>(pc, k0 + kb, d, rb);
  };
  const auto store = [&](int st, int64_t k0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool in = k0 + kb + u < d;
      const double a = in && xr >= 0 ? ra[u] : 0.0, b = in && xc >= 0 ? rb[u] : 0.0;
      As[st][kb + u][gcol(kb + u, row)] = a;
      Bs[st][kb + u][gcol(kb + u, row)] = b;
      sr2 = fma(a, a, sr2);
      sc2 = fma(b, b, sc2);
    }
  };
  dbl4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
  fetch(0);
  store(0, 0);
  __syncthreads();
  const int64_t nk = (d + GK - 1) / GK;
  for (int64_t kt = 0; kt < nk; ++kt) {
    const int cur = (int)(kt & 1);
    const bool more = kt + 1 < nk;
    if (more) fetch((kt + 1) * GK);
#pragma unroll
    for (int kk = 0; kk < GK; kk += 4) {
      const double a0 = As[cur][kk + lk][gcol(kk, wi + li)];
      const double a1 = As[cur][kk + lk][gcol(kk, wi + 16 + li)];
      const double b0 = Bs[cur][kk + lk][gcol(kk, wj + li)];
      const double b1 = Bs[cur][kk + lk][gcol(kk, wj + 16 + li)];
      acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
    }
    if (more) {
      store(cur ^ 1, (kt + 1) * GK);
      __syncthreads();
    }
  }
  // squared norms: the four threads of a row
  sr2 += __shfl_xor(sr2, 1, kWave);
  sc2 += __shfl_xor(sc2, 1, kWave);
  sr2 += __shfl_xor(sr2, 2, kWave);
  sc2 += __shfl_xor(sc2, 2, kWave);
  if ((t & 3) == 0) {
    nr[row] = sr2;
    nc[row] = sc2;
  }
  __syncthreads();
  out += (int64_t)q * sout_q;
  constexpr int TS = GT + 1;
  static_assert(GT * TS <= 4 * GK * (GT + GPAD), "the tile's entries fit the stages");
  for (int s = 0; s < S; ++s) {
    const double f = f2.v[s];
    double* o = out + (int64_t)s * sout_s;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2; ++bj) {
        const int lj = wj + bj * 16 + li;
        const int32_t cj = ci[lj];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int lr = wi + bi * 16 + 4 * r + lk;
          const int32_t rj = ri[lr];
          double v = nr[lr] + nc[lj] - 2.0 * acc[bi][bj][r];
          v = v > 0.0 ? v : 0.0;
          v = (rj < 0 || cj < 0) ? 0.0 : (rj == cj ? 1.0 : exp_neg(-v * f));
          if constexpr (SYM) {
            sh[lr * TS + lj] = v;
          } else {
            const int64_t gi = i0 + lr, gj = j0 + lj;
            if (gi < m && gj < p) o[gi * ld + gj] = v;
          }
        }
      }
    if constexpr (SYM) {
      // both sides in whole row pieces; on the diagonal tile each side stores
      // its own half, so that the two entries of a pair are one value
      __syncthreads();
#pragma unroll 4
      for (int u = 0; u < 16; ++u) {
        const int e = 16 * w + u;
        const int64_t gi = i0 + e, gj = j0 + lane;
        if (gi < m && gj < p && gi >= gj) o[gi * ld + gj] = sh[e * TS + lane];
      }
#pragma unroll 4
      for (int u = 0; u < 16; ++u) {
        const int e = 16 * w + u;
        const int64_t gi = i0 + lane, gj = j0 + e;
        if (gi < m && gi > gj) o[gj * ld + gi] = sh[lane * TS + e];
      }
      __syncthreads();
    }
  }
}

int rbf_blocks(hipStream_t s, const double* X, int64_t d, int64_t ldx, const int32_t* idx_r,
               int64_t sr, int64_t m, const int32_t* idx_c, int64_t sc, int64_t p, int nb,
               const double* inv2s2, int S, double* out, int64_t sout_s, int64_t sout_q,
               int64_t ld) {
  if (m <= 0 || p <= 0 || nb <= 0) return 0;
  if (S < 1 || S > MAXS) {
    set_error("rbf_blocks: at most 8 bandwidths per launch");
    return KMP_EINVAL;
  }
  Small8 f2{};
  for (int i = 0; i < S; ++i) f2.v[i] = inv2s2[i];
  const dim3 grid((unsigned)ceil_div(m, GT), (unsigned)ceil_div(p, GT), (unsigned)nb);
  const bool pairs = d % 2 == 0 && ldx % 2 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0;
  const bool sym = idx_r == idx_c && m == p && sr == sc;
#define KMP_GRAM_CASE(P, Y)                                                                       \
  if (pairs == P && sym == Y)                                                                     \
    hipLaunchKernelGGL((rbf_blocks_kernel<P, Y>), grid, dim3(256), 0, s, X, d, ldx, idx_r, sr, m, \
                       idx_c, sc, p, f2, S, out, sout_s, sout_q, ld);
  KMP_GRAM_CASE(true, true)
  KMP_GRAM_CASE(true, false)
  KMP_GRAM_CASE(false, true)
  KMP_GRAM_CASE(false, false)
#undef KMP_GRAM_CASE
  KMP_LAUNCH_CHECK();
  return 0;
}

}  // namespace kmp
