// Grouped products A B (row-major, packed) in two forms that add every
// element's products in one order (k in fours, increasing), so that they give
// the same bits:
//  - a wavefront per 16 x 16 block over the whole K, its operands straight from
//    memory into the matrix-core registers, SPD slices of 16 k in flight,
//    without LDS or a barrier, where there are few blocks;
//  - tiles of 32 x 64 or 64 x 64 through LDS.
// us per call (launch and wait included), against 32 x 64 tiles with checked
// loads, whose branches held back the loads behind them:
//   groups x M x N x K    blocks  wavefronts  32 x 64  64 x 64  before
//   6 x 2420 x 5 x 1759      912      54         93      100      84
//   3 x 1001 x 30 x 1501     378      47         71      102      86
//   1 x 2400 x 50 x 2400     600      71        103      147     131
//   1 x 3000 x 128 x 3000   1504     120        123      176     171
//   5 x 2400 x 50 x 2400    3000     184        137      157     167
//   2 x 1000^3              7938     158        108       99     120
//   10 x 3000 x 128 x 3000 15040     865        631      571     685
// The first form is bound by its loads through the second-level cache, the
// last by the matrix cores (40 TFLOP/s on 128 columns, 58 at 4096^3).
#include "kmp_common.h"
#include "kmp_kernels.h"

namespace kmp {

typedef double sdbl4 __attribute__((ext_vector_type(4)));

namespace {
constexpr int SPD = 4;             // slices in flight

// Transposes lane group against register: on entry register s of lane group
// lk (lanes 16 lk ..) holds k = 4 lk + s, on exit k = 4 s + lk. permlane32
// swaps the upper half of its first operand with the lower half of its
// second, permlane16 the odd rows of 16 lanes with the even ones.
__device__ __forceinline__ void swap_rows32(double& a, double& b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a);
  const unsigned long long y = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  a = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
  b = __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ void swap_rows16(double& a, double& b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a);
  const unsigned long long y = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  a = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
  b = __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ void transpose4(double (&v)[4]) {
  swap_rows32(v[0], v[2]);
  swap_rows32(v[1], v[3]);
  swap_rows16(v[0], v[1]);
  swap_rows16(v[2], v[3]);
}

// C = A B for batch b (blockIdx.z): A M x K, B K x N, C M x N, any M, N, K >=
// 1. Wavefront unit u = 4 blockIdx.x + w: column block u mod cblk, row block
// u / cblk. Rows and columns past the end repeat the last one and are not
// stored. PAIRS: K even and A 16-byte aligned.
template <bool PAIRS>
__global__ __launch_bounds__(256) void skinny_product_kernel(int M, int N, int K, int cblk,
                                                             const double* __restrict__ A,
                                                             const double* __restrict__ B,
                                                             double* __restrict__ C) {
  const int64_t b = blockIdx.z;
  A += b * M * K;
  B += b * K * N;
  C += b * M * N;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int u = 4 * (int)blockIdx.x + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i0 = 16 * (u / cblk), j0 = 16 * (u % cblk);
  if (i0 >= M) return;
  const double* pa = A + (int64_t)min(i0 + li, M - 1) * K + 4 * lk;
  const double* pb = B + (int64_t)lk * N + min(j0 + li, N - 1);
  const int nc = K / 16;
  double av[SPD][4], bv[SPD][4];
  const auto fetch = [&](int c, double (&a)[4], double (&v)[4]) {
    const int k = 16 * min(c, nc - 1);            // past the end: the last slice again, unused
    if constexpr (PAIRS) {
      const double2 p = *reinterpret_cast<const double2*>(pa + k);
      const double2 q = *reinterpret_cast<const double2*>(pa + k + 2);
      a[0] = p.x; a[1] = p.y; a[2] = q.x; a[3] = q.y;
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) a[s] = pa[k + s];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = pb[(int64_t)(k + 4 * s) * N];
  };
  sdbl4 acc = {0.0, 0.0, 0.0, 0.0};
  const auto products = [&](double (&a)[4], const double (&v)[4]) {
    transpose4(a);
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], v[s], acc, 0, 0, 0);
  };
  if (nc > 0) {
#pragma unroll
    for (int p = 0; p < SPD; ++p) fetch(p, av[p], bv[p]);
    int c = 0;
    for (; c + SPD <= nc; c += SPD) {
#pragma unroll
      for (int p = 0; p < SPD; ++p) {
        products(av[p], bv[p]);
        fetch(c + SPD + p, av[p], bv[p]);
      }
    }
#pragma unroll
    for (int p = 0; p < SPD - 1; ++p)
      if (c + p < nc) products(av[p], bv[p]);
  }
  if (K % 16 != 0) {                              // the last, partial slice: zeros past K
    const int k0 = 16 * nc;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = k0 + 4 * s + lk;
      const double v = k < K ? pb[(int64_t)(k0 + 4 * s) * N] : 0.0;
      const double a = k < K ? pa[k - 4 * lk] : 0.0;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, v, acc, 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = i0 + mfma_row(lane, r), j = j0 + li;
    if (i < M && j < N) C[(int64_t)i * N + j] = acc[r];
  }
}

// The same product in tiles of BM x 64 per workgroup, the wavefronts in a 2 x
// 2 arrangement over (BM/2) x 32 pieces, slices of 16 k through two LDS
// stages and two register sets: each slice's loads are issued two slices
// before they are stored to LDS, no branch or arithmetic stands between
// (addresses past the end are clamped, k past K zeroed at the LDS store; the
// count of slices is rounded up to even). lds_at spreads a store's lanes over
// the banks: a thread stages APT consecutive k of one row.
constexpr int TK = 16, TC = 64;
template <int BM, bool PAIRS>
__global__ __launch_bounds__(256) void tile_product_kernel(int M, int N, int K,
                                                           const double* __restrict__ A,
                                                           const double* __restrict__ B,
                                                           double* __restrict__ C) {
  constexpr int MB = BM / 32, APT = BM * TK / 256;
  __shared__ double As[2][TK][BM + 4];
  __shared__ double Bs[2][TK][TC + 4];
  const int64_t b = blockIdx.z;
  A += b * M * K;
  B += b * K * N;
  C += b * M * N;
  const int i0 = BM * blockIdx.x, j0 = TC * blockIdx.y;
  const int t = threadIdx.x, lane = t & 63, li = lane & 15, lk = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wi = (w & 1) * (BM / 2), wj = (w >> 1) * 32;
  const bool use0 = j0 + wj < N, use1 = j0 + wj + 16 < N;
  const auto lds_at = [](int k, int c) { return c ^ (((k / APT) & 3) << 2); };
  const int ar = t / (TK / APT), ak = (t % (TK / APT)) * APT;   // A: row, first k
  const int bj = t & 63, bk = t >> 6;                           // B: column, k = bk + 4 q
  const double* pa = A + (int64_t)min(i0 + ar, M - 1) * K;
  const double* pb = B + min(j0 + bj, N - 1);
  double a0[APT], b0[4], a1[APT], b1[4];
  const auto fetch = [&](int kt, double (&a)[APT], double (&v)[4]) {
    const int k = TK * kt + ak;
    if constexpr (PAIRS) {
#pragma unroll
      for (int q = 0; q < APT; q += 2) {
        const double2 p = *reinterpret_cast<const double2*>(pa + min(k + q, K - 2));
        a[q] = p.x;
        a[q + 1] = p.y;
      }
    } else {
#pragma unroll
      for (int q = 0; q < APT; ++q) a[q] = pa[min(k + q, K - 1)];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = pb[(int64_t)min(TK * kt + bk + 4 * q, K - 1) * N];
  };
  const auto store = [&](int kt, const double (&a)[APT], const double (&v)[4], int st) {
#pragma unroll
    for (int q = 0; q < APT; ++q)
      As[st][ak + q][lds_at(ak + q, ar)] = TK * kt + ak + q < K ? a[q] : 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) Bs[st][bk + 4 * q][bj] = TK * kt + bk + 4 * q < K ? v[q] : 0.0;
  };
  sdbl4 acc[MB][2];
#pragma unroll
  for (int x = 0; x < MB; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = sdbl4{0.0, 0.0, 0.0, 0.0};
  const auto products = [&](int st) {
    if (!use0) return;
#pragma unroll
    for (int kk = 0; kk < TK; kk += 4) {
      double av[MB];
#pragma unroll
      for (int x = 0; x < MB; ++x) av[x] = As[st][kk + lk][lds_at(kk + lk, wi + 16 * x + li)];
      const double v0 = Bs[st][kk + lk][wj + li], v1 = Bs[st][kk + lk][wj + 16 + li];
#pragma unroll
      for (int x = 0; x < MB; ++x) {
        acc[x][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x], v0, acc[x][0], 0, 0, 0);
        if (use1) acc[x][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x], v1, acc[x][1], 0, 0, 0);
      }
    }
  };
  const int nk = (K + TK - 1) / TK;
  fetch(0, a0, b0);
  store(0, a0, b0, 0);
  fetch(1, a0, b0);
  // slice 1's loads stay older than slice 2's (the waits count in issue order)
  __builtin_amdgcn_sched_barrier(0);
  fetch(2, a1, b1);
  __syncthreads();
  for (int kt = 0; kt < nk; kt += 2) {
    store(kt + 1, a0, b0, 1);
    fetch(kt + 3, a0, b0);
    products(0);
    __syncthreads();
    store(kt + 2, a1, b1, 0);
    fetch(kt + 4, a1, b1);
    products(1);
    __syncthreads();
  }
#pragma unroll
  for (int x = 0; x < MB; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + wi + 16 * x + mfma_row(lane, r), j = j0 + wj + 16 * y + li;
        if (i < M && j < N) C[(int64_t)i * N + j] = acc[x][y][r];
      }
}
}  // namespace

int grouped_product(hipStream_t s, int G, int M, int N, int K, const double* A, const double* B,
                    double* C) {
  const bool pairs = K % 2 == 0 && (reinterpret_cast<uintptr_t>(A) & 15) == 0;
  const int cblk = (int)ceil_div(N, 16);
  const int64_t units = ceil_div(M, 16) * cblk;
  // the lines between the forms: see the table above
  const int rows = units * G <= 2048 ? 16 : units * G <= 4096 ? 32 : 64;
  const dim3 grid = rows == 16 ? dim3((unsigned)ceil_div(units, 4), 1, (unsigned)G)
                               : dim3((unsigned)ceil_div(M, rows), (unsigned)ceil_div(N, TC), (unsigned)G);
#define KMP_PRODUCT_CASE(P)                                                                    \
  if (pairs == P) {                                                                            \
    if (rows == 16)                                                                            \
      hipLaunchKernelGGL(skinny_product_kernel<P>, grid, dim3(256), 0, s, M, N, K, cblk, A, B, C); \
    else if (rows == 32)                                                                       \
      hipLaunchKernelGGL((tile_product_kernel<32, P>), grid, dim3(256), 0, s, M, N, K, A, B, C); \
    else                                                                                       \
      hipLaunchKernelGGL((tile_product_kernel<64, P>), grid, dim3(256), 0, s, M, N, K, A, B, C); \
  }
  KMP_PRODUCT_CASE(true)
  KMP_PRODUCT_CASE(false)
#undef KMP_PRODUCT_CASE
  KMP_LAUNCH_CHECK();
  return 0;
}

}  // namespace kmp
