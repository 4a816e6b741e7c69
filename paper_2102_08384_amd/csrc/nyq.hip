// Midpoint P_l on half of the separations: the planes x = N/2 and y = N/2, where the mirror of an index
// is not the opposite separation and the part of g that the other cells drop counts (k_iy_half).
//   nyq_rows   inverse x transform of the rows y = N/2
//   nyq        A_{l nu} of these cells, from the complementary parts of g and of the weights
// A few times N^2 cells per field: latency-bound, a few microseconds each.
#include "kernels.h"

#include "coeffs.h"
#include "dev_core.h"

namespace pw {

template <int L, int K, bool ALLP, typename R> struct MidReweight;
#include "mix_gen.inc"

// Row (p, z) of nyy (half spectrum along x) to real space, N/8 lanes each
template <typename R, int N>
__global__ void __launch_bounds__(FxShape<N>::THREADS)
k_nyq_rows(const cplx<R> *__restrict__ in, R *__restrict__ out, int nrows, int rs, const cplx<R> *__restrict__ tw) {
  constexpr int T = FxShape<N>::T, ROWS = FxShape<N>::ROWS, LN = N + N / 8;
  __shared__ cplx<R> lds[ROWS * LN];
  const int rl = threadIdx.x / T, t = threadIdx.x % T;
  const int row = blockIdx.x * ROWS + rl;
  const bool live = row < nrows;
  cplx<R> *my = lds + rl * LN;
  auto at = [my](int i) -> cplx<R> & { return my[i + (i >> 3)]; };
  auto sync = []() { __syncthreads(); };
  const cplx<R> *src = in + (size_t)(live ? row : 0) * rs;
  cplx<R> v[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int k = t + s * T;
    cplx<R> h = src[k <= N / 2 ? k : N - k];
    if (k == 0 || k == N / 2) h.y = 0;
    v[s] = k <= N / 2 ? h : cconj(h);
  }
  fft_pencil<R, N, true>(v, t, tw, at, sync);
  if (live)
#pragma unroll
    for (int s = 0; s < 8; ++s) out[(size_t)row * N + t + s * T] = v[s].x;
}

template <typename R, int N>
static void nyq_rows_launch(hipStream_t s, const void *in, void *out, int nrows, int rs, const void *tw) {
  constexpr int ROWS = FxShape<N>::ROWS;
  hipLaunchKernelGGL((k_nyq_rows<R, N>), dim3((unsigned)((nrows + ROWS - 1) / ROWS)), dim3(FxShape<N>::THREADS), 0, s,
                     (const cplx<R> *)in, (R *)out, nrows, rs, (const cplx<R> *)tw);
}

void launch_nyq_rows(hipStream_t s, int prec, int N, const void *nyy, void *yx, int nfields, int rs, const void *tw) {
  const int nrows = nfields * (N / 2 + 1);
  if (nrows <= 0) return;
  if (prec == 0) {
    PW_DISPATCH_N(nyq_rows_launch, float, s, nyy, yx, nrows, rs, tw)
  } else {
    PW_DISPATCH_N(nyq_rows_launch, double, s, nyy, yx, nrows, rs, tw)
  }
}

// One thread per cell: blockIdx.y = 0 the cells (N/2, y, z), 1 the cells (x, N/2, z); 0 < z < N/2 (the
// values at the other z are never read)
template <typename R, int L, int K, bool ALLP>
__global__ void __launch_bounds__(128)
k_nyq(const R *__restrict__ nyx, const R *__restrict__ yx, R *__restrict__ ax, R *__restrict__ ay, int N, R scale, R Hu) {
  using MR = MidReweight<L, K, ALLP, R>;
  constexpr int NG = MR::NG, NA = MR::NA, F = kMixFields, NDP = ALLP ? K + 1 : K / 2 + 1;
  const int ncell = (N / 2 + 1) * N, i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ncell) return;
  const int z = i / N, j = i % N;
  const bool rows = blockIdx.y != 0;
  const R *src = (rows ? yx : nyx) + i;
  R *dst = (rows ? ay : ax) + i;
  if (z == 0 || z == N / 2 || (!rows && j == N / 2)) {  // (the rows y = N/2 hold the cell x = N/2 too)
    for (int a = 0; a < NA; ++a) dst[(size_t)a * ncell] = 0;
    return;
  }
  const int x = rows ? j : N / 2, y = rows ? N / 2 : j;
  const int sx = x < N / 2 ? x : x - N, sy = y < N / 2 ? y : y - N;
  const R dx = (R)sx * Hu, dy = (R)sy * Hu, dz = (R)z * Hu;
  const R d2 = dx * dx + dy * dy + dz * dz, ir = (R)1 / sqrt(d2), dstep = ALLP ? sqrt(d2) : d2;
  R Dp[NDP], yD[(K + 1) * (K + 1)], y2[(K + 1) * (K + 1)], A[NA];
  Dp[0] = 1;
#pragma unroll
  for (int a = 1; a < NDP; ++a) Dp[a] = Dp[a - 1] * dstep;
  MR::dirs(dx * ir, dy * ir, dz * ir, yD);
  MR::dirs(x == N / 2 ? dx * ir : -dx * ir, y == N / 2 ? dy * ir : -dy * ir, -dz * ir, y2);
  MR::parity_part(yD, y2, true);
#pragma unroll
  for (int a = 0; a < NA; ++a) A[a] = 0;
  for_each_const<MR::NCH>([&](auto ic) {
    constexpr int C = decltype(ic)::value;
    R g[F];
#pragma unroll
    for (int f = 0; f < F; ++f)
      if (C * F + f < NG) g[f] = src[(size_t)(C * F + f) * ncell] * scale;
    MR::template chunk<C>(g, yD, Dp, A);
  });
#pragma unroll
  for (int a = 0; a < NA; ++a) dst[(size_t)a * ncell] = A[a];
}

void launch_nyq(hipStream_t s, int prec, int N, int lmax, int order, int all_parity, const void *nyx, const void *yx,
                void *ax, void *ay, double scale, double Hu) {
  const dim3 grid((unsigned)(((N / 2 + 1) * N + 127) / 128), 2);
#define PW_NQ(L, K, AP)                                                                                          \
  if (lmax == L && order == K && (all_parity != 0) == AP) {                                                      \
    if (prec == 0)                                                                                               \
      hipLaunchKernelGGL((k_nyq<float, L, K, AP>), grid, dim3(128), 0, s, (const float *)nyx, (const float *)yx,  \
                         (float *)ax, (float *)ay, N, (float)scale, (float)Hu);                                  \
    else                                                                                                         \
      hipLaunchKernelGGL((k_nyq<double, L, K, AP>), grid, dim3(128), 0, s, (const double *)nyx, (const double *)yx, \
                         (double *)ax, (double *)ay, N, scale, Hu);                                              \
    return;                                                                                                      \
  }
#ifndef PW_NO_SHAPES  // (a build for host checks launches nothing)
  PW_MIX_SHAPES(PW_NQ)
#endif
#undef PW_NQ
}

}  // namespace pw
