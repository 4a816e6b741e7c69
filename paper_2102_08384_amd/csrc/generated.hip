// HIP kernels whose couplings are straight-line code generated at build time from the FP64
// host coefficient generator (contract_gen.inc):
//   contract_bis_reg  bisector P_l contraction with every field value of a mode in VGPRs
//                     (Section 5.2 boxed estimator, real-harmonic basis)
//   targets           bisector xi_l per-mode targets T_{l nu} (Section 6 boxed estimator)
#include "kernels.h"

#include "dev_core.h"

namespace pw {

__constant__ ShConst c_sh_gen;

void upload_sh_const_generated(const ShConst &c) {
  (void)hipMemcpyToSymbol(HIP_SYMBOL(c_sh_gen), &c, sizeof(ShConst));
}

template <int L, int B, typename R> struct BisContract {
  static constexpr bool kGenerated = false;
};
#include "contract_gen.inc"

// Register-resident variant: the coupling for (LMAX, BMAX) is straight-line code generated at
// build time (BisContract<L, B, R>::run), so all field values of a mode stay in VGPRs.  With
// ORD the terms of each order beta go to accumulators of their own (run_orders): rows
// beta * (LMAX/2 + 1) + l/2, then the mode count and the |k| sum.

template <typename R, int LMAX, int BMAX, bool ORD>
__global__ void __launch_bounds__(256)
k_contract_bis_reg(const cplx<R> *__restrict__ spec, int64_t nmodes, int64_t mstride,
                   const uint32_t *__restrict__ modecoord,
                   int N, const int *__restrict__ bin_of_s2, int64_t n_s2, int nbins, double kf,
                   const R *__restrict__ winv, double *__restrict__ acc, const Batch ba) {
  using CT = BisContract<LMAX, BMAX, R>;
  if (ba.n) {  // catalog blockIdx.z of a batch
    const BatchSlot &bs = ba.s[blockIdx.z];
    spec = (const cplx<R> *)bs.A;
    acc = bs.acc;
  }
  constexpr int NF = CT::NF;
  constexpr int NSH = (LMAX + 1) * (LMAX + 1);
  constexpr int NE = ORD ? CT::NO * (LMAX / 2 + 1) : LMAX / 2 + 1;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double *bacc = reinterpret_cast<double *>(smem_raw);
  const int nacc = (NE + 2) * nbins;
  for (int i = threadIdx.x; i < nacc; i += blockDim.x) bacc[i] = 0.0;
  __syncthreads();
  const int half = N / 2;
  for (int64_t mode = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; mode < nmodes;
       mode += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t mc = modecoord[mode];
    const int kx = mc & 0x7ff, ky = (mc >> 11) & 0x7ff, kz = (mc >> 22) & 0x3ff;
    const int sx = (kx == half) ? -half : kx;
    const int sy = (ky < half) ? ky : ky - N;
    const int sz = (kz < half) ? kz : kz - N;
    const int64_t s2 = (int64_t)sx * sx + (int64_t)sy * sy + (int64_t)sz * sz;
    const int b = (s2 < n_s2) ? bin_of_s2[s2] : -1;
    if (b < 0) continue;
    cplx<R> a[NF];
#pragma unroll
    for (int p = 0; p < NF; ++p) a[p] = load_nt<true>(spec + (size_t)p * mstride + mode);
    const bool pair = (kx != 0 && kx != half);
    R wdir[NSH];
#pragma unroll
    for (int i = 0; i < NSH; ++i) wdir[i] = 0;
    {
      R ux = 0, uy = 0, uz = 1;
      const R ir = s2 > 0 ? (R)1 / sqrt((R)s2) : (R)0;
      if (s2 > 0) { ux = (R)sx * ir; uy = (R)sy * ir; uz = (R)sz * ir; }
      real_sh_even<R, LMAX>(c_sh_gen, ux, uy, uz, wdir);
      if (pair) {
        const int my = (ky == half) ? sy : -sy;
        const int mz = (kz == half) ? sz : -sz;
        R wm[NSH];
#pragma unroll
        for (int i = 0; i < NSH; ++i) wm[i] = 0;
        real_sh_even<R, LMAX>(c_sh_gen, (R)(-sx) * ir, (R)my * ir, (R)mz * ir, wm);
#pragma unroll
        for (int i = 0; i < NSH; ++i) wdir[i] += wm[i];
      }
    }
    R E[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) E[i] = 0;
    if constexpr (ORD) CT::run_orders(a, wdir, E);
    else CT::run(a, wdir, E);
    if (winv) {
      const R iw = winv[kx] * winv[ky] * winv[kz];
      const R iw2 = iw * iw;
#pragma unroll
      for (int i = 0; i < NE; ++i) E[i] *= iw2;
    }
    const double mult = pair ? 2.0 : 1.0;
#pragma unroll
    for (int i = 0; i < NE; ++i) atomicAdd(&bacc[i * nbins + b], (double)E[i]);
    atomicAdd(&bacc[NE * nbins + b], mult);
    atomicAdd(&bacc[(NE + 1) * nbins + b], mult * kf * sqrt((double)s2));
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nacc; i += blockDim.x)
    if (bacc[i] != 0.0) atomicAdd(&acc[i], bacc[i]);
}

template <typename R, int L, int B>
static bool contract_reg_launch(hipStream_t s, const void *spec, int64_t nmodes, int64_t mstride,
                                const uint32_t *modecoord,
                                int N, const int *bin_of_s2, int64_t n_s2, int nbins, double kf,
                                const void *winv, double *acc, int orders, const Batch *batch, ColTune tune) {
  if constexpr (BisContract<L, B, R>::kGenerated) {
    Batch ba;
    ba.n = 0;
    if (batch) ba = *batch;
    const int nb = ba.n ? ba.n : 1;
    int64_t want = (nmodes + 255) / 256;
    // workgroups per catalog: the tuned count, else up to 4096 over all catalogs
    const int64_t cap = tune.blocks > 0 ? tune.blocks : (4096 / nb > 0 ? 4096 / nb : 1);
    unsigned blocks = (unsigned)(want < cap ? (want > 0 ? want : 1) : cap);
    const int ne = (orders ? B + 1 : 1) * (L / 2 + 1);
    size_t sh = (size_t)(ne + 2) * nbins * sizeof(double);
    if (orders)
      hipLaunchKernelGGL((k_contract_bis_reg<R, L, B, true>), dim3(blocks, 1, nb), dim3(256), sh, s,
                         (const cplx<R> *)spec, nmodes, mstride, modecoord, N, bin_of_s2, n_s2, nbins, kf,
                         (const R *)winv, acc, ba);
    else
      hipLaunchKernelGGL((k_contract_bis_reg<R, L, B, false>), dim3(blocks, 1, nb), dim3(256), sh, s,
                         (const cplx<R> *)spec, nmodes, mstride, modecoord, N, bin_of_s2, n_s2, nbins, kf,
                         (const R *)winv, acc, ba);
    return true;
  } else {
    return false;
  }
}

template <typename R>
static bool contract_reg_dispatch(int lmax, int bmax, hipStream_t s, const void *spec, int64_t nmodes,
                                  int64_t mstride,
                                  const uint32_t *modecoord, int N, const int *bin_of_s2, int64_t n_s2,
                                  int nbins, double kf, const void *winv, double *acc, int orders,
                                  const Batch *batch, ColTune tune) {
#define PW_CR(L, B)                                                                                \
  if (lmax == L && bmax == B)                                                                      \
    return contract_reg_launch<R, L, B>(s, spec, nmodes, mstride, modecoord, N, bin_of_s2, n_s2, nbins, kf, winv, \
                                        acc, orders, batch, tune);
  PW_CR(0, 0) PW_CR(0, 1) PW_CR(0, 2) PW_CR(2, 0) PW_CR(2, 1) PW_CR(2, 2)
  PW_CR(4, 0) PW_CR(4, 1) PW_CR(4, 2) PW_CR(6, 0) PW_CR(6, 1) PW_CR(6, 2)
#undef PW_CR
  return false;
}

bool launch_contract_bis_generated(hipStream_t s, int prec, int lmax, int bmax, const void *spec, int64_t nmodes,
                                   int64_t mstride, const uint32_t *modecoord, int N, const int *bin_of_s2, int64_t n_s2,
                                   int nbins, double kf, const void *winv, double *acc, int orders,
                                   const Batch *batch, ColTune tune) {
  return prec == 0 ? contract_reg_dispatch<float>(lmax, bmax, s, spec, nmodes, mstride, modecoord, N, bin_of_s2,
                                                  n_s2, nbins, kf, winv, acc, orders, batch, tune)
                   : contract_reg_dispatch<double>(lmax, bmax, s, spec, nmodes, mstride, modecoord, N, bin_of_s2,
                                                   n_s2, nbins, kf, winv, acc, orders, batch, tune);
}

// ------------------------------------------------------------------------------ generated
bool bis_contract_generated(int lmax, int bmax) {
#define PW_BG(L, B) if (lmax == L && bmax == B) return BisContract<L, B, float>::kGenerated;
  PW_BG(0, 0) PW_BG(0, 1) PW_BG(0, 2) PW_BG(2, 0) PW_BG(2, 1) PW_BG(2, 2)
  PW_BG(4, 0) PW_BG(4, 1) PW_BG(4, 2) PW_BG(6, 0) PW_BG(6, 1) PW_BG(6, 2)
#undef PW_BG
  return false;
}

int mid_reweight_nfields(int lmax, int order, int all_parity) {
  for (const MidShape &m : kMidShapes)
    if (m.L == lmax && m.K == order && m.all == (all_parity ? 1 : 0)) return m.NG;
  return -1;
}

bool mid_reweight_generated(int lmax, int order, int all_parity) {
  return mid_reweight_nfields(lmax, order, all_parity) >= 0;
}

// Bisector xi targets over the full spectra: one thread per mode.
template <typename R, int LMAX, int BMAX>
__global__ void __launch_bounds__(256)
k_targets(const cplx<R> *__restrict__ spec, int64_t nmodes, int64_t mstride, int N, int rs,
          const R *__restrict__ winv, R *__restrict__ T) {
  using CT = BisContract<LMAX, BMAX, R>;
  constexpr int NF = CT::NF;
  constexpr int NT = (LMAX + 1) * (LMAX + 2) / 2;   // targets of even l <= LMAX
  constexpr int NSH = (LMAX + 1) * (LMAX + 1);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nmodes;
       i += (int64_t)gridDim.x * blockDim.x) {
    cplx<R> a[NF];
#pragma unroll
    for (int p = 0; p < NF; ++p) a[p] = load_nt<true>(spec + (size_t)p * mstride + i);
    R full[NSH];
    CT::targets(a, full);
    R iw2 = (R)1;
    if (winv) {
      // mode i = (g N + kz) C + c of pencil q = g C + c
      constexpr int C = 128 / (int)sizeof(cplx<R>);
      const int64_t row = i / C, g = row / N, q = g * C + (i - row * C);
      const int kz = (int)(row - g * N), ky = (int)(q / rs), kx = (int)(q - (int64_t)ky * rs);
      const R iw = winv[kx] * winv[ky] * winv[kz];
      iw2 = iw * iw;
    }
#pragma unroll
    for (int l = 0, o = 0; l <= LMAX; l += 2)
#pragma unroll
      for (int nu = -l; nu <= l; ++nu, ++o) T[(size_t)o * nmodes + i] = full[l * l + l + nu] * iw2;
    (void)NT;
  }
}

template <typename R, int L, int B>
static bool targets_launch(hipStream_t s, const void *spec, int64_t nmodes, int64_t mstride, int N, int rs,
                           const void *winv, void *T) {
  if constexpr (BisContract<L, B, R>::kGenerated) {
    int64_t want = (nmodes + 255) / 256;
    unsigned blocks = (unsigned)(want < 65536 ? (want > 0 ? want : 1) : 65536);
    hipLaunchKernelGGL((k_targets<R, L, B>), dim3(blocks), dim3(256), 0, s, (const cplx<R> *)spec, nmodes, mstride, N,
                       rs, (const R *)winv, (R *)T);
    return true;
  } else {
    return false;
  }
}

void launch_targets(hipStream_t s, int prec, int N, int lmax, int bmax, const void *spec, int64_t nmodes,
                    int64_t mstride, int rs, const void *winv, void *T) {
#define PW_TG(L, B)                                                                               \
  if (lmax == L && bmax == B) {                                                                   \
    if (prec == 0) targets_launch<float, L, B>(s, spec, nmodes, mstride, N, rs, winv, T);         \
    else targets_launch<double, L, B>(s, spec, nmodes, mstride, N, rs, winv, T);                  \
    return;                                                                                       \
  }
  PW_TG(0, 0) PW_TG(0, 1) PW_TG(0, 2) PW_TG(2, 0) PW_TG(2, 1) PW_TG(2, 2)
  PW_TG(4, 0) PW_TG(4, 1) PW_TG(4, 2) PW_TG(6, 0) PW_TG(6, 1) PW_TG(6, 2)
#undef PW_TG
}

// ------------------------------------------------------------------------------ mix (by mesh size)
#define PW_MIX_ARGS                                                                                \
  hipStream_t s, int prec, int lmax, int order, int all_parity, const void *in, void *out, int rs, \
      int nkx, int rso, double scale, double Hu, const void *tw, const void *ax, const void *ay
void launch_mix_16(PW_MIX_ARGS);
void launch_mix_32(PW_MIX_ARGS);
void launch_mix_64(PW_MIX_ARGS);
void launch_mix_128(PW_MIX_ARGS);
void launch_mix_256(PW_MIX_ARGS);
void launch_mix_512(PW_MIX_ARGS);

void launch_mix(hipStream_t s, int prec, int N, int lmax, int order, int all_parity, const void *in, void *out, int rs,
                int nkx, int rso, double scale, double Hu, const void *tw, const void *ax, const void *ay) {
  switch (N) {
#define PW_MIX_CASE(n) \
  case n: launch_mix_##n(s, prec, lmax, order, all_parity, in, out, rs, nkx, rso, scale, Hu, tw, ax, ay); break;
    PW_MIX_CASE(16) PW_MIX_CASE(32) PW_MIX_CASE(64) PW_MIX_CASE(128) PW_MIX_CASE(256) PW_MIX_CASE(512)
#undef PW_MIX_CASE
    default: break;
  }
}

}  // namespace pw
