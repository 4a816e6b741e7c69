// Midpoint P_l, real-space step (gfx950, wave64): one pass over the rows of the separation grid
//   inverse x transform of every g field, A_{l nu}(D) = sum Phi' y(D^) |D|^alpha g (Section 3.3,
//   Appendix D; all-parity: Section 3.2), forward x transform of every A field.
// Compiled once per mesh size (PW_MIX_N), so that the generated shapes build side by side.
#include "kernels.h"

#include "coeffs.h"
#include "dev_core.h"

#ifndef PW_MIX_N
#error "PW_MIX_N: the mesh size of this build"
#endif

namespace pw {

template <int L, int K, bool ALLP, typename R> struct MidReweight;
#include "mix_gen.inc"

// A workgroup holds one cell per thread: NT / N rows (z, y), N <= 256, or one row of 512.  The g
// fields go through in steps of kMixFields = 16: eight pairs per row, each the two real fields of
// one complex transform, one pair per N/8 lanes (Z = Ha + i Hb is built from the two half spectra
// in registers, the mirrored half by a cross-lane permute).  The transform's exchanges and its
// real results use the pair's own 2N reals of LDS; then every thread adds the step's terms to the
// A values of its cell, which stay in registers.  Two LDS buffers alternate, so a step has one
// barrier, and the next step's spectra are loaded while the current one is added up.  At the end
// the A rows go back through LDS and are transformed in pairs, pruned to kx < nkx.
//
// What bounds it: the read of the half spectra (n_g N/2 complex values per row) and about the same
// time of VALU work (the transforms and the generated terms).  As three passes (inverse x to real
// g fields, re-weighting, forward x of A) the g fields were written and read again.  Measured, FP32,
// ell_max 4, order 4, three passes -> this one: 256^3 3.76 -> 1.48 ms (all-parity, 130 g fields:
// 6.24 -> 2.65 ms), 512^3 26.5 -> 13.8 ms; on the half z >= 0 of the rows, with the two kernels of
// nyq.hip: 0.80 (1.38) and 7.1 ms.
//
// Exchange swizzle: element i of a pair's N complex values sits at i ^ ((i >> 5) & 7) ^
// (((i >> 6) & 3) << 3): the radix-8 stages' stores (strides 8 and 64 / N) and the reads (stride
// 1) of 32 lanes then fall on different banks without padding.
template <typename R, int N> struct MixShape {
  static constexpr int T = N / 8;
  static constexpr int NT = N <= 256 ? 256 : N;
  static constexpr int ROWS = NT / N;
  static constexpr int BUF = ROWS * kMixFields * N;  // reals of one LDS buffer
  // FP32 wavefronts per SIMD: four where 128 registers hold a step (parity-even; at 512 also
  // all-parity, whose 512-thread workgroups would otherwise sit one to a CU), else three
  template <int K, bool ALLP> static constexpr int waves() {
    return sizeof(R) == 8 ? 1 : (K <= 4 && (!ALLP || N == 512)) ? 4 : 3;
  }
};

template <typename R, int N, int L, int K, bool ALLP>
__global__ void __launch_bounds__((MixShape<R, N>::NT))
__attribute__((amdgpu_waves_per_eu((MixShape<R, N>::template waves<K, ALLP>()), 8)))
k_mix(const cplx<R> *__restrict__ in, cplx<R> *__restrict__ out, int rs, int nkx, int rso, R scale, R Hu,
      const cplx<R> *__restrict__ tw, const R *__restrict__ ax, const R *__restrict__ ay) {
  typedef MixShape<R, N> S;
  constexpr int T = S::T, F = kMixFields;
  using MR = MidReweight<L, K, ALLP, R>;
  constexpr int NG = MR::NG, NA = MR::NA, NCH = MR::NCH;
  __shared__ __align__(16) R lds[2 * S::BUF];
  const int tid = threadIdx.x;
  const int t = tid & (T - 1), grp = tid / T, j = grp & 7, rl = grp >> 3;  // pair j of row rl
  const int partner = (tid & 63 & ~(T - 1)) | ((T - t) & (T - 1));         // lane T - t of the group
  const size_t row = (size_t)blockIdx.x * S::ROWS + rl;                    // z * N + y
  constexpr bool HALF = N >= kMidHalfMesh;  // rows z = 0 .. N/2 (see k_iy_half), else every z
  constexpr int NZ = HALF ? N / 2 + 1 : N;
  const size_t fin = (size_t)NZ * N * rs, fout = (size_t)NZ * N * rso;
  FftTw<R, N> twr;
  twr.load(t, tw);
  int buf = 0;
  auto region = [&]() -> cplx<R> * {
    return reinterpret_cast<cplx<R> *>(lds + buf * S::BUF + (rl * F + 2 * j) * N);
  };
  auto sync = []() { wave_lds_sync(); };
  // half spectra of a pair: kx = t + s T (s < 4), and kx = N/2 on lane 0
  cplx<R> ha[4], hb[4];
  R na = 0, nb = 0;
  auto fetch = [&](int c) {
    const int f = c * F + 2 * j;
    const cplx<R> *pa = in + (size_t)f * fin + row * rs, *pb = pa + fin;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      ha[s] = f < NG ? load_nt<!keep_loads<R>(N)>(pa + t + s * T) : mk<R>(0, 0);
      hb[s] = f + 1 < NG ? load_nt<!keep_loads<R>(N)>(pb + t + s * T) : mk<R>(0, 0);
    }
    if (t == 0) {
      na = f < NG ? pa[N / 2].x : (R)0;
      nb = f + 1 < NG ? pb[N / 2].x : (R)0;
    }
  };
  fetch(0);
  // the thread's own cell: direction and powers of |D|
  const int x = tid & (N - 1), rc = tid / N;
  const size_t crow = (size_t)blockIdx.x * S::ROWS + rc;
  constexpr int NDP = ALLP ? K + 1 : K / 2 + 1;
  R yD[(K + 1) * (K + 1)], Dp[NDP], A[NA];
  {
    const int y = (int)(crow & (N - 1)), z = (int)(crow / N);
    const int sx = x < N / 2 ? x : x - N, sy = y < N / 2 ? y : y - N, sz = z < N / 2 ? z : z - N;
    const R dx = (R)sx * Hu, dy = (R)sy * Hu, dz = (R)sz * Hu;  // D / unit
    const R d2 = dx * dx + dy * dy + dz * dz;
    Dp[0] = 1;
    const R dstep = ALLP ? sqrt(d2) : d2;
#pragma unroll
    for (int i = 1; i < NDP; ++i) Dp[i] = Dp[i - 1] * dstep;
    // D = 0: |D|^alpha = 0 for every alpha > 0, so the direction is immaterial
    const R ir = d2 > (R)0 ? (R)1 / sqrt(d2) : (R)0;
    MR::dirs(dx * ir, dy * ir, d2 > (R)0 ? dz * ir : (R)1, yD);
    if (HALF && z > 0 && z < N / 2 && (x == N / 2 || y == N / 2)) {
      // the mirrored index stands for (sx, ..) where x = N/2: the part of y_J1 of J1's parity
      R y2[(K + 1) * (K + 1)];
      MR::dirs(x == N / 2 ? dx * ir : -dx * ir, y == N / 2 ? dy * ir : -dy * ir, -dz * ir, y2);
      MR::parity_part(yD, y2, false);
    }
  }
#pragma unroll
  for (int i = 0; i < NA; ++i) A[i] = 0;

  auto step = [&](auto ic) {
    constexpr int C = decltype(ic)::value;
    cplx<R> *reg = region();
    auto at = [reg](int i) -> cplx<R> & { return reg[i ^ ((i >> 5) & 7) ^ (((i >> 6) & 3) << 3)]; };
    if (C * F + 2 * j < NG) {
      cplx<R> v[8];
#pragma unroll
      for (int s = 0; s < 4; ++s) v[s] = mk<R>(ha[s].x - hb[s].y, ha[s].y + hb[s].x);
      // Z(N - k) = conj(Ha(k)) + i conj(Hb(k)): v[s], s >= 4, wants k = T (8 - s) - t, held by lane
      // T - t at 7 - s, or (t = 0) by lane 0 itself at 8 - s, k = N/2 at s = 4
      cplx<R> m[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) m[s] = mk<R>(ha[s].x + hb[s].y, hb[s].x - ha[s].y);
#pragma unroll
      for (int s = 4; s < 8; ++s) {
        const cplx<R> own = s == 4 ? mk<R>(na, nb) : m[(8 - s) & 3];
        const cplx<R> pub = t == 0 ? own : m[7 - s];
        v[s] = lane_fetch<R>(partner, pub);
      }
      if (t == 0) v[0] = mk<R>(ha[0].x, hb[0].x);  // kx = 0 keeps real parts
      fft_pencil<R, N, true>(v, t, twr, at, sync);
      R *ga = reinterpret_cast<R *>(reg);
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        ga[t + s * T] = v[s].x * scale;
        ga[N + t + s * T] = v[s].y * scale;
      }
    }
    if constexpr (C + 1 < NCH) fetch(C + 1);
    __syncthreads();
    R g[F];
    const R *col = lds + buf * S::BUF + rc * F * N + x;
#pragma unroll
    for (int i = 0; i < F; ++i)
      if (C * F + i < NG) g[i] = col[i * N];
    MR::template chunk<C>(g, yD, Dp, A);
    // pins the sums here (sunk to their use after the last step, they keep every step's g values
    // live), and makes the next step form its products y(D^) |D|^alpha anew
#pragma unroll
    for (int i = 0; i < NA; ++i) asm volatile("" : "+v"(A[i]));
#pragma unroll
    for (int i = 1; i < NDP; ++i) asm volatile("" : "+v"(Dp[i]));
    buf ^= 1;  // (the next step's transforms write the other buffer; its barrier covers these reads)
  };
  for_each_const<NCH>(step);
  if (HALF) {  // the other parts on the planes x = N/2 and y = N/2
    const int y = (int)(crow & (N - 1)), z = (int)(crow / N);
    if (z > 0 && z < N / 2 && (x == N / 2 || y == N / 2)) {
      const R *src = y == N / 2 ? ay + (size_t)z * N + x : ax + (size_t)z * N + y;
#pragma unroll
      for (int i = 0; i < NA; ++i) A[i] += src[(size_t)i * NZ * N];
    }
  }

  // forward transforms of the A rows, kMixFields rows at a time
  for_each_const<(NA + F - 1) / F>([&](auto ic) {
    constexpr int C = decltype(ic)::value;
    R *col = lds + buf * S::BUF + rc * F * N + x;
#pragma unroll
    for (int i = 0; i < F; ++i)
      if (C * F + i < NA) col[i * N] = A[C * F + i < NA ? C * F + i : 0];
    __syncthreads();
    const int f = C * F + 2 * j;
    if (f < NA) {
      const bool two = f + 1 < NA;
      cplx<R> *reg = region();
      auto at = [reg](int i) -> cplx<R> & { return reg[i ^ ((i >> 5) & 7) ^ (((i >> 6) & 3) << 3)]; };
      const R *ga = reinterpret_cast<const R *>(reg);
      cplx<R> v[8];
      // (the inputs carry the factor 1/2 of the two-real-field separation)
#pragma unroll
      for (int s = 0; s < 8; ++s)
        v[s] = mk<R>((R)0.5 * ga[t + s * T], two ? (R)0.5 * ga[N + t + s * T] : (R)0);
      sync();
      fft_pencil<R, N, false>(v, t, twr, at, sync);
      cplx<R> *oa = out + (size_t)f * fout + row * rso, *ob = oa + fout;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (T * s >= rso) break;
        const cplx<R> pub = t == 0 ? v[(8 - s) & 7] : v[7 - s];
        const cplx<R> b = lane_fetch<R>(partner, pub), a = v[s];
        const int kx = t + T * s;
        if (kx < rso) {
          const bool keep = kx < nkx;
          oa[kx] = keep ? mk<R>(a.x + b.x, a.y - b.y) : mk<R>(0, 0);
          if (two) ob[kx] = keep ? mk<R>(a.y + b.y, b.x - a.x) : mk<R>(0, 0);
        }
      }
      for (int kx = N / 2 + t; kx < rso; kx += T) {  // kx = N/2 pairs with itself; padding beyond
        const bool keep = kx == N / 2 && kx < nkx;
        oa[kx] = keep ? mk<R>(v[4].x + v[4].x, (R)0) : mk<R>(0, 0);
        if (two) ob[kx] = keep ? mk<R>(v[4].y + v[4].y, (R)0) : mk<R>(0, 0);
      }
    }
    buf ^= 1;
  });
}

template <typename R, int N, int L, int K, bool ALLP>
static void mix_launch(hipStream_t s, const void *in, void *out, int rs, int nkx, int rso, double scale, double Hu,
                       const void *tw, const void *ax, const void *ay) {
  typedef MixShape<R, N> S;
  hipLaunchKernelGGL((k_mix<R, N, L, K, ALLP>), dim3((unsigned)((N >= kMidHalfMesh ? N / 2 + 1 : N) * N / S::ROWS)), dim3(S::NT), 0, s,
                     (const cplx<R> *)in, (cplx<R> *)out, rs, nkx, rso, (R)scale, (R)Hu, (const cplx<R> *)tw,
                     (const R *)ax, (const R *)ay);
}

#define PW_CAT2(a, b) a##b
#define PW_CAT(a, b) PW_CAT2(a, b)
void PW_CAT(launch_mix_, PW_MIX_N)(hipStream_t s, int prec, int lmax, int order, int all_parity, const void *in,
                                   void *out, int rs, int nkx, int rso, double scale, double Hu, const void *tw,
                                   const void *ax, const void *ay) {
#define PW_MX(L, K, AP)                                                                          \
  if (lmax == L && order == K && (all_parity != 0) == AP) {                                      \
    if (prec == 0) mix_launch<float, PW_MIX_N, L, K, AP>(s, in, out, rs, nkx, rso, scale, Hu, tw, ax, ay);  \
    else mix_launch<double, PW_MIX_N, L, K, AP>(s, in, out, rs, nkx, rso, scale, Hu, tw, ax, ay);           \
    return;                                                                                      \
  }
#ifndef PW_NO_SHAPES  // (a build for host checks launches nothing)
  PW_MIX_SHAPES(PW_MX)
#endif
#undef PW_MX
}

}  // namespace pw
