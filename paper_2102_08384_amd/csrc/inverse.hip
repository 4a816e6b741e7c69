// HIP kernels of the inverse-transform paths (gfx950, wave64).
//
//   iz             bisector xi_l: inverse FFT along z of the real targets, two to a transform;
//                  output pruned to the retained planes z >= 0
//   fziz           midpoint g fields: forward FFT along z, the product conj(D) Q / W^2
//                  (Section 3.2) and the inverse FFT along z in one pass over each pencil
//   fziz_half      the same for xi_l, whose sums need only the part of g that is even (or odd) in D:
//                  two fields to an inverse transform, planes z >= 0
//   iy_half        midpoint P_l: inverse y pass of the part of g even (or odd) in D, planes z >= 0
//   ix             xi_l: complex-to-real inverse FFT along x of field pairs, weighted by
//                  |D|^alpha y_J^mu(D^) times the per-field multipole coefficient and binned into
//                  r-shells in FP64 (Section 4.3 midpoint estimator, Section 6 bisector estimator)
//   contract_mid   midpoint P_l contraction sum_nu y_l^nu(k^) Re[G + A] (Section 3.3 boxed
//                  estimator in the real-harmonic basis) with FP64 shell sums
//   finalize_xi    xi_l = (4 pi / I) sum / (N_a H^3)
#include "kernels.h"

#include <algorithm>
#include <type_traits>

#include "dev_core.h"

namespace pw {

__constant__ ShConst c_sh_inv;

void upload_sh_const_inverse(const ShConst &c) {
  (void)hipMemcpyToSymbol(HIP_SYMBOL(c_sh_inv), &c, sizeof(ShConst));
}

// ------------------------------------------------------------------------------ half sets
// xi_l sums w_f(D) g_f(D) over whole shells of separations, D and -D alike, and every weight
// |D|^alpha y_J^mu(D^) has the parity of J: only the part of g of that parity counts, and the half
// z >= 0 of the separations, counted twice off the self-mirrored planes z = 0 and z = N/2, holds it.
// The even part's spectrum is Re G, the odd part's i Im G, so one complex transform along z carries
// two fields: with Z = IFT[s_a + i s_b] of real s_a, s_b (s = Re G or Im G, each scaled by 1/2),
//   h_a(z) = Z(z) + conj Z(-z),  h_b(z) = -i (Z(z) - conj Z(-z)),
// and an odd field's h is multiplied by i.

// On entry lane t holds v[s] = Z(t + s T); `at` is this pencil's LDS row, free on entry and on exit
// (the caller's next exchange comes after the closing barrier).  fn(z, h_a, h_b) is called for
// the planes z = t + s T <= zmax of this lane.
template <typename R, int T, int N, typename At, typename Fn>
__device__ __forceinline__ void split_half(const cplx<R> v[8], int t, int zmax, At at, Fn fn) {
#pragma unroll
  for (int s = 4; s < 8; ++s) {  // mirrors of 1 .. N/2
    const int z = t + s * T;
    if (N - z <= zmax) at(z) = v[s];
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    const int z = t + s * T;
    if (z <= zmax && z <= N / 2) {
      const cplx<R> w = z == 0 ? v[0] : at(N - z);
      fn(z, mk<R>(v[s].x + w.x, v[s].y - w.y), mk<R>(v[s].y + w.y, w.x - v[s].x));
    }
  }
  __syncthreads();
}

// ------------------------------------------------------------------------------ iz
// Bisector targets are real, T(-k) = T(k): Z = IFT[(T_a + i T_b) / 2], bound by the read of the targets
// and the exchanges' barriers.  Two targets to a transform and half the planes, through this pass and
// the inverse y and x passes: a bisector xi_l of 512^3 went from 25.8 to 25.0 ms.
template <typename R, int N>
__global__ void __launch_bounds__((ColShape<R, N>::THREADS))
k_iz(const R *__restrict__ in, cplx<R> *__restrict__ out, int nfields, int64_t npen, int nz,
     const cplx<R> *__restrict__ tw) {
  constexpr int T = ColShape<R, N>::T, C = ColShape<R, N>::C;
  __shared__ cplx<R> lds[N * (C + 1)];
  const int c = threadIdx.x % C, t = threadIdx.x / C;
  const int64_t q = (int64_t)blockIdx.x * C + c;
  auto at = [c](int i) -> cplx<R> & { return lds[i * (C + 1) + c]; };
  auto sync = []() { __syncthreads(); };
  FftTw<R, N> twr;
  twr.load(t, tw);
  wait_vmem();
  // the pair's values of this lane, the next pair's loaded while the current one is transformed
  // (npen is a multiple of C: every pencil of the group exists)
  R xa[8], xb[8];
  const R *mine = in + (size_t)blockIdx.x * N * C + t * C + c;
  const size_t fstride = (size_t)npen * N;
  auto fetch = [&](int p) {
    const R *src = mine + (size_t)p * fstride;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      xa[s] = load_real_nt<!keep_loads<R>(N)>(src + s * T * C);
      xb[s] = p + 1 < nfields ? load_real_nt<!keep_loads<R>(N)>(src + fstride + s * T * C) : (R)0;
    }
  };
  fetch(0);
  for (int p = 0; p < nfields; p += 2) {
    cplx<R> v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = mk<R>((R)0.5 * xa[s], (R)0.5 * xb[s]);
    if (p + 2 < nfields) fetch(p + 2);
    fft_pencil<R, N, true>(v, t, twr, at, sync);
    cplx<R> *oa = out + (size_t)p * nz * npen + q, *ob = oa + (size_t)nz * npen;
    const bool two = p + 1 < nfields;
    split_half<R, T, N>(v, t, nz - 1, at, [&](int z, cplx<R> ha, cplx<R> hb) {
      oa[(size_t)z * npen] = ha;
      if (two) ob[(size_t)z * npen] = hb;
    });
  }
}

template <typename R, int N>
static void iz_launch(hipStream_t s, const void *in, void *out, int nfields, int64_t npen, int nz, const void *tw) {
  constexpr int C = ColShape<R, N>::C;
  hipLaunchKernelGGL((k_iz<R, N>), dim3((unsigned)((npen + C - 1) / C)), dim3(ColShape<R, N>::THREADS), 0, s,
                     (const R *)in, (cplx<R> *)out, nfields, npen, nz, (const cplx<R> *)tw);
}

void launch_iz(hipStream_t s, int prec, int N, const void *in, void *out, int nfields, int64_t npen, int nz,
               const void *tw) {
  if (nfields <= 0 || npen <= 0) return;
  if (prec == 0) {
    PW_DISPATCH_N(iz_launch, float, s, in, out, nfields, npen, nz, tw)
  } else {
    PW_DISPATCH_N(iz_launch, double, s, in, out, nfields, npen, nz, tw)
  }
}

// ------------------------------------------------------------------------------ fziz
// Midpoint g fields (Section 3.2): the forward z pass, the product conj(D) Q / W^2 and the
// inverse z pass all act along one pencil (kx, ky), so one kernel does the three and the full
// spectra never go through HBM.  Input: the y-pass output of full sets, [field][z][pencil q]
// (q = ky * rs + kx, every pencil N long; pencils kx >= nkx are zero padding).  Field 0 is
// Q_{0,0,0}; D = d_scale * its transform.  Fields p < n_inplace stay in k-space: the contraction reads
// the real part of their product on the modes of the k-sphere only, so that is what is stored, as
// reals, in the sphere's [group][kz slot][pencil] layout (sph; field stride sph.mstride; the C pencils
// of a block are one of its groups, or lie outside it and skip these fields).  Against full complex
// products, FP32, order 4, bins to |n| = 127: 256^3 1.86 -> 1.76 ms, 512^3 17.6 -> 16.3 ms (there 81% of
// the blocks lie outside the sphere).  The other fields go back to z and leave the retained
// planes at out[p - n_inplace][zrank[z]][q].  A block owns C adjacent pencils and one group of fields
// [p0, p1); it transforms field 0 first (every group does) and prefetches the next field's
// loads across each transform.  conj(D) / W^2 waits in LDS (each lane its own 8 values), which
// keeps the N = 512 FP32 form within 128 VGPRs.  Loads and the z-side stores are raw buffer
// accesses whose per-lane offsets (empty planes, padding pencils and planes outside the
// r-bins masked out) are fixed for the whole kernel, so the per-field work is the transforms.
template <typename R, int N>
__global__ void __launch_bounds__((ColShape<R, N>::THREADS))
k_fziz(const cplx<R> *__restrict__ in, R *__restrict__ prod, const SphereSet sph, cplx<R> *__restrict__ out,
       int nfields, int n_inplace, int fpb, int64_t npen, int rs, R d_scale, const R *__restrict__ winv,
       const int *__restrict__ zrank, int nz, const cplx<R> *__restrict__ tw, const int *__restrict__ planemask) {
  constexpr int T = ColShape<R, N>::T, C = ColShape<R, N>::C, NT = ColShape<R, N>::THREADS;
  constexpr int64_t E = sizeof(cplx<R>);
  __shared__ cplx<R> lds[N * (C + 1)];
  __shared__ cplx<R> dls[8 * NT];
  const int c = threadIdx.x % C, t = threadIdx.x / C;
  const int64_t q0 = (int64_t)blockIdx.x * C;
  const int64_t q = q0 + c;
  const int p0 = blockIdx.y * fpb;
  const int p1 = min(nfields, p0 + fpb);
  if (p0 >= p1) return;  // uniform
  // the block's group of the k-sphere: first slot m0 and kz slots S (0: outside it)
  int64_t m0 = 0;
  int S = 0;
  if (n_inplace > 0) {
    const int ky = (int)(q0 / rs), kx = (int)(q0 - (int64_t)ky * rs);
    if (kx < sph.ycnt[ky]) {
      const int64_t g = (sph.yoff[ky] + kx) / C;
      m0 = sph.goff[g];
      S = sph.gsize[g];
    }
  }
  const int skip = S ? 0 : n_inplace;  // fields below it leave nothing in this block
  if (p1 <= skip) return;  // uniform
  FftTw<R, N> twr;
  twr.load(t, tw);
  const bool has = q < npen;
  // byte offsets: input plane z = t + s T of pencil q sits at lo[s] + s * sT in its field, and
  // the output row of a retained plane z at zo[s] in its output field
  const uint32_t sT = (uint32_t)(T * npen * E);
  const uint32_t lane_in = (uint32_t)((t * npen + q) * E);
  // wave-uniform bit s of wload / wstore: some lane of the wave loads / stores plane t + s T (a
  // wave spans 4 adjacent planes, so empty planes and planes outside the r-bins skip whole
  // instructions, not only lanes)
  uint32_t lo[8], zo[8], wload = 0, wstore = 0;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int z = t + s * T;
    lo[s] = (has && (!planemask || planemask[z])) ? lane_in : kOob;
    const int zr = zrank ? zrank[z] : -1;
    zo[s] = (has && zr >= 0) ? (uint32_t)((zr * npen + q) * E) : kOob;
    if (__builtin_amdgcn_ballot_w64(lo[s] != kOob)) wload |= 1u << s;
    if (__builtin_amdgcn_ballot_w64(zo[s] != kOob)) wstore |= 1u << s;
  }
  const uint32_t in_bytes = (uint32_t)(N * npen * E);
  const uint32_t out_bytes = (uint32_t)(nz * npen * E);
  R iwxy = (R)1;
  if (winv && has) {
    const int qky = (int)(q / rs), qkx = (int)(q - (int64_t)qky * rs);
    iwxy = winv[qkx] * winv[qky];
  }
  wait_vmem();
  auto load = [&](int p, cplx<R> *v) {
    const __amdgpu_buffer_rsrc_t r = buf_rsrc(in + (size_t)p * N * npen, in_bytes);
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = (wload >> s & 1) ? buf_load<R, load_policy<R>(N)>(r, lo[s], (uint32_t)s * sT) : mk<R>(0, 0);
  };
  auto at = [c](int i) -> cplx<R> & { return lds[i * (C + 1) + c]; };
  auto sync = []() { __syncthreads(); };
  cplx<R> nxt[8];
  const int pf = max(max(p0, 1), skip);  // first field after D's own
  // field p's product (in v, kz = t + s T): stored in k-space, or transformed back to z
  auto finish = [&](int p, cplx<R> *v) {
    if (p < n_inplace) {
      // kz = j for slots j <= h, kz = N - S + j above (slot rows C apart; when S == N, h covers all)
      R *dst = prod + (size_t)p * sph.mstride + m0;
      const __amdgpu_buffer_rsrc_t rl = buf_rsrc(dst, 0x7fffffffu), rh = buf_rsrc(dst - (size_t)(N - S) * C, 0x7fffffffu);
      const uint32_t lane = (uint32_t)((t * C + c) * sizeof(R));
      const int h = S == N ? N : (S - 1) / 2;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int kz = t + s * T;
        const uint32_t so = (uint32_t)(s * T * C * sizeof(R));
        buf_store_real<R>(v[s].x, rl, kz <= h ? lane : kOob, so);
        buf_store_real<R>(v[s].x, rh, (kz > h && kz >= N - h) ? lane : kOob, so);
      }
    } else {
      fft_pencil<R, N, true>(v, t, twr, at, sync);
      const __amdgpu_buffer_rsrc_t r = buf_rsrc(out + (size_t)(p - n_inplace) * nz * npen, out_bytes);
#pragma unroll
      for (int s = 0; s < 8; ++s)
        if (wstore >> s & 1) buf_store<R, store_policy(N)>(v[s], r, zo[s], 0);
    }
  };
  // conj(D) / W^2 on every mode, D = d_scale Q_000~; field 0's own product is then
  // d_scale |Q_000~|^2 / W^2
  {
    cplx<R> d[8], v[8];
    load(0, d);
    if (pf < p1) load(pf, nxt);
    fft_pencil<R, N, false>(d, t, twr, at, sync);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const R iw = iwxy * (winv ? winv[t + s * T] : (R)1);
      const R f = d_scale * iw * iw;
      v[s] = mk<R>(f * (d[s].x * d[s].x + d[s].y * d[s].y), (R)0);
      dls[s * NT + threadIdx.x] = mk<R>(d[s].x * f, -d[s].y * f);
    }
    if (p0 == 0 && skip == 0) finish(0, v);
  }
  for (int p = pf; p < p1; ++p) {
    cplx<R> v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = nxt[s];
    if (p + 1 < p1) load(p + 1, nxt);
    fft_pencil<R, N, false>(v, t, twr, at, sync);
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = cmul(dls[s * NT + threadIdx.x], v[s]);
    finish(p, v);
  }
}

template <typename R, int N>
static void fziz_launch(hipStream_t s, const void *in, void *prod, const SphereSet &sph, void *out, int nfields, int n_inplace,
                        int64_t npen, int rs, double d_scale, const void *winv, const int *zrank, int nz,
                        const void *tw, const int *planemask, ColTune tune) {
  constexpr int C = ColShape<R, N>::C;
  const unsigned ng = (unsigned)((npen + C - 1) / C);
  int fpb = tune.fpb;
  if (fpb <= 0) {
    // field groups fill the chip on small meshes; each group transforms D again, so keep >= 8
    // fields per group
    int G = field_groups(nfields, (int)std::min<int64_t>(ng, 1 << 20));
    G = std::max(1, std::min(G, nfields / 8));
    fpb = (nfields + G - 1) / G;
  }
  fpb = std::min(fpb, nfields);
  dim3 grid(ng, (nfields + fpb - 1) / fpb);
  hipLaunchKernelGGL((k_fziz<R, N>), grid, dim3(ColShape<R, N>::THREADS), 0, s, (const cplx<R> *)in,
                     (R *)prod, sph, (cplx<R> *)out, nfields, n_inplace, fpb, npen, rs, (R)d_scale,
                     (const R *)winv, zrank, nz, (const cplx<R> *)tw, planemask);
}

void launch_fziz(hipStream_t s, int prec, int N, const void *in, void *prod, const SphereSet &sph, void *out,
                 int nfields, int n_inplace, int64_t npen, int rs, double d_scale, const void *winv, const int *zrank, int nz, const void *tw,
                 const int *planemask, ColTune tune) {
  if (nfields <= 0 || npen <= 0) return;
  if (prec == 0) {
    PW_DISPATCH_N(fziz_launch, float, s, in, prod, sph, out, nfields, n_inplace, npen, rs, d_scale, winv, zrank, nz,
                  tw, planemask, tune)
  } else {
    PW_DISPATCH_N(fziz_launch, double, s, in, prod, sph, out, nfields, n_inplace, npen, rs, d_scale, winv, zrank, nz,
                  tw, planemask, tune)
  }
}

// ------------------------------------------------------------------------------ fziz_half
// k_fziz for xi_l (see half sets): fields p, p + 1 are transformed forward and multiplied by
// conj(D) / W^2 one after the other, the real (imaginary: odd_of[p] != 0) parts kept, and go back
// together.  Three transforms for two fields in place of four, and half the planes stored.  The pass
// is bound by its VALU work: at 512^3 (FP32, 88 fields, 36 planes) 13.6 -> 11.5 ms, with the inverse y
// and x passes after it 1.56 -> 0.82 and 1.21 -> 0.73 ms.
template <typename R, int N>
__global__ void __launch_bounds__((ColShape<R, N>::THREADS))
k_fziz_half(const cplx<R> *__restrict__ in, cplx<R> *__restrict__ out, int nfields, int fpb, int64_t npen, int rs,
            R d_scale, const R *__restrict__ winv, const int *__restrict__ odd_of, int nz,
            const cplx<R> *__restrict__ tw, const int *__restrict__ planemask) {
  constexpr int T = ColShape<R, N>::T, C = ColShape<R, N>::C, NT = ColShape<R, N>::THREADS;
  constexpr int64_t E = sizeof(cplx<R>);
  __shared__ cplx<R> lds[N * (C + 1)];
  __shared__ cplx<R> dls[8 * NT];  // each lane its own 8 values of conj(D) / W^2
  const int c = threadIdx.x % C, t = threadIdx.x / C;
  const int64_t q = (int64_t)blockIdx.x * C + c;
  const int p0 = blockIdx.y * fpb;
  const int p1 = min(nfields, p0 + fpb);
  if (p0 >= p1) return;  // uniform
  FftTw<R, N> twr;
  twr.load(t, tw);
  const bool has = q < npen;
  // input planes as in k_fziz: byte offsets fixed for the kernel, empty planes out of range
  const uint32_t sT = (uint32_t)(T * npen * E);
  const uint32_t lane_in = (uint32_t)((t * npen + q) * E);
  uint32_t lo[8], wload = 0;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    lo[s] = (has && (!planemask || planemask[t + s * T])) ? lane_in : kOob;
    if (__builtin_amdgcn_ballot_w64(lo[s] != kOob)) wload |= 1u << s;
  }
  const uint32_t in_bytes = (uint32_t)(N * npen * E), out_bytes = (uint32_t)(nz * npen * E);
  R iwxy = (R)1;
  if (winv && has) {
    const int qky = (int)(q / rs), qkx = (int)(q - (int64_t)qky * rs);
    iwxy = winv[qkx] * winv[qky];
  }
  wait_vmem();
  auto load = [&](int p, cplx<R> *v) {
    const __amdgpu_buffer_rsrc_t r = buf_rsrc(in + (size_t)p * N * npen, in_bytes);
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = (wload >> s & 1) ? buf_load<R, load_policy<R>(N)>(r, lo[s], (uint32_t)s * sT) : mk<R>(0, 0);
  };
  auto at = [c](int i) -> cplx<R> & { return lds[i * (C + 1) + c]; };
  auto sync = []() { __syncthreads(); };
  cplx<R> nxt[8];
  {
    cplx<R> d[8];
    load(0, d);
    load(p0, nxt);
    fft_pencil<R, N, false>(d, t, twr, at, sync);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const R iw = iwxy * (winv ? winv[t + s * T] : (R)1);
      const R f = (R)0.5 * d_scale * iw * iw;
      dls[s * NT + threadIdx.x] = mk<R>(d[s].x * f, -d[s].y * f);
    }
  }
  for (int p = p0; p < p1; p += 2) {
    const bool two = p + 1 < p1;
    const int odd_a = odd_of ? odd_of[p] : 0, odd_b = (odd_of && two) ? odd_of[p + 1] : 0;
    cplx<R> v[8];
    R sa[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = nxt[s];
    if (two) load(p + 1, nxt);
    fft_pencil<R, N, false>(v, t, twr, at, sync);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const cplx<R> g = cmul(dls[s * NT + threadIdx.x], v[s]);
      sa[s] = odd_a ? g.y : g.x;
    }
    if (two) {
#pragma unroll
      for (int s = 0; s < 8; ++s) v[s] = nxt[s];
      if (p + 2 < p1) load(p + 2, nxt);
      fft_pencil<R, N, false>(v, t, twr, at, sync);
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const cplx<R> g = cmul(dls[s * NT + threadIdx.x], v[s]);
        v[s] = mk<R>(sa[s], odd_b ? g.y : g.x);
      }
    } else {
#pragma unroll
      for (int s = 0; s < 8; ++s) v[s] = mk<R>(sa[s], (R)0);
    }
    fft_pencil<R, N, true>(v, t, twr, at, sync);
    const __amdgpu_buffer_rsrc_t ra = buf_rsrc(out + (size_t)p * nz * npen, out_bytes);
    const __amdgpu_buffer_rsrc_t rb = buf_rsrc(out + (size_t)(p + 1) * nz * npen, out_bytes);
    split_half<R, T, N>(v, t, nz - 1, at, [&](int z, cplx<R> ha, cplx<R> hb) {
      const uint32_t zo = has ? (uint32_t)((z * npen + q) * E) : kOob;
      buf_store<R, store_policy(N)>(odd_a ? mk<R>(-ha.y, ha.x) : ha, ra, zo, 0);
      if (two) buf_store<R, store_policy(N)>(odd_b ? mk<R>(-hb.y, hb.x) : hb, rb, zo, 0);
    });
  }
}

template <typename R, int N>
static void fziz_half_launch(hipStream_t s, const void *in, void *out, int nfields, int64_t npen, int rs,
                             double d_scale, const void *winv, const int *odd_of, int nz, const void *tw,
                             const int *planemask, ColTune tune) {
  constexpr int C = ColShape<R, N>::C;
  const unsigned ng = (unsigned)((npen + C - 1) / C);
  int fpb = tune.fpb;
  if (fpb <= 0) {
    // (as in fziz_launch)
    int G = field_groups(nfields, (int)std::min<int64_t>(ng, 1 << 20));
    G = std::max(1, std::min(G, nfields / 8));
    fpb = (nfields + G - 1) / G;
  }
  fpb = (std::min(fpb, nfields) + 1) / 2 * 2;  // whole pairs
  dim3 grid(ng, (nfields + fpb - 1) / fpb);
  hipLaunchKernelGGL((k_fziz_half<R, N>), grid, dim3(ColShape<R, N>::THREADS), 0, s, (const cplx<R> *)in,
                     (cplx<R> *)out, nfields, fpb, npen, rs, (R)d_scale, (const R *)winv, odd_of, nz,
                     (const cplx<R> *)tw, planemask);
}

void launch_fziz_half(hipStream_t s, int prec, int N, const void *in, void *out, int nfields, int64_t npen, int rs,
                      double d_scale, const void *winv, const int *odd_of, int nz, const void *tw,
                      const int *planemask, ColTune tune) {
  if (nfields <= 0 || npen <= 0) return;
  if (prec == 0) {
    PW_DISPATCH_N(fziz_half_launch, float, s, in, out, nfields, npen, rs, d_scale, winv, odd_of, nz, tw, planemask, tune)
  } else {
    PW_DISPATCH_N(fziz_half_launch, double, s, in, out, nfields, npen, rs, d_scale, winv, odd_of, nz, tw, planemask, tune)
  }
}

// ------------------------------------------------------------------------------ iy_half
// Midpoint P_l: only Re FT[A] counts, the transform of the part of A even under D -> -D (indices mod
// N), and a weight |D|^alpha y_J1 has the parity of alpha: A's even part takes the even or odd part
// of each g (odd_of), and the planes z <= N/2 hold it.  The part is formed before the transform,
//   h'(kx, ky, z) = (h(z) +- conj h(-z)) / 2,
// so this pass reads both planes, transforms once and writes half of what it reads.  The planes
// z = 0 and N/2, their own mirrors, stay whole (their odd part drops out with Im FT).
// On the planes x = N/2 and y = N/2 the index mirror is not -D (the signed index of N/2 is -N/2), so
// there the complementary part counts too, with the weights' complementary part.  Its values come
// out on the way: summed over ky with (-1)^ky for y = N/2 (nyy[p][z][kx], still to be transformed
// along x), and over kx with (-1)^kx, then transformed along y, for x = N/2 (nyx[p][z][y]).
// Bound by HBM; 73 fields, FP32, against the pass over whole planes: 256^3 2.07 -> 1.56 ms, 512^3 15.4 ->
// 11.6 ms, and the passes after it halve.
template <typename R, int N>
__global__ void __launch_bounds__((ColShape<R, N>::THREADS))
k_iy_half(const cplx<R> *__restrict__ in, cplx<R> *__restrict__ out, R *__restrict__ nyx, cplx<R> *__restrict__ nyy,
          int nfields, int fpb, int nkx, int rs, const int *__restrict__ odd_of, const cplx<R> *__restrict__ tw) {
  constexpr int T = ColShape<R, N>::T, C = ColShape<R, N>::C, NT = ColShape<R, N>::THREADS;
  constexpr int NW = (NT + 63) / 64, NZ = N / 2 + 1;
  constexpr uint32_t E = sizeof(cplx<R>);
  constexpr int LB = N * (C + 1);  // one exchange buffer; two alternate (one barrier per exchange)
  __shared__ cplx<R> lds[2 * LB];
  __shared__ cplx<R> red[2][NW][C];
  const int c = threadIdx.x % C, t = threadIdx.x / C, wv = threadIdx.x / 64;
  const int z = blockIdx.x, zm = (N - z) & (N - 1);
  const bool self = z == zm;  // uniform
  const int p0 = blockIdx.y * fpb, p1 = min(nfields, p0 + fpb);
  const int ncb = (nkx + C - 1) / C, nitems = (p1 - p0) * ncb;
  if (nitems <= 0) return;
  FftTw<R, N> twr;
  twr.load(t, tw);
  wait_vmem();
  const uint32_t lane = (uint32_t)(t * rs + c) * E, sT = (uint32_t)(T * rs) * E;
  const size_t plane = (size_t)N * rs;
  const uint32_t bytes = (uint32_t)(plane * E);
  auto load = [&](int p, int cb, cplx<R> *a, cplx<R> *b) {
    const uint32_t lo = cb * C + c < nkx ? lane : kOob;
    const __amdgpu_buffer_rsrc_t ra = buf_rsrc(in + ((size_t)p * N + z) * plane + cb * C, bytes);
#pragma unroll
    for (int s = 0; s < 8; ++s) a[s] = buf_load<R, load_policy<R>(N)>(ra, lo, (uint32_t)s * sT);
    if (!self) {
      const __amdgpu_buffer_rsrc_t rb = buf_rsrc(in + ((size_t)p * N + zm) * plane + cb * C, bytes);
#pragma unroll
      for (int s = 0; s < 8; ++s) b[s] = buf_load<R, load_policy<R>(N)>(rb, lo, (uint32_t)s * sT);
    }
  };
  int lb = 0;
  auto at = [c, &lb](int i) -> cplx<R> & { return lds[lb * LB + i * (C + 1) + c]; };
  auto sync = []() { __syncthreads(); };
  auto flip = [&lb]() { lb ^= 1; };
  cplx<R> S[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) S[s] = mk<R>(0, 0);
  int p = p0, cb = 0;
  cplx<R> na[8], nb[8];
  load(p, cb, na, nb);
  for (int it = 0; it < nitems; ++it) {
    const int pc = p, cbc = cb, kx = cb * C + c;
    const bool last = cb + 1 == ncb;
    cplx<R> v[8];
    if (self) {
#pragma unroll
      for (int s = 0; s < 8; ++s) v[s] = na[s];
    } else {
      // v: the part of the field's parity; u: the other one
      const R sg = (odd_of && odd_of[pc]) ? (R)-0.5 : (R)0.5;
      const R wx = kx < nkx ? ((kx == 0 || kx == N / 2) ? (R)1 : (R)2) * ((c & 1) ? (R)-1 : (R)1) : (R)0;
      cplx<R> r = mk<R>(0, 0);
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const cplx<R> a = na[s], b = nb[s];
        v[s] = mk<R>((R)0.5 * a.x + sg * b.x, (R)0.5 * a.y - sg * b.y);
        const cplx<R> u = mk<R>((R)0.5 * a.x - sg * b.x, (R)0.5 * a.y + sg * b.y);
        S[s].x += wx * u.x;
        S[s].y += wx * u.y;
        r = cadd(r, u);
      }
      if (t & 1) r = mk<R>(-r.x, -r.y);  // (T is even: the sign of row t + s T is that of t)
#pragma unroll
      for (int off = C; off < (NT < 64 ? NT : 64); off <<= 1) {
        r.x += __shfl_xor(r.x, off);
        r.y += __shfl_xor(r.y, off);
      }
      if ((threadIdx.x & 63) < C) red[it & 1][wv][c] = r;
    }
    if (++cb == ncb) {
      cb = 0;
      ++p;
    }
    if (it + 1 < nitems) load(p, cb, na, nb);
    fft_pencil_db<R, N, true>(v, t, twr, at, sync, flip);
    const __amdgpu_buffer_rsrc_t w = buf_rsrc(out + ((size_t)pc * NZ + z) * plane + cbc * C, bytes);
#pragma unroll
    for (int s = 0; s < 8; ++s) buf_store<R, store_policy(N)>(v[s], w, lane, (uint32_t)s * sT);
    if (!self) {
      // (the transform's barriers lie between every wave's row of red and this read, and the next
      // item's between this read and that row's next write: two rows alternate)
      if (t == 0) {
        cplx<R> r = red[it & 1][0][c];
        for (int i = 1; i < NW; ++i) r = cadd(r, red[it & 1][i][c]);
        nyy[((size_t)pc * NZ + z) * rs + kx] = r;
      }
      if (last) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
#pragma unroll
          for (int off = 1; off < C; off <<= 1) {
            S[s].x += __shfl_xor(S[s].x, off);
            S[s].y += __shfl_xor(S[s].y, off);
          }
          v[s] = S[s];
          S[s] = mk<R>(0, 0);
        }
        fft_pencil_db<R, N, true>(v, t, twr, at, sync, flip);
        if (c == 0) {
          R *dst = nyx + ((size_t)pc * NZ + z) * N;
#pragma unroll
          for (int s = 0; s < 8; ++s) dst[t + s * T] = v[s].x;
        }
      }
    }
  }
}

template <typename R, int N>
static void iy_half_launch(hipStream_t s, const void *in, void *out, void *nyx, void *nyy, int nfields, int nkx, int rs,
                           const int *odd_of, const void *tw, ColTune tune) {
  int fpb = tune.fpb;
  if (fpb <= 0) {
    const int G = field_groups(nfields, N / 2 + 1);
    fpb = (nfields + G - 1) / G;
  }
  fpb = std::min(fpb, nfields);
  hipLaunchKernelGGL((k_iy_half<R, N>), dim3(N / 2 + 1, (nfields + fpb - 1) / fpb), dim3(ColShape<R, N>::THREADS), 0, s,
                     (const cplx<R> *)in, (cplx<R> *)out, (R *)nyx, (cplx<R> *)nyy, nfields, fpb, nkx, rs, odd_of,
                     (const cplx<R> *)tw);
}

void launch_iy_half(hipStream_t s, int prec, int N, const void *in, void *out, void *nyx, void *nyy, int nfields,
                    int nkx, int rs, const int *odd_of, const void *tw, ColTune tune) {
  if (nfields <= 0) return;
  if (prec == 0) {
    PW_DISPATCH_N(iy_half_launch, float, s, in, out, nyx, nyy, nfields, nkx, rs, odd_of, tw, tune)
  } else {
    PW_DISPATCH_N(iy_half_launch, double, s, in, out, nyx, nyy, nfields, nkx, rs, odd_of, tw, tune)
  }
}

// ------------------------------------------------------------------------------ ix
constexpr int kMaxEll = 5;  // multipoles 0, 2, .., 8

template <typename R, int N>
__global__ void __launch_bounds__(FxShape<N>::THREADS)
k_ix(const cplx<R> *__restrict__ in, int rs, const FieldJob *__restrict__ jobs, int njobs,
     const R *__restrict__ coef, int nell, int half, int nz, int ny, const int *__restrict__ zidx,
     const int *__restrict__ yidx, R Hu, double Hd, R scale, const int *__restrict__ bin_of_s2, int64_t n_s2,
     int nbins, double *__restrict__ acc, const cplx<R> *__restrict__ tw) {
  constexpr int T = FxShape<N>::T, ROWS = FxShape<N>::ROWS, NKX = N / 2 + 1;
  constexpr int LN = N + N / 8;
  __shared__ cplx<R> lds[ROWS * LN];
  extern __shared__ double bacc[];  // (nell + 2) * nbins
  const int rl = threadIdx.x / T, t = threadIdx.x % T;
  const int64_t nrows = (int64_t)nz * ny;
  const int64_t row = (int64_t)blockIdx.x * ROWS + rl;
  const bool live = row < nrows;
  const int zr = live ? (int)(row / ny) : 0, yr = live ? (int)(row - (int64_t)zr * ny) : 0;
  const int z = zidx[zr], y = yidx[yr];
  cplx<R> *my = lds + rl * LN;
  auto at = [my](int i) -> cplx<R> & { return my[i + (i >> 3)]; };
  auto sync = []() { __syncthreads(); };
  const int sy = y < N / 2 ? y : y - N, sz = z < N / 2 ? z : z - N;

  // geometry of the eight cells this lane holds
  R ux[8], uy[8], uz[8], dm[8];
  int bin[8];
  // The sums over the jobs run in FP64: in FP32 their rounding is the largest of the inverse passes, and half
  // of the separations average it half as often as all would (FP32 error of xi_2, all-parity order 4 at
  // 128^3, against FP64: all planes 1.9e-7 of |xi_0|, half with FP32 sums 4.3e-7, this 1.1e-7).  The kernel runs one
  // wave per SIMD either way (256 VGPRs); 512^3: 0.73 ms with both.
  double X[kMaxEll][8];
  const int nacc = (nell + 2) * nbins;
  for (int i = threadIdx.x; i < nacc; i += blockDim.x) bacc[i] = 0.0;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int x = t + s * T;
    const int sx = x < N / 2 ? x : x - N;
    const int64_t s2 = (int64_t)sx * sx + (int64_t)sy * sy + (int64_t)sz * sz;
    bin[s] = (live && s2 < n_s2) ? bin_of_s2[s2] : -1;
    dm[s] = Hu * sqrt((R)s2);  // |D| / unit
    if (s2 > 0) {
      const R ir = (R)1 / sqrt((R)s2);
      ux[s] = (R)sx * ir; uy[s] = (R)sy * ir; uz[s] = (R)sz * ir;
    } else {
      ux[s] = 0; uy[s] = 0; uz[s] = 1;
    }
#pragma unroll
    for (int l = 0; l < kMaxEll; ++l) X[l][s] = 0;
  }
  ShRec8<R> rec;
  rec.init();
  const size_t fstride = (size_t)nrows * rs;  // rows padded to rs
  // this workgroup's share of the jobs (grid y): the sums are linear in them
  const int jb0 = njobs * (int)blockIdx.y / (int)gridDim.y, jb1 = njobs * ((int)blockIdx.y + 1) / (int)gridDim.y;
  for (int jb = jb0; jb < jb1; ++jb) {
    const FieldJob J = jobs[jb];
    const cplx<R> *ha = in + (size_t)J.pa * fstride + (size_t)row * rs;
    const cplx<R> *hb = in + (size_t)(J.pb < 0 ? 0 : J.pb) * fstride + (size_t)row * rs;
    // Z = Ha + i Hb on the full x range from the half spectra (Ha(-k) = conj Ha(k) after the
    // y and z inverse passes of a real field); the self-conjugate kx = 0, N/2 keep real parts.
    for (int kx = t; kx < NKX; kx += T) {
      const cplx<R> a = live ? ha[kx] : mk<R>(0, 0);
      const cplx<R> b = (live && J.pb >= 0) ? hb[kx] : mk<R>(0, 0);
      if (kx == 0 || kx == N / 2) {
        at(kx) = mk<R>(a.x, b.x);
      } else {
        at(kx) = mk<R>(a.x - b.y, a.y + b.x);
        at(N - kx) = mk<R>(a.x + b.y, b.x - a.y);
      }
    }
    sync();
    cplx<R> v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = at(t + s * T);
    sync();
    fft_pencil<R, N, true>(v, t, tw, at, sync);
    R ya[8], yb[8];
    if (J.kind == 0) {
      rec.set_m(J.m, ux, uy);
      rec.advance(c_sh_inv, J.Ja, uz);
      const R n = sh_n<R>(c_sh_inv, J.Ja, J.m);
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        R w = n * rec.q0[s];
        for (int a = 0; a < J.alpha; ++a) w *= dm[s];
        ya[s] = w * rec.cr[s];
        yb[s] = w * rec.ci[s];
      }
    } else {
      rec.set_m(0, ux, uy);
      rec.advance(c_sh_inv, J.Ja, uz);
      const R na = sh_n<R>(c_sh_inv, J.Ja, 0);
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        R w = na * rec.q0[s];
        for (int a = 0; a < J.alpha; ++a) w *= dm[s];
        ya[s] = w;
        yb[s] = 0;
      }
      if (J.Jb >= 0) {
        rec.advance(c_sh_inv, J.Jb, uz);
        const R nb = sh_n<R>(c_sh_inv, J.Jb, 0);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          R w = nb * rec.q0[s];
          for (int a = 0; a < J.alpha_b; ++a) w *= dm[s];
          yb[s] = w;
        }
      }
    }
    const R *ca = coef + (size_t)jb * 2 * nell, *cb = ca + nell;
#pragma unroll
    for (int l = 0; l < kMaxEll; ++l) {
      if (l < nell) {
        const R fa = ca[l], fb = cb[l];
#pragma unroll
        for (int s = 0; s < 8; ++s) X[l][s] += (double)(fa * ya[s]) * v[s].x + (double)(fb * yb[s]) * v[s].y;
      }
    }
  }
  sync();  // bacc cleared by every thread before any accumulation
  const double mult = (half && z != 0 && z != N / 2) ? 2.0 : 1.0;  // -D has the same terms
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int b = bin[s];
    if (b < 0) continue;
    const int x = t + s * T;
    const int sx = x < N / 2 ? x : x - N;
    const double s2 = (double)sx * sx + (double)sy * sy + (double)sz * sz;
#pragma unroll
    for (int l = 0; l < kMaxEll; ++l)
      if (l < nell) atomicAdd(&bacc[l * nbins + b], mult * X[l][s] * (double)scale);
    if (blockIdx.y == 0) {  // each cell is counted once
      atomicAdd(&bacc[nell * nbins + b], mult);
      atomicAdd(&bacc[(nell + 1) * nbins + b], mult * Hd * sqrt(s2));
    }
  }
  sync();
  for (int i = threadIdx.x; i < nacc; i += blockDim.x)
    if (bacc[i] != 0.0) atomicAdd(&acc[i], bacc[i]);
}

template <typename R, int N>
static void ix_launch(hipStream_t s, const void *in, int rs, const FieldJob *jobs, int njobs, const void *coef,
                      int nell, int half, int nz, int ny, const int *zidx, const int *yidx, double H, double unit, double scale,
                      const int *bin_of_s2, int64_t n_s2, int nbins, double *acc, const void *tw) {
  constexpr int ROWS = FxShape<N>::ROWS;
  const int64_t nrows = (int64_t)nz * ny;
  // Few rows lie inside the r-bins of a coarse mesh (9 x 17 at 128^3 for bins to 200 in a box of 2900:
  // 20 workgroups), each a chain over every job: the jobs are shared out over grid y until a thousand
  // workgroups run, at least three jobs each: with 28 targets 80 -> 30 us.  At 512^3 the rows alone fill the
  // chip (640 workgroups of two waves per SIMD) and sharing them out three ways was slower (1.22 -> 1.27 ms).
  const unsigned nblk = (unsigned)((nrows + ROWS - 1) / ROWS);
  dim3 grid(nblk, std::max(1u, std::min(1024u / nblk, (unsigned)njobs / 3u)));
  const size_t sh = (size_t)(nell + 2) * nbins * sizeof(double);
  hipLaunchKernelGGL((k_ix<R, N>), grid, dim3(FxShape<N>::THREADS), sh, s, (const cplx<R> *)in, rs, jobs, njobs,
                     (const R *)coef, nell, half, nz, ny, zidx, yidx, (R)(H / unit), H, (R)scale, bin_of_s2, n_s2, nbins, acc,
                     (const cplx<R> *)tw);
}

void launch_ix(hipStream_t s, int prec, int N, const void *in, int rs, const FieldJob *jobs, int njobs,
               const void *coef, int nell, int half, int nz, int ny, const int *zidx, const int *yidx, double H, double unit,
               double scale, const int *bin_of_s2, int64_t n_s2, int nbins, double *acc, const void *tw) {
  if (njobs <= 0 || nz <= 0 || ny <= 0 || nell > kMaxEll) return;
  if (prec == 0) {
    PW_DISPATCH_N(ix_launch, float, s, in, rs, jobs, njobs, coef, nell, half, nz, ny, zidx, yidx, H, unit, scale,
                  bin_of_s2, n_s2, nbins, acc, tw)
  } else {
    PW_DISPATCH_N(ix_launch, double, s, in, rs, jobs, njobs, coef, nell, half, nz, ny, zidx, yidx, H, unit, scale,
                  bin_of_s2, n_s2, nbins, acc, tw)
  }
}

// ------------------------------------------------------------------------------ contract_mid
// One thread per retained mode of the half spectrum; a mode with 0 < kx < N/2 also stands for
// its mirror (conjugate values, same real parts) whose direction is that of (-n) mod N.
template <typename R, int LMAX>
__global__ void __launch_bounds__(256)
k_contract_mid(const R *__restrict__ G, const R *__restrict__ A, int64_t nmodes, int64_t mstride,
               const uint32_t *__restrict__ modecoord, int N, const int *__restrict__ bin_of_s2, int64_t n_s2,
               int nbins, double kf, double *__restrict__ acc) {
  constexpr int NSH = (LMAX + 1) * (LMAX + 1);
  constexpr int NE = LMAX / 2 + 1;
  extern __shared__ double bacc[];
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
    const bool pair = (kx != 0 && kx != half);
    R wdir[NSH];
#pragma unroll
    for (int i = 0; i < NSH; ++i) wdir[i] = 0;
    {
      R ux = 0, uy = 0, uz = 1;
      const R ir = s2 > 0 ? (R)1 / sqrt((R)s2) : (R)0;
      if (s2 > 0) { ux = (R)sx * ir; uy = (R)sy * ir; uz = (R)sz * ir; }
      real_sh_even<R, LMAX>(c_sh_inv, ux, uy, uz, wdir);
      if (pair) {
        const int my = (ky == half) ? sy : -sy;
        const int mz = (kz == half) ? sz : -sz;
        R wm[NSH];
#pragma unroll
        for (int i = 0; i < NSH; ++i) wm[i] = 0;
        real_sh_even<R, LMAX>(c_sh_inv, (R)(-sx) * ir, (R)my * ir, (R)mz * ir, wm);
#pragma unroll
        for (int i = 0; i < NSH; ++i) wdir[i] += wm[i];
      }
    }
    R E[NE];
#pragma unroll
    for (int l = 0, o = 0; l <= LMAX; l += 2) {
      R e = 0;
#pragma unroll
      for (int nu = -l; nu <= l; ++nu, ++o) {
        R v = __builtin_nontemporal_load(G + (size_t)o * mstride + mode);
        if (l >= 2 && A) v += __builtin_nontemporal_load(A + (size_t)(o - 1) * mstride + mode);
        e += wdir[l * l + l + nu] * v;
      }
      E[l / 2] = e;
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

void launch_contract_mid(hipStream_t s, int prec, int lmax, const void *G, const void *A,
                         int64_t nmodes, int64_t mstride, const uint32_t *modecoord, int N, const int *bin_of_s2,
                         int64_t n_s2, int nbins, double kf, double *acc) {
  if (nmodes <= 0) return;
  int64_t want = (nmodes + 255) / 256;
  unsigned blocks = (unsigned)(want < 4096 ? (want > 0 ? want : 1) : 4096);
  size_t sh = (size_t)(lmax / 2 + 3) * nbins * sizeof(double);
#define PW_CM(R, L)                                                                                \
  hipLaunchKernelGGL((k_contract_mid<R, L>), dim3(blocks), dim3(256), sh, s, (const R *)G, \
                     (const R *)A, nmodes, mstride, modecoord, N, bin_of_s2, n_s2, nbins, kf, acc);
  if (prec == 0) {
    switch (lmax) {
      case 0: PW_CM(float, 0) break;
      case 2: PW_CM(float, 2) break;
      case 4: PW_CM(float, 4) break;
      case 6: PW_CM(float, 6) break;
      default: PW_CM(float, 8) break;
    }
  } else {
    switch (lmax) {
      case 0: PW_CM(double, 0) break;
      case 2: PW_CM(double, 2) break;
      case 4: PW_CM(double, 4) break;
      case 6: PW_CM(double, 6) break;
      default: PW_CM(double, 8) break;
    }
  }
#undef PW_CM
}

// ------------------------------------------------------------------------------ finalize_xi
__global__ void k_finalize_xi(const double *acc, int nell, int nbins, double cell_volume, const DevNorm *norm,
                              double *out) {
  const double fourpi = 12.566370614359172953850573533118;
  const double I = norm->I;
  for (int i = threadIdx.x; i < (nell + 1) * nbins; i += blockDim.x) {
    const int l = i / nbins, b = i % nbins;
    const double cnt = acc[nell * nbins + b];
    if (l < nell) {
      out[l * nbins + b] = (cnt > 0) ? fourpi / I * acc[l * nbins + b] / (cnt * cell_volume) : 0.0;
    } else {
      out[nell * nbins + b] = (cnt > 0) ? acc[(nell + 1) * nbins + b] / cnt : 0.0;  // mean |D|
      out[(nell + 1) * nbins + b] = cnt;
    }
  }
}

void launch_finalize_xi(hipStream_t s, const double *acc, int nell, int nbins, double cell_volume,
                        const DevNorm *norm, double *out) {
  hipLaunchKernelGGL(k_finalize_xi, dim3(1), dim3(256), 0, s, acc, nell, nbins, cell_volume, norm, out);
}

}  // namespace pw
