// 1D lines of the non-circular modes, of any length, as right-angle transforms
// (ra_device.hpp): a line of L points is N >= L complex points, N a power of
// two, at the frequencies f + 1/4.
//
//  * conv1d_ra, bwd1d_ra: forward, and backward, of lines up to 8192 points in
//    one pass, a workgroup per line, the spectra in registers (the backward's
//    three at one workgroup of two wavefronts per SIMD);
//  * lines beyond (forward and backward) in three passes, N = N1 x N2 with
//    n = n1 N2 + n2 and f = f1 + N1 f2:
//      columns   over n1 at the frequencies f1 + 1/4, then the twiddle
//                exp(-2 pi i n2 (f1 + 1/4) / N);
//      core      rows f1: plain transforms over n2, the pointwise products
//                with the shortcut folded in, inverse, the twiddle back;
//      columns   inverse, exp(+2 pi i n1 / (4 N1)), real part, gates, store.
//    A bin has no mirror, so a core workgroup needs one row of each signal
//    (the packed real transform needs the rows f1 and N1 - f1 together).
//
// Single pass: bound by the LDS exchanges and the vector units (1024 lines of
// 8192 points move 0.15 GB in fp32, 30 us at 5.1 TB/s).  The packed
// real transform on 2 P points, which these replace, untangled its mirror bins
// through LDS, and the lengths that are no powers of two went through copies
// embedded in a circular grid.  Forward, 1024 x 8192 points, fp32: 92.9 -> 72.8
// us; backward, bf16, centered, 1024 x 8192: 919.7 -> 137.5; 1024 x 8000 linear:
// 806.9 -> 127.9.  One line per workgroup leaves short calls to the latency of
// the chain: 64 lines of 4096 points 10.5 -> 8.9 us.
//
// Three passes: bound by the traffic of the spectra (forward: u and k written
// and read, y written and read, 48 bytes a point against 8 of the tensors).
// 256 lines of 2^20 points, bf16, with the filter's own kernel: 3812 -> 3343
// us, 15.7 GB; the columns of u and k 51 us, the core 44 and the inverse columns 28
// per launch of five lines, of which two run side by side.  512 lines of 16384
// points, backward, bf16: 421 -> 275 us; lengths that are no powers of two
// (embedded copies before) 3.1 to 7 times faster.
#include "fourstep.hpp"
#include "ra_mp.hpp"

namespace hyenand {

namespace {

// exp(-2 pi i e / (4 E)), E points per lane (2 to 16)
template <int E>
__device__ __forceinline__ float2 ra_root(int e) {
  return make_float2(kCos64[e * (16 / E)], -kSin64[e * (16 / E)]);
}

// exp(-2 pi i n / (4 N)) at n = t + (N / E) e: the root r of e with what its rounding
// leaves, times 1 + d, d = exp(-2 pi i t / (4 N)) - 1 of the lane.  d and the
// remainder are small, so only the last sum rounds; the product of r and one or
// two table entries rounds three to six times.  Relative L2 against 64 bits, fp32
// lines, forward: 512 points 1.91e-7 -> 1.65e-7, 2048 2.06e-7 -> 1.80e-7, 8192
// 2.37e-7 -> 2.17e-7 (packed real transforms: 1.70, 1.90, 2.06e-7); it costs 1 to
// 4 % (1024 x 2048 points 13.6 -> 14.1 us).
template <int E>
__device__ __forceinline__ float2 ra_weight(float2 d, int e) {
  const float2 r = ra_root<E>(e);
  const float lx = kCos64Lo[e * (16 / E)], ly = -kSin64Lo[e * (16 / E)];  // r's own rounding
  return make_float2(r.x + fmaf(d.x, r.x, fmaf(-d.y, r.y, lx)), r.y + fmaf(d.x, r.y, fmaf(d.y, r.x, ly)));
}

// ---------------------------------------------------------------------------
// single-pass backward
// ---------------------------------------------------------------------------
// Points per lane.  8 shortens the chain of a line, 16 takes a pass and an
// exchange less: fp32 lines of 4096 points, 64 of them 9.1 (8) against 9.9 us,
// 1024 of them 28.2 against 27.7 (2048 points: 15.9 against 14.5).  Calls of up
// to two workgroups per CU take 8, more take 16; up to 1024 points 8 is the
// better one at any count.  The backward's three spectra: 1024 x 4096 points
// 76 (8) against 55 us, 1024 x 1024 points 21.0 against 23.5.
constexpr int ra1_e(int N) { return N > 1024 ? 16 : 8; }
constexpr int64_t kRaShortCall = 512;
constexpr int ra1_nt(int N) { return N / ra1_e(N); }  // of the backward

// Whether a kernel can scale its lines (norm): the mixed plan has circular lines
// of up to 4096 points forward (KC), others of up to about 1500 backward.  In the
// other kernels the code would cost 1 to 2 % (backward of 8192 points, bf16: 125.4
// -> 127.6 us).
template <int N, bool KC>
constexpr bool kRa1Norm = KC && N <= 4096;
template <int N>
constexpr bool kRa1BwdNorm = N <= 2048;

// norm: u, k and h scaled by powers of two (ra_device.hpp); the scratch of the
// magnitudes is free again after the next barrier.
template <int N, bool KC, typename TS>
__global__ void __launch_bounds__(ra1_nt(N)) __attribute__((amdgpu_waves_per_eu(2)))
    bwd1d_ra(const TS* __restrict__ x1, const TS* __restrict__ x2, const TS* __restrict__ v,
             const TS* __restrict__ k, const TS* __restrict__ Dp, const TS* __restrict__ gy, TS* __restrict__ gx1,
             TS* __restrict__ gx2, TS* __restrict__ gv, TS* __restrict__ gk, float* __restrict__ partial, int C, int L,
             int norm) {
  constexpr int E = ra1_e(N), T = N / E, NT = T;
  static_assert(NT >= 64, "a wavefront or more");
  __shared__ float2 S[pad16_size(N)];
  __shared__ float2 twl[PassTw<N, E>::kCount];
  __shared__ float red[NT / 64];
  const int t = threadIdx.x;
  PassTw<N, E>::fill(twl, t, NT);
  const int64_t line = blockIdx.x;
  const int c = (int)(line % C);
  const int64_t base = line * L;
  const int KL = KC ? 2 * L - 1 : L;
  const TS* const kl = k + line * KL;
  const ScrPad16 sc{S};
  constexpr float scale = 1.f / (float)N;
  float2 wt = kTwDelta[t * (8192 / N)];
  auto om = [&](int e) { return ra_weight<E>(wt, e); };  // at n = t + T e

  float xa[E], xv[E], xg[E];
  float2 wu[E], wh[E], wk[E];
  float hu = 0.f;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = t + T * e;
    const bool in = n < L;
    xa[e] = ra_ld_sel(x1 + base, n, in);
    xv[e] = ra_ld_sel(v + base, n, in);
    xg[e] = ra_ld_sel(gy + base, n, in);
    wh[e].x = ra_ld_sel(x2 + base, n, in);
    if constexpr (KC) wk[e] = make_float2(ra_ld_sel(kl + L - 1, n, in), ra_ld_sel(kl + L - 1, n - N, n > N - L));
    else wk[e] = make_float2(ra_ld_sel(kl, n, in), 0.f);
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    wh[e].x *= xg[e];
    wu[e].x = xa[e] * xv[e];
    hu = fmaf(wh[e].x, wu[e].x, hu);
  }
  const float Dv = ld1(Dp + c);
  int eu = 0, eh = 0, ek = 0;
  if (kRa1BwdNorm<N> && norm) {
    RaMags<NT / 64, 3> mags;
    mags.s = reinterpret_cast<uint32_t*>(S);
    uint32_t m[3] = {0, 0, 0};
#pragma unroll
    for (int e = 0; e < E; ++e) {
      m[0] = ra_umax(m[0], ra_mag(wu[e].x));
      m[1] = ra_umax(m[1], ra_mag(wh[e].x));
      m[2] = ra_umax(m[2], ra_umax(ra_mag(wk[e].x), ra_mag(wk[e].y)));
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) mags.put(i, m[i], t);
    mags.sync();
    eu = mags.get(0), eh = mags.get(1), ek = imax(mags.get(2), ra_exponent(ra_mag(Dv)));
#pragma unroll
    for (int e = 0; e < E; ++e) {
      wu[e].x *= ra_pow2(-eu);
      wh[e].x *= ra_pow2(-eh);
    }
  }
  const float ks = scale * ra_pow2(-ek);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    wu[e] = c_scale(om(e), wu[e].x);
    wh[e] = c_scale(om(e), wh[e].x);
    wk[e] = KC ? c_mul(c_scale(wk[e], ks), om(e)) : c_scale(om(e), wk[e].x * ks);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) hu += __shfl_xor(hu, o, 64);
  if ((t & 63) == 0) red[t >> 6] = hu;
  __syncthreads();  // the twiddles and the sums
  if (t == 0) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) s += red[i];
    partial[line] = s;
  }
  // not kept across the transforms: formed again from wt for the outputs
  asm volatile("" : "+v"(wt.x), "+v"(wt.y));
  BlockFFT<N, E, false>::run(wu, t, sc, true, twl);
  BlockFFT<N, E, false>::run(wh, t, sc, true, twl);
  BlockFFT<N, E, false>::run(wk, t, sc, true, twl);
  const float Ds = ks * Dv;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const float2 kd = make_float2(wk[e].x + Ds, wk[e].y);
    wk[e] = c_scale(c_mulc(wh[e], wu[e]), scale);
    wu[e] = c_mul(wu[e], kd);
    wh[e] = c_mulc(wh[e], kd);
  }
  // point n of the ring element: z conj(om)
  BlockFFT<N, E, true>::run(wu, t, sc, true, twl);
  if (kRa1BwdNorm<N> && norm) ra_ldexp(wu, eu + ek);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = t + T * e;
    const float2 o = om(e);
    if (n < L) st1(gx2 + base + n, xg[e] * fmaf(wu[e].x, o.x, wu[e].y * o.y));
  }
  asm volatile("" : "+v"(wt.x), "+v"(wt.y));
  BlockFFT<N, E, true>::run(wh, t, sc, true, twl);
  if (kRa1BwdNorm<N> && norm) ra_ldexp(wh, eh + ek);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = t + T * e;
    const float2 o = om(e);
    const float g = fmaf(wh[e].x, o.x, wh[e].y * o.y);
    if (n < L) {
      st1(gx1 + base + n, g * xv[e]);
      st1(gv + base + n, g * xa[e]);
    }
  }
  asm volatile("" : "+v"(wt.x), "+v"(wt.y));
  BlockFFT<N, E, true>::run(wk, t, sc, true, twl);
  if (kRa1BwdNorm<N> && norm) ra_ldexp(wk, eu + eh);
  TS* const gkl = gk + line * KL;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = t + T * e;
    const float2 o = om(e);
    if (n < L) st1(gkl + (KC ? L - 1 : 0) + n, fmaf(wk[e].x, o.x, wk[e].y * o.y));
    if (KC && n > N - L) st1(gkl + L - 1 - N + n, fmaf(wk[e].y, o.x, -wk[e].x * o.y));
  }
}

// Forward: u and k are transformed in turn by the same lanes, so their spectra
// meet in registers.
template <int N, int E, bool KC, typename TS, bool ACT>
__global__ void __launch_bounds__(N / E) __attribute__((amdgpu_waves_per_eu(N / E == 512 ? 4 : 2)))
    conv1d_ra(const TS* __restrict__ x1, const TS* __restrict__ x2, const TS* __restrict__ v,
              const TS* __restrict__ k, const TS* __restrict__ Dp, TS* __restrict__ y, int C, int kC, int L,
              int periodic, int norm, ActIn ain) {
  constexpr int T = N / E, NT = T;
  __shared__ float2 S[pad16_size(N)];
  __shared__ float2 twl[PassTw<N, E>::kCount];
  const int t = threadIdx.x;
  const int64_t line = blockIdx.x;
  const int c = (int)(line % C);
  const int64_t base = line * L;
  // the displacements n >= 0 and n - N < 0 of a kernel on the double grid
  const TS* const kl = k + k_line(line, kC) * (KC && !periodic ? 2 * L - 1 : L);
  const int reo = KC && !periodic ? L - 1 : 0, imo = (periodic ? L : L - 1) - N;
  const ScrPad16 sc{S};
  constexpr float scale = 1.f / (float)N;
  float2 wt = kTwDelta[t * (8192 / N)];
  auto om = [&](int e) { return ra_weight<E>(wt, e); };
  float2 wu[E], wk[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = t + T * e;
    wk[e] = make_float2(ra_ld_sel(kl + reo, n, n < L), KC ? ra_ld_sel(kl, n + imo, n > N - L) : 0.f);
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = t + T * e;
    wu[e] = make_float2(ra_ld_sel(x1 + base, n, n < L), ra_ld_sel(v + base, n, n < L));
  }
  PassTw<N, E>::fill(twl, t, NT);
  const Gates<ACT> G = line_gates<ACT, TS>(ain, line, C);
  const float Dv = ld1(Dp + c);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    float u = wu[e].x * wu[e].y;
    if constexpr (ACT) u = t + T * e < L ? G.u1(wu[e].x, wu[e].y, t + T * e) : 0.f;
    wu[e].x = u;
  }
  int eu = 0, ek = 0;
  if (kRa1Norm<N, KC> && norm) {
    RaMags<NT / 64, 2> mags;
    mags.s = reinterpret_cast<uint32_t*>(S);
    uint32_t m[2] = {0, 0};
#pragma unroll
    for (int e = 0; e < E; ++e) {
      m[0] = ra_umax(m[0], ra_mag(wu[e].x));
      m[1] = ra_umax(m[1], KC ? ra_umax(ra_mag(wk[e].x), ra_mag(wk[e].y)) : ra_mag(wk[e].x));
    }
    mags.put(0, m[0], t);
    mags.put(1, m[1], t);
    mags.sync();
    eu = mags.get(0), ek = imax(mags.get(1), ra_exponent(ra_mag(Dv)));
#pragma unroll
    for (int e = 0; e < E; ++e) wu[e].x *= ra_pow2(-eu);
  }
  const float ks = scale * ra_pow2(-ek);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    wk[e] = KC ? c_mul(c_scale(wk[e], ks), om(e)) : c_scale(om(e), wk[e].x * ks);
    wu[e] = c_scale(om(e), wu[e].x);
  }
  asm volatile("" : "+v"(wt.x), "+v"(wt.y));
  __syncthreads();
  BlockFFT<N, E, false>::run(wk, t, sc, true, twl);
  BlockFFT<N, E, false>::run(wu, t, sc, true, twl);
  const float Ds = ks * Dv;
#pragma unroll
  for (int e = 0; e < E; ++e) wu[e] = gated_product(wu[e], wk[e], Ds);
  float g[E];
#pragma unroll
  for (int e = 0; e < E; ++e) g[e] = ra_ld_sel(x2 + base, t + T * e, t + T * e < L);
  BlockFFT<N, E, true>::run(wu, t, sc, true, twl);
  if (kRa1Norm<N, KC> && norm) ra_ldexp(wu, eu + ek);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = t + T * e;
    const float2 o = om(e);
    if (n < L) st1(y + base + n, G.g1(g[e]) * fmaf(wu[e].x, o.x, wu[e].y * o.y));
  }
}

template <int N, int E, typename TS>
hipError_t fwd1d_e(const FftConvArgs& a, bool norm, hipStream_t s) {
  if (norm && !kRa1Norm<N, true>) return hipErrorInvalidValue;  // no line of the mixed plan
#define HY_F(KC, ACT)                                                                                          \
  hipLaunchKernelGGL((conv1d_ra<N, E, KC, TS, ACT>), dim3((unsigned)a.lines), dim3(N / E), 0, s, (const TS*)a.x1, \
                     (const TS*)a.x2, (const TS*)a.v, (const TS*)a.k, (const TS*)a.D, (TS*)a.y, (int)a.C, a.kC, \
                     (int)a.L[0], (int)a.periodic, (int)norm, a.act_in)
  if (a.centered || a.periodic) {
    if (a.act) HY_F(true, true);
    else HY_F(true, false);
  } else if (norm) {
    return hipErrorInvalidValue;
  } else if (a.act) {
    HY_F(false, true);
  } else {
    HY_F(false, false);
  }
#undef HY_F
  return hipGetLastError();
}
template <int N, typename TS>
hipError_t fwd1d_t(const FftConvArgs& a, bool norm, hipStream_t s) {
  if constexpr (N == 2048 || N == 4096) {
    if (a.lines <= kRaShortCall) return fwd1d_e<N, 8, TS>(a, norm, s);
  }
  return fwd1d_e<N, ra1_e(N), TS>(a, norm, s);
}

template <int N, typename TS>
hipError_t bwd1d_t(const FftConvBwdArgs& b, bool norm, hipStream_t s) {
  const FftConvArgs& a = b.f;
  if (norm && !kRa1BwdNorm<N>) return hipErrorInvalidValue;  // no line of the mixed plan
#define HY_B(KC)                                                                                                  \
  hipLaunchKernelGGL((bwd1d_ra<N, KC, TS>), dim3((unsigned)a.lines), dim3(ra1_nt(N)), 0, s, (const TS*)a.x1,      \
                     (const TS*)a.x2, (const TS*)a.v, (const TS*)a.k, (const TS*)a.D, (const TS*)b.gy,            \
                     (TS*)b.gx1, (TS*)b.gx2, (TS*)b.gv, (TS*)b.gk, b.partial, (int)a.C, (int)a.L[0], (int)norm)
  if (a.centered) HY_B(true);
  else HY_B(false);
#undef HY_B
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// three passes
// ---------------------------------------------------------------------------
constexpr int kRaN2 = 4096;
struct RaLine {
  int64_t L, N;
  int N1, kmode, log4N;  // log2 (4 N)
};

// a tile of TL adjacent columns of N1 points: as wide as two tiles fit in a CU
// (runs of TL values of the tensors), 64 lanes (N1 up to 16), 128, 256 or 512 (from
// N1 = 128 on)
template <int N1>
struct RaColsCfg {
  static constexpr int tl(int cap) { return cap > 1 && N1 * (cap + 1) * 8 > 76 * 1024 ? tl(cap / 2) : cap; }
  static constexpr int E = imin(16, N1), T = N1 / E;
  static constexpr int TL = imin(tl(64), 1024 / T);
  static constexpr int NT = imax(64, TL * T);
  static constexpr int TLP = TL + 1;
};

// exp(-+2 pi i m / 2^log) for log of 13 to 24, m < 2^log: the coarse entry c and the
// fine angle's sine s, c + c (exp(-i s) - 1) with cos - 1 = -s^2 / 2 (s < 1.6e-3).
template <bool INV>
__device__ __forceinline__ float2 ra_twiddle_rt(uint32_t m, int log) {
  const uint32_t b = m << (24 - log);
  const float2 c = kTwCoarse[b >> 12];
  const float y = kTwFine[b & 4095u].y, x = -0.5f * y * y;
  const float2 w = make_float2(c.x + (c.x * x - c.y * y), c.y + (c.x * y + c.y * x));
  return INV ? c_conj(w) : w;
}

// v[e] times scale exp(-+2 pi i (m0 + step e) / 2^log): chains of eight products
// from entries of their own, since the rounding of the step grows along a chain.
// Relative L2 against 64 bits, fp32 lines of 2^20 points, forward: 3.68e-7, with
// one chain of 16 from two rounded table entries 4.61e-7 (packed real transforms:
// 3.97e-7).  64 such lines: 896 -> 884 us, backward 2426 -> 2062.
template <int E, bool INV>
__device__ __forceinline__ void ra_twiddle_run(float2 (&v)[E], uint32_t m0, uint32_t step, int log, float scale) {
  constexpr int CH = imin(E, 8);
  const float2 s = ra_twiddle_rt<INV>(step, log);
#pragma unroll
  for (int b = 0; b < E; b += CH) {
    float2 w = c_scale(ra_twiddle_rt<INV>(m0 + (uint32_t)b * step, log), scale);
#pragma unroll
    for (int e = 0; e < CH; ++e) {
      v[b + e] = c_mul(v[b + e], w);
      if (e + 1 < CH) w = c_mul(w, s);
    }
  }
}

// PassTw<N1, E>'s tables for the frequencies f1 + 1/4
template <int N1, int E, int NS = 1>
__device__ __forceinline__ void ra_fill(float2* lds, int tid, int nt) {
  using Tw = PassTw<N1, E>;
  if constexpr (NS < N1) {
    constexpr int R = Tw::radix(NS);
    if constexpr (NS > 1) {
      constexpr int off = Tw::offset(NS), cnt = Tw::rows(NS) * NS;
      for (int i = tid; i < cnt; i += nt) {
        const int q = i / NS, jm = i - q * NS;
        const int r = Tw::full(NS) ? q + 1 : (1 << q);
        lds[off + i] = twiddle<ilog2(4 * NS * R), false>((uint32_t)((4 * jm + 1) * r));
      }
    }
    ra_fill<N1, E, NS * R>(lds, tid, nt);
  }
}

// Tiles whose rows are 64 bytes of the tensors: tiles 2 q and 2 q + 1 of a
// signal share every cache line, so they run on one XCD in consecutive slots
// (fs_pair_tiles); with three signals in turn the plain order is the faster.
template <int NTILE, int RUN>
__device__ __forceinline__ unsigned ra_pair_tiles(unsigned b, unsigned nsig) {
  if constexpr (RUN >= 128 || NTILE % 16 != 0) return b;
  return nsig == 1 ? fs_pair_tiles<1>(b) : (nsig == 2 ? fs_pair_tiles<2>(b) : b);
}

// Workgroups: (line, tile, signal).  KERN: k on the double grid (signal 0).
template <int N1, bool KERN, typename TS, bool ACT>
__global__ void __launch_bounds__((RaColsCfg<N1>::NT))
    ra_cols_fwd(RaSignals sg, float2* __restrict__ ws, RaLine g, int64_t line0, int64_t per, int kC, ActIn ain, int C) {
  using Cf = RaColsCfg<N1>;
  constexpr int E = Cf::E, T = Cf::T, NT = Cf::NT, TL = Cf::TL, TLP = Cf::TLP, N2 = kRaN2, NTILE = N2 / TL;
  __shared__ float2 tile[N1 * TLP];
  __shared__ float2 twl[imax(1, PassTw<N1, E>::kCount)];
  const int tid = threadIdx.x;
  ra_fill<N1, E>(twl, tid, NT);
  const unsigned nsig = KERN ? 1 : sg.n, bid = ra_pair_tiles<NTILE, TL * sizeof(TS)>(blockIdx.x, nsig);
  const unsigned sig = bid % nsig, rest = bid / nsig;
  const int64_t line = rest / NTILE, gl = line0 + line;
  const int col = (int)(rest % NTILE) * TL + tid % TL, t = tid / TL;
  const bool act = t < T;
  const TS* const w0 = KERN ? nullptr : (const TS*)sg.w[sig];
  const int64_t kl = g.kmode == RA_CENTERED ? 2 * g.L - 1 : g.L;
  const TS* const x = (const TS*)sg.x[sig] + (w0 ? gl * g.L : k_line(gl, kC) * kl);
  const TS* const w = w0 ? w0 + gl * g.L : nullptr;
  const Gates<ACT> G = line_gates<ACT, TS>(ain, gl, C);
  float2 z[E];
  if constexpr (KERN) {
    const int64_t reo = g.kmode == RA_CENTERED ? g.L - 1 : 0, imo = (g.kmode == RA_CENTERED ? g.L - 1 : g.L) - g.N;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int64_t n = (int64_t)(t + T * e) * N2 + col;
      z[e] = make_float2(ra_ld_sel(x + reo, n, act && n < g.L), ra_ld_sel(x + reo, n + imo - reo, act && n > g.N - g.L));
    }
#pragma unroll
    for (int e = 0; e < E; ++e) z[e] = c_mul(z[e], ra_root<E>(e));
  } else {
    float a[E], b[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int64_t n = (int64_t)(t + T * e) * N2 + col;
      a[e] = ra_ld_sel(x, n, act && n < g.L);
      b[e] = 1.f;
    }
    if (w) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int64_t n = (int64_t)(t + T * e) * N2 + col;
        b[e] = ra_ld_sel(w, n, act && n < g.L);
      }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      float u = a[e] * b[e];
      if constexpr (ACT) {
        const int64_t n = (int64_t)(t + T * e) * N2 + col;
        if (w) u = act && n < g.L ? G.u1(a[e], b[e], n) : 0.f;
      }
      z[e] = c_scale(ra_root<E>(e), u);
    }
  }
  __syncthreads();
  BlockFFT<N1, E, false>::run(z, t, ScrS<TLP>{tile + tid % TL}, act, twl);
  if (act) {
    // exp(-2 pi i n2 (f1 + 1/4) / N), f1 = t + T e
    ra_twiddle_run<E, false>(z, (uint32_t)col * (uint32_t)(4 * t + 1), (uint32_t)col * (uint32_t)(4 * T), g.log4N, 1.f);
    float2* const A = ws + sg.off[sig] + line * per + col;
#pragma unroll
    for (int e = 0; e < E; ++e) A[(int64_t)(t + T * e) * N2] = z[e];
  }
}

// Workgroups: (line, row f1).  U at 0, H at N (BWD), K after them.
// points per lane: three signals of 16 spill or leave two wavefronts per SIMD
// (64 lines of 2^18 points, fp32, backward 662 us; 8 per lane 645 us); two of
// 16 take one exchange less than of 8 (64 x 2^20, bf16: 854 against 920 us)
template <bool BWD>
constexpr int ra_core_e() {
  return BWD ? 8 : 16;
}

template <bool BWD>
__global__ void __launch_bounds__(kRaN2 / ra_core_e<BWD>())
    ra_line_core(float2* __restrict__ ws, const void* __restrict__ Dp, int dbf16, RaLine g, int64_t line0, int C,
                 int64_t per, float scale) {
  constexpr int N2 = kRaN2, E = ra_core_e<BWD>(), T = N2 / E;
  __shared__ float2 S[pad16_size(N2)];
  __shared__ float2 twl[PassTw<N2, E>::kCount];
  const int t = threadIdx.x;
  PassTw<N2, E>::fill(twl, t, T);
  const int f1 = (int)(blockIdx.x % (unsigned)g.N1);
  const int64_t line = blockIdx.x / (unsigned)g.N1;
  const int c = (int)((line0 + line) % C);
  const float D = dbf16 ? ld1((const uint16_t*)Dp + c) : ld1((const float*)Dp + c);
  float2* const U = ws + line * per + (int64_t)f1 * N2 + t;
  float2* const H = U + g.N;
  float2* const K = U + (BWD ? 2 : 1) * g.N;
  const ScrPad16 sc{S};
  float2 wu[E], wk[E], wh[BWD ? E : 1];
#pragma unroll
  for (int e = 0; e < E; ++e) wu[e] = U[T * e];
#pragma unroll
  for (int e = 0; e < E; ++e) wk[e] = K[T * e];
  if constexpr (BWD) {
#pragma unroll
    for (int e = 0; e < E; ++e) wh[e] = H[T * e];
  }
  __syncthreads();
  BlockFFT<N2, E, false>::run(wu, t, sc, true, twl);
  BlockFFT<N2, E, false>::run(wk, t, sc, true, twl);
  if constexpr (BWD) BlockFFT<N2, E, false>::run(wh, t, sc, true, twl);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const float2 kd = make_float2(wk[e].x + D, wk[e].y);
    if constexpr (BWD) {
      wk[e] = c_mulc(wh[e], wu[e]);
      wh[e] = c_mulc(wh[e], kd);
    }
    wu[e] = c_mul(wu[e], kd);
  }
  // exp(+2 pi i n2 (f1 + 1/4) / N), n2 = t + T e, with the normalisation
  const uint32_t m0 = (uint32_t)t * (uint32_t)(4 * f1 + 1), step = (uint32_t)T * (uint32_t)(4 * f1 + 1);
  BlockFFT<N2, E, true>::run(wu, t, sc, true, twl);
  ra_twiddle_run<E, true>(wu, m0, step, g.log4N, scale);
#pragma unroll
  for (int e = 0; e < E; ++e) U[T * e] = wu[e];
  if constexpr (BWD) {
    BlockFFT<N2, E, true>::run(wh, t, sc, true, twl);
    ra_twiddle_run<E, true>(wh, m0, step, g.log4N, scale);
#pragma unroll
    for (int e = 0; e < E; ++e) H[T * e] = wh[e];
    BlockFFT<N2, E, true>::run(wk, t, sc, true, twl);
    ra_twiddle_run<E, true>(wk, m0, step, g.log4N, scale);
#pragma unroll
    for (int e = 0; e < E; ++e) K[T * e] = wk[e];
  }
}

// Workgroups: (line, tile, output).
template <int N1, typename TS, bool ACT>
__global__ void __launch_bounds__((RaColsCfg<N1>::NT))
    ra_cols_inv(RaIos ios, const float2* __restrict__ ws, RaLine g, int64_t line0, int64_t per) {
  using Cf = RaColsCfg<N1>;
  constexpr int E = Cf::E, T = Cf::T, NT = Cf::NT, TL = Cf::TL, TLP = Cf::TLP, N2 = kRaN2, NTILE = N2 / TL;
  __shared__ float2 tile[N1 * TLP];
  __shared__ float2 twl[imax(1, PassTw<N1, E>::kCount)];
  const int tid = threadIdx.x;
  PassTw<N1, E>::fill(twl, tid, NT);
  const unsigned bid = ra_pair_tiles<NTILE, TL * sizeof(TS)>(blockIdx.x, ios.n);
  const unsigned which = bid % (unsigned)ios.n, rest = bid / (unsigned)ios.n;
  const int64_t line = rest / NTILE, gl = line0 + line;
  const int col = (int)(rest % NTILE) * TL + tid % TL, t = tid / TL;
  const bool act = t < T;
  const RaOut out = ios.io[which].out;
  const float2* const B = ws + ios.io[which].off + line * per + col;
  const TS* const p = (const TS*)ios.io[which].p;
  const TS* const q = (const TS*)ios.io[which].q;
  TS* const o1 = (TS*)ios.io[which].o;
  TS* const o2 = (TS*)ios.io[which].o2;
  const int64_t n0 = (int64_t)t * N2 + col, step = (int64_t)T * N2, base = gl * g.L;
  float2 z[E];
  RaGates<E> gt;
#pragma unroll
  for (int e = 0; e < E; ++e) z[e] = B[act ? (int64_t)(t + T * e) * N2 : 0];
  gt.load(out, p, q, base, n0, step, g.L, act);
  __syncthreads();
  BlockFFT<N1, E, true>::run(z, t, ScrS<TLP>{tile + tid % TL}, act, twl);
  if (!act) return;
  const float2 wt = kTwDelta[t * (8192 / N1)];
  auto om = [&](int e) { return c_conj(ra_weight<E>(wt, e)); };  // exp(+2 pi i n1 / (4 N1)), n1 = t + T e
  auto re = [&](int e) {
    const float2 o = om(e);
    return fmaf(z[e].x, o.x, -z[e].y * o.y);
  };
  if (out == RA_GK && g.kmode == RA_CENTERED) {
    TS* const d = o1 + gl * (2 * g.L - 1) + g.L - 1;  // displacement 0
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int64_t n = n0 + step * e;
      const float2 o = om(e);
      if (n < g.L) st1(d + n, re(e));
      if (n > g.N - g.L) st1(d + n - g.N, fmaf(z[e].x, o.y, z[e].y * o.x));
    }
  } else {
    gt.template store<ACT>(out, o1, o2, base, n0, step, g.L, re);
  }
}

struct RaLinePass {
  const FftConvArgs* a;
  RaLine g;
  float2* ws;
  int64_t per, line0;
  int nl;
  hipStream_t s;
};

template <int N1, typename TS>
hipError_t cols_signals(const RaLinePass& p, const RaSignals& sg, bool kern) {
  using Cf = RaColsCfg<N1>;
  const FftConvArgs& a = *p.a;
  const dim3 grid((unsigned)((int64_t)p.nl * (kRaN2 / Cf::TL) * sg.n));
#define HY_C(KERN, ACT)                                                                                        \
  hipLaunchKernelGGL((ra_cols_fwd<N1, KERN, TS, ACT>), grid, dim3(Cf::NT), 0, p.s, sg, p.ws, p.g, p.line0, p.per, \
                     a.kC, a.act_in, (int)a.C)
  if (kern) HY_C(true, false);
  else if (a.act) HY_C(false, true);
  else HY_C(false, false);
#undef HY_C
  return hipGetLastError();
}
template <int N1, typename TS>
hipError_t cols_inverse(const RaLinePass& p, const RaIos& ios) {
  using Cf = RaColsCfg<N1>;
  const dim3 grid((unsigned)((int64_t)p.nl * (kRaN2 / Cf::TL) * ios.n));
  if (p.a->act)
    hipLaunchKernelGGL((ra_cols_inv<N1, TS, true>), grid, dim3(Cf::NT), 0, p.s, ios, p.ws, p.g, p.line0, p.per);
  else
    hipLaunchKernelGGL((ra_cols_inv<N1, TS, false>), grid, dim3(Cf::NT), 0, p.s, ios, p.ws, p.g, p.line0, p.per);
  return hipGetLastError();
}

#define HY_N1_SWITCH(FN, ...)                                                                  \
  switch (p.g.N1) {                                                                            \
    case 4: return p.a->bf16 ? FN<4, uint16_t>(__VA_ARGS__) : FN<4, float>(__VA_ARGS__);       \
    case 8: return p.a->bf16 ? FN<8, uint16_t>(__VA_ARGS__) : FN<8, float>(__VA_ARGS__);       \
    case 16: return p.a->bf16 ? FN<16, uint16_t>(__VA_ARGS__) : FN<16, float>(__VA_ARGS__);    \
    case 32: return p.a->bf16 ? FN<32, uint16_t>(__VA_ARGS__) : FN<32, float>(__VA_ARGS__);    \
    case 64: return p.a->bf16 ? FN<64, uint16_t>(__VA_ARGS__) : FN<64, float>(__VA_ARGS__);    \
    case 128: return p.a->bf16 ? FN<128, uint16_t>(__VA_ARGS__) : FN<128, float>(__VA_ARGS__); \
    case 256: return p.a->bf16 ? FN<256, uint16_t>(__VA_ARGS__) : FN<256, float>(__VA_ARGS__); \
    case 512: return p.a->bf16 ? FN<512, uint16_t>(__VA_ARGS__) : FN<512, float>(__VA_ARGS__); \
    default: return hipErrorInvalidValue;                                                      \
  }
hipError_t d_cols_signals(const RaLinePass& p, const RaSignals& sg, bool kern) { HY_N1_SWITCH(cols_signals, p, sg, kern) }
hipError_t d_cols_inverse(const RaLinePass& p, const RaIos& ios) { HY_N1_SWITCH(cols_inverse, p, ios) }

RaLine line_geom(const FftConvArgs& a) {
  RaLine g;
  g.L = a.L[0];
  g.N = a.P[0] / 2;
  g.N1 = (int)(g.N / kRaN2);
  g.kmode = a.periodic ? RA_PERIODIC : (a.centered ? RA_CENTERED : RA_LINEAR);
  g.log4N = ilog2_rt(4 * g.N);
  return g;
}

// the columns of the signals and of k (at ws + koff), then the core
hipError_t transform(const RaLinePass& p, RaSignals sg, bool bwd) {
  const FftConvArgs& a = *p.a;
  const int64_t koff = (bwd ? 2 : 1) * p.g.N;
  hipError_t e;
  if (p.g.kmode == RA_LINEAR) {
    sg.x[sg.n] = a.k;
    sg.w[sg.n] = nullptr;
    sg.off[sg.n++] = koff;
    e = d_cols_signals(p, sg, false);
  } else {
    e = d_cols_signals(p, sg, false);
    if (e == hipSuccess) e = d_cols_signals(p, RaSignals{{a.k}, {nullptr}, {koff}, 1}, true);
  }
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)((int64_t)p.nl * p.g.N1));
  const float scale = (float)(1.0 / (double)p.g.N);
  if (bwd)
    hipLaunchKernelGGL((ra_line_core<true>), grid, dim3(kRaN2 / ra_core_e<true>()), 0, p.s, p.ws, a.D, (int)a.bf16, p.g, p.line0, (int)a.C,
                       p.per, scale);
  else
    hipLaunchKernelGGL((ra_line_core<false>), grid, dim3(kRaN2 / ra_core_e<false>()), 0, p.s, p.ws, a.D, (int)a.bf16, p.g, p.line0, (int)a.C,
                       p.per, scale);
  return hipGetLastError();
}

}  // namespace

bool ra1d_supported(const FftConvArgs& a) {
  return a.ndim == 1 && !a.circular && a.L[0] >= 2 && a.P[0] >= 1024 && a.P[0] <= 16384;
}

hipError_t launch_ra1d(const FftConvArgs& a, bool norm, hipStream_t s) {
  switch (a.P[0] / 2) {
#define HY_CASE(n) \
  case n: return a.bf16 ? fwd1d_t<n, uint16_t>(a, norm, s) : fwd1d_t<n, float>(a, norm, s);
    HY_CASE(512) HY_CASE(1024) HY_CASE(2048) HY_CASE(4096) HY_CASE(8192)
#undef HY_CASE
    default: return hipErrorInvalidValue;
  }
}

bool ra1d_backward_supported(const FftConvArgs& a) {
  return ra1d_supported(a) && !a.periodic;
}

hipError_t launch_ra1d_backward(const FftConvBwdArgs& b, bool norm, hipStream_t s) {
  switch (b.f.P[0] / 2) {
#define HY_CASE(n) \
  case n: return b.f.bf16 ? bwd1d_t<n, uint16_t>(b, norm, s) : bwd1d_t<n, float>(b, norm, s);
    HY_CASE(512) HY_CASE(1024) HY_CASE(2048) HY_CASE(4096) HY_CASE(8192)
#undef HY_CASE
    default: return hipErrorInvalidValue;
  }
}

// lines of 2^14 to 2^21 complex points; the fused modal filter keeps its own
// passes (conv_fourstep.hip)
bool ra_line_supported(const FftConvArgs& a) {
  return a.ndim == 1 && !a.circular && a.modal.M == 0 && a.P[0] >= (1 << 15) && a.P[0] <= (1 << 22);
}
size_t ra_line_bytes_per_line(const FftConvArgs& a, bool backward) {
  return (size_t)(a.P[0] / 2) * (backward ? 3 : 2) * sizeof(float2);
}

hipError_t launch_ra_line(const FftConvArgs& a, int64_t line0, int64_t nl, void* ws, hipStream_t s) {
  if (!ra_line_supported(a) || nl < 1 || line0 < 0 || line0 + nl > a.lines) return hipErrorInvalidValue;
  const RaLine g = line_geom(a);
  const RaLinePass p{&a, g, (float2*)ws, 2 * g.N, line0, (int)nl, s};
  const hipError_t e = transform(p, RaSignals{{a.x1}, {a.v}, {0}, 1}, false);
  return e == hipSuccess ? d_cols_inverse(p, RaIos{{{RA_Y, a.x2, nullptr, a.y, nullptr, 0}}, 1}) : e;
}

hipError_t launch_ra_line_backward(const FftConvBwdArgs& b, int64_t line0, int64_t nl, void* ws, hipStream_t s) {
  const FftConvArgs& a = b.f;
  if (!ra_line_supported(a) || a.periodic || nl < 1 || line0 < 0 || line0 + nl > a.lines) return hipErrorInvalidValue;
  const RaLine g = line_geom(a);
  const RaLinePass p{&a, g, (float2*)ws, 3 * g.N, line0, (int)nl, s};
  const hipError_t e = transform(p, RaSignals{{a.x1, b.gy}, {a.v, a.x2}, {0, g.N}, 2}, true);
  if (e != hipSuccess) return e;
  return d_cols_inverse(p, RaIos{{{RA_GX2, b.gy, nullptr, b.gx2, nullptr, 0},
                                  {RA_GU, a.v, a.x1, b.gx1, b.gv, g.N},
                                  {RA_GK, nullptr, nullptr, b.gk, nullptr, 2 * g.N}}, 3});
}

}  // namespace hyenand
