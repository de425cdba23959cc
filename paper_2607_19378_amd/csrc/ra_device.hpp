// Right-angle transforms: the building blocks of the non-circular plans.
//
// A linear convolution of real lines of L points needs only the ring
// C[x] / (x^N + i), N >= L: its complex elements hold 2N real coefficients, the
// product of two real lines is y[n] - i y[N + n], and the wanted outputs n < N
// are the real part.  The ring's evaluation points are the N roots of x^N = -i,
// so a transform is a DFT of N points at the frequencies f + 1/4,
//   X[f] = sum_n x[n] exp(-2 pi i n (f + 1/4) / N),
// half the points of the zero-padded real transform, and its bins have no
// mirror bins: no untangling, no packing, no DC / Nyquist column, and products
// are pointwise.  A kernel with displacements d in (-N, N) is the line
// k[n] + i k[n - N] (x^-N = i), conj(K) is the reversed kernel, and a
// correlation sum_n h[n] u[n - d] comes back in g[n] as Re (d = n) and
// Im (d = n - N).
//
// In the Stockham passes the shift of 1/4 costs nothing: pass (NS, R) uses
// exp(-2 pi i r (jm + 1/4) / (NS R)) in place of exp(-2 pi i r jm / (NS R)),
// and the first pass (jm = 0, real inputs) scales its inputs by constants.
// The inverse multiplies its outputs by exp(+2 pi i n / (4 N)): the part of
// that which depends on the lane joins the last pass's twiddles, the rest are
// constants.
//
// Every transform here is held by one wavefront: T lanes per line, E points
// per lane, 64 / T lines per wavefront, one exchange through LDS slots that
// only this wavefront touches between two barriers of the workgroup, so the
// exchange needs no barrier (a wavefront's LDS accesses are performed in
// order).  The layouts below keep the exchanges free of bank conflicts
// (64 banks of 4 bytes: 64 lanes of 8 bytes, two lanes per bank pair; columns of
// narrow rows excepted).
#pragma once

#include "kernels.hpp"

namespace hyenand {
namespace {

// ---------------------------------------------------------------------------
// Magnitudes of a line.  The sums of a transform leave fp32's range where the
// inputs come near its ends (196 values of 1e37, a kernel of 1e-36 under the
// normalisation of 1 / N), although u k does not.  The mixed-radix kernels scale
// u, k and h of a line, exactly, by powers of two to magnitudes near 1 and undo
// it at the store; in their place these kernels do too (norm).  Everywhere else
// it would cost without need: 6 to 17 % of 28^2 to 57 x 40 images, 8 % of 64
// lines of 3000 points.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t ra_umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
// the bits of |x|, ordered like the values; NaN above all
__device__ __forceinline__ uint32_t ra_mag(float x) { return __float_as_uint(fabsf(x)); }
// largest of a wavefront (every lane active), in every lane: maxima over rows of
// 16 lanes, then across the rows
__device__ __forceinline__ uint32_t ra_wave_max(uint32_t m) {
#define HY_DPP(ctrl, rows) m = ra_umax(m, (uint32_t)__builtin_amdgcn_update_dpp((int)m, (int)m, ctrl, rows, 0xf, false))
  HY_DPP(0x111, 0xf);  // row_shr:1, 2, 4, 8
  HY_DPP(0x112, 0xf);
  HY_DPP(0x114, 0xf);
  HY_DPP(0x118, 0xf);
  HY_DPP(0x142, 0xa);  // row_bcast:15, 31
  HY_DPP(0x143, 0xc);
#undef HY_DPP
  return (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
}
// Exponent e of the magnitude with bits b: b 2^-e in [1/2, 1), 0 for 0, infinity
// and NaN; within [-100, 112], so that 2^-e and 2^-e / 2^14 are normal numbers
// (what that leaves unscaled is within 2^16 of 1).
__device__ __forceinline__ int ra_exponent(uint32_t b) {
  const int e = __builtin_amdgcn_frexp_expf(__uint_as_float(b));
  return e < -100 ? -100 : (e > 112 ? 112 : e);
}
template <int E>
__device__ __forceinline__ void ra_ldexp(float2 (&w)[E], int e) {
#pragma unroll
  for (int i = 0; i < E; ++i) w[i] = make_float2(ldexpf(w[i].x, e), ldexpf(w[i].y, e));
}
__device__ __forceinline__ float ra_pow2(int e) { return __uint_as_float((uint32_t)(127 + e) << 23); }
// The exponents of NS signals' largest magnitudes over a workgroup of W
// wavefronts: put (every lane, its magnitude), a barrier of the workgroup, get.
// A single wavefront needs neither LDS nor the barrier.
template <int W, int NS>
struct RaMags {
  uint32_t one[NS];
  uint32_t* s;  // NS W words of LDS
  __device__ __forceinline__ void put(int i, uint32_t m, int tid) {
    m = ra_wave_max(m);
    if constexpr (W == 1) one[i] = m;
    else if ((tid & 63) == 0) s[i * W + (tid >> 6)] = m;
  }
  __device__ __forceinline__ void sync() const {
    if constexpr (W > 1) __syncthreads();
  }
  __device__ __forceinline__ int get(int i) const {
    uint32_t b;
    if constexpr (W == 1) {
      b = one[i];
    } else {
      b = s[i * W];
#pragma unroll
      for (int j = 1; j < W; ++j) b = ra_umax(b, s[i * W + j]);
    }
    return __builtin_amdgcn_readfirstlane(ra_exponent(b));
  }
};

// Orders this wavefront's LDS accesses for the compiler; the hardware
// performs them in order.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// Rows: N points (16 to 512), E = 8 per lane up to 64 points, 16 beyond.
// Point p of a row sits in slot p + p / E of a pitch of N + N / E slots: the
// writes of a pass (slots (E + 1) t + r) and the reads t + T e both spread over
// all banks.
// ---------------------------------------------------------------------------
//
// F = 2: the bins 2 j + p of a row of 2 N points, as the N-point transform of
// the folded row x[n] + x[n + N] exp(-i pi (p + 1/4)) at the frequencies
// j + (p + 1/4) / 2.  p is wave-uniform; F = 1 has p = 0.
template <int N, int F = 1>
struct RaRow {
  static_assert(is_pow2(N) && N >= 16 && N <= 512, "row length");
  static_assert(F == 1 || (F == 2 && N == 64), "folded rows");
  static constexpr int E = N <= 64 ? 8 : 16, T = N / E;  // lanes per row
  static constexpr int PITCH = N + N / E;
  static constexpr int R2 = imin(E, N / E), NB2 = E / R2;              // second pass
  static constexpr bool kThree = R2 * E < N;                           // 512 points: a third pass
  static constexpr int R3 = kThree ? N / (E * R2) : 1, NB3 = E / R3;
  static constexpr int RL = kThree ? R3 : R2, NBL = kThree ? NB3 : NB2;  // last pass
  // slot of point t + T e, less t + t / E
  static constexpr int off(int e) { return T * e + (T * e) / E; }
  static __device__ __forceinline__ int slot(int p) { return p + p / E; }

  // forward: exp(-2 pi i r (jm + sh) / (NS R)), r >= 1, sh = (p + 1/4) / F;
  // folded rows also the first pass's exp(-2 pi i e sh / E)
  struct FwdTw {
    float2 w2[NB2][R2], w3[kThree ? NB3 : 1][R3], first[F > 1 ? E : 1];
    __device__ __forceinline__ void load(int t, int p = 0) {
      if constexpr (F > 1) {
#pragma unroll
        for (int e = 1; e < E; ++e) first[e] = twiddle<ilog2(4 * F * E), false>((uint32_t)(e * (4 * p + 1)));
      }
#pragma unroll
      for (int b = 0; b < NB2; ++b)
#pragma unroll
        for (int r = 1; r < R2; ++r)
          w2[b][r] = twiddle<ilog2(4 * F * E * R2), false>((uint32_t)((4 * F * ((t + T * b) & (E - 1)) + 4 * p + 1) * r));
      if constexpr (kThree) {
#pragma unroll
        for (int b = 0; b < NB3; ++b)
#pragma unroll
          for (int r = 1; r < R3; ++r) w3[b][r] = twiddle<ilog2(4 * N), false>((uint32_t)((4 * (t + T * b) + 1) * r));
      }
    }
  };
  // inverse: exp(+2 pi i jm r / (NS R)), and in the last pass (NS R = N)
  // exp(+2 pi i jm (r + 1/4) / N), r >= 0
  struct InvTw {
    float2 w2[NB2][R2], w3[kThree ? NB3 : 1][R3];
    __device__ __forceinline__ void load(int t) {
      static_assert(F == 1, "folded rows are not inverted");
#pragma unroll
      for (int b = 0; b < NB2; ++b)
#pragma unroll
        for (int r = 0; r < R2; ++r) {
          const int jm = (t + T * b) & (E - 1);
          if constexpr (kThree) w2[b][r] = twiddle<ilog2(E * R2), true>((uint32_t)(jm * r));
          else w2[b][r] = twiddle<ilog2(4 * N), true>((uint32_t)(jm * (4 * r + 1)));
        }
      if constexpr (kThree) {
#pragma unroll
        for (int b = 0; b < NB3; ++b)
#pragma unroll
          for (int r = 0; r < R3; ++r) w3[b][r] = twiddle<ilog2(4 * N), true>((uint32_t)((t + T * b) * (4 * r + 1)));
      }
    }
  };

  // the first pass's constants exp(-2 pi i e / (4 E)) on a real or complex input;
  // 16 points per lane (the rows of passes that memory bounds) also take what the
  // constants' rounding leaves
  static constexpr bool kLo = E == 16;
  static __device__ __forceinline__ float lead_c(int e) { return E == 8 ? kCos32[e] : kCos64[e]; }
  static __device__ __forceinline__ float lead_s(int e) { return E == 8 ? kSin32[e] : kSin64[e]; }
  static __device__ __forceinline__ float2 lead(float x, int e) {
    if (!kLo || e == 0) return make_float2(x * lead_c(e), -x * lead_s(e));
    return make_float2(fmaf(x, lead_c(e), x * kCos64Lo[e]), -fmaf(x, lead_s(e), x * kSin64Lo[e]));
  }
  static __device__ __forceinline__ float2 lead(float2 x, int e) {
    if (e == 0) return x;
    const float c = lead_c(e), s = lead_s(e);
    if (!kLo) return make_float2(fmaf(x.x, c, x.y * s), fmaf(x.y, c, -x.x * s));
    const float cl = kCos64Lo[e], sl = kSin64Lo[e];
    return make_float2(fmaf(x.x, c, fmaf(x.y, s, fmaf(x.x, cl, x.y * sl))),
                       fmaf(x.y, c, fmaf(-x.x, s, fmaf(x.y, cl, -x.x * sl))));
  }

  // folded rows: point n from x[n] (a) and x[n + N] (b), both real or complex
  static __device__ __forceinline__ float2 fold(float2 a, float2 b, int p, const FwdTw& tw, int e) {
    const float s = p ? -0.70710678118654752f : 0.70710678118654752f;  // exp(-i pi (p + 1/4)) = s (1 - i)
    const float2 z = make_float2(fmaf(s, b.x + b.y, a.x), fmaf(s, b.y - b.x, a.y));
    return e ? c_mul(z, tw.first[e]) : z;
  }
  // exchange after pass (NS, R): butterfly j = t + T b leaves its output r at
  // position (j - jm) R + jm + NS r
  template <int NS, int R>
  static __device__ __forceinline__ void exchange(float2 (&w)[E], int t, float2* row) {
    constexpr int NB = E / R;
    static_assert(NB == 1, "a pass before an exchange has one butterfly per lane");
    wave_sync();
    const int jm = t & (NS - 1);
    float2* const pw = row + slot((t - jm) * R + jm);
    // NS r: a multiple of E, or (first pass) inside the E slots from a multiple of E on
#pragma unroll
    for (int r = 0; r < R; ++r) pw[NS * r + (NS * r) / E] = w[r];
    wave_sync();
    const float2* const pr = row + slot(t);
#pragma unroll
    for (int e = 0; e < E; ++e) w[e] = pr[off(e)];
    wave_sync();
  }
  template <int R, int NB, bool INV, bool FIRST>
  static __device__ __forceinline__ void pass(float2 (&w)[E], const float2 (&tw)[NB][R]) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float2 x[R];
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = (r || FIRST) ? c_mul(w[b + NB * r], tw[b][r]) : w[b];
      dft<R, INV>(x);
#pragma unroll
      for (int r = 0; r < R; ++r) w[b + NB * r] = x[r];
    }
  }

  // w[e] = lead(point t + T e); leaves bin t + T e in w[e]
  static __device__ __forceinline__ void forward(float2 (&w)[E], int t, float2* row, const FwdTw& tw) {
    dft<E, false>(w);
    exchange<1, E>(w, t, row);
    pass<R2, NB2, false, false>(w, tw.w2);
    if constexpr (kThree) {
      exchange<E, R2>(w, t, row);
      pass<R3, NB3, false, false>(w, tw.w3);
    }
  }
  // bin t + T e in w[e]; leaves point t + T e up to exp(2 pi i r / (4 RL)),
  // r = e / NBL, which re() and im() apply
  static __device__ __forceinline__ void inverse(float2 (&w)[E], int t, float2* row, const InvTw& tw) {
    dft<E, true>(w);
    exchange<1, E>(w, t, row);
    pass<R2, NB2, true, !kThree>(w, tw.w2);
    if constexpr (kThree) {
      exchange<E, R2>(w, t, row);
      pass<R3, NB3, true, true>(w, tw.w3);
    }
  }
  // cos, sin of 2 pi (e / NBL) / (4 RL), and what their rounding leaves.  A
  // constant's error is the same at every N / RL-th point of every row, so it
  // weighs more than the roundings around it.  Relative L2 against 64 bits, fp32:
  // 64 x 64 linear 1.83e-7 -> 1.71e-7, 57 x 40 centered 1.82e-7 -> 1.71e-7, 200 x
  // 150 centered 2.18e-7 -> 2.02e-7 (packed real transforms: 1.77, 1.75, 2.11e-7), in
  // the same time to 1 %.  The first pass's constants at 8 points per lane would take
  // 6 to 8 % more off the error, and 1 % more time on 64 x 64 images.
  static constexpr float root_c(int e) { return RL == 16 ? kCos64[e / NBL] : kCos32[(e / NBL) * (8 / imin(RL, 8))]; }
  static constexpr float root_s(int e) { return RL == 16 ? kSin64[e / NBL] : kSin32[(e / NBL) * (8 / imin(RL, 8))]; }
  static constexpr float root_cl(int e) { return RL == 16 ? kCos64Lo[e / NBL] : kCos32Lo[(e / NBL) * (8 / imin(RL, 8))]; }
  static constexpr float root_sl(int e) { return RL == 16 ? kSin64Lo[e / NBL] : kSin32Lo[(e / NBL) * (8 / imin(RL, 8))]; }
  static __device__ __forceinline__ float re(float2 z, int e) {
    return e / NBL ? fmaf(z.x, root_c(e), fmaf(-z.y, root_s(e), fmaf(z.x, root_cl(e), -z.y * root_sl(e)))) : z.x;
  }
  static __device__ __forceinline__ float im(float2 z, int e) {
    return e / NBL ? fmaf(z.x, root_s(e), fmaf(z.y, root_c(e), fmaf(z.x, root_sl(e), z.y * root_cl(e)))) : z.y;
  }
};

// ---------------------------------------------------------------------------
// Columns: P points (16 to 128) of the rows of a region, ordinary transforms.
// A wavefront holds 64 / T adjacent columns; their slots in the P rows of the
// region are its own.  Row n of the region holds point n of the column before
// and after; the exchange stores point p in row rho(p), p with its low two
// bits turned by p / E, so that the lanes of a first pass (p = E t + r) and
// of its reads (p = t + T e) fall on different rows modulo 4.
// ---------------------------------------------------------------------------
template <int P, class Row>
struct RaCol {
  static_assert(P == 16 || P == 32 || P == 64 || P == 128, "column length");
  static constexpr int PITCH = Row::PITCH;
  static constexpr int E = P == 128 ? 16 : 8, T = P / E;
  static constexpr int CW = 64 / T;            // columns per wavefront
  static constexpr int R = T, NB = E / R;      // last pass
  static constexpr int LE = ilog2(E);

  static __device__ __forceinline__ void exchange(float2 (&w)[E], int t, float2* col) {
    wave_sync();
    float2* pw[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) pw[q] = col + (E * t + ((q + t) & 3)) * PITCH;
#pragma unroll
    for (int r = 0; r < E; ++r) pw[r & 3][(r & ~3) * PITCH] = w[r];
    wave_sync();
    const float2* pr[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) pr[q] = col + ((t & ~3) + ((t + q) & 3)) * PITCH;
#pragma unroll
    for (int e = 0; e < E; ++e) w[e] = pr[((T * e) + ((T * e) >> LE)) & 3][((T * e) & ~3) * PITCH];
    wave_sync();
  }

  // the last pass's twiddles exp(-2 pi i r (t + T b) / P)
  struct Tw {
    float2 w[NB][R];
    __device__ __forceinline__ void load(int t) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 1; r < R; ++r) w[b][r] = pass_twiddle<E, R, false>((uint32_t)(t + T * b), r);
    }
  };

  // points (bins) t + T e in w[e], in and out
  template <bool INV>
  static __device__ __forceinline__ void run(float2 (&w)[E], int t, float2* col, const Tw& tw) {
    dft<E, INV>(w);
    exchange(w, t, col);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float2 x[R];
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = !r ? w[b] : (INV ? c_mulc(w[b + NB * r], tw.w[b][r]) : c_mul(w[b + NB * r], tw.w[b][r]));
      dft<R, INV>(x);
#pragma unroll
      for (int r = 0; r < R; ++r) w[b + NB * r] = x[r];
    }
  }
};

}  // namespace
}  // namespace hyenand
