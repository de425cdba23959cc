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
// (64 banks of 4 bytes: 64 lanes of 8 bytes, two lanes per bank pair).
#pragma once

#include "kernels.hpp"

namespace hyenand {
namespace {

// Orders this wavefront's LDS accesses for the compiler; the hardware
// performs them in order.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A lane number the compiler cannot see through: twiddles indexed by it are
// loaded where they are used, not hoisted out of a loop over images into
// registers that live through all of it.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// ---------------------------------------------------------------------------
// Rows: N points (16, 32 or 64), 8 per lane.  Point p of a row sits in slot
// p + p / 8 of a pitch of 9 N / 8 slots: lane (row l, t) writes slots 9 t + r
// of the first pass and reads t + T e, and both spread over all banks.
// ---------------------------------------------------------------------------
template <int N>
struct RaRow {
  static_assert(N == 16 || N == 32 || N == 64, "row length");
  static constexpr int E = 8, T = N / E;       // lanes per row
  static constexpr int PITCH = N + N / 8;
  static constexpr int R = N / E, NB = E / R;  // last pass: NB butterflies of radix R per lane
  static constexpr int kRoot = 32 / (4 * R);   // exp(2 pi i r / (4 R)) in 32nds of a turn
  // slot of point t + T e, less t
  static constexpr int off(int e) { return T * e + (T * e) / 8; }

  // exp(-2 pi i r (j + 1/4) / N), j = t + T b the butterfly, r = 1 .. R - 1
  struct FwdTw {
    float2 w[NB][R];
    __device__ __forceinline__ void load(int t) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 1; r < R; ++r) w[b][r] = twiddle<ilog2(4 * N), false>((uint32_t)((4 * (t + T * b) + 1) * r));
    }
  };
  // exp(+2 pi i j (r + 1/4) / N), r = 0 .. R - 1
  struct InvTw {
    float2 w[NB][R];
    __device__ __forceinline__ void load(int t) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < R; ++r) w[b][r] = twiddle<ilog2(4 * N), true>((uint32_t)((t + T * b) * (4 * r + 1)));
    }
  };

  // the first pass's constants exp(-2 pi i e / 32) on a real or complex input
  static __device__ __forceinline__ float2 lead(float x, int e) { return make_float2(x * kCos32[e], -x * kSin32[e]); }
  static __device__ __forceinline__ float2 lead(float2 x, int e) { return mul_root<32, false>(x, e); }

  static __device__ __forceinline__ void exchange(float2 (&w)[E], int t, float2* row) {
    wave_sync();
    float2* const pw = row + 9 * t;
#pragma unroll
    for (int r = 0; r < E; ++r) pw[r] = w[r];
    wave_sync();
    const float2* const pr = row + t;
#pragma unroll
    for (int e = 0; e < E; ++e) w[e] = pr[off(e)];
    wave_sync();
  }

  // w[e] = lead(point t + T e); leaves bin t + T e in w[e]
  static __device__ __forceinline__ void forward(float2 (&w)[E], int t, float2* row, const FwdTw& tw) {
    dft<E, false>(w);
    exchange(w, t, row);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float2 x[R];
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = r ? c_mul(w[b + NB * r], tw.w[b][r]) : w[b];
      dft<R, false>(x);
#pragma unroll
      for (int r = 0; r < R; ++r) w[b + NB * r] = x[r];
    }
  }
  // bin t + T e in w[e]; leaves point t + T e up to exp(2 pi i r / (4 R)),
  // r = e / NB, which re() and im() apply
  static __device__ __forceinline__ void inverse(float2 (&w)[E], int t, float2* row, const InvTw& tw) {
    dft<E, true>(w);
    exchange(w, t, row);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float2 x[R];
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = c_mul(w[b + NB * r], tw.w[b][r]);
      dft<R, true>(x);
#pragma unroll
      for (int r = 0; r < R; ++r) w[b + NB * r] = x[r];
    }
  }
  static __device__ __forceinline__ float re(float2 z, int e) {
    const int j = (e / NB) * kRoot;
    return j ? fmaf(z.x, kCos32[j], -z.y * kSin32[j]) : z.x;
  }
  static __device__ __forceinline__ float im(float2 z, int e) {
    const int j = (e / NB) * kRoot;
    return j ? fmaf(z.x, kSin32[j], z.y * kCos32[j]) : z.y;
  }
};

// ---------------------------------------------------------------------------
// Columns: P points (32, 64 or 128) along axis 0, ordinary transforms.  A
// wavefront holds 64 / T adjacent columns; their slots in the P rows of the
// region are its own.  Row n of the region holds point n of the column before
// and after; the exchange stores point p in row rho(p), p with its low two
// bits turned by p / E, so that the lanes of a first pass (p = E t + r) and
// of its reads (p = t + T e) fall on different rows modulo 4.
// ---------------------------------------------------------------------------
template <int P, int PITCH>
struct RaCol {
  static_assert(P == 32 || P == 64 || P == 128, "column length");
  static constexpr int E = P == 128 ? 16 : 8, T = P / E;
  static constexpr int CW = 64 / T;            // columns per wavefront
  static constexpr int R = T, NB = E / R;      // last pass
  static constexpr int LE = ilog2(E);

  static __device__ __forceinline__ int slot(int col) { return col + (col >> 3); }

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
    for (int e = 0; e < E; ++e) w[e] = pr[((T * e) >> LE) & 3][T * e * PITCH];
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
