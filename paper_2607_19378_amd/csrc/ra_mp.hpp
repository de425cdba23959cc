// Geometry shared by the multi-pass kernels on right-angle rows
// (conv_ra_slab.hip, conv_ra_mp.hip): non-circular 2D and 3D grids of any
// extents, forward and backward.
//
// Rows (the last axis) are transformed in N complex points, N a power of two
// >= LL; axes 0 and 1 as zero-padded transforms of P0 and P1 points, powers of
// two >= 2 L - 1.  A spectrum is [planes][P1][N], N a multiple of 16 complex
// values: every row is whole cache lines, without padding.  Only points inside
// the L_d are read and only they are written back; the planes of a spectrum
// are the L0 that can be nonzero, or the 2 L0 - 1 displacements of a kernel on
// the double grid (centered, or a circular kernel repeated over the
// displacements -(L - 1) .. L - 1).
#pragma once

#include "ra_device.hpp"

namespace hyenand {

enum RaKernel { RA_LINEAR = 0, RA_CENTERED = 1, RA_PERIODIC = 2 };

struct RaGeom {
  int L0, P0, L1, P1, LL, N;  // L1 = P1 = 1 in 2D
  int kmode;                  // RaKernel
  int KP;                     // planes of K: L0 (linear) or 2 L0 - 1
  bool slab;                  // 3D: axis-1 and row transforms of a plane in one pass
  int64_t half, halfK;        // complex entries of U (and H) and of K per line
  int64_t data, kpts;         // points of a line of the tensors and of k
};

// which gradients an inverse pass writes
enum RaOut { RA_Y = 0, RA_GX2 = 1, RA_GU = 2, RA_GK = 3 };

// pointers of one pass; the meaning per output: RA_Y p = x2, o = y; RA_GX2
// p = gy, o = gx2; RA_GU p = v, q = x1, o = gx1, o2 = gv; RA_GK o = gk
struct RaIo {
  RaOut out;
  const void *p, *q;
  void *o, *o2;
  int64_t off;  // of the spectrum
};
struct RaIos {
  RaIo io[3];
  int n;
};

struct RaPass {
  const FftConvArgs* a;
  RaGeom g;
  float2* ws;      // first line's spectra
  int64_t per;     // complex entries between lines
  int64_t line0;
  int nl;
  hipStream_t s;
};

// a signal of a plane: gate(x, w), or x alone (w null: a linear kernel), into
// the spectrum at ws + off
struct RaSignals {
  const void* x[3];
  const void* w[3];
  int64_t off[3];
  int n;
};
hipError_t ra_slab_signals(const RaPass& p, const RaSignals& sg, bool act);
hipError_t ra_slab_kernel(const RaPass& p, int64_t off);  // k on the double grid
hipError_t ra_slab_inverse(const RaPass& p, const RaIo& io);
bool ra_slab_takes(int P1, int N);

namespace {

// row of a kernel on the double grid: point n of the complex line is
// re + i im, re = p[reo + n] (n < LL), im = p[imo + n] (n > N - LL, displacement n - N)
struct RaKRow {
  int64_t row;  // offset of the row, or -1 (no displacement)
  int reo, imo;
};
// d0, d1: displacements along axes 0 and 1
__device__ __forceinline__ RaKRow ra_krow(const RaGeom& g, int d0, int d1) {
  RaKRow r;
  if (g.kmode == RA_CENTERED) {
    r.row = ((int64_t)(d0 + g.L0 - 1) * (2 * g.L1 - 1) + (d1 + g.L1 - 1)) * (2 * g.LL - 1);
    r.reo = g.LL - 1;
    r.imo = g.LL - 1 - g.N;
  } else {  // periodic
    r.row = ((int64_t)(d0 < 0 ? d0 + g.L0 : d0) * g.L1 + (d1 < 0 ? d1 + g.L1 : d1)) * g.LL;
    r.reo = 0;
    r.imo = g.LL - g.N;
  }
  return r;
}
// p[i], or 0 where not in (p[0] is read instead).
template <typename TS>
__device__ __forceinline__ float ra_ld_sel(const TS* p, int64_t i, bool in) {
  const float v = ld1(p + (in ? i : 0));
  return in ? v : 0.f;
}
// The same where many lanes are out (a kernel row fills part of its line):
// fp32 loads under their condition (rows of 200 x 150 kernels 140 -> 78 us).
// The compiler would widen a conditional bf16 load under its condition, so
// each would be waited for before the next is issued.
template <typename TS>
__device__ __forceinline__ float ra_ld_in(const TS* p, int64_t i, bool in) {
  if constexpr (sizeof(TS) == 4) return in ? ld1(p + i) : 0.f;
  return ra_ld_sel(p, i, in);
}
template <typename TS>
__device__ __forceinline__ float2 ra_kvalue(const TS* kl, const RaKRow& r, const RaGeom& g, int n) {
  const TS* const p = kl + r.row + r.reo;
  return make_float2(ra_ld_in(p, n, n < g.LL), ra_ld_in(p, n + r.imo - r.reo, n > g.N - g.LL));
}

// Rows between memory and LDS in 16-byte accesses.  A wavefront's rows are
// consecutive, so their nrows LL values are one run; LL has to be a multiple of
// the V values of an access (the tensors are 16-byte aligned, so the run is
// too).  Row i's values sit at s + i * 2 PITCH (floats), where the row's
// transform has its exchange slots.
template <typename TS>
struct RaVec {
  static constexpr int V = 16 / sizeof(TS);
};
__device__ __forceinline__ void ra_ld(const float* p, float (&v)[4]) {
  const float4 a = ld4(p);
  v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w;
}
__device__ __forceinline__ void ra_ld(const uint16_t* p, float (&v)[8]) {
  const uint4 a = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ void ra_st(float* p, const float (&v)[4]) { st4(p, make_float4(v[0], v[1], v[2], v[3])); }
__device__ __forceinline__ void ra_st(uint16_t* p, const float (&v)[8]) {
  *reinterpret_cast<uint4*>(p) =
      make_uint4(bf16_pack(v[0], v[1]), bf16_pack(v[2], v[3]), bf16_pack(v[4], v[5]), bf16_pack(v[6], v[7]));
}
// s and the rows in it are 16-byte aligned (the callers' arrays are declared so).
// values x w (w null: x) of nrows rows from x and w on
template <int PITCH, int RW, int NMAX, typename TS>
__device__ __forceinline__ void ra_rows_in(const TS* x, const TS* w, int nrows, int LL, float* s, int lane) {
  static_assert(PITCH * sizeof(float2) % 16 == 0, "rows at 16-byte offsets");
  constexpr int V = RaVec<TS>::V, ITER = (RW * NMAX / V + 63) / 64;
  const unsigned vr = (unsigned)LL / V, total = (unsigned)nrows * vr;
  wave_sync();
#pragma unroll
  for (int j = 0; j < ITER; ++j) {
    const unsigned i = (unsigned)lane + 64u * j;
    if (i < total) {
      float a[V], b[V];
      ra_ld(x + (size_t)i * V, a);
      if (w) {
        ra_ld(w + (size_t)i * V, b);
#pragma unroll
        for (int k = 0; k < V; ++k) a[k] *= b[k];
      }
      const unsigned r = i / vr;
      float* const d = s + r * (2 * PITCH) + (i - r * vr) * V;
#pragma unroll
      for (int k = 0; k < V; k += 4) *reinterpret_cast<float4*>(d + k) = make_float4(a[k], a[k + 1], a[k + 2], a[k + 3]);
    }
  }
  wave_sync();
}
// o = g(p) value (RA_Y: the outer gate), p value (RA_GX2), the values (RA_GK),
// or o = p value and o2 = q value (RA_GU), for nrows rows from those pointers on
template <int PITCH, int RW, int NMAX, bool ACT, typename TS>
__device__ __forceinline__ void ra_rows_out(RaOut out, const TS* p, const TS* q, TS* o, TS* o2, int nrows, int LL,
                                            const float* s, int lane) {
  static_assert(PITCH * sizeof(float2) % 16 == 0, "rows at 16-byte offsets");
  constexpr int V = RaVec<TS>::V, ITER = (RW * NMAX / V + 63) / 64;
  const unsigned vr = (unsigned)LL / V, total = (unsigned)nrows * vr;
  wave_sync();
#pragma unroll
  for (int j = 0; j < ITER; ++j) {
    const unsigned i = (unsigned)lane + 64u * j;
    if (i < total) {
      const size_t at = (size_t)i * V;
      float a[V], b[V], z[V];
      if (out != RA_GK) ra_ld(p + at, a);
      if (out == RA_GU) ra_ld(q + at, b);
      const unsigned r = i / vr;
      const float* const d = s + r * (2 * PITCH) + (i - r * vr) * V;
#pragma unroll
      for (int k = 0; k < V; k += 4) {
        const float4 f = *reinterpret_cast<const float4*>(d + k);
        z[k] = f.x, z[k + 1] = f.y, z[k + 2] = f.z, z[k + 3] = f.w;
      }
      if (out == RA_GU) {
#pragma unroll
        for (int k = 0; k < V; ++k) b[k] *= z[k];
        ra_st(o2 + at, b);
      }
      if (out != RA_GK) {
#pragma unroll
        for (int k = 0; k < V; ++k) z[k] *= out == RA_Y ? Gates<ACT>{}.g1(a[k]) : a[k];
      }
      ra_st(o + at, z);
    }
  }
  wave_sync();
}

// The gates of a lane's points i + step e, fetched before the inverse
// transform, and the points' store after it (n < LL).
template <int E>
struct RaGates {
  float p[E], q[E];
  template <typename TS>
  __device__ __forceinline__ void load(RaOut out, const TS* pp, const TS* qq, int64_t base, int64_t n0, int64_t step,
                                       int64_t L, bool act) {
    if (out == RA_GK) return;
#pragma unroll
    for (int e = 0; e < E; ++e) p[e] = ra_ld_in(pp + base, n0 + step * e, act && n0 + step * e < L);
    if (out == RA_GU) {
#pragma unroll
      for (int e = 0; e < E; ++e) q[e] = ra_ld_in(qq + base, n0 + step * e, act && n0 + step * e < L);
    }
  }
  template <bool ACT, typename TS, class Re>
  __device__ __forceinline__ void store(RaOut out, TS* o1, TS* o2, int64_t base, int64_t n0, int64_t step, int64_t L,
                                        const Re& re) const {
    TS* const a = o1 + base + n0;
    if (out == RA_GU) {
      TS* const b = o2 + base + n0;
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (n0 + step * e < L) {
          const float z = re(e);
          st1(a + step * e, z * p[e]);
          st1(b + step * e, z * q[e]);
        }
    } else if (out == RA_GK) {
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (n0 + step * e < L) st1(a + step * e, re(e));
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (n0 + step * e < L) st1(a + step * e, (out == RA_Y ? Gates<ACT>{}.g1(p[e]) : p[e]) * re(e));
    }
  }
};

}  // namespace
}  // namespace hyenand
