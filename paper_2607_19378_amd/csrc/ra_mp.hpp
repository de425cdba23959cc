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
  const void *p, *q;
  void *o, *o2;
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
hipError_t ra_slab_inverse(const RaPass& p, RaOut out, const RaIo& io, int64_t off);
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
template <typename TS>
__device__ __forceinline__ float2 ra_kvalue(const TS* kl, const RaKRow& r, const RaGeom& g, int n) {
  return make_float2(n < g.LL ? ld1(kl + r.row + r.reo + n) : 0.f, n > g.N - g.LL ? ld1(kl + r.row + r.imo + n) : 0.f);
}

// one point of an inverse pass: z at data point o (line base + index)
template <RaOut OUT, typename TS, bool ACT>
__device__ __forceinline__ void ra_store(const TS* p, const TS* q, TS* o1, TS* o2, int64_t o, float z) {
  if constexpr (OUT == RA_Y) st1(o1 + o, Gates<ACT>{}.g1(ld1(p + o)) * z);
  if constexpr (OUT == RA_GX2) st1(o1 + o, ld1(p + o) * z);
  if constexpr (OUT == RA_GU) {
    st1(o1 + o, z * ld1(p + o));
    st1(o2 + o, z * ld1(q + o));
  }
}

}  // namespace
}  // namespace hyenand
