// Multi-pass plan of the non-circular 2D and 3D grids beyond the single-pass
// kernels, of any extents, on right-angle rows (ra_mp.hpp), forward and
// backward:
//
//   rows       u = x1 v (and h = gy x2), k: the rows along the last axis, one
//              wavefront per row group, straight between memory and registers;
//   axis 1     (3D) columns of every plane; where a plane fits in LDS rows and
//              axis 1 are one slab pass (conv_ra_slab.hip);
//   core       columns along axis 0: forward, the pointwise products with the
//              shortcut folded in (U (K + D); backward also conj(K + D) H and
//              conj(U) H), inverse, in place;
//   axis 1, rows  inverse; gates; store.
//
// Only points of the grid are read and written: no embedded copies, no rows or
// planes of zeros, no padding bins.  A ragged grid costs its transform grid's
// columns, not its copies: the embedded plan moved five (backward nine)
// tensors on the padded grid and transformed all of it.
#include <stdlib.h>
#include <string.h>

#include "multipass.hpp"
#include "ra_mp.hpp"

namespace hyenand {

namespace {

// ---------------------------------------------------------------------------
// rows
// ---------------------------------------------------------------------------
constexpr int kRaNT = 256;
constexpr int kRaRowBlocks = 4096;  // a wavefront takes several row groups: its twiddles are loaded once

template <int N>
struct RaRowsCfg {
  using Row = RaRow<N>;
  static constexpr int RW = 64 / Row::T;  // rows per wavefront
  static constexpr int RB = RW * (kRaNT / 64);
};

// KERN: k on the double grid (signal 0); else the gated signals and, w null,
// linear kernels, workgroup by workgroup in turn.  vec: rows come in 16-byte
// accesses through the rows' LDS slots; otherwise point by point.
template <int N, bool KERN, typename TS, bool ACT>
__global__ void __launch_bounds__(kRaNT)
    ra_rows_fwd(RaSignals sg, float2* __restrict__ ws, RaGeom g, int64_t line0, int nl, int64_t per, int kC, int vec,
                ActIn ain, int C) {
  using Cf = RaRowsCfg<N>;
  using Row = typename Cf::Row;
  constexpr int E = Row::E, T = Row::T;
  __shared__ __align__(16) float2 S[Cf::RB * Row::PITCH];  // 16-byte accesses of rows
  const int tid = threadIdx.x, lane = tid & 63;
  const int rr = tid / T, t = tid % T;
  float2* const row = S + rr * Row::PITCH;
  float* const wrow = reinterpret_cast<float*>(S + (tid >> 6) * Cf::RW * Row::PITCH);  // this wavefront's rows
  typename Row::FwdTw tw;
  tw.load(t);
  const unsigned nsig = KERN ? 1 : sg.n, nb = gridDim.x / nsig;
  const unsigned sig = blockIdx.x % nsig;
  const TS* const x = (const TS*)sg.x[sig];
  const TS* const w = KERN ? nullptr : (const TS*)sg.w[sig];
  const bool act_gate = ACT && w;
  const bool vrow = !KERN && vec && !act_gate && (w || !kC);
  const uint32_t n1s = KERN ? 2 * g.L1 - 1 : g.L1;               // rows of a plane
  const uint32_t rows = (KERN ? g.KP : g.L0) * n1s;               // rows of a line
  const uint32_t total = rows * (uint32_t)nl;
  for (uint32_t r0 = blockIdx.x / nsig * Cf::RB; r0 < total; r0 += nb * Cf::RB) {
    const uint32_t r = r0 + rr;
    const bool act = r < total;
    const uint32_t line = act ? r / rows : 0, lr = act ? r - line * rows : 0;
    const uint32_t pl = lr / n1s, i1 = lr - pl * n1s;
    const int64_t gl = line0 + line;
    float2 v[E];
    int64_t dst = sg.off[sig] + line * per;
    if constexpr (KERN) {
      const int d1 = (int)i1 - (g.L1 - 1);
      const RaKRow kr = ra_krow(g, (int)pl - (g.L0 - 1), d1);
      const TS* const kl = x + k_line(gl, kC) * g.kpts;
      float2 z[E];
#pragma unroll
      for (int e = 0; e < E; ++e) z[e] = act ? ra_kvalue(kl, kr, g, t + T * e) : czero();
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = Row::lead(z[e], e);
      dst += ((int64_t)pl * g.P1 + (d1 < 0 ? d1 + g.P1 : d1)) * N;
    } else {
      if (vrow) {
        const uint32_t rw = r0 + (uint32_t)(tid >> 6) * Cf::RW;  // the wavefront's first row
        const int nrows = rw < total ? (int)(total - rw < (uint32_t)Cf::RW ? total - rw : Cf::RW) : 0;
        const int64_t o = line0 * g.data + (int64_t)rw * g.LL;
        ra_rows_in<Row::PITCH, Cf::RW, N>(x + o, w ? w + o : nullptr, nrows, g.LL, wrow, lane);
        const float* const rf = reinterpret_cast<const float*>(row) + t;
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = Row::lead(act && t + T * e < g.LL ? rf[T * e] : 0.f, e);
      } else {
        const int64_t o = (int64_t)lr * g.LL + t;
        const TS* const a = x + (w ? gl : k_line(gl, kC)) * g.data + o;
        const TS* const b = w + (w ? gl * g.data + o : 0);
        const Gates<ACT> G = line_gates<ACT, TS>(ain, gl, C);
        float p[E], q[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
          p[e] = ra_ld_in(a - t, t + T * e, act && t + T * e < g.LL);
          q[e] = 1.f;
        }
        if (w) {
#pragma unroll
          for (int e = 0; e < E; ++e) q[e] = ra_ld_in(b - t, t + T * e, act && t + T * e < g.LL);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
          float u = p[e] * q[e];
          if (act_gate) u = act && t + T * e < g.LL ? G.u1(p[e], q[e], o + T * e) : 0.f;
          v[e] = Row::lead(u, e);
        }
      }
      dst += ((int64_t)pl * g.P1 + i1) * N;
    }
    Row::forward(v, t, row, tw);
    if (act) {
#pragma unroll
      for (int e = 0; e < E; ++e) ws[dst + t + T * e] = v[e];
    }
  }
}

// the inverse of one spectrum (forward) or of z, gu and gk in turn (BWD)
template <int N, bool BWD, typename TS, bool ACT>
__global__ void __launch_bounds__(kRaNT)
    ra_rows_inv(RaIos ios, const float2* __restrict__ ws, RaGeom g, int64_t line0, int nl, int64_t per, int vec) {
  using Cf = RaRowsCfg<N>;
  using Row = typename Cf::Row;
  constexpr int E = Row::E, T = Row::T;
  __shared__ __align__(16) float2 S[Cf::RB * Row::PITCH];  // 16-byte accesses of rows
  const int tid = threadIdx.x, lane = tid & 63;
  const int rr = tid / T, t = tid % T;
  float2* const row = S + rr * Row::PITCH;
  float* const wrow = reinterpret_cast<float*>(S + (tid >> 6) * Cf::RW * Row::PITCH);
  typename Row::InvTw tw;
  tw.load(t);
  const unsigned n = BWD ? ios.n : 1, nb = gridDim.x / n, which = blockIdx.x % n;
  const RaOut out = BWD ? ios.io[which].out : RA_Y;
  const TS* const p = (const TS*)ios.io[which].p;
  const TS* const q = (const TS*)ios.io[which].q;
  TS* const o1 = (TS*)ios.io[which].o;
  TS* const o2 = (TS*)ios.io[which].o2;
  const bool dbl = BWD && out == RA_GK && g.kmode != RA_LINEAR;
  const uint32_t n1s = dbl ? 2 * g.L1 - 1 : g.L1;
  const uint32_t rows = (dbl ? g.KP : g.L0) * n1s;
  const uint32_t total = rows * (uint32_t)nl;
  for (uint32_t r0 = blockIdx.x / n * Cf::RB; r0 < total; r0 += nb * Cf::RB) {
    const uint32_t r = r0 + rr;
    const bool act = r < total;
    const uint32_t line = act ? r / rows : 0, lr = act ? r - line * rows : 0;
    const uint32_t pl = lr / n1s, i1 = lr - pl * n1s;
    const int64_t gl = line0 + line;
    const int d1 = dbl ? (int)i1 - (g.L1 - 1) : (int)i1;
    const float2* const src =
        ws + ios.io[which].off + line * per + ((int64_t)pl * g.P1 + (d1 < 0 ? d1 + g.P1 : d1)) * N + t;
    float2 v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = src[T * e];
    const int64_t o0 = gl * g.data + (int64_t)lr * g.LL;  // the row's first point (not dbl)
    RaGates<E> gt;
    if (!vec && !dbl) gt.load(out, p, q, o0, t, T, g.LL, act);
    Row::inverse(v, t, row, tw);
    if (dbl) {
      if (act) {
        const RaKRow kr = ra_krow(g, (int)pl - (g.L0 - 1), d1);
        TS* const d = o1 + gl * g.kpts + kr.row;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int m = t + T * e;
          if (m < g.LL) st1(d + kr.reo + m, Row::re(v[e], e));
          if (m > g.N - g.LL) st1(d + kr.imo + m, Row::im(v[e], e));
        }
      }
    } else if (vec) {
      float* const rf = reinterpret_cast<float*>(row) + t;
#pragma unroll
      for (int e = 0; e < E; ++e) rf[T * e] = Row::re(v[e], e);
      const uint32_t rw = r0 + (uint32_t)(tid >> 6) * Cf::RW;
      const int nrows = rw < total ? (int)(total - rw < (uint32_t)Cf::RW ? total - rw : Cf::RW) : 0;
      const int64_t o = line0 * g.data + (int64_t)rw * g.LL;
      ra_rows_out<Row::PITCH, Cf::RW, N, ACT>(out, p + o, q + o, o1 + o, o2 + o, nrows, g.LL, wrow, lane);
    } else if (act) {
      gt.template store<ACT>(out, o1, o2, o0, t, T, g.LL, [&](int e) { return Row::re(v[e], e); });
    }
  }
}

// ---------------------------------------------------------------------------
// axis 1 (3D, planes beyond the slab passes): columns of P1 points of every
// plane, in place; rows n < L1 (and, dbl, n > P1 - L1) are data
// ---------------------------------------------------------------------------
template <int P1, bool INV>
__global__ void __launch_bounds__(kTileNT)
    ra_axis1(float2* __restrict__ ws, int N, int planes, int L1, int dbl, int64_t per) {
  using Cf = TileCfg<P1, 1>;
  constexpr int TL = Cf::TL, TLP = Cf::TLP, E = Cf::E, T = Cf::T, NT = kTileNT;
  __shared__ float2 tile[P1 * TLP];
  __shared__ float2 twl[imax(1, PassTw<P1, E>::kCount)];
  PassTw<P1, E>::fill(twl, threadIdx.x, NT);
  const unsigned ntile = (unsigned)((N + TL - 1) / TL);
  const unsigned tl = blockIdx.x % ntile, rest = blockIdx.x / ntile;
  const int64_t line = rest / (unsigned)planes;
  const int pl = (int)(rest % (unsigned)planes);
  const int tid = threadIdx.x;
  const int cc = tid % (NT / T), t = tid / (NT / T);
  const bool act = cc < TL && (int)tl * TL + cc < N;
  float2* const g = ws + line * per + (int64_t)pl * P1 * N + (act ? tl * TL + cc : 0);
  auto data = [&](int n) { return n < L1 || (dbl && n > P1 - L1); };
  float2 w[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = t + T * e;
    w[e] = act && (INV || data(n)) ? g[(int64_t)n * N] : czero();
  }
  static_assert(NT / T >= TL, "one round of columns");
  BlockFFT<P1, E, INV>::run(w, t, ScrS<TLP>{tile + (cc < TL ? cc : 0)}, cc < TL, twl);
  if (act) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int n = t + T * e;
      if (!INV || data(n)) g[(int64_t)n * N] = w[e];
    }
  }
}

// ---------------------------------------------------------------------------
// core: columns of P0 points along axis 0, one workgroup per (line, tile of
// TL adjacent columns of the [planes][ncols] view).  Plane n < L0 of the data;
// of a kernel on the double grid also n > P0 - L0 (displacement n - P0), kept
// in planes n + KP - L0 and n - P0 + KP - L0.
// ---------------------------------------------------------------------------
template <int P0, bool BWD>
struct RaCoreCfg {
  static constexpr int NT = mp_core_nt(P0);
  static constexpr int TL = mp_tl(P0, 1, mp_core_small(P0) ? kTileKB / 2 : kTileKB);
  static constexpr int E = mp_e(P0, TL, NT);
  static constexpr int T = P0 / E;
  static constexpr int TLP = TL + 1;
};

template <int P0, bool DBL, bool BWD>
__global__ void __launch_bounds__(mp_core_nt(P0))
    ra_core(float2* __restrict__ ws, const void* __restrict__ Dp, int dbf16, RaGeom g, int64_t line0, int C,
            int64_t per, float scale) {
  using Cf = RaCoreCfg<P0, BWD>;
  constexpr int TL = Cf::TL, TLP = Cf::TLP, E = Cf::E, T = Cf::T, NT = Cf::NT, PH = P0 / 2;
  __shared__ float2 tile[P0 * TLP];
  __shared__ float2 twl[imax(1, PassTw<P0, E>::kCount)];
  const int ncols = g.P1 * g.N;
  const unsigned ntile = (unsigned)((ncols + TL - 1) / TL);
  const unsigned tl = blockIdx.x % ntile;
  const int64_t line = blockIdx.x / ntile;
  const int tid = threadIdx.x;
  PassTw<P0, E>::fill(twl, tid, NT);
  const int c = (int)((line0 + line) % C);
  const float D = dbf16 ? ld1((const uint16_t*)Dp + c) : ld1((const float*)Dp + c);
  static_assert(NT / T >= TL, "one round of columns");
  const int cc = tid % TL, t = tid / TL;
  const bool act = t < T;
  const int col = (int)tl * TL + cc;
  const bool cv = act && col < ncols;
  float2* const uc = ws + line * per + (cv ? col : 0);
  float2* const hc = uc + g.half;
  float2* const kc = uc + (BWD ? 2 : 1) * g.half;
  const int koff = g.KP - g.L0;
  auto kplane = [&](int n) { return n < g.L0 ? n + koff : (DBL && n > P0 - g.L0 ? n - P0 + koff : -1); };
  const ScrS<TLP> sc{tile + cc};
  float2 wu[E], wk[E], wh[BWD ? E : 1];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = t + T * e;
    wu[e] = n < PH && cv && n < g.L0 ? uc[(int64_t)n * ncols] : czero();
    if constexpr (BWD) wh[e] = n < PH && cv && n < g.L0 ? hc[(int64_t)n * ncols] : czero();
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = t + T * e;
    const int kp = kplane(n);
    wk[e] = (DBL || n < PH) && cv && kp >= 0 ? kc[(int64_t)kp * ncols] : czero();
  }
  BlockFFT<P0, E, false>::run(wu, t, sc, act, twl);
  BlockFFT<P0, E, false>::run(wk, t, sc, act, twl);
  if constexpr (BWD) BlockFFT<P0, E, false>::run(wh, t, sc, act, twl);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const float2 kd = make_float2(wk[e].x + D, wk[e].y);
    if constexpr (BWD) {
      wk[e] = c_scale(c_mulc(wh[e], wu[e]), scale);
      wh[e] = c_scale(c_mulc(wh[e], kd), scale);
    }
    wu[e] = c_scale(c_mul(wu[e], kd), scale);
  }
  BlockFFT<P0, E, true>::run(wu, t, sc, act, twl);
  if constexpr (BWD) {
    BlockFFT<P0, E, true>::run(wh, t, sc, act, twl);
    BlockFFT<P0, E, true>::run(wk, t, sc, act, twl);
  }
  if (cv) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int n = t + T * e;
      if (n < PH && n < g.L0) {
        uc[(int64_t)n * ncols] = wu[e];
        if constexpr (BWD) hc[(int64_t)n * ncols] = wh[e];
      }
      if constexpr (BWD) {
        const int kp = kplane(n);
        if (kp >= 0) kc[(int64_t)kp * ncols] = wk[e];
      }
    }
  }
}

// gD: sums of h u over parts of a line, in a fixed order
constexpr int kHuPts = 8192;
template <typename TS>
__global__ void __launch_bounds__(256)
    ra_hu(const TS* __restrict__ x1, const TS* __restrict__ v, const TS* __restrict__ gy, const TS* __restrict__ x2,
          float* __restrict__ partial, int64_t data, int parts) {
  __shared__ float red[4];
  const int64_t line = blockIdx.x / (unsigned)parts;
  const int part = (int)(blockIdx.x % (unsigned)parts);
  const int64_t step = (data + parts - 1) / parts, i0 = part * step;
  const int64_t end = i0 + step < data ? i0 + step : data;
  float s = 0.f;
  for (int64_t i = i0 + threadIdx.x; i < end; i += 256) {
    const int64_t o = line * data + i;
    s += (ld1(x1 + o) * ld1(v + o)) * (ld1(gy + o) * ld1(x2 + o));
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
RaGeom ra_geom(const FftConvArgs& a) {
  RaGeom g;
  const int last = a.ndim - 1;
  g.L0 = (int)a.L[0];
  g.P0 = (int)a.P[0];
  g.L1 = a.ndim == 3 ? (int)a.L[1] : 1;
  g.P1 = a.ndim == 3 ? (int)a.P[1] : 1;
  g.LL = (int)a.L[last];
  g.N = imax(16, (int)(a.P[last] / 2));
  // (rows of 8 points or less: the slab passes' 32-point rows would not fit in
  // the workspace that is asked for; HYENAND_SLAB=0 keeps to the passes per axis)
  const char* const slab = getenv("HYENAND_SLAB");
  g.slab = a.ndim == 3 && a.P[last] >= 32 && ra_slab_takes(g.P1, imax(32, g.N)) && !(slab && strcmp(slab, "0") == 0);
  if (g.slab) g.N = imax(32, g.N);
  g.kmode = a.periodic ? RA_PERIODIC : (a.centered ? RA_CENTERED : RA_LINEAR);
  g.KP = g.kmode == RA_LINEAR ? g.L0 : 2 * g.L0 - 1;
  g.half = (int64_t)g.L0 * g.P1 * g.N;
  g.halfK = (int64_t)g.KP * g.P1 * g.N;
  g.data = (int64_t)g.L0 * g.L1 * g.LL;
  g.kpts = g.kmode == RA_CENTERED ? (int64_t)(2 * g.L0 - 1) * (2 * g.L1 - 1) * (2 * g.LL - 1) : g.data;
  return g;
}

unsigned row_blocks(int64_t rows, int rb) {
  const int64_t n = (rows + rb - 1) / rb;
  return (unsigned)(n < kRaRowBlocks ? n : kRaRowBlocks);
}

template <typename TS>
int ra_vec(const RaGeom& g) {
  return g.LL % RaVec<TS>::V == 0;
}

template <int N, typename TS>
hipError_t rows_signals(const RaPass& p, const RaSignals& sg, bool act) {
  const FftConvArgs& a = *p.a;
  const dim3 grid(row_blocks((int64_t)p.nl * p.g.L0 * p.g.L1, RaRowsCfg<N>::RB) * sg.n);
  if (act)
    hipLaunchKernelGGL((ra_rows_fwd<N, false, TS, true>), grid, dim3(kRaNT), 0, p.s, sg, p.ws, p.g, p.line0, p.nl,
                       p.per, a.kC, ra_vec<TS>(p.g), a.act_in, (int)a.C);
  else
    hipLaunchKernelGGL((ra_rows_fwd<N, false, TS, false>), grid, dim3(kRaNT), 0, p.s, sg, p.ws, p.g, p.line0, p.nl,
                       p.per, a.kC, ra_vec<TS>(p.g), a.act_in, (int)a.C);
  return hipGetLastError();
}
template <int N, typename TS>
hipError_t rows_kernel(const RaPass& p, int64_t off) {
  const FftConvArgs& a = *p.a;
  const dim3 grid(row_blocks((int64_t)p.nl * p.g.KP * (2 * p.g.L1 - 1), RaRowsCfg<N>::RB));
  const RaSignals sg{{a.k}, {nullptr}, {off}, 1};
  hipLaunchKernelGGL((ra_rows_fwd<N, true, TS, false>), grid, dim3(kRaNT), 0, p.s, sg, p.ws, p.g, p.line0, p.nl,
                     p.per, a.kC, 0, a.act_in, (int)a.C);
  return hipGetLastError();
}
template <int N, typename TS>
hipError_t rows_inverse(const RaPass& p, const RaIos& ios) {
  const int64_t rows = (int64_t)p.nl * p.g.KP * (p.g.kmode == RA_LINEAR ? p.g.L1 : 2 * p.g.L1 - 1);  // the most of any
  const bool bwd = ios.io[0].out != RA_Y;
  const dim3 grid(row_blocks(bwd ? rows : (int64_t)p.nl * p.g.L0 * p.g.L1, RaRowsCfg<N>::RB) * ios.n);
#define HY_INV(BWD, ACT)                                                                                       \
  hipLaunchKernelGGL((ra_rows_inv<N, BWD, TS, ACT>), grid, dim3(kRaNT), 0, p.s, ios, p.ws, p.g, p.line0, p.nl, \
                     p.per, ra_vec<TS>(p.g))
  if (bwd) HY_INV(true, false);
  else if (p.a->act) HY_INV(false, true);
  else HY_INV(false, false);
#undef HY_INV
  return hipGetLastError();
}

#define HY_N_SWITCH(FN, ...)                                                                     \
  switch (p.g.N) {                                                                               \
    case 16: return p.a->bf16 ? FN<16, uint16_t>(__VA_ARGS__) : FN<16, float>(__VA_ARGS__);      \
    case 32: return p.a->bf16 ? FN<32, uint16_t>(__VA_ARGS__) : FN<32, float>(__VA_ARGS__);      \
    case 64: return p.a->bf16 ? FN<64, uint16_t>(__VA_ARGS__) : FN<64, float>(__VA_ARGS__);      \
    case 128: return p.a->bf16 ? FN<128, uint16_t>(__VA_ARGS__) : FN<128, float>(__VA_ARGS__);   \
    case 256: return p.a->bf16 ? FN<256, uint16_t>(__VA_ARGS__) : FN<256, float>(__VA_ARGS__);   \
    case 512: return p.a->bf16 ? FN<512, uint16_t>(__VA_ARGS__) : FN<512, float>(__VA_ARGS__);   \
    default: return hipErrorInvalidValue;                                                        \
  }
hipError_t d_rows_signals(const RaPass& p, const RaSignals& sg, bool act) { HY_N_SWITCH(rows_signals, p, sg, act) }
hipError_t d_rows_kernel(const RaPass& p, int64_t off) { HY_N_SWITCH(rows_kernel, p, off) }
hipError_t d_rows_inverse(const RaPass& p, const RaIos& ios) { HY_N_SWITCH(rows_inverse, p, ios) }

template <int P1>
hipError_t axis1(const RaPass& p, bool inv, int planes, bool dbl, int64_t off) {
  constexpr int TL = TileCfg<P1, 1>::TL;
  const dim3 grid((unsigned)((int64_t)p.nl * planes * ((p.g.N + TL - 1) / TL)));
  if (inv)
    hipLaunchKernelGGL((ra_axis1<P1, true>), grid, dim3(kTileNT), 0, p.s, p.ws + off, p.g.N, planes, p.g.L1, (int)dbl, p.per);
  else
    hipLaunchKernelGGL((ra_axis1<P1, false>), grid, dim3(kTileNT), 0, p.s, p.ws + off, p.g.N, planes, p.g.L1, (int)dbl, p.per);
  return hipGetLastError();
}
template <int P0>
hipError_t core(const RaPass& p, bool bwd) {
  constexpr int TL = RaCoreCfg<P0, false>::TL, NT = RaCoreCfg<P0, false>::NT;
  const FftConvArgs& a = *p.a;
  const int ncols = p.g.P1 * p.g.N;
  const dim3 grid((unsigned)((int64_t)p.nl * ((ncols + TL - 1) / TL)));
  const float scale = (float)(1.0 / ((double)p.g.P0 * (double)p.g.P1 * (double)p.g.N));
#define HY_CORE(DBL, BWD)                                                                                        \
  hipLaunchKernelGGL((ra_core<P0, DBL, BWD>), grid, dim3(NT), 0, p.s, p.ws, a.D, (int)a.bf16, p.g, p.line0, (int)a.C, \
                     p.per, scale)
  if (p.g.kmode != RA_LINEAR) {
    if (bwd) HY_CORE(true, true);
    else HY_CORE(true, false);
  } else {
    if (bwd) HY_CORE(false, true);
    else HY_CORE(false, false);
  }
#undef HY_CORE
  return hipGetLastError();
}
#define HY_P_SWITCH(P, FN, ...)                   \
  switch (P) {                                    \
    case 2: return FN<2>(__VA_ARGS__);            \
    case 4: return FN<4>(__VA_ARGS__);            \
    case 8: return FN<8>(__VA_ARGS__);            \
    case 16: return FN<16>(__VA_ARGS__);          \
    case 32: return FN<32>(__VA_ARGS__);          \
    case 64: return FN<64>(__VA_ARGS__);          \
    case 128: return FN<128>(__VA_ARGS__);        \
    case 256: return FN<256>(__VA_ARGS__);        \
    case 512: return FN<512>(__VA_ARGS__);        \
    case 1024: return FN<1024>(__VA_ARGS__);      \
    default: return hipErrorInvalidValue;         \
  }
hipError_t d_axis1(const RaPass& p, bool inv, int planes, bool dbl, int64_t off) {
  HY_P_SWITCH(p.g.P1, axis1, p, inv, planes, dbl, off)
}
hipError_t d_core(const RaPass& p, bool bwd) { HY_P_SWITCH(p.g.P0, core, p, bwd) }

// forward transforms of axes 1 and 2 of the signals and of k (at ws + koff; a
// linear k is one signal more)
hipError_t forward_axes(const RaPass& p, RaSignals sg, bool act, int64_t koff) {
  const bool lin = p.g.kmode == RA_LINEAR;
  if (lin) {
    sg.x[sg.n] = p.a->k;
    sg.w[sg.n] = nullptr;
    sg.off[sg.n++] = koff;
  }
  hipError_t e = hipSuccess;
  if (p.g.slab) {
    e = ra_slab_signals(p, sg, act);
    return e == hipSuccess && !lin ? ra_slab_kernel(p, koff) : e;
  }
  e = d_rows_signals(p, sg, act);
  for (int i = 0; i < sg.n && e == hipSuccess && p.g.P1 > 1; ++i) e = d_axis1(p, false, p.g.L0, false, sg.off[i]);
  if (!lin) {
    if (e == hipSuccess) e = d_rows_kernel(p, koff);
    if (e == hipSuccess && p.g.P1 > 1) e = d_axis1(p, false, p.g.KP, true, koff);
  }
  return e;
}
hipError_t inverse_axes(const RaPass& p, const RaIos& ios) {
  hipError_t e = hipSuccess;
  for (int i = 0; i < ios.n && e == hipSuccess; ++i) {
    const bool dbl = ios.io[i].out == RA_GK && p.g.kmode != RA_LINEAR;
    if (p.g.slab) e = ra_slab_inverse(p, ios.io[i]);
    else if (p.g.P1 > 1) e = d_axis1(p, true, dbl ? p.g.KP : p.g.L0, dbl, ios.io[i].off);
  }
  return e == hipSuccess && !p.g.slab ? d_rows_inverse(p, ios) : e;
}

int64_t line_points(const FftConvArgs& a) {
  int64_t n = 1;
  for (int d = 0; d < a.ndim; ++d) n *= a.L[d];
  return n;
}

RaPass make_pass(const FftConvArgs& a, const RaGeom& g, bool bwd, int64_t line0, int64_t nl, void* ws, hipStream_t s) {
  RaPass p;
  p.a = &a;
  p.g = g;
  p.ws = (float2*)ws;
  p.per = (bwd ? 2 : 1) * g.half + g.halfK;
  p.line0 = line0;
  p.nl = (int)nl;
  p.s = s;
  return p;
}

}  // namespace

bool ra_mp_supported(const FftConvArgs& a) {
  if ((a.ndim != 2 && a.ndim != 3) || a.circular) return false;
  for (int d = 0; d < a.ndim; ++d)
    if (a.L[d] < 2 || a.P[d] < 2 || a.P[d] > kMaxP) return false;
  return true;
}

size_t ra_mp_bytes_per_line(const FftConvArgs& a, bool backward) {
  const RaGeom g = ra_geom(a);
  return (size_t)((backward ? 2 : 1) * g.half + g.halfK) * sizeof(float2);
}

hipError_t launch_ra_mp(const FftConvArgs& a, int64_t line0, int64_t nl, void* ws, hipStream_t s) {
  if (!ra_mp_supported(a) || nl < 1 || line0 < 0 || line0 + nl > a.lines) return hipErrorInvalidValue;
  const RaPass p = make_pass(a, ra_geom(a), false, line0, nl, ws, s);
  hipError_t e;
  if ((e = forward_axes(p, RaSignals{{a.x1}, {a.v}, {0}, 1}, a.act, p.g.half)) != hipSuccess) return e;
  if ((e = d_core(p, false)) != hipSuccess) return e;
  return inverse_axes(p, RaIos{{{RA_Y, a.x2, nullptr, a.y, nullptr, 0}}, 1});
}

// the periodic kernel's gradient gathers two displacements per axis, which
// these passes do not
bool ra_mp_backward_supported(const FftConvArgs& a) { return ra_mp_supported(a) && !a.periodic; }

hipError_t launch_ra_mp_backward(const FftConvBwdArgs& b, int64_t line0, int64_t nl, void* ws, hipStream_t s) {
  const FftConvArgs& a = b.f;
  if (!ra_mp_backward_supported(a) || nl < 1 || line0 < 0 || line0 + nl > a.lines) return hipErrorInvalidValue;
  const RaPass p = make_pass(a, ra_geom(a), true, line0, nl, ws, s);
  const int64_t h = p.g.half;
  hipError_t e;
  if ((e = forward_axes(p, RaSignals{{a.x1, b.gy}, {a.v, a.x2}, {0, h}, 2}, false, 2 * h)) != hipSuccess) return e;
  if ((e = d_core(p, true)) != hipSuccess) return e;
  return inverse_axes(p, RaIos{{{RA_GX2, b.gy, nullptr, b.gx2, nullptr, 0},
                                {RA_GU, a.v, a.x1, b.gx1, b.gv, h},
                                {RA_GK, nullptr, nullptr, b.gk, nullptr, 2 * h}}, 3});
}

int64_t ra_mp_partials_per_line(const FftConvArgs& a) {
  const int64_t n = (line_points(a) + kHuPts - 1) / kHuPts;
  return n < 64 ? n : 64;
}

hipError_t launch_ra_mp_hu(const FftConvBwdArgs& b, float* partial, hipStream_t s) {
  const FftConvArgs& a = b.f;
  const int parts = (int)ra_mp_partials_per_line(a);
  const int64_t data = line_points(a);
  const dim3 grid((unsigned)(a.lines * parts));
  if (a.bf16)
    hipLaunchKernelGGL((ra_hu<uint16_t>), grid, dim3(256), 0, s, (const uint16_t*)a.x1, (const uint16_t*)a.v,
                       (const uint16_t*)b.gy, (const uint16_t*)a.x2, partial, data, parts);
  else
    hipLaunchKernelGGL((ra_hu<float>), grid, dim3(256), 0, s, (const float*)a.x1, (const float*)a.v, (const float*)b.gy,
                       (const float*)a.x2, partial, data, parts);
  return hipGetLastError();
}

}  // namespace hyenand
