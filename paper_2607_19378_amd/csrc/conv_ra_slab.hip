// Slab passes of the non-circular 3D plan on right-angle rows (ra_mp.hpp):
// the row and axis-1 transforms of a plane in one pass, the plane in LDS.
//
// Axis 1 has P1 = 2 PH points of which L1 <= PH can be nonzero: the even bins
// are the length-PH transform of x[n] (+ x[n + PH]), the odd ones that of the
// same times exp(-2 pi i n / P1) (- instead of +), so the region holds PH rows
// and both transforms run in place.  A kernel on the double grid has rows in
// both halves; they take the region one after the other.
//
// These passes move a plane's spectrum between LDS and memory once each; one
// wavefront holds whole rows, then whole columns, with a barrier where rows
// turn into columns.
#include "ra_mp.hpp"

namespace hyenand {

namespace {

// Rows beyond 64 points enter as two foldings of 64, a workgroup each: the
// region then leaves room for a second workgroup on the CU (unfolded, 1024
// lanes and 139 KB: 34.8 us for the 128 planes of a signal of 128^3 points).
// Their bins are stored in that order, bin f in column (f mod 2) 64 + f / 2.
// The inverse sums over all bins, so it runs unfolded (two foldings in turn
// spilled 392 bytes).
constexpr int slab_foldings(int N) { return N > 64 ? 2 : 1; }

template <int P1, int N, int FOLD>
struct SlabRa {
  static constexpr int F = FOLD;
  using Row = RaRow<N / F, F>;
  static constexpr int NC = N / F;         // columns of a workgroup
  static constexpr int PH = P1 / 2;
  using Col = RaCol<PH, Row>;
  static constexpr int NT = NC * Col::T;   // one round of columns
  static constexpr int RPR = NT / Row::T;  // rows per round
  static constexpr int NR = imax(1, PH / RPR);
  static_assert(NT >= 64 && NT <= 1024, "workgroup");
};
template <int P1, int N>
using SlabFwd = SlabRa<P1, N, slab_foldings(N)>;
template <int P1, int N>
using SlabInv = SlabRa<P1, N, 1>;

// A plane's P1 x N bins in the workspace: the core transforms every (axis-1
// bin, column) alike, so the order is free.  [column / CW][parity of the axis-1
// bin][bin / 2][column mod CW], CW the columns of a wavefront: a wavefront's
// loads and stores are 512-byte runs (bins in rows of N: 64-byte ones).
template <int P1, int CW>
__device__ __forceinline__ int slab_bin(int col) {
  return col / CW * (P1 * CW) + col % CW;
}

// Wavefronts per SIMD asked for (the VGPR cap: 6 is 80, 4 is 128).  Planes of up to
// 128 axis-1 bins fit several times in the LDS of a CU, and 6 wavefronts of them hide
// more latency than 4.  Not where rows have 65 to 128 points, in the inverse and in a
// kernel's planes (FULL): their points (two foldings or both halves) do not fit in 80
// VGPRs, and 7 to 66 spilled (at 128 at most 5, in gk).  32 volumes of 64 x 64 x 128,
// centered, bf16: 6 for all 960 us, 4 in those inverses 875, in both 737; backward
// 1740, 1581, 1415.  P1 = 256 needs 1024 lanes, so 4, and spills 2 to 9.
template <int P1, int N>
constexpr int slab_waves(bool many) {
  return P1 <= 128 && !(many && N > 64) ? 6 : 4;
}

// FULL: a kernel on the double grid (signal 0), planes of 2 L0 - 1
// displacements; else the gated signals and, w null, linear kernels.
// Workgroups: (line, plane, signal, folding).
template <int P1, int N, bool FULL, typename TS, bool ACT>
__global__ void __launch_bounds__((SlabFwd<P1, N>::NT)) __attribute__((amdgpu_waves_per_eu(slab_waves<P1, N>(FULL))))
    ra_slab_fwd(RaSignals sg, float2* __restrict__ ws, RaGeom g, int64_t line0, int64_t per, int kC, int vec, ActIn ain,
                int C) {
  using S_ = SlabFwd<P1, N>;
  using Row = typename S_::Row;
  using Col = typename S_::Col;
  constexpr int F = S_::F, PH = S_::PH, PITCH = Row::PITCH, TR = Row::T, ER = Row::E, E = Col::E, TC = Col::T;
  constexpr int RPR = S_::RPR, NC = S_::NC;
  __shared__ __align__(16) float2 S[PH * PITCH];  // 16-byte accesses of rows
  const unsigned planes = FULL ? g.KP : g.L0;
  unsigned bid = blockIdx.x;
  const int p = F > 1 ? (int)(bid % F) : 0;
  bid /= F;
  const int sig = FULL ? 0 : (int)(bid % (unsigned)sg.n);
  if (!FULL) bid /= (unsigned)sg.n;
  const int pl = (int)(bid % planes);
  const int64_t line = bid / planes, gl = line0 + line;
  const int tid = threadIdx.x;
  const int rr = tid / TR, tr = tid % TR;
  const int lane = tid & 63;
  const int col = (tid >> 6) * Col::CW + lane % Col::CW, tc = lane / Col::CW;
  float2* const cp = S + Row::slot(col);
  typename Row::FwdTw ftw;
  ftw.load(tr, p);

  const TS* const w0 = (const TS*)sg.w[sig];
  const bool gated = !FULL && w0 != nullptr;
  const TS* const kl = (const TS*)sg.x[sig] + (gated ? gl * g.data : k_line(gl, kC) * g.kpts);
  const TS* const wl = gated ? w0 + gl * g.data : nullptr;
  const Gates<ACT> G = line_gates<ACT, TS>(ain, gl, C);
  constexpr int RW = 64 / TR;  // rows of a wavefront
  const bool vrow = !FULL && vec && !(ACT && gated);
  // the rows of one half of axis 1: n1 = r, or (FULL) displacement r - PH
  auto rows = [&](int hf) {
#pragma unroll
    for (int q = 0; q < S_::NR; ++q) {
      const int r = q * RPR + rr;
      const int d1 = hf ? r - PH : r;
      if (vrow) {
        const int rw = q * RPR + (tid >> 6) * RW;  // the wavefront's first row
        const int64_t o = ((int64_t)pl * g.L1 + rw) * g.LL;
        ra_rows_in<PITCH, RW, N>(kl + o, gated ? wl + o : nullptr, imax(0, imin(RW, g.L1 - rw)), g.LL,
                                 reinterpret_cast<float*>(S + rw * PITCH), lane);
      }
      if (r < PH && (hf ? d1 > -g.L1 : r < g.L1)) {
        float2 v[ER];
        if constexpr (FULL) {
          const RaKRow kr = ra_krow(g, pl - (g.L0 - 1), d1);
          float2 z[F][ER];
#pragma unroll
          for (int f = 0; f < F; ++f)
#pragma unroll
            for (int e = 0; e < ER; ++e) z[f][e] = ra_kvalue(kl, kr, g, tr + TR * e + f * NC);
#pragma unroll
          for (int e = 0; e < ER; ++e) {
            if constexpr (F > 1) v[e] = Row::fold(z[0][e], z[F - 1][e], p, ftw, e);
            else v[e] = Row::lead(z[0][e], e);
          }
        } else {
          const int64_t o = ((int64_t)pl * g.L1 + r) * g.LL + tr;
          float a[F][ER], b[F][ER];
#pragma unroll
          for (int f = 0; f < F; ++f)
#pragma unroll
            for (int e = 0; e < ER; ++e) {
              const int n = TR * e + f * NC;
              const bool in = tr + n < g.LL;
              b[f][e] = 1.f;
              if (vrow) {
                const float u = reinterpret_cast<const float*>(S + r * PITCH)[tr + n];
                a[f][e] = in ? u : 0.f;
              } else {
                a[f][e] = ra_ld_in(kl + o - tr, tr + n, in);
                if (gated) b[f][e] = ra_ld_in(wl + o - tr, tr + n, in);
              }
            }
#pragma unroll
          for (int e = 0; e < ER; ++e) {
            float u[F];
#pragma unroll
            for (int f = 0; f < F; ++f) {
              const int n = TR * e + f * NC;
              u[f] = a[f][e] * b[f][e];
              if constexpr (ACT) {
                if (gated) u[f] = tr + n < g.LL ? G.u1(a[f][e], b[f][e], o + n) : 0.f;
              }
            }
            if constexpr (F > 1) v[e] = Row::fold(make_float2(u[0], 0.f), make_float2(u[F - 1], 0.f), p, ftw, e);
            else v[e] = Row::lead(u[0], e);
          }
        }
        float2* const row = S + r * PITCH;
        Row::forward(v, tr, row, ftw);
        float2* const pw = row + Row::slot(tr);
#pragma unroll
        for (int e = 0; e < ER; ++e) pw[Row::off(e)] = v[e];
      }
    }
  };
  rows(0);
  __syncthreads();
  typename Col::Tw ctw;
  ctw.load(tc);
  float2 ev[E], od[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = tc + TC * e;
    ev[e] = n < g.L1 ? cp[n * PITCH] : czero();
    if constexpr (!FULL) od[e] = c_mul(ev[e], twiddle<ilog2(P1), false>((uint32_t)n));
  }
  if constexpr (FULL) {
    __syncthreads();
    rows(1);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int n = tc + TC * e;
      const float2 z = n > PH - g.L1 ? cp[n * PITCH] : czero();
      od[e] = c_mul(c_sub(ev[e], z), twiddle<ilog2(P1), false>((uint32_t)n));
      ev[e] = c_add(ev[e], z);
    }
  }
  float2* const out = ws + sg.off[sig] + line * per + (int64_t)pl * P1 * N + slab_bin<P1, Col::CW>(p * NC + col) + tc * Col::CW;
  Col::template run<false>(ev, tc, cp, ctw);
#pragma unroll
  for (int e = 0; e < E; ++e) out[TC * e * Col::CW] = ev[e];
  Col::template run<false>(od, tc, cp, ctw);
#pragma unroll
  for (int e = 0; e < E; ++e) out[(PH + TC * e) * Col::CW] = od[e];
}

// Workgroups: (line, plane), for a gk on the double grid (line, plane, half of
// axis 1).
template <int P1, int N, RaOut OUT, typename TS, bool ACT>
__global__ void __launch_bounds__((SlabInv<P1, N>::NT)) __attribute__((amdgpu_waves_per_eu(slab_waves<P1, N>(true))))
    ra_slab_inv(const float2* __restrict__ ws, const TS* __restrict__ p, const TS* __restrict__ q,
                TS* __restrict__ o1, TS* __restrict__ o2, RaGeom g, int64_t line0, int64_t per, int vec) {
  using S_ = SlabInv<P1, N>;
  using Row = typename S_::Row;
  using Col = typename S_::Col;
  constexpr int PH = S_::PH, PITCH = Row::PITCH, TR = Row::T, ER = Row::E, E = Col::E, TC = Col::T, RPR = S_::RPR;
  constexpr int F = slab_foldings(N);
  __shared__ __align__(16) float2 S[PH * PITCH];  // 16-byte accesses of rows
  const bool dbl = OUT == RA_GK && g.kmode != RA_LINEAR;
  const unsigned planes = OUT == RA_GK ? g.KP : g.L0;
  unsigned bid = blockIdx.x;
  const int hf = dbl ? (int)(bid & 1) : 0;
  if (dbl) bid >>= 1;
  const int pl = (int)(bid % planes);
  const int64_t line = bid / planes, gl = line0 + line;
  const int tid = threadIdx.x;
  const int rr = tid / TR, tr = tid % TR;
  const int lane = tid & 63;
  const int col = (tid >> 6) * Col::CW + lane % Col::CW, tc = lane / Col::CW;
  float2* const cp = S + Row::slot(col);
  {
    const float2* const in = ws + line * per + (int64_t)pl * P1 * N + slab_bin<P1, Col::CW>(col) + tc * Col::CW;
    float2 ev[E], od[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      ev[e] = in[TC * e * Col::CW];
      od[e] = in[(PH + TC * e) * Col::CW];
    }
    typename Col::Tw ctw;
    ctw.load(tc);
    Col::template run<true>(ev, tc, cp, ctw);
    Col::template run<true>(od, tc, cp, ctw);
    wave_sync();
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int n = tc + TC * e;
      const float2 z = c_mul(od[e], twiddle<ilog2(P1), true>((uint32_t)n));
      cp[n * PITCH] = OUT == RA_GK && hf ? c_sub(ev[e], z) : c_add(ev[e], z);  // point n + PH or n
    }
  }
  typename Row::InvTw itw;
  itw.load(tr);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < S_::NR; ++i) {
    const int r = i * RPR + rr;
    const int d1 = OUT == RA_GK && hf ? r - PH : r;
    if (r < PH && (d1 < 0 ? d1 > -g.L1 : r < g.L1)) {
      float2* const row = S + r * PITCH;
      float2 v[ER];
      if constexpr (F == 1) {
        const float2* const pr = row + Row::slot(tr);
#pragma unroll
        for (int e = 0; e < ER; ++e) v[e] = pr[Row::off(e)];
      } else {
        // bin tr + TR e from column (tr mod 2) N / 2 + tr / 2 + TR e / 2
        static_assert(TR % 2 == 0 && TR / 2 <= ER, "folded order");
        const float2* const pr = row + Row::slot((tr & 1) * (N / 2) + (tr >> 1));
#pragma unroll
        for (int e = 0; e < ER; ++e) v[e] = pr[(TR / 2) * e + (TR / 2 * e) / ER];
      }
      const int64_t lr = (int64_t)pl * g.L1 + r;
      RaGates<ER> gt;
      if (!vec && !dbl) gt.load(OUT, p, q, gl * g.data + lr * g.LL, tr, TR, g.LL, true);
      Row::inverse(v, tr, row, itw);
      if (vec && !dbl) {
        wave_sync();
        float* const rf = reinterpret_cast<float*>(row) + tr;
#pragma unroll
        for (int e = 0; e < ER; ++e) rf[TR * e] = Row::re(v[e], e);
        continue;
      }
      if (dbl) {
        const RaKRow kr = ra_krow(g, pl - (g.L0 - 1), d1);
        TS* const d = o1 + gl * g.kpts + kr.row;
#pragma unroll
        for (int e = 0; e < ER; ++e) {
          const int n = tr + TR * e;
          if (n < g.LL) st1(d + kr.reo + n, Row::re(v[e], e));
          if (n > g.N - g.LL) st1(d + kr.imo + n, Row::im(v[e], e));
        }
      } else {
        gt.template store<ACT>(OUT, o1, o2, gl * g.data + lr * g.LL, tr, TR, g.LL,
                               [&](int e) { return Row::re(v[e], e); });
      }
    }
  }
  if (vec && !dbl) {
    constexpr int RW = 64 / TR;
#pragma unroll
    for (int i = 0; i < S_::NR; ++i) {
      const int rw = i * RPR + (tid >> 6) * RW;
      const int64_t o = gl * g.data + ((int64_t)pl * g.L1 + rw) * g.LL;
      ra_rows_out<PITCH, RW, N, ACT>(OUT, p + o, q + o, o1 + o, o2 + o, imax(0, imin(RW, g.L1 - rw)), g.LL,
                                     reinterpret_cast<const float*>(S + rw * PITCH), lane);
    }
  }
}

template <int P1, int N, typename TS>
hipError_t slab_signals(const RaPass& p, const RaSignals& sg, bool act) {
  constexpr int NT = SlabFwd<P1, N>::NT, F = SlabFwd<P1, N>::F;
  const FftConvArgs& a = *p.a;
  // (shared kernels start at k_line's line, as aligned as any other)
  const int kvec = p.g.LL % RaVec<TS>::V == 0;
  const dim3 grid((unsigned)((int64_t)p.nl * p.g.L0 * sg.n * F));
  if (act)
    hipLaunchKernelGGL((ra_slab_fwd<P1, N, false, TS, true>), grid, dim3(NT), 0, p.s, sg, p.ws, p.g, p.line0, p.per,
                       a.kC, kvec, a.act_in, (int)a.C);
  else
    hipLaunchKernelGGL((ra_slab_fwd<P1, N, false, TS, false>), grid, dim3(NT), 0, p.s, sg, p.ws, p.g, p.line0, p.per,
                       a.kC, kvec, a.act_in, (int)a.C);
  return hipGetLastError();
}

template <int P1, int N, typename TS>
hipError_t slab_kernel(const RaPass& p, int64_t off) {
  constexpr int NT = SlabFwd<P1, N>::NT, F = SlabFwd<P1, N>::F;
  const FftConvArgs& a = *p.a;
  const RaSignals sg{{a.k}, {nullptr}, {off}, 1};
  const int kvec = 0;
  hipLaunchKernelGGL((ra_slab_fwd<P1, N, true, TS, false>), dim3((unsigned)((int64_t)p.nl * p.g.KP * F)), dim3(NT), 0,
                     p.s, sg, p.ws, p.g, p.line0, p.per, a.kC, kvec, a.act_in, (int)a.C);
  return hipGetLastError();
}

template <int P1, int N, typename TS>
hipError_t slab_inverse(const RaPass& p, const RaIo& io) {
  constexpr int NT = SlabInv<P1, N>::NT;
  const RaOut out = io.out;
  const bool dbl = out == RA_GK && p.g.kmode != RA_LINEAR;
  const dim3 grid((unsigned)((int64_t)p.nl * (out == RA_GK ? p.g.KP : p.g.L0) * (dbl ? 2 : 1)));
#define HY_INV(OUT, ACT)                                                                                      \
  hipLaunchKernelGGL((ra_slab_inv<P1, N, OUT, TS, ACT>), grid, dim3(NT), 0, p.s, p.ws + io.off, (const TS*)io.p, \
                     (const TS*)io.q, (TS*)io.o, (TS*)io.o2, p.g, p.line0, p.per, \
                     (int)(p.g.LL % RaVec<TS>::V == 0))
  if (out == RA_Y) {
    if (p.a->act) HY_INV(RA_Y, true);
    else HY_INV(RA_Y, false);
  } else if (out == RA_GX2) {
    HY_INV(RA_GX2, false);
  } else if (out == RA_GU) {
    HY_INV(RA_GU, false);
  } else {
    HY_INV(RA_GK, false);
  }
#undef HY_INV
  return hipGetLastError();
}

#define HY_SLAB_SIZES(X) \
  X(32, 32) X(32, 64) X(32, 128) X(64, 32) X(64, 64) X(64, 128) X(128, 32) X(128, 64) X(128, 128) \
  X(256, 32) X(256, 64) X(256, 128)

}  // namespace

bool ra_slab_takes(int P1, int N) { return P1 >= 32 && P1 <= 256 && N >= 32 && N <= 128; }

#define HY_CASE(p1, n)             \
  if (p.g.P1 == p1 && p.g.N == n)  \
    return p.a->bf16 ? HY_FN(p1, n, uint16_t) : HY_FN(p1, n, float);
hipError_t ra_slab_signals(const RaPass& p, const RaSignals& sg, bool act) {
#define HY_FN(P1, N, TS) slab_signals<P1, N, TS>(p, sg, act)
  HY_SLAB_SIZES(HY_CASE)
#undef HY_FN
  return hipErrorInvalidValue;
}
hipError_t ra_slab_kernel(const RaPass& p, int64_t off) {
#define HY_FN(P1, N, TS) slab_kernel<P1, N, TS>(p, off)
  HY_SLAB_SIZES(HY_CASE)
#undef HY_FN
  return hipErrorInvalidValue;
}
hipError_t ra_slab_inverse(const RaPass& p, const RaIo& io) {
#define HY_FN(P1, N, TS) slab_inverse<P1, N, TS>(p, io)
  HY_SLAB_SIZES(HY_CASE)
#undef HY_FN
  return hipErrorInvalidValue;
}
#undef HY_CASE

}  // namespace hyenand
