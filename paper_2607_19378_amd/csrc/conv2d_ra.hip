// Single-pass 2D kernels of the non-circular modes (linear and centered),
// forward and backward, on right-angle row transforms (ra_device.hpp): the
// whole image stays in LDS, HBM sees each tensor once.
//
// Rows (axis 1) are transformed in the ring x^N = -i, N = P1 / 2 complex points
// for L1 = N reals; columns (axis 0) as ordinary zero-padded transforms of
// P0 = 2 L0 points.  Every bin column is an ordinary complex column: products
// are pointwise, and no pass untangles mirror bins.  One wavefront holds whole
// rows, then whole columns, so a barrier is needed only where rows turn into
// columns and back (two per image in the linear forward kernel).
//
// What bounds them (8 x 256 images of 64 x 64, fp32): the forward kernel issues
// 25.5 M VALU instructions, 41.5 us, and moves 168 MB, 33 us at a large copy's 5.1
// TB/s; two images per CU (74 KB of LDS each, 109 VGPRs) overlap the two.  The
// packed real transforms that these replace issued 29.8 M and met 21 barriers:
// linear forward 64.7 -> 56.3 us, the operator on centered kernels 165 -> 118 us
// (bf16), linear backward 220 -> 147 us, and centered backward 1566 us (embedded in
// the circular 128 x 128 grid) -> 222 us.  The backward holds three spectra in
// registers (230 VGPRs): one image per CU, its loads, arithmetic and stores in turn;
// at 128 VGPRs it spills (360 us).  The forward of ragged extents in 128 x 128
// transforms spills 8 to 10 of its 128 VGPRs (36 to 44 bytes a lane; 57 x 40, fp32,
// centered: 60.6 us).  Keeping a workgroup resident and fetching the next image's
// inputs during the inverse rows spilled too (80 us forward).
#include "ra_mp.hpp"

namespace hyenand {

namespace {

template <int P0, int N>
struct Ra2D {
  using Row = RaRow<N>;
  static constexpr int L0 = P0 / 2, L1 = N;
  static constexpr int PITCH = Row::PITCH;
  using Col = RaCol<P0, Row>;
  static constexpr int NT = N * Col::T;         // one round of columns
  static constexpr int RPR = NT / Row::T;       // rows per round
  static constexpr int NR = (P0 + RPR - 1) / RPR;  // rounds of P0 rows (two for 128 columns points, else one)
  static_assert(P0 % RPR == 0 && (NR == 1 || RPR == L0), "rounds hold whole signals or both");
};

// Rows of an image and of its kernel in the region.  RAG: M0 x M1 points in the
// corner of the L0 x L1 that the transforms take, the rest zeros.
template <bool RAG, int P0, int N>
struct RaImage {
  int m0, m1;
  bool per;  // k of a circular mode: displacement d is point d mod M
  __device__ __forceinline__ RaImage(int M0, int M1, bool p) : m0(RAG ? M0 : P0 / 2), m1(RAG ? M1 : N), per(RAG && p) {}
  __device__ __forceinline__ bool row(int r) const { return !RAG || r < m0; }
  __device__ __forceinline__ bool in(int r, int n) const { return !RAG || (r < m0 && n < m1); }
  __device__ __forceinline__ int points() const { return m0 * m1; }
  template <bool KC>
  __device__ __forceinline__ int kpoints() const {
    return KC && !per ? (2 * m0 - 1) * (2 * m1 - 1) : m0 * m1;
  }
  // value i (of a row at p), zero outside the image
  template <typename TS>
  __device__ __forceinline__ float ld(const TS* p, int i, bool inside) const {
    return RAG ? ra_ld_sel(p, i, inside) : ld1(p + i);
  }
  // centered kernels: row g0 of the double grid holds a displacement, and which
  __device__ __forceinline__ bool krow(int g0) const { return RAG ? g0 < m0 || g0 > P0 - m0 : g0 != P0 / 2; }
  __device__ __forceinline__ int kofs(int g0) const {
    if (per) return (g0 < P0 / 2 ? g0 : g0 - P0 + m0) * m1;
    return (g0 < P0 / 2 ? g0 + m0 - 1 : g0 - P0 + m0 - 1) * (2 * m1 - 1);
  }
  // column n: displacements n and n - N
  __device__ __forceinline__ bool kre(int n) const { return !RAG || n < m1; }
  __device__ __forceinline__ bool kim(int n) const { return RAG ? n > N - m1 : n > 0; }
  __device__ __forceinline__ int kre_ofs(int n) const { return per ? n : n + m1 - 1; }
  __device__ __forceinline__ int kim_ofs(int n) const { return per ? n - N + m1 : n - N + m1 - 1; }
  // k of one line: the points of row g0, column n
  template <bool KC, typename TS>
  __device__ __forceinline__ float2 kernel_point(const TS* kl, int g0, int n, float scale) const {
    if constexpr (!KC) {
      return make_float2(ld(kl, g0 * m1 + n, in(g0, n)) * scale, 0.f);
    } else if constexpr (RAG) {
      const bool r = krow(g0);
      const int o = kofs(g0);
      return make_float2(ld(kl, o + kre_ofs(n), r && kre(n)) * scale, ld(kl, o + kim_ofs(n), r && kim(n)) * scale);
    } else {
      float2 z = czero();
      if (krow(g0)) {  // row L0 holds no displacement
        const TS* kr = kl + kofs(g0);
        z.x = ld1(kr + kre_ofs(n)) * scale;
        if (kim(n)) z.y = ld1(kr + kim_ofs(n)) * scale;
      }
      return z;
    }
  }
};

// Whether the forward kernel can scale a line (norm): the mixed plan's images of
// these transforms.  Beyond them (from 33 x 17 points) that plan's 2048 transform
// points are passed, and the code would cost 57 x 40 images 10 % in registers.
template <int P0, int N, bool RAG>
constexpr bool kRa2Norm = RAG && P0 < 128 && N < 64;

// KH as in the circular kernel: 0 transforms each image's own k, 1 writes the
// spectrum of each channel's k to khat[c][n][col] and stops, 2 reads it.
template <int P0, int N, bool KC, typename TS, bool ACT, int KH, bool RAG>
__global__ void __launch_bounds__((Ra2D<P0, N>::NT)) __attribute__((amdgpu_waves_per_eu(4)))
    conv2d_ra(const TS* __restrict__ x1, const TS* __restrict__ x2, const TS* __restrict__ v,
              const TS* __restrict__ k, const TS* __restrict__ Dp, TS* __restrict__ y, int C, int kC, ActIn ain,
              float2* __restrict__ khat, int M0, int M1, bool per, bool norm) {
  static_assert(KH == 0 || (!KC && !ACT && !RAG), "kept spectra: linear, plain gates, powers of two");
  using F = Ra2D<P0, N>;
  using Row = typename F::Row;
  using Col = typename F::Col;
  constexpr int L0 = F::L0, PITCH = F::PITCH, RPR = F::RPR, NR = F::NR, TR = Row::T;
  const RaImage<RAG, P0, N> im(M0, M1, per);
  constexpr int E = Col::E, TC = Col::T;
  constexpr float scale = 1.f / ((float)P0 * (float)N);  // of the unnormalised inverses, a power of two
  __shared__ float2 S[P0 * PITCH];
  constexpr bool NORM = kRa2Norm<P0, N, RAG>;
  constexpr int W = F::NT / 64;
  __shared__ uint32_t magw[NORM ? 2 * W : 1];
  int img = blockIdx.x;
  if constexpr (KH == 2) {
    // the B images of a channel in consecutive slots of one XCD (workgroup j
    // runs on XCD j mod 8): its spectrum comes into that L2 once
    if ((C & 7) == 0) {
      const int nb = (int)gridDim.x / C, x = img & 7, q = img >> 3;
      img = (q % nb) * C + (q / nb) * 8 + x;
    }
  }
  const int c = img % C;
  const int tid = threadIdx.x;
  const int rr = tid / TR, tr = tid % TR;                     // row of a round, lane of the row
  const int lane = tid & 63;
  const int col = (tid >> 6) * Col::CW + lane % Col::CW, tc = lane / Col::CW;  // column, lane of the column
  float2* const cp = S + Row::slot(col);
  const int r = rr % L0;                          // data row of this lane
  const bool has_u = NR == 2 || rr < L0;          // with one round, lanes rr >= L0 take K's rows
  const size_t base = (size_t)img * im.points();
  const int rb = r * im.m1 + tr;  // its first point
  const TS* const kl = k + (size_t)k_line(img, kC) * im.template kpoints<KC>();
  const Gates<ACT> G = line_gates<ACT, TS>(ain, img, C);

  typename Row::FwdTw ftw;
  ftw.load(tr);
  auto load_u = [&](float (&a)[8], float (&b)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool in = im.in(r, tr + TR * e);
      a[e] = im.ld(x1 + base, rb + TR * e, in);
      b[e] = im.ld(v + base, rb + TR * e, in);
    }
  };
  auto gate_u = [&](float (&a)[8], const float (&b)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool in = im.in(r, tr + TR * e);
      const float u = G.u1(a[e], b[e], in ? rb + TR * e : 0);
      a[e] = in ? u : 0.f;
    }
  };
  auto lead_u = [&](const float (&a)[8], float s, float2 (&w)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = Row::lead(NORM ? a[e] * s : a[e], e);
  };
  // NORM: unscaled until the magnitudes are known
  auto load_k = [&](int g0, float2 (&w)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = im.template kernel_point<KC>(kl, g0, tr + TR * e, NORM ? 1.f : scale);
  };
  auto lead_k = [&](float2 (&w)[8], float s) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (NORM) w[e] = c_scale(w[e], s);
      w[e] = KC ? Row::lead(w[e], e) : Row::lead(w[e].x, e);
    }
  };
  // norm: the exponents of the largest |u| (0) and of the largest of |k| (1) and |D|
  const float Dv = KH == 1 ? 0.f : ld1(Dp + c);
  RaMags<W, 2> mags;
  mags.s = magw;
  auto u_mag = [&](const float (&a)[8]) {
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) m = ra_umax(m, ra_mag(a[e]));
    return m;
  };
  auto k_mag = [&](const float2 (&w)[8]) {
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      m = ra_umax(m, ra_mag(w[e].x));
      if constexpr (KC) m = ra_umax(m, ra_mag(w[e].y));
    }
    return m;
  };
  int eu = 0, ek = 0;
  auto row_fwd = [&](int slot_row, float2 (&w)[8]) {
    float2* const row = S + slot_row * PITCH;
    Row::forward(w, tr, row, ftw);
#pragma unroll
    for (int e = 0; e < 8; ++e) row[tr + Row::off(e)] = w[e];
  };

  float2 wu[E], wk[E];
  typename Col::Tw ctw;
  if constexpr (KC) {
    // U's rows first; each lane keeps the U values of its column while K's
    // P0 rows take the region
    {
      float a[8] = {}, b[8];
      if (has_u) {
        load_u(a, b);
        gate_u(a, b);
      }
      if (NORM && norm) {
        mags.put(0, u_mag(a), tid);
        mags.sync();
        eu = mags.get(0);
      }
      if (has_u) {
        float2 w[8];
        lead_u(a, ra_pow2(-eu), w);
        row_fwd(rr, w);
      }
    }
    float2 wr[NR][8];
#pragma unroll
    for (int q = 0; q < NR; ++q) load_k(q * RPR + rr, wr[q]);
    if (NORM && norm) {
      uint32_t m = 0;
#pragma unroll
      for (int q = 0; q < NR; ++q) m = ra_umax(m, k_mag(wr[q]));
      mags.put(1, m, tid);
    }
    __syncthreads();
    if (NORM && norm) ek = imax(mags.get(1), ra_exponent(ra_mag(Dv)));
#pragma unroll
    for (int e = 0; e < E / 2; ++e) wu[e] = cp[(tc + TC * e) * PITCH];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      lead_k(wr[q], scale * ra_pow2(-ek));
      row_fwd(q * RPR + rr, wr[q]);
    }
    __syncthreads();
    ctw.load(tc);
#pragma unroll
    for (int e = 0; e < E; ++e) wk[e] = cp[(tc + TC * e) * PITCH];
  } else {
    // U in rows [0, L0) of the region, K in [L0, P0)
    if constexpr (NR == 2) {
      float a[8], b[8];
      float2 wr[8];
      if constexpr (KH != 2) load_k(rr, wr);
      if constexpr (KH != 1) load_u(a, b);
      static_assert(!NORM, "two rounds of rows");
      if constexpr (KH != 2) {
        lead_k(wr, 1.f);
        row_fwd(L0 + rr, wr);
      }
      if constexpr (KH != 1) {
        gate_u(a, b);
        lead_u(a, 1.f, wr);
        row_fwd(rr, wr);
      }
    } else if constexpr (NORM) {
      float a[8] = {}, b[8];
      float2 w[8] = {};
      if (has_u) {
        load_u(a, b);
        gate_u(a, b);
      } else {
        load_k(r, w);
      }
      if (NORM && norm) {
        mags.put(0, u_mag(a), tid);
        mags.put(1, k_mag(w), tid);
        mags.sync();
        eu = mags.get(0);
        ek = imax(mags.get(1), ra_exponent(ra_mag(Dv)));
      }
      if (has_u) lead_u(a, ra_pow2(-eu), w);
      else lead_k(w, scale * ra_pow2(-ek));
      row_fwd(rr, w);
    } else if (KH == 0 || (KH == 1) == !has_u) {
      float2 w[8];
      if (!has_u) {
        load_k(r, w);
        lead_k(w, 1.f);
      } else {
        float a[8], b[8];
        load_u(a, b);
        gate_u(a, b);
        lead_u(a, 1.f, w);
      }
      row_fwd(rr, w);
    }
    __syncthreads();
    ctw.load(tc);
    if constexpr (KH != 1) {
#pragma unroll
      for (int e = 0; e < E / 2; ++e) wu[e] = cp[(tc + TC * e) * PITCH];
    }
    if constexpr (KH != 2) {
#pragma unroll
      for (int e = 0; e < E / 2; ++e) wk[e] = cp[(L0 + tc + TC * e) * PITCH];
#pragma unroll
      for (int e = E / 2; e < E; ++e) wk[e] = czero();
    }
  }

  // columns: forward, product with the folded shortcut, inverse, crop
  float2* const kh = khat + ((size_t)c * P0 + tc) * N + col;
  if constexpr (KH == 2) {
#pragma unroll
    for (int e = 0; e < E; ++e) wk[e] = kh[TC * e * N];
  } else {
    Col::template run<false>(wk, tc, cp, ctw);
  }
  if constexpr (KH == 1) {
#pragma unroll
    for (int e = 0; e < E; ++e) kh[TC * e * N] = wk[e];
    return;
  }
#pragma unroll
  for (int e = E / 2; e < E; ++e) wu[e] = czero();
  Col::template run<false>(wu, tc, cp, ctw);
  const float Ds = NORM ? Dv * (scale * ra_pow2(-ek)) : scale * Dv;
#pragma unroll
  for (int e = 0; e < E; ++e) wu[e] = gated_product(wu[e], wk[e], Ds);
  // the outer gate and the inverse rows' twiddles arrive meanwhile
  float g[8];
  typename Row::InvTw itw;
  if (has_u) {
#pragma unroll
    for (int e = 0; e < 8; ++e) g[e] = im.ld(x2 + base, rb + TR * e, im.in(r, tr + TR * e));
    itw.load(tr);
  }
  Col::template run<true>(wu, tc, cp, ctw);
  wave_sync();
#pragma unroll
  for (int e = 0; e < E / 2; ++e) cp[(tc + TC * e) * PITCH] = wu[e];

  // inverse rows, outer gate, store
  __syncthreads();
  if (!has_u) return;
  float2* const row = S + rr * PITCH;
  float2 w[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) w[e] = row[tr + Row::off(e)];
  Row::inverse(w, tr, row, itw);
  if (NORM && norm) ra_ldexp(w, eu + ek);
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (im.in(r, tr + TR * e)) st1(y + base + rb + TR * e, G.g1(g[e]) * Row::re(w[e], e));
}

// Backward (conv_backward.hip states the products): U and H take the region
// side by side, then K; the three products' inverses return z and gu together,
// then gk.  x1, v and gy stay in registers from staging to the epilogue (the
// lane that stages row r of u and h stores row r of the gradients).
template <int P0, int N, bool KC, typename TS, bool RAG>
__global__ void __launch_bounds__((Ra2D<P0, N>::NT)) __attribute__((amdgpu_waves_per_eu(2)))
    bwd2d_ra(const TS* __restrict__ x1, const TS* __restrict__ x2, const TS* __restrict__ v,
             const TS* __restrict__ k, const TS* __restrict__ Dp, const TS* __restrict__ gy, TS* __restrict__ gx1,
             TS* __restrict__ gx2, TS* __restrict__ gv, TS* __restrict__ gk, float* __restrict__ partial, int C, int M0, int M1,
             bool norm) {
  using F = Ra2D<P0, N>;
  using Row = typename F::Row;
  using Col = typename F::Col;
  constexpr int L0 = F::L0, PITCH = F::PITCH, RPR = F::RPR, NR = F::NR, TR = Row::T, NT = F::NT;
  const RaImage<RAG, P0, N> im(M0, M1, false);
  constexpr int E = Col::E, TC = Col::T;
  constexpr float scale = 1.f / ((float)P0 * (float)N);
  __shared__ float2 S[P0 * PITCH];
  __shared__ float red[imax(1, NT / 64)];
  constexpr int W = NT / 64;
  __shared__ uint32_t magw[RAG ? 3 * W : 1];
  RaMags<W, 3> mags;  // norm: |u|, |h|, |k|
  mags.s = magw;
  int eu = 0, eh = 0, ek = 0;
  const int img = blockIdx.x;
  const int c = img % C;
  const size_t base = (size_t)img * im.points();
  const TS* const kl = k + (size_t)img * im.template kpoints<KC>();
  TS* const gkl = gk + (size_t)img * im.template kpoints<KC>();
  const int tid = threadIdx.x;
  const int rr = tid / TR, tr = tid % TR;
  const int lane = tid & 63;
  const int col = (tid >> 6) * Col::CW + lane % Col::CW, tc = lane / Col::CW;
  float2* const cp = S + Row::slot(col);
  const int r = rr % L0;                        // data row of this lane
  const int rb = r * im.m1 + tr;                // its first point

  // rows of u [0, L0) and h [L0, P0)
  float xa[8], xv[8], xg[8];
  typename Row::FwdTw ftw;
  ftw.load(tr);
  auto row_fwd = [&](int slot_row, float2 (&w)[8]) {
    float2* const row = S + slot_row * PITCH;
    Row::forward(w, tr, row, ftw);
#pragma unroll
    for (int e = 0; e < 8; ++e) row[tr + Row::off(e)] = w[e];
  };
  {
    float xe[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool in = im.in(r, tr + TR * e);
      xa[e] = im.ld(x1 + base, rb + TR * e, in);
      xv[e] = im.ld(v + base, rb + TR * e, in);
      xg[e] = im.ld(gy + base, rb + TR * e, in);
      xe[e] = im.ld(x2 + base, rb + TR * e, in);
    }
    float hu = 0.f;
    if (RAG && norm) {
      uint32_t mu = 0, mh = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        mu = ra_umax(mu, ra_mag(xa[e] * xv[e]));
        mh = ra_umax(mh, ra_mag(xg[e] * xe[e]));
      }
      mags.put(0, mu, tid);
      mags.put(1, mh, tid);
      mags.sync();
      eu = mags.get(0);
      eh = mags.get(1);
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const bool ish = q * RPR + rr >= L0;
      const float s = ra_pow2(ish ? -eh : -eu);
      float2 w[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = ish ? xg[e] * xe[e] : xa[e] * xv[e];
        w[e] = Row::lead(RAG ? x * s : x, e);
      }
      row_fwd(q * RPR + rr, w);
    }
    if (rr < L0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) hu += (xa[e] * xv[e]) * (xg[e] * xe[e]);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) hu += __shfl_xor(hu, o, 64);
    if (lane == 0) red[tid >> 6] = hu;
  }
  // K's rows are fetched while the columns of U and H are read
  constexpr int NK = KC ? NR : 1;  // rounds of K's rows
  float2 wr[NK][8];
  uint32_t mk = 0;
#pragma unroll
  for (int q = 0; q < NK; ++q) {
    const int g0 = q * RPR + rr;
    if (KC || g0 < L0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        wr[q][e] = im.template kernel_point<KC>(kl, g0, tr + TR * e, RAG ? 1.f : scale);
        if constexpr (RAG) mk = ra_umax(mk, ra_umax(ra_mag(wr[q][e].x), ra_mag(wr[q][e].y)));
      }
    }
  }
  const float Dv = ld1(Dp + c);
  if (RAG && norm) mags.put(2, mk, tid);
  __syncthreads();
  if (RAG && norm) ek = imax(mags.get(2), ra_exponent(ra_mag(Dv)));
  const float ks = scale * ra_pow2(-ek);
  if (tid == 0) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) s += red[i];
    partial[img] = s;
  }
  float2 wu[E], wh[E], wk[E];
#pragma unroll
  for (int e = 0; e < E / 2; ++e) {
    wu[e] = cp[(tc + TC * e) * PITCH];
    wh[e] = cp[(L0 + tc + TC * e) * PITCH];
    wu[E / 2 + e] = wh[E / 2 + e] = czero();
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NK; ++q) {
    const int g0 = q * RPR + rr;
    if (KC || g0 < L0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (RAG) wr[q][e] = c_scale(wr[q][e], ks);
        wr[q][e] = KC ? Row::lead(wr[q][e], e) : Row::lead(wr[q][e].x, e);
      }
      row_fwd(g0, wr[q]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e) wk[e] = (KC || e < E / 2) ? cp[(tc + TC * e) * PITCH] : czero();

  // columns: three forward transforms, the products, inverse of z and gu
  typename Col::Tw ctw;
  ctw.load(tc);
  Col::template run<false>(wk, tc, cp, ctw);
  Col::template run<false>(wu, tc, cp, ctw);
  Col::template run<false>(wh, tc, cp, ctw);
  {
    const float Ds = Dv * ks;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const float2 kd = make_float2(wk[e].x + Ds, wk[e].y);
      wk[e] = c_scale(c_mulc(wh[e], wu[e]), scale);  // gk: H conj U
      wu[e] = c_mul(wu[e], kd);                      // z: U (K + D)
      wh[e] = c_mulc(wh[e], kd);                     // gu: H conj(K + D)
    }
  }
  Col::template run<true>(wu, tc, cp, ctw);
  Col::template run<true>(wh, tc, cp, ctw);
  wave_sync();
#pragma unroll
  for (int e = 0; e < E / 2; ++e) {
    cp[(tc + TC * e) * PITCH] = wu[e];
    cp[(L0 + tc + TC * e) * PITCH] = wh[e];
  }
  typename Row::InvTw itw;
  itw.load(tr);
  __syncthreads();

  // rows of z and gu; gx2 = gy z, gx1 = gu v, gv = gu x1
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    float2* const row = S + (q * RPR + rr) * PITCH;
    const bool isgu = q * RPR + rr >= L0;
    float2 w[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = row[tr + Row::off(e)];
    Row::inverse(w, tr, row, itw);
    if (RAG && norm) ra_ldexp(w, (isgu ? eh : eu) + ek);
    if (isgu) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float g = Row::re(w[e], e);
        if (!im.in(r, tr + TR * e)) continue;
        st1(gx1 + base + rb + TR * e, g * xv[e]);
        st1(gv + base + rb + TR * e, g * xa[e]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (im.in(r, tr + TR * e)) st1(gx2 + base + rb + TR * e, Row::re(w[e], e) * xg[e]);
    }
  }
  __syncthreads();

  // gk: inverse columns (all P0 rows centered), rows, displacements
  Col::template run<true>(wk, tc, cp, ctw);
  wave_sync();
#pragma unroll
  for (int e = 0; e < (KC ? E : E / 2); ++e) cp[(tc + TC * e) * PITCH] = wk[e];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NK; ++q) {
    const int g0 = q * RPR + rr;
    if (KC || g0 < L0) {
      float2* const row = S + g0 * PITCH;
      float2 w[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) w[e] = row[tr + Row::off(e)];
      Row::inverse(w, tr, row, itw);
      if (RAG && norm) ra_ldexp(w, eu + eh);
      if constexpr (!KC) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (im.in(g0, tr + TR * e)) st1(gkl + g0 * im.m1 + tr + TR * e, Row::re(w[e], e));
      } else if (im.krow(g0)) {
        TS* const kr = gkl + im.kofs(g0);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int n = tr + TR * e;
          if (im.kre(n)) st1(kr + im.kre_ofs(n), Row::re(w[e], e));
          if (im.kim(n)) st1(kr + im.kim_ofs(n), Row::im(w[e], e));
        }
      }
    }
  }
}

template <int P0, int N, typename TS, bool RAG>
hipError_t launch_fwd_t(const FftConvArgs& a, bool norm, hipStream_t s) {
  constexpr int NT = Ra2D<P0, N>::NT;
  if (norm && !kRa2Norm<P0, N, RAG>) return hipErrorInvalidValue;  // no shape of the mixed plan
#define HY_RA(KC, ACT, KH, GRID)                                                                               \
  hipLaunchKernelGGL((conv2d_ra<P0, N, KC, TS, ACT, KH, RAG>), dim3((unsigned)(GRID)), dim3(NT), 0, s,              \
                     (const TS*)a.x1, (const TS*)a.x2, (const TS*)a.v, (const TS*)a.k, (const TS*)a.D,         \
                     (TS*)a.y, (int)a.C, a.kC, a.act_in, a.khat, (int)a.L[0], (int)a.L[1], a.periodic, norm)
  if (a.centered || a.periodic) {
    if (a.act) HY_RA(true, true, 0, a.lines);
    else HY_RA(true, false, 0, a.lines);
  } else if (a.act) {
    HY_RA(false, true, 0, a.lines);
  } else if (RAG || !a.khat) {
    HY_RA(false, false, 0, a.lines);
  } else if constexpr (!RAG) {
    if (a.khat_pass != 2) HY_RA(false, false, 1, a.C);
    if (a.khat_pass != 1) HY_RA(false, false, 2, a.lines);
  }
#undef HY_RA
  return hipGetLastError();
}

template <int P0, int N, typename TS, bool RAG>
hipError_t launch_bwd_t(const FftConvBwdArgs& b, bool norm, hipStream_t s) {
  const FftConvArgs& a = b.f;
  constexpr int NT = Ra2D<P0, N>::NT;
#define HY_RA(KC)                                                                                                 \
  hipLaunchKernelGGL((bwd2d_ra<P0, N, KC, TS, RAG>), dim3((unsigned)a.lines), dim3(NT), 0, s, (const TS*)a.x1,         \
                     (const TS*)a.x2, (const TS*)a.v, (const TS*)a.k, (const TS*)a.D, (const TS*)b.gy,            \
                     (TS*)b.gx1, (TS*)b.gx2, (TS*)b.gv, (TS*)b.gk, b.partial, (int)a.C, (int)a.L[0], (int)a.L[1], norm)
  if (a.centered) HY_RA(true);
  else HY_RA(false);
#undef HY_RA
  return hipGetLastError();
}

#define HY_RA2D_SIZES(X) X(32, 32) X(64, 64) X(128, 128) X(64, 128) X(128, 64) X(32, 64) X(64, 32)

}  // namespace

bool ra2d_supported(const FftConvArgs& a) {
  if (a.ndim != 2 || a.circular || a.rl) return false;
#define HY_CASE(p0, p1) if (a.P[0] == p0 && a.P[1] == p1) return true;
  HY_RA2D_SIZES(HY_CASE)
#undef HY_CASE
  return false;
}

// Images of other extents run in the corner of the transforms of the next ones
// (9 to 64 points an axis), forward and backward, also where the mixed-radix
// kernels would transform fewer points: those wait at a workgroup barrier for
// every factor and compute their indexes from run-time radixes.  8 x 256
// images, fp32, centered, forward and backward: 17 x 17 (four times the points)
// 30.6 -> 21.9 and 56.7 -> 41.5 us; 28 x 28 62.2 -> 21.8 and 134 -> 45.3; 57 x
// 40 (packed real transforms, and embedded) 273 -> 60.6 and 1330 -> 166; 16 x
// 384 of 9 x 9 27.1 -> 16.4 and 55.9 -> 31.3, of 14 x 14 44.3 -> 17.4 and 89.4
// -> 38.8.
bool ra2d_ragged(const FftConvArgs& a) {
  if (a.ndim != 2 || a.circular || !a.rl) return false;
#define HY_CASE(p0, p1) if (a.P[0] == p0 && a.P[1] == p1) return true;
  HY_RA2D_SIZES(HY_CASE)
#undef HY_CASE
  return false;
}

hipError_t launch_ra2d(const FftConvArgs& a, bool norm, hipStream_t s) {
#define HY_CASE(p0, p1)                                                                                        \
  if (a.P[0] == p0 && a.P[1] == p1) {                                                                          \
    if (a.rl)                                                                                                  \
      return a.bf16 ? launch_fwd_t<p0, p1 / 2, uint16_t, true>(a, norm, s) : launch_fwd_t<p0, p1 / 2, float, true>(a, norm, s); \
    return a.bf16 ? launch_fwd_t<p0, p1 / 2, uint16_t, false>(a, norm, s) : launch_fwd_t<p0, p1 / 2, float, false>(a, norm, s); \
  }
  HY_RA2D_SIZES(HY_CASE)
#undef HY_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_ra2d_backward(const FftConvBwdArgs& b, bool norm, hipStream_t s) {
  const FftConvArgs& a = b.f;
#define HY_CASE(p0, p1)                                                                                        \
  if (a.P[0] == p0 && a.P[1] == p1) {                                                                          \
    if (a.rl)                                                                                                  \
      return a.bf16 ? launch_bwd_t<p0, p1 / 2, uint16_t, true>(b, norm, s) : launch_bwd_t<p0, p1 / 2, float, true>(b, norm, s); \
    return a.bf16 ? launch_bwd_t<p0, p1 / 2, uint16_t, false>(b, norm, s) : launch_bwd_t<p0, p1 / 2, float, false>(b, norm, s); \
  }
  HY_RA2D_SIZES(HY_CASE)
#undef HY_CASE
  return hipErrorInvalidValue;
}

}  // namespace hyenand
