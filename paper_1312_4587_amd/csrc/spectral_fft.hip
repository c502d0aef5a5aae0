// Spectral Neumann Poisson solve (Eqs. (8)-(12)) with hand-written FFTs.
//
// The 2-D transforms are separable; the solve is three passes over the map,
// each one block per pair of rows (or columns), the 1-D transforms done in
// LDS by the whole block:
//   A  rows:    DCT-II along x of rho           -> bT[u][iy] (written transposed)
//   B  columns: DCT-II along y, scale by c_u c_v / n^2 / (w_u^2 + w_v^2 + eps)
//               (zero at (0,0): the DC is removed), then DCT-III along y
//               (-> P) and the sine transform along y weighted by w_v (-> Q)
//                                               -> P[iy][u], Q[iy][u]
//   C  rows:    DCT-III along x of P (-> psi) and of Q (-> Ey), sine
//               transform along x of w_u P (-> Ex); energy sum rho*psi.
// Difference mode (for the exact density gradient) replaces the fields by
// the differences of psi between neighbouring bin centres,
//   Dx(iy, ix) = psi(iy, ix+1) - psi(iy, ix),  Dy(iy, ix) = psi(iy+1, ix) - psi(iy, ix),
// taken in the spectral domain: cos(w (i + 3/2)) - cos(w (i + 1/2)) =
// (cos w - 1) cos(w (i + 1/2)) - sin w sin(w (i + 1/2)), so each difference is
// a DCT-III with weights cos w - 1 minus a sine transform with weights sin w.
// Both weights vanish at low frequency, so the small differences come out
// with float32 accuracy relative to themselves instead of to psi.  Pass B
// then outputs R = DCT-III((cos w_v - 1) G) - sine(sin w_v G) in place of Q,
// and pass C gives Dy = DCT-III(R) and Dx from P the same way along x.
// A length-n DCT-II is an n-point complex FFT of the even/odd reordered
// sequence followed by a quarter-sample twiddle (Makhoul's algorithm); two
// real sequences share one complex FFT as its real and imaginary parts.  A
// DCT-III runs the same steps backwards.  The sine transform is a DCT-III of
// the reversed coefficients with alternating output signs:
//   sum_{k>=1} b_k sin(pi k (2i+1)/2n) = (-1)^i sum_{k>=1} b_{n-k} cos(pi k (2i+1)/2n).
// The 1-D FFT is a Stockham autosort radix-4 (one radix-2 stage first when
// log2 n is odd), in place in LDS, every stage reading all its inputs into
// registers before a barrier and writing after it.  The independent
// transforms of a pass share the stages.  Each pass issues all its global
// loads (rows and tables) before touching LDS, so a block waits on memory
// once rather than once per loop trip.
#include "fft_device.hpp"

namespace fftpl {

namespace {

// ---------------------------------------------------------------------------
// Pass A: rows -> bT (transposed), row sums in double; optional overflow sums.
// ---------------------------------------------------------------------------
template <int N, int NB>
__global__ void __launch_bounds__(FftShape<N>::NT)
    k_rows_dct2(SpecBatch<NB> sb, const float2* __restrict__ tw_g,
                const float2* __restrict__ cs_g) {
  // design blockIdx.y of the batch
  const SpecReq& rq = sb.r[blockIdx.y];
  const float* __restrict__ rho = rq.rho;
  const float* __restrict__ base = rq.base;
  const float* __restrict__ cap = rq.cap;
  const float rho_t = rq.rho_t;
  double* __restrict__ tau_part = rq.tau_part;
  constexpr int NT = FftShape<N>::NT;
  constexpr int PER = (N + NT - 1) / NT;
  __shared__ RowsLds<N, NT> lds;
  const int tid = threadIdx.x;
  const int pair = xcd_block(blockIdx.x, gridDim.x);
  const int r1 = 2 * pair, r2 = r1 + 1;
  float a1[PER], a2[PER], b1[PER], b2[PER], c1[PER], c2[PER];
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int i = min(tid + NT * t, N - 1);
    a1[t] = rho[(int64_t)r1 * N + i];
    a2[t] = rho[(int64_t)r2 * N + i];
  }
  // (pointer tests hoisted out of the loops so that the loads issue together)
  if (tau_part && base) {
#pragma unroll
    for (int t = 0; t < PER; ++t) {
      const int i = min(tid + NT * t, N - 1);
      b1[t] = base[(int64_t)r1 * N + i];
      b2[t] = base[(int64_t)r2 * N + i];
    }
  } else {
#pragma unroll
    for (int t = 0; t < PER; ++t) b1[t] = b2[t] = 0.0f;
  }
  if (tau_part && cap) {
#pragma unroll
    for (int t = 0; t < PER; ++t) {
      const int i = min(tid + NT * t, N - 1);
      c1[t] = cap[(int64_t)r1 * N + i];
      c2[t] = cap[(int64_t)r2 * N + i];
    }
  } else {
#pragma unroll
    for (int t = 0; t < PER; ++t) {
      c1[t] = fmaxf(0.0f, rho_t - fminf(rho_t, b1[t]));
      c2[t] = fmaxf(0.0f, rho_t - fminf(rho_t, b2[t]));
    }
  }
  stage_tables<N, NT, false>(lds.tw, tw_g, lds.cs, cs_g, nullptr, nullptr, tid);
  rows_dct2<N, NT>(a1, a2, b1, b2, c1, c2, r1, tid, lds, rq.bT, rq.rowsum, tau_part);
}

// ---------------------------------------------------------------------------
// Pass B: columns u1 = 2q, u2 = 2q+1 (rows of bT).  Column 0 is rebuilt from
// the double row sums minus their mean so that the DC never enters float32.
// ---------------------------------------------------------------------------
template <int N, bool DIFF, int NB>
__global__ void __launch_bounds__(FftShape<N>::NT)
    k_cols_solve(SpecBatch<NB> sb, const float2* __restrict__ tw_g,
                 const float2* __restrict__ cs_g, const float* __restrict__ wf_g) {
  const SpecReq& rq = sb.r[blockIdx.y];
  const float* __restrict__ bT = rq.bT;
  const double* __restrict__ rowsum = rq.rowsum;
  float* __restrict__ P = rq.P;
  float* __restrict__ Q = rq.Q;
  const float eps = rq.eps;
  constexpr int NT = FftShape<N>::NT;
  constexpr int PER = (N + NT - 1) / NT, PK = (N / 2 + NT) / NT;
  __shared__ float2 buf0[N];
  __shared__ float2 buf1[N];
  __shared__ float2 buf2[DIFF ? N : 1];
  __shared__ float2 tw[N];
  __shared__ float2 cs[N / 2 + 1];
  __shared__ float wf[N];
  __shared__ double red[NT / kWave];
  const int tid = threadIdx.x;
  const int q = xcd_block(blockIdx.x, gridDim.x);
  const int u1 = 2 * q, u2 = u1 + 1;
  float c1[PER], c2[PER];
  if (u1 == 0) {
    double rs[PER];
    double s[1] = {0.0};
#pragma unroll
    for (int t = 0; t < PER; ++t) {
      rs[t] = rowsum[min(tid + NT * t, N - 1)];
      if (N % NT == 0 || tid + NT * t < N) s[0] += rs[t];
    }
    block_sums<NT, 1>(s, red, tid);
    const double mean0 = s[0] / N;
#pragma unroll
    for (int t = 0; t < PER; ++t) c1[t] = (float)(rs[t] - mean0);
  } else {
#pragma unroll
    for (int t = 0; t < PER; ++t) c1[t] = bT[(int64_t)u1 * N + min(tid + NT * t, N - 1)];
  }
#pragma unroll
  for (int t = 0; t < PER; ++t) c2[t] = bT[(int64_t)u2 * N + min(tid + NT * t, N - 1)];
  stage_tables<N, NT, true>(tw, tw_g, cs, cs_g, wf, wf_g, tid);
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int i = tid + NT * t;
    if (N % NT == 0 || i < N) buf0[mk_pos<N>(i)] = make_float2(c1[t], c2[t]);
  }
  block_lds_sync<NT>();
  block_fft<N, NT, false, 1>(buf0, nullptr, nullptr, nullptr, tw, tid);
  const float inv_n2 = 1.0f / ((float)N * (float)N);
  const float wu1 = wf[u1], wu2 = wf[u2];
  const float f1 = (u1 == 0 ? 1.0f : 2.0f) * inv_n2, f2 = 2.0f * inv_n2;
#pragma unroll
  for (int t = 0; t < PK; ++t) {
    const int k = tid + NT * t;
    if (k > N / 2) continue;
    const int kp = (N - k) & (N - 1);
    const float2 c = cs[k];
    float x1k, x2k, x1kp, x2kp;
    dct2_pair(buf0[k], buf0[kp], c, x1k, x2k, x1kp, x2kp);
    const float wk = wf[k], wkp = wf[kp];
    const float ck = (k == 0 ? 1.0f : 2.0f), ckp = (kp == 0 ? 1.0f : 2.0f);
    float g1k = x1k * (f1 * ck) / (wu1 * wu1 + wk * wk + eps);
    float g1kp = x1kp * (f1 * ckp) / (wu1 * wu1 + wkp * wkp + eps);
    const float g2k = x2k * (f2 * ck) / (wu2 * wu2 + wk * wk + eps);
    const float g2kp = x2kp * (f2 * ckp) / (wu2 * wu2 + wkp * wkp + eps);
    if (u1 == 0 && k == 0) g1k = 0.0f;   // a_00 := 0
    // P: DCT-III of G.  Q: DCT-III of Yb with Yb_k = w_{n-k} G_{n-k} (k >= 1),
    // Yb_0 = 0.  The two columns' P share one complex FFT and their Q another:
    // sequences packed together must have similar magnitudes (P ~ 1/w^2 is far
    // larger than Q ~ 1/w), or the rounding of one swamps the other.
    const bool k0 = (k == 0);
    float2 h1, h1p, h2, h2p;
    dct3_herm(g1k, g1kp, c, k0, h1, h1p);
    dct3_herm(g2k, g2kp, c, k0, h2, h2p);
    buf0[k] = pack2(h1, h2);
    if (!k0 && k != N / 2) buf0[kp] = pack2(h1p, h2p);
    if (!DIFF) {
      dct3_herm(k0 ? 0.0f : wkp * g1kp, k0 ? 0.0f : wk * g1k, c, k0, h1, h1p);
      dct3_herm(k0 ? 0.0f : wkp * g2kp, k0 ? 0.0f : wk * g2k, c, k0, h2, h2p);
      buf1[k] = pack2(h1, h2);
      if (!k0 && k != N / 2) buf1[kp] = pack2(h1p, h2p);
    } else {
      // R = DCT-III((cos w - 1) G) (buf1) - sine transform of sin(w) G (buf2)
      float dmk, dmkp, sw;
      diff_weights(c, dmk, dmkp, sw);
      dct3_herm(dmk * g1k, dmkp * g1kp, c, k0, h1, h1p);
      dct3_herm(dmk * g2k, dmkp * g2kp, c, k0, h2, h2p);
      buf1[k] = pack2(h1, h2);
      if (!k0 && k != N / 2) buf1[kp] = pack2(h1p, h2p);
      dct3_herm(k0 ? 0.0f : sw * g1kp, k0 ? 0.0f : sw * g1k, c, k0, h1, h1p);
      dct3_herm(k0 ? 0.0f : sw * g2kp, k0 ? 0.0f : sw * g2k, c, k0, h2, h2p);
      buf2[k] = pack2(h1, h2);
      if (!k0 && k != N / 2) buf2[kp] = pack2(h1p, h2p);
    }
  }
  block_lds_sync<NT>();
  block_fft<N, NT, true, DIFF ? 3 : 2>(buf0, buf1, buf2, nullptr, tw, tid);
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int iy = tid + NT * t;
    if (N % NT != 0 && iy >= N) continue;
    const int mpos = mk_pos<N>(iy);
    const float2 zp = buf0[mpos], zq = buf1[mpos];
    const float sg = (iy & 1) ? -1.0f : 1.0f;
    *reinterpret_cast<float2*>(&P[(int64_t)iy * N + u1]) = zp;
    if (!DIFF) {
      *reinterpret_cast<float2*>(&Q[(int64_t)iy * N + u1]) = make_float2(sg * zq.x, sg * zq.y);
    } else {
      const float2 zs = buf2[mpos];
      *reinterpret_cast<float2*>(&Q[(int64_t)iy * N + u1]) =
          make_float2(zq.x - sg * zs.x, zq.y - sg * zs.y);
    }
  }
}

// ---------------------------------------------------------------------------
// Pass C: rows r1 = 2p, r2 = 2p+1 of P and Q -> psi, Ex, Ey; energy.
// ---------------------------------------------------------------------------
template <int N, bool DIFF, int NB>
__global__ void __launch_bounds__(FftShape<N>::NT)
    k_rows_inverse(SpecBatch<NB> sb, const float2* __restrict__ tw_g,
                   const float2* __restrict__ cs_g, const float* __restrict__ wf_g) {
  const SpecReq& rq = sb.r[blockIdx.y];
  const float* __restrict__ P = rq.P;
  const float* __restrict__ Q = rq.Q;
  const float* __restrict__ rho = rq.rho;
  float* __restrict__ psi = rq.psi;
  float* __restrict__ ex = rq.ex;
  float* __restrict__ ey = rq.ey;
  float2* __restrict__ exy = rq.exy;
  double* __restrict__ energy = rq.en_part;
  constexpr int NT = FftShape<N>::NT;
  constexpr int PER = (N + NT - 1) / NT, PK = (N / 2 + NT) / NT;
  __shared__ float2 bufa[N];
  __shared__ float2 bufb[N];
  __shared__ float2 bufc[N];
  __shared__ float2 bufd[DIFF ? N : 1];
  __shared__ float2 tw[N];
  __shared__ float2 cs[N / 2 + 1];
  __shared__ float wf[N];
  __shared__ float rows[4 * N];
  __shared__ double red[NT / kWave];
  const int tid = threadIdx.x;
  const int pr = xcd_block(blockIdx.x, gridDim.x);
  const int r1 = 2 * pr, r2 = r1 + 1;
  // rows P[r1], P[r2], Q[r1], Q[r2] (and rho for the energy): all loads first
  float v[4][PER], e1[PER], e2[PER];
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int i = min(tid + NT * t, N - 1);
    v[0][t] = P[(int64_t)r1 * N + i];
    v[1][t] = P[(int64_t)r2 * N + i];
    v[2][t] = Q[(int64_t)r1 * N + i];
    v[3][t] = Q[(int64_t)r2 * N + i];
  }
  if (energy) {
#pragma unroll
    for (int t = 0; t < PER; ++t) {
      const int i = min(tid + NT * t, N - 1);
      e1[t] = rho[(int64_t)r1 * N + i];
      e2[t] = rho[(int64_t)r2 * N + i];
    }
  }
  stage_tables<N, NT, true>(tw, tw_g, cs, cs_g, wf, wf_g, tid);
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int i = tid + NT * t;
    if (N % NT == 0 || i < N) {
#pragma unroll
      for (int r = 0; r < 4; ++r) rows[r * N + i] = v[r][t];
    }
  }
  block_lds_sync<NT>();
  const float* P1 = rows;
  const float* P2 = rows + N;
  const float* Q1 = rows + 2 * N;
  const float* Q2 = rows + 3 * N;
#pragma unroll
  for (int t = 0; t < PK; ++t) {
    const int k = tid + NT * t;
    if (k > N / 2) continue;
    const int kp = (N - k) & (N - 1);
    const bool k0 = (k == 0), self = k0 || k == N / 2;
    const float2 c = cs[k];
    const float wk = wf[k], wkp = wf[kp];
    const float p1k = P1[k], p1kp = P1[kp], p2k = P2[k], p2kp = P2[kp];
    // like-magnitude pairs share a complex FFT: (psi r1, psi r2), (Ey r1, Ey r2),
    // (Ex r1, Ex r2)
    float2 ha, hap, hb, hbp;
    dct3_herm(p1k, p1kp, c, k0, ha, hap);
    dct3_herm(p2k, p2kp, c, k0, hb, hbp);
    bufa[k] = pack2(ha, hb);
    if (!self) bufa[kp] = pack2(hap, hbp);
    dct3_herm(Q1[k], Q1[kp], c, k0, ha, hap);
    dct3_herm(Q2[k], Q2[kp], c, k0, hb, hbp);
    bufb[k] = pack2(ha, hb);
    if (!self) bufb[kp] = pack2(hap, hbp);
    if (!DIFF) {
      dct3_herm(k0 ? 0.0f : wkp * p1kp, k0 ? 0.0f : wk * p1k, c, k0, ha, hap);
      dct3_herm(k0 ? 0.0f : wkp * p2kp, k0 ? 0.0f : wk * p2k, c, k0, hb, hbp);
      bufc[k] = pack2(ha, hb);
      if (!self) bufc[kp] = pack2(hap, hbp);
    } else {
      // Dx = DCT-III((cos w - 1) P) (bufc) - sine transform of sin(w) P (bufd)
      float dmk, dmkp, sw;
      diff_weights(c, dmk, dmkp, sw);
      dct3_herm(dmk * p1k, dmkp * p1kp, c, k0, ha, hap);
      dct3_herm(dmk * p2k, dmkp * p2kp, c, k0, hb, hbp);
      bufc[k] = pack2(ha, hb);
      if (!self) bufc[kp] = pack2(hap, hbp);
      dct3_herm(k0 ? 0.0f : sw * p1kp, k0 ? 0.0f : sw * p1k, c, k0, ha, hap);
      dct3_herm(k0 ? 0.0f : sw * p2kp, k0 ? 0.0f : sw * p2k, c, k0, hb, hbp);
      bufd[k] = pack2(ha, hb);
      if (!self) bufd[kp] = pack2(hap, hbp);
    }
  }
  block_lds_sync<NT>();
  block_fft<N, NT, true, DIFF ? 4 : 3>(bufa, bufb, bufc, bufd, tw, tid);
  double en[1] = {0.0};
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int ix = tid + NT * t;
    if (N % NT != 0 && ix >= N) continue;
    const int mpos = mk_pos<N>(ix);
    const float2 za = bufa[mpos], zb = bufb[mpos];
    const float sg = (ix & 1) ? -1.0f : 1.0f;
    float2 zc = bufc[mpos];
    if (DIFF) {
      // (Dx, Dy) instead of (Ex, Ey): zc holds Dx after the sign below
      const float2 zd = bufd[mpos];
      zc = make_float2(sg * (zc.x - sg * zd.x), sg * (zc.y - sg * zd.y));
    }
    const int64_t o1 = (int64_t)r1 * N + ix, o2 = (int64_t)r2 * N + ix;
    if (psi) {
      psi[o1] = za.x;
      psi[o2] = za.y;
    }
    if (ex) {
      ex[o1] = sg * zc.x;
      ex[o2] = sg * zc.y;
    }
    if (ey) {
      ey[o1] = zb.x;
      ey[o2] = zb.y;
    }
    if (exy) {
      exy[o1] = make_float2(sg * zc.x, zb.x);
      exy[o2] = make_float2(sg * zc.y, zb.y);
    }
    if (energy) en[0] += (double)e1[t] * za.x + (double)e2[t] * za.y;
  }
  if (energy) {
    block_sums<NT, 1>(en, red, tid);
    if (tid == 0) energy[pr] = en[0];   // per-block partial
  }
}

template <int N, int NB>
hipError_t run_fft_nb(Plan& p, const SpecBatch<NB>& sb, bool diff, bool rows, hipStream_t s) {
  const dim3 grid(N / 2, sb.count), block(FftShape<N>::NT);
  hipError_t e = hipSuccess;
  if (rows) {
    hipLaunchKernelGGL((k_rows_dct2<N, NB>), grid, block, 0, s, sb, p.fft_tw, p.dct_cs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    plan_mark(p, "k_rows_dct2", s);
  }
  if (diff)
    hipLaunchKernelGGL((k_cols_solve<N, true, NB>), grid, block, 0, s, sb, p.fft_tw, p.dct_cs,
                       p.wfreq);
  else
    hipLaunchKernelGGL((k_cols_solve<N, false, NB>), grid, block, 0, s, sb, p.fft_tw,
                       p.dct_cs, p.wfreq);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  plan_mark(p, "k_cols_solve", s);
  if (diff)
    hipLaunchKernelGGL((k_rows_inverse<N, true, NB>), grid, block, 0, s, sb, p.fft_tw,
                       p.dct_cs, p.wfreq);
  else
    hipLaunchKernelGGL((k_rows_inverse<N, false, NB>), grid, block, 0, s, sb, p.fft_tw,
                       p.dct_cs, p.wfreq);
  e = hipGetLastError();
  plan_mark(p, "k_rows_inverse", s);
  return e;
}

}  // namespace

// The descriptor of request a for the plan's batch slot `slot`.
SpecReq spec_req(Plan& p, const SpectralArgs& a, int slot) {
  const size_t nn = (size_t)p.n * p.n;
  SpecReq q;
  q.rho = a.rho;
  q.psi = a.psi;
  q.ex = a.ex;
  q.ey = a.ey;
  q.exy = reinterpret_cast<float2*>(a.exy);
  q.bT = p.tmp0 + slot * nn;
  q.rowsum = p.rowsum + (size_t)slot * p.n;
  q.P = p.tmp1 + slot * nn;
  q.Q = p.tmp2 + slot * nn;
  q.base = a.base;
  q.cap = a.cap;
  q.rho_t = a.rho_t;
  q.eps = a.eps;
  q.en_part = a.en_part;
  q.tau_part = a.tau_part;
  return q;
}

namespace {

template <int N>
hipError_t run_fft(Plan& p, const SpectralArgs* a, int count, bool rows, hipStream_t s) {
  if (count == 1) {
    SpecBatch<1> sb;
    sb.count = 1;
    sb.r[0] = spec_req(p, a[0], 0);
    return run_fft_nb<N, 1>(p, sb, a[0].diff, rows, s);
  }
  SpecBatch<kMaxBatch> sb;
  sb.count = count;
  for (int i = 0; i < count; ++i) sb.r[i] = spec_req(p, a[i], i);
  return run_fft_nb<N, kMaxBatch>(p, sb, a[0].diff, rows, s);
}

}  // namespace

hipError_t spectral_fft_batch(Plan& p, const SpectralArgs* a, int count, hipStream_t s,
                              bool rows) {
  if (count <= 0) return hipSuccess;
  if (count > p.max_batch) return hipErrorInvalidValue;
  for (int i = 1; i < count; ++i)
    if (a[i].diff != a[0].diff) return hipErrorInvalidValue;
  switch (p.n) {
    case 8: return run_fft<8>(p, a, count, rows, s);
    case 16: return run_fft<16>(p, a, count, rows, s);
    case 32: return run_fft<32>(p, a, count, rows, s);
    case 64: return run_fft<64>(p, a, count, rows, s);
    case 128: return run_fft<128>(p, a, count, rows, s);
    case 256: return run_fft<256>(p, a, count, rows, s);
    case 512: return run_fft<512>(p, a, count, rows, s);
    case 1024: return run_fft<1024>(p, a, count, rows, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t spectral_fft(Plan& p, const SpectralArgs& a, hipStream_t s) {
  return spectral_fft_batch(p, &a, 1, s);
}

}  // namespace fftpl
