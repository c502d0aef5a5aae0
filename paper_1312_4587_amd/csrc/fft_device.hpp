// Device code of the FFT solve shared by its passes and the compact evaluation
// kernels: 1-D transforms of a block in LDS, their pre- and post-processing,
// and the row transform of the first pass.
#pragma once

#include "fftpl_internal.hpp"

namespace fftpl {

constexpr int ilog2c(int v) { return v <= 1 ? 0 : 1 + ilog2c(v / 2); }

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Position of sample i in the even/odd reordered sequence.
template <int N>
__device__ __forceinline__ int mk_pos(int i) {
  return (i & 1) ? N - ((i + 1) >> 1) : (i >> 1);
}

// Threads per block for a length-N transform: one radix-4 butterfly per
// thread and stage at N = 1024 (four wavefronts), never less than one
// wavefront.
template <int N>
struct FftShape {
  static constexpr int NT = N / 4 >= 256 ? 256 : (N / 4 >= kWave ? N / 4 : kWave);
};

template <int NT>
__device__ __forceinline__ void block_lds_sync() {
  if constexpr (NT > kWave)
    __syncthreads();
  else
    wave_lds_sync();
}

// Unnormalised in-place DFTs of NB buffers of length N (b0..b{NB-1}) by a
// block of NT threads.  The buffers go through the stages together, so one
// barrier per stage serves all of them and each twiddle is read once for all.
// INV selects exp(+).  tw[t] = exp(-2 pi i t / N).
template <int N, int NT, bool INV, int NB>
__device__ __forceinline__ void block_fft(float2* b0, float2* b1, float2* b2, float2* b3,
                                          const float2* __restrict__ tw, int tid) {
  float2* const bufs[4] = {b0, b1, b2, b3};
  constexpr int LOG = ilog2c(N);
  int ns = 1;
  if constexpr (LOG & 1) {
    constexpr int B = N / 2;
    constexpr int PER = (B + NT - 1) / NT;
    float2 v0[NB][PER], v1[NB][PER];
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int t = 0; t < PER; ++t) {
        const int j = tid + NT * t;
        if (B % NT == 0 || j < B) {
          v0[q][t] = bufs[q][j];
          v1[q][t] = bufs[q][j + B];
        }
      }
    block_lds_sync<NT>();
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int t = 0; t < PER; ++t) {
        const int j = tid + NT * t;
        if (B % NT == 0 || j < B) {
          bufs[q][2 * j] = make_float2(v0[q][t].x + v1[q][t].x, v0[q][t].y + v1[q][t].y);
          bufs[q][2 * j + 1] = make_float2(v0[q][t].x - v1[q][t].x, v0[q][t].y - v1[q][t].y);
        }
      }
    block_lds_sync<NT>();
    ns = 2;
  }
  constexpr int B = N / 4;
  constexpr int PER = (B + NT - 1) / NT;
#pragma unroll
  for (int st = 0; st < LOG / 2; ++st) {
    float2 v[NB][PER][4];
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int t = 0; t < PER; ++t) {
        const int j = tid + NT * t;
        if (B % NT == 0 || j < B) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[q][t][r] = bufs[q][j + r * B];
        }
      }
    block_lds_sync<NT>();
    const int stride = N / (4 * ns);
#pragma unroll
    for (int t = 0; t < PER; ++t) {
      const int j = tid + NT * t;
      if (B % NT == 0 || j < B) {
        const int k = j & (ns - 1);
        float2 w[4];
        if (ns > 1) {
#pragma unroll
          for (int r = 1; r < 4; ++r) {
            w[r] = tw[k * r * stride];
            if (INV) w[r].y = -w[r].y;
          }
        }
        const int o = (j - k) * 4 + k;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
          float2* u = v[q][t];
          if (ns > 1) {
#pragma unroll
            for (int r = 1; r < 4; ++r) u[r] = cmul(u[r], w[r]);
          }
          const float2 t0 = make_float2(u[0].x + u[2].x, u[0].y + u[2].y);
          const float2 t1 = make_float2(u[0].x - u[2].x, u[0].y - u[2].y);
          const float2 t2 = make_float2(u[1].x + u[3].x, u[1].y + u[3].y);
          const float2 d = make_float2(u[1].x - u[3].x, u[1].y - u[3].y);
          // forward: t3 = -i * d ; inverse: t3 = +i * d
          const float2 t3 = INV ? make_float2(-d.y, d.x) : make_float2(d.y, -d.x);
          float2* b = bufs[q];
          b[o] = make_float2(t0.x + t2.x, t0.y + t2.y);
          b[o + ns] = make_float2(t1.x + t3.x, t1.y + t3.y);
          b[o + 2 * ns] = make_float2(t0.x - t2.x, t0.y - t2.y);
          b[o + 3 * ns] = make_float2(t1.x - t3.x, t1.y - t3.y);
        }
      }
    }
    block_lds_sync<NT>();
    ns *= 4;
  }
}

// Copy the twiddle table, the quarter-sample table cs and (WF) the frequency
// table wf into LDS.  All global loads are issued before the first LDS write,
// so the block waits on memory once; the caller synchronises.
template <int N, int NT, bool WF>
__device__ __forceinline__ void stage_tables(float2* tw, const float2* __restrict__ tw_g,
                                             float2* cs, const float2* __restrict__ cs_g,
                                             float* wf, const float* __restrict__ wf_g,
                                             int tid) {
  constexpr int PT = (N + NT - 1) / NT, PC = (N / 2 + NT) / NT;
  float2 a[PT], c[PC];
  float f[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    const int i = min(tid + NT * t, N - 1);
    a[t] = tw_g[i];
    if (WF) f[t] = wf_g[i];
  }
#pragma unroll
  for (int t = 0; t < PC; ++t) c[t] = cs_g[min(tid + NT * t, N / 2)];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    const int i = tid + NT * t;
    if (N % NT == 0 || i < N) {
      tw[i] = a[t];
      if (WF) wf[i] = f[t];
    }
  }
#pragma unroll
  for (int t = 0; t < PC; ++t) {
    const int i = tid + NT * t;
    if (i <= N / 2) cs[i] = c[t];
  }
}

// Sums over the block of K per-thread doubles, added in a fixed order, so
// every thread gets the same bits.  red holds K * NT / 64 doubles of LDS.
template <int NT, int K>
__device__ __forceinline__ void block_sums(double (&v)[K], double* red, int tid) {
  constexpr int NW = NT / kWave;
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = wave_sum_dpp_d(v[k]);
  if constexpr (NW > 1) {
    if ((tid & (kWave - 1)) == 0) {
#pragma unroll
      for (int k = 0; k < K; ++k) red[k * NW + tid / kWave] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += red[k * NW + w];
      v[k] = s;
    }
  }
}

// Forward post-processing for the pair (k, n-k) of a two-real-sequence FFT
// V = FFT(v1 + i v2): returns the DCT-II outputs X1, X2 at k and n-k.
// cs = (cos, sin)(pi k / 2n).
__device__ __forceinline__ void dct2_pair(float2 A, float2 B, float2 cs, float& x1k,
                                          float& x2k, float& x1kp, float& x2kp) {
  const float v1x = 0.5f * (A.x + B.x), v1y = 0.5f * (A.y - B.y);
  const float v2x = 0.5f * (A.y + B.y), v2y = -0.5f * (A.x - B.x);
  x1k = cs.x * v1x + cs.y * v1y;
  x2k = cs.x * v2x + cs.y * v2y;
  x1kp = cs.y * v1x - cs.x * v1y;
  x2kp = cs.y * v2x - cs.x * v2y;
}

// Hermitian input of a DCT-III of real coefficients Y at the pair (k, n-k):
// H_k = exp(i pi k / 2n) (Y_k - i Y_{n-k}) / 2, H_{n-k} = conj(H_k), H_0 = Y_0.
__device__ __forceinline__ void dct3_herm(float yk, float ykp, float2 cs, bool k0,
                                          float2& hk, float2& hkp) {
  if (k0) {
    hk = make_float2(yk, 0.0f);
    hkp = hk;
    return;
  }
  hk = make_float2(0.5f * (cs.x * yk + cs.y * ykp), 0.5f * (cs.y * yk - cs.x * ykp));
  hkp = make_float2(hk.x, -hk.y);
}

// z = ha + i hb
__device__ __forceinline__ float2 pack2(float2 ha, float2 hb) {
  return make_float2(ha.x - hb.y, ha.y + hb.x);
}

// Difference-mode weights at the pair (k, n-k) from cs = (cos, sin)(pi k / 2n):
// cos w_k - 1 = -2 sin^2(w_k / 2), cos w_{n-k} - 1 = -2 cos^2(w_k / 2),
// sin w_k = sin w_{n-k} = 2 sin(w_k / 2) cos(w_k / 2).
__device__ __forceinline__ void diff_weights(float2 cs, float& dm_k, float& dm_kp, float& sw) {
  dm_k = -2.0f * cs.y * cs.y;
  dm_kp = -2.0f * cs.x * cs.x;
  sw = 2.0f * cs.y * cs.x;
}

// LDS of the row transform of one row pair by NT threads.
template <int N, int NT>
struct RowsLds {
  double red[4 * (NT / kWave)];
  float2 buf[N];
  float2 tw[N];
  float2 cs[N / 2 + 1];
};

// First pass on the row pair (r1, r1 + 1) held by NT threads, thread tid with
// samples tid + NT t: a the rows' values, b and c the fixed charge and the
// capacity there (read for the overflow sums, tau_part set).  Writes the
// transposed DCT-II rows of bT, the double row sums and the overflow pair.
template <int N, int NT>
__device__ __forceinline__ void rows_dct2(
    const float (&a1)[(N + NT - 1) / NT], const float (&a2)[(N + NT - 1) / NT],
    const float (&b1)[(N + NT - 1) / NT], const float (&b2)[(N + NT - 1) / NT],
    const float (&c1)[(N + NT - 1) / NT], const float (&c2)[(N + NT - 1) / NT], int r1, int tid,
    RowsLds<N, NT>& lds, float* __restrict__ bT, double* __restrict__ rowsum,
    double* __restrict__ tau_part) {
  constexpr int PER = (N + NT - 1) / NT, PK = (N / 2 + NT) / NT;
  const int r2 = r1 + 1;
  double s[4] = {0.0, 0.0, 0.0, 0.0};   // row sums r1, r2; overflow; movable
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    if (N % NT == 0 || tid + NT * t < N) {
      s[0] += a1[t];
      s[1] += a2[t];
      if (tau_part) {
        const float m1 = a1[t] - b1[t], m2 = a2[t] - b2[t];
        s[2] += fmaxf(0.0f, m1 - c1[t]);
        s[2] += fmaxf(0.0f, m2 - c2[t]);
        s[3] += m1;
        s[3] += m2;
      }
    }
  }
  block_sums<NT, 4>(s, lds.red, tid);
  if (tid == 0) {
    rowsum[r1] = s[0];
    rowsum[r2] = s[1];
    if (tau_part) {
      tau_part[r1] = s[2];
      tau_part[r1 + 1] = s[3];
    }
  }
  const float m1 = (float)(s[0] / N), m2 = (float)(s[1] / N);
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int i = tid + NT * t;
    if (N % NT == 0 || i < N) lds.buf[mk_pos<N>(i)] = make_float2(a1[t] - m1, a2[t] - m2);
  }
  block_lds_sync<NT>();
  block_fft<N, NT, false, 1>(lds.buf, nullptr, nullptr, nullptr, lds.tw, tid);
#pragma unroll
  for (int t = 0; t < PK; ++t) {
    const int k = tid + NT * t;
    if (k > N / 2) continue;
    const int kp = (N - k) & (N - 1);
    float x1k, x2k, x1kp, x2kp;
    dct2_pair(lds.buf[k], lds.buf[kp], lds.cs[k], x1k, x2k, x1kp, x2kp);
    if (k == 0) {
      x1k = (float)s[0];
      x2k = (float)s[1];
    }
    *reinterpret_cast<float2*>(&bT[(int64_t)k * N + r1]) = make_float2(x1k, x2k);
    if (k != 0 && k != N / 2)
      *reinterpret_cast<float2*>(&bT[(int64_t)kp * N + r1]) = make_float2(x1kp, x2kp);
  }
}

}  // namespace fftpl
