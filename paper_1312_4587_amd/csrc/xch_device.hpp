// Device code of the pin exchange shared by its own kernels and the compact
// evaluation kernels: one net block, and the fixed-point pin sums of one cell
// block.
#pragma once

#include <math.h>

#include "fftpl_internal.hpp"

namespace fftpl {

constexpr int kXchSmallDeg = 8;   // degree handled by one thread
// B positions per thread of a net block: for blocks of up to kXchPinLds2 pins,
// or up to kXchPinCap
constexpr int kStageS = (kXchPinLds2 + kXchWaThreads - 1) / kXchWaThreads;
constexpr int kStageL = (kXchPinCap + kXchWaThreads - 1) / kXchWaThreads;
constexpr int kStageHold = 4;   // of them staged together in the compact kernels

// Weighted-average terms of one axis with the exponentials computed once:
// e+ = exp((X - M)/gamma), e- = exp((L - X)/gamma) (fast exp2-based exp: the
// arguments are <= 0 and the terms that matter are near 0).
__device__ __forceinline__ float fexp(float v) { return __expf(v); }

// T[a] = (x, y) of pin a's cell, over part b % SPLIT of the A range of cell block
// b / SPLIT, by NT threads; the cells' positions staged in win[CELLS].
template <int NT, int CELLS, int SPLIT>
__device__ __forceinline__ void spread_part(const XchReq& rq, int b, float2* win) {
  const int m = rq.m, cpb = rq.cpb;
  const int32_t* __restrict__ cb_a_ptr = rq.cb_a_ptr;
  const uint16_t* __restrict__ lc = rq.lc;
  const float* __restrict__ x = rq.x;
  const float* __restrict__ y = rq.y;
  float2* __restrict__ T = rq.T;
  const int cb = b / SPLIT, part = b % SPLIT;
  const int t = threadIdx.x;
  const int c0 = cb * cpb;
  const int nc = min(cpb, m - c0);
  {
    constexpr int W = CELLS / NT;
    float xv[W], yv[W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
      const int i = c0 + min(t + k * NT, nc - 1);
      xv[k] = x[i];
      yv[k] = y[i];
    }
#pragma unroll
    for (int k = 0; k < W; ++k)
      if (t + k * NT < nc) win[t + k * NT] = make_float2(xv[k], yv[k]);
  }
  __syncthreads();
  const int b0 = cb_a_ptr[cb], b1 = cb_a_ptr[cb + 1];
  const int len = (b1 - b0 + SPLIT - 1) / SPLIT;
  const int a0 = b0 + part * len, a1 = min(b1, a0 + len);
  if (a0 >= a1) return;
  // pairs of consecutive A positions aligned to 2, consecutive pairs on
  // consecutive lanes: one 4-byte load of their cell indices and one 16-byte
  // store of their positions per pair, both coalesced across the wavefront;
  // a pair straddling either end of the range is stored only inside it (its
  // index load stays inside the index allocation)
  const int g0 = a0 >> 1, g1 = (a1 + 1) >> 1;
  const uint32_t* lc2 = reinterpret_cast<const uint32_t*>(lc);
  float4* T2 = reinterpret_cast<float4*>(T);
  constexpr int U = 8;
  for (int g = g0 + t; g < g1; g += U * NT) {
    uint32_t q[U];
#pragma unroll
    for (int k = 0; k < U; ++k) q[k] = lc2[min(g + k * NT, g1 - 1)];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int gg = g + k * NT;
      if (gg >= g1) continue;
      const float2 v0 = win[min((int)(q[k] & 0xffffu), CELLS - 1)];
      const float2 v1 = win[min((int)(q[k] >> 16), CELLS - 1)];
      const int a = gg * 2;
      if (a >= a0 && a + 2 <= a1) {
        T2[gg] = make_float4(v0.x, v0.y, v1.x, v1.y);
      } else {
        if (a >= a0) T[a] = v0;
        if (a + 1 < a1) T[a + 1] = v1;
      }
    }
  }
}

// One net block: cell positions and pin offsets staged in LDS in CSR order,
// nets evaluated from LDS, gradients written to the pins' A positions in T.
// The positions come from T (written there by the spread, and overwritten by
// the gradients), or DIRECT from x and y by pin_cell: a design whose positions
// fit the L2 of every XCD needs no spread, and its pins are read in CSR order.
// LDS: pos[cap], off[cap] (dynamic, 16 bytes per pin of the block).
// LSE: the log-sum-exp model in place of the weighted average (same sums;
// the gradient is e+/S+ - e-/S-, the value (M - L) + gamma (ln S+ + ln S-)).
// Staging goes HOLD pins per thread at a time: with HOLD < STAGE chunks past the
// block's last pin are skipped, and only the first chunk's A positions are kept
// for the write-back (fewer registers, for blocks of mostly one chunk).
template <int STAGE, int HOLD, bool LSE, bool DIRECT>
__device__ __forceinline__ void wa_block(const XchReq& rq, int k, float2* smem) {
  constexpr int NW = kXchWaThreads, kSmall = kXchSmallDeg;
  const int t = threadIdx.x, nblk = rq.nnb;
  const int num_pins = rq.num_pins, cap = rq.cap;
  const int32_t* __restrict__ net_ptr = rq.net_ptr;
  const int32_t* __restrict__ nb_net_ptr = rq.nb_net_ptr;
  const uint32_t* __restrict__ nmeta = rq.nmeta;
  const int32_t* __restrict__ a_of_b = rq.a_of_b;
  const uint16_t* __restrict__ lcsr = rq.lcsr;
  const float* __restrict__ pin_dx = rq.pin_dx;
  const float* __restrict__ pin_dy = rq.pin_dy;
  const float gamma = rq.dgamma ? rq.dgamma[0] : rq.gamma;
  const float inv_gamma = rq.dgamma ? 1.0f / gamma : rq.inv_gamma;
  float2* __restrict__ T = rq.T;
  double* __restrict__ part = rq.part;
  double* __restrict__ net_wl = rq.net_wl;
  double* __restrict__ net_hp = rq.net_hp;
  float2* pos = smem;
  float2* off = smem + cap;
  __shared__ uint32_t bigmeta[NW];   // extents of the last NW nets of the order
  __shared__ int q_big, q_small;     // work counters
  const int lane = t & (kWave - 1), wv = t / kWave;
  const int e0 = nb_net_ptr[k], e1 = nb_net_ptr[k + 1];
  const int p0 = net_ptr[e0], p1 = net_ptr[e1];
  const int np = p1 - p0;
  double acc_wa = 0.0, acc_hp = 0.0;
  if (np > 0 && np <= cap && np <= STAGE * NW) {
    // 0. net extents, read before the staging loads so that the latency of
    // both overlaps: the last NW entries of the order (the large nets, largest
    // first) for LDS, and this wavefront's first chunk of small nets.
    const int nn = e1 - e0;
    constexpr int NWV = NW / kWave;
    const uint32_t* meta = nmeta + e0;
    const uint32_t mbig = meta[max(nn - 1 - t, 0)];
    const uint32_t msm0 = meta[min(wv * kWave + lane, nn - 1)];
    // 1. stage: off[csr offset] = pin offset (coalesced), pos[csr offset] =
    // cell position read from T in B order (runs of consecutive A positions).
    // Loads are unconditional (index clamped into the block) so that each
    // batch is in flight at once; only the LDS stores are masked.
    // (DIRECT: both in CSR order, positions by the pins' cells)
    int av[HOLD], lv[HOLD];
    const int blast = p1 - 1;
    if constexpr (DIRECT) {
      const int32_t* __restrict__ pin_cell = rq.pin_cell;
      const float* __restrict__ x = rq.x;
      const float* __restrict__ y = rq.y;
      const float2* __restrict__ xy = rq.xy;
      const unsigned mlast = (unsigned)(rq.m - 1);
#pragma unroll
      for (int j0 = 0; j0 < STAGE; j0 += HOLD) {
        if (j0 * NW >= np) break;
        float dx[HOLD], dy[HOLD];
        float2 q[HOLD];
        int c[HOLD];
#pragma unroll
        for (int j = 0; j < HOLD; ++j) {
          const int b = min(p0 + t + (j0 + j) * NW, blast);
          c[j] = pin_cell[b];
          dx[j] = pin_dx[b];
          dy[j] = pin_dy[b];
          if (j0 == 0) {
            av[j] = a_of_b[b];
            lv[j] = lcsr[b];
          }
        }
#pragma unroll
        for (int j = 0; j < HOLD; ++j) c[j] = (int)min((unsigned)c[j], mlast);
        if (xy) {
#pragma unroll
          for (int j = 0; j < HOLD; ++j) q[j] = xy[c[j]];
        } else {
#pragma unroll
          for (int j = 0; j < HOLD; ++j) q[j] = make_float2(x[c[j]], y[c[j]]);
        }
#pragma unroll
        for (int j = 0; j < HOLD; ++j) {
          const int l = t + (j0 + j) * NW;
          if (p0 + l < p1) {
            off[l] = make_float2(dx[j], dy[j]);
            pos[l] = q[j];
          }
        }
      }
    } else {
#pragma unroll
      for (int j0 = 0; j0 < STAGE; j0 += HOLD) {
        if (HOLD < STAGE && j0 * NW >= np) break;
        float dx[HOLD], dy[HOLD];
        int ai[HOLD], li[HOLD];
#pragma unroll
        for (int j = 0; j < HOLD; ++j) {
          const int b = min(p0 + t + (j0 + j) * NW, blast);
          ai[j] = a_of_b[b];
          li[j] = lcsr[b];
          dx[j] = pin_dx[b];
          dy[j] = pin_dy[b];
        }
#pragma unroll
        for (int j = 0; j < HOLD; ++j) {
          ai[j] = min((unsigned)ai[j], (unsigned)(num_pins - 1));
          li[j] = min(li[j], cap - 1);
        }
        float2 q[HOLD];
#pragma unroll
        for (int j = 0; j < HOLD; ++j) q[j] = T[ai[j]];
#pragma unroll
        for (int j = 0; j < HOLD; ++j) {
          const int l = t + (j0 + j) * NW;
          if (p0 + l < p1) {
            off[l] = make_float2(dx[j], dy[j]);
            pos[li[j]] = q[j];
          }
          if (j0 == 0) {
            av[j] = ai[j];
            lv[j] = li[j];
          }
        }
      }
    }
    bigmeta[t] = mbig;
    if (t == 0) {
      q_big = 0;
      q_small = NWV;   // chunks 0..NWV-1 are the wavefronts' first ones
    }
    __syncthreads();

    // 2. nets in degree order, work handed out by block-wide counters so
    // that every wavefront stays busy until the block's nets run out.  Nets
    // above kSmall sit at the back of the order, largest class last: each is
    // taken by one wavefront, largest first (three passes over its pins in
    // LDS: pass 1 turns positions into pin coordinates relative to the first
    // pin's cell, pass 3 overwrites them with the gradient).  Then the
    // others: one lane per net, a wavefront per chunk of kWave nets of
    // (nearly) equal degree, loops as long as the chunk's largest degree.
    for (;;) {
      int j = 0;
      if (lane == 0) j = atomicAdd(&q_big, 1);
      j = __builtin_amdgcn_readfirstlane(j);
      if (j >= nn) break;
      // beyond the NW staged extents (more than NW large nets): from memory
      const uint32_t mj = j < NW ? bigmeta[j] : meta[nn - 1 - j];
      const int deg = (int)(mj & 0xffffu);
      if (deg <= kSmall) break;   // every net left is small
      // extents come from the index; kept inside the staged pins whatever it
      // holds, so a block never leaves its LDS
      const int b0 = min((int)(mj >> 16), np - 1), b1 = min(b0 + deg, np);
      const float2 r = pos[b0];
      wave_lds_sync();
      constexpr int H = 4;   // pins per lane whose LDS loads are issued together
      float mx = -INFINITY, lx = INFINITY, my = -INFINITY, ly = INFINITY;
      for (int l = b0 + lane; l < b1; l += H * kWave) {
        float2 c[H], d[H];
#pragma unroll
        for (int u = 0; u < H; ++u) {
          const int li = min(l + u * kWave, b1 - 1);
          c[u] = pos[li];
          d[u] = off[li];
        }
#pragma unroll
        for (int u = 0; u < H; ++u) {
          if (l + u * kWave < b1) {
            const float X = (c[u].x - r.x) + d[u].x, Y = (c[u].y - r.y) + d[u].y;
            pos[l + u * kWave] = make_float2(X, Y);
            mx = fmaxf(mx, X);
            lx = fminf(lx, X);
            my = fmaxf(my, Y);
            ly = fminf(ly, Y);
          }
        }
      }
      mx = wave_max_dpp(mx);
      lx = wave_min_dpp(lx);
      my = wave_max_dpp(my);
      ly = wave_min_dpp(ly);
      wave_lds_sync();
      float spx = 0.f, tpx = 0.f, smx = 0.f, tmx = 0.f;
      float spy = 0.f, tpy = 0.f, smy = 0.f, tmy = 0.f;
      for (int l = b0 + lane; l < b1; l += H * kWave) {
        float2 c[H];
#pragma unroll
        for (int u = 0; u < H; ++u) c[u] = pos[min(l + u * kWave, b1 - 1)];
#pragma unroll
        for (int u = 0; u < H; ++u) {
          if (l + u * kWave < b1) {
            float dd = c[u].x - mx, ee = fexp(dd * inv_gamma);
            spx += ee;
            tpx += dd * ee;
            dd = c[u].x - lx;
            ee = fexp(-dd * inv_gamma);
            smx += ee;
            tmx += dd * ee;
            dd = c[u].y - my;
            ee = fexp(dd * inv_gamma);
            spy += ee;
            tpy += dd * ee;
            dd = c[u].y - ly;
            ee = fexp(-dd * inv_gamma);
            smy += ee;
            tmy += dd * ee;
          }
        }
      }
      spx = wave_sum_dpp(spx);
      tpx = wave_sum_dpp(tpx);
      smx = wave_sum_dpp(smx);
      tmx = wave_sum_dpp(tmx);
      spy = wave_sum_dpp(spy);
      tpy = wave_sum_dpp(tpy);
      smy = wave_sum_dpp(smy);
      tmy = wave_sum_dpp(tmy);
      const float rspx = 1.0f / spx, rsmx = 1.0f / smx;
      const float rspy = 1.0f / spy, rsmy = 1.0f / smy;
      const float wpx = tpx * rspx, wmx = tmx * rsmx;
      const float wpy = tpy * rspy, wmy = tmy * rsmy;
      for (int l = b0 + lane; l < b1; l += H * kWave) {
        float2 c[H];
#pragma unroll
        for (int u = 0; u < H; ++u) c[u] = pos[min(l + u * kWave, b1 - 1)];
#pragma unroll
        for (int u = 0; u < H; ++u) {
          if (l + u * kWave < b1) {
            const float dpx = c[u].x - mx, dmx = c[u].x - lx;
            const float dpy = c[u].y - my, dmy = c[u].y - ly;
            if (LSE)
              pos[l + u * kWave] = make_float2(
                  fexp(dpx * inv_gamma) * rspx - fexp(-dmx * inv_gamma) * rsmx,
                  fexp(dpy * inv_gamma) * rspy - fexp(-dmy * inv_gamma) * rsmy);
            else
              pos[l + u * kWave] = make_float2(
                  fexp(dpx * inv_gamma) * rspx * (1.0f + (dpx - wpx) * inv_gamma) -
                      fexp(-dmx * inv_gamma) * rsmx * (1.0f - (dmx - wmx) * inv_gamma),
                  fexp(dpy * inv_gamma) * rspy * (1.0f + (dpy - wpy) * inv_gamma) -
                      fexp(-dmy * inv_gamma) * rsmy * (1.0f - (dmy - wmy) * inv_gamma));
          }
        }
      }
      if (lane == 0) {
        const double vw = net_wl_value<LSE>(mx, lx, wpx, wmx, spx, smx, gamma) +
                          net_wl_value<LSE>(my, ly, wpy, wmy, spy, smy, gamma);
        const double vh = (double)(mx - lx) + (double)(my - ly);
        acc_wa += vw;
        acc_hp += vh;
        if (net_wl) {
          net_wl[p0 + b0] = vw;
          net_hp[p0 + b0] = vh;
        }
      }
    }

    // small nets: chunk c holds order entries c * kWave + lane; a
    // wavefront's first chunk is its own (extents read before staging), the
    // rest come from the counter, each one's extents read while the previous
    // chunk is evaluated
    int cc = wv;
    uint32_t mcur = msm0;
    for (;;) {
      if (cc * kWave >= nn) break;
      int cn = 0;
      if (lane == 0) cn = atomicAdd(&q_small, 1);
      cn = __builtin_amdgcn_readfirstlane(cn);
      uint32_t mnext = 0u;
      if (cn * kWave < nn) mnext = meta[min(cn * kWave + lane, nn - 1)];
      const int li = cc * kWave + lane;
      int deg = li < nn ? (int)(mcur & 0xffffu) : 0;
      if (deg > kSmall) deg = 0;   // done above
      // kept inside the staged pins whatever the index holds
      const int l0 = min((int)(mcur >> 16), np - 1);
      deg = min(deg, np - l0);
      // the chunk's largest small degree, uniform across the wavefront
      const int wdeg = wave_max_dpp_i(deg);
      if (deg == 1) {
        // a one-pin net: no gradient, zero wirelength and half-perimeter
        pos[l0] = make_float2(0.0f, 0.0f);
        if (net_wl) {
          net_wl[p0 + l0] = 0.0;
          net_hp[p0 + l0] = 0.0;
        }
      }
      if (wdeg >= 2) {
        float px[kSmall], py[kSmall];
        const float2 r = pos[deg >= 1 ? l0 : 0];
        float mx = -INFINITY, lx = INFINITY, my = -INFINITY, ly = INFINITY;
#pragma unroll
        for (int j = 0; j < kSmall; ++j) {
          if (j < wdeg) {
            px[j] = 0.0f;
            py[j] = 0.0f;
            if (j < deg) {
              const float2 c = pos[l0 + j], d = off[l0 + j];
              px[j] = (c.x - r.x) + d.x;
              py[j] = (c.y - r.y) + d.y;
              mx = fmaxf(mx, px[j]);
              lx = fminf(lx, px[j]);
              my = fmaxf(my, py[j]);
              ly = fminf(ly, py[j]);
            }
          }
        }
        float epx[kSmall], emx[kSmall], epy[kSmall], emy[kSmall];
        float spx = 0.f, tpx = 0.f, smx = 0.f, tmx = 0.f;
        float spy = 0.f, tpy = 0.f, smy = 0.f, tmy = 0.f;
#pragma unroll
        for (int j = 0; j < kSmall; ++j) {
          if (j < wdeg) {
            const bool in = j < deg;
            const float dpx = px[j] - mx, dmx = px[j] - lx;
            const float dpy = py[j] - my, dmy = py[j] - ly;
            epx[j] = in ? fexp(dpx * inv_gamma) : 0.0f;
            emx[j] = in ? fexp(-dmx * inv_gamma) : 0.0f;
            epy[j] = in ? fexp(dpy * inv_gamma) : 0.0f;
            emy[j] = in ? fexp(-dmy * inv_gamma) : 0.0f;
            spx += epx[j];
            tpx += dpx * epx[j];
            smx += emx[j];
            tmx += dmx * emx[j];
            spy += epy[j];
            tpy += dpy * epy[j];
            smy += emy[j];
            tmy += dmy * emy[j];
          }
        }
        if (deg >= 2) {
          const float rspx = 1.0f / spx, rsmx = 1.0f / smx;
          const float rspy = 1.0f / spy, rsmy = 1.0f / smy;
          const float wpx = tpx * rspx, wmx = tmx * rsmx;
          const float wpy = tpy * rspy, wmy = tmy * rsmy;
#pragma unroll
          for (int j = 0; j < kSmall; ++j) {
            if (j < wdeg && j < deg) {
              const float dpx = px[j] - mx, dmx = px[j] - lx;
              const float dpy = py[j] - my, dmy = py[j] - ly;
              if (LSE)
                pos[l0 + j] = make_float2(epx[j] * rspx - emx[j] * rsmx,
                                          epy[j] * rspy - emy[j] * rsmy);
              else
                pos[l0 + j] = make_float2(
                    epx[j] * rspx * (1.0f + (dpx - wpx) * inv_gamma) -
                        emx[j] * rsmx * (1.0f - (dmx - wmx) * inv_gamma),
                    epy[j] * rspy * (1.0f + (dpy - wpy) * inv_gamma) -
                        emy[j] * rsmy * (1.0f - (dmy - wmy) * inv_gamma));
            }
          }
          const double vw = net_wl_value<LSE>(mx, lx, wpx, wmx, spx, smx, gamma) +
                            net_wl_value<LSE>(my, ly, wpy, wmy, spy, smy, gamma);
          const double vh = (double)(mx - lx) + (double)(my - ly);
          acc_wa += vw;
          acc_hp += vh;
          if (net_wl) {
            net_wl[p0 + l0] = vw;
            net_hp[p0 + l0] = vh;
          }
        }
      }
      cc = cn;
      mcur = mnext;
    }
    __syncthreads();

    // 3. gradients to the pins' A positions
#pragma unroll
    for (int j0 = 0; j0 < STAGE; j0 += HOLD) {
      if (HOLD < STAGE && j0 * NW >= np) break;
#pragma unroll
      for (int j = 0; j < HOLD; ++j) {
        if (j0 > 0) {
          const int b = min(p0 + t + (j0 + j) * NW, blast);
          av[j] = a_of_b[b];
          lv[j] = lcsr[b];
        }
      }
#pragma unroll
      for (int j = 0; j < HOLD; ++j)
        if (p0 + t + (j0 + j) * NW < p1)
          T[min((unsigned)av[j], (unsigned)(num_pins - 1))] = pos[min(lv[j], cap - 1)];
    }
  }
  // the block's totals: both sums through one barrier
  __shared__ double red[2][NW / kWave];
  acc_wa = wave_sum_dpp_d(acc_wa);
  acc_hp = wave_sum_dpp_d(acc_hp);
  if (lane == 0) {
    red[0][wv] = acc_wa;
    red[1][wv] = acc_hp;
  }
  __syncthreads();
  if (t < 2) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NW / kWave; ++w) s += red[t][w];
    part[t == 0 ? k : nblk + k] = s;
  }
}

// Adds the gradients T of a cell block's A range [a0, a1) to its cells'
// fixed-point accumulators ax, ay (units of 1 / scale; cleared by the caller) by
// NTS threads; a non-finite gradient marks its cell in bad.  prefetch() issues
// the first group's loads, before the clear.
template <int NTS, int CELLS>
struct PinSums {
  static constexpr int U = 4, STEP = U * NTS;
  // two groups of U pairs per thread in flight: the next group's loads are
  // issued before the current group's adds
  uint32_t q[U], qn[U];
  float4 v[U], vn[U];
  const uint32_t* lc2;
  const float4* T2;
  int a0, a1, g1, g;
  __device__ __forceinline__ void fetch(uint32_t (&qq)[U], float4 (&vv)[U], int gi) {
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int gg = min(gi + k * NTS, g1 - 1);
      qq[k] = lc2[gg];
      vv[k] = T2[gg];
    }
  }
  // pairs of consecutive A positions aligned to 2, consecutive pairs on
  // consecutive lanes (one 4-byte load of their cell indices and one 16-byte
  // load of their gradients, coalesced); positions outside the range are
  // skipped (the loads of a straddling pair stay inside the allocations)
  __device__ __forceinline__ void prefetch(const uint16_t* lc, const float2* T, int a0_, int a1_) {
    lc2 = reinterpret_cast<const uint32_t*>(lc);
    T2 = reinterpret_cast<const float4*>(T);
    a0 = a0_;
    a1 = a1_;
    g1 = (a1 + 1) >> 1;
    g = (a0 >> 1) + (int)threadIdx.x;
    if (g < g1) fetch(q, v, g);
  }
  __device__ __forceinline__ void add(float scale, unsigned long long* ax, unsigned long long* ay,
                                      unsigned char* bad) {
    for (; g < g1; g += STEP) {
      if (g + STEP < g1) fetch(qn, vn, g + STEP);
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int gg = g + k * NTS;
        if (gg >= g1) continue;
        const int a = gg * 2;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          if (a + e < a0 || a + e >= a1) continue;
          const int l = min((int)(e ? q[k] >> 16 : q[k] & 0xffffu), CELLS - 1);
          const float gxv = e ? v[k].z : v[k].x, gyv = e ? v[k].w : v[k].y;
          if (fabsf(gxv) <= 3.0e38f && fabsf(gyv) <= 3.0e38f) {
            atomicAdd(&ax[l], (unsigned long long)(long long)__float2int_rn(gxv * scale));
            atomicAdd(&ay[l], (unsigned long long)(long long)__float2int_rn(gyv * scale));
          } else {
            bad[l] = 1;
          }
        }
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        q[k] = qn[k];
        v[k] = vn[k];
      }
    }
  }
};

// One cell's fixed-point sum back to float.
__device__ __forceinline__ float pin_sum(unsigned long long a, unsigned char bad,
                                         double inv_scale) {
  return bad ? __builtin_nanf("") : (float)((double)(long long)a * inv_scale);
}

}  // namespace fftpl
