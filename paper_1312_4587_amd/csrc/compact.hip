// The compact evaluation: the exchange path of designs whose kernels are all
// shorter than the work of launching them.
//
// The general exchange path runs nine kernels on two streams.  Up to a million
// cells each of them lasts 3 to 30 us, much of it the latency of a few dependent
// loads, and the host enqueues the nine launches and the four cross-stream event
// calls in 75 to 89 us, for small designs longer than the device evaluates.  Here the
// same steps take four to six launches (more with the matrix-core solve) on the
// caller's stream alone:
//   place  the counting sort of the cells by band (k_band_place), skipped up to
//          kScanCells cells (n <= 512), whose band blocks read every cell; past
//          kCompactDirectCells cells or kCompactDirectPins pins with the spread
//          beside it (k_compact_place);
//   mid    band blocks: scatter of a row pair, and for FFT plans its row transform
//          straight from LDS (past n = 512 of up to four rows, the row pass on its
//          own, as for n < 64); beside them in the same launch the net blocks, which
//          up to that many cells and pins read the positions by cell, from the L2 of
//          every XCD, so that neither a spread nor a second stream is needed;
//   solve  the column and the inverse row pass (or the matrix-core solve);
//   cells  per cell the density gradient gathered from the field map (it fits the
//          L2 too, or nearly) and the sum of its pins' gradients; one more block
//          per design sums the scalars.
// Every per-cell, per-bin and per-net value is computed by the same code and
// in the same order as on the general path.
// Per evaluation, general -> compact, one after another: 2k cells (n = 64) 77.8
// -> 20.3 us, 30k (n = 256, exact, LSE) 71.5 -> 29.1, 200k (n = 512) 78.3 -> 49.1,
// 500k (n = 1024) 106 -> 88, clustered 111 -> 85, eight of 17k to 62k cells in a batch
// 172 -> 61.  What bounds it now is the device: at 200k cells place 7, mid 21, columns
// 7, inverse rows 6, cells 9 us; at 500k place 11, mid 26, rows 9, columns 13, inverse
// rows 10, cells 19.
#include <algorithm>

#include "band_device.hpp"
#include "fft_device.hpp"
#include "xch_device.hpp"

namespace fftpl {

namespace {

constexpr int NT = kXchWaThreads;   // the net blocks' threads, and the band blocks'
constexpr int KB = 4;               // band entries a thread takes together
constexpr int kList = 4 * NT;       // cells of a scanning band block's list
// bins of a band: a row pair for n <= 512, up to four rows above
constexpr int kBinsPair = 2 * kCompactPairN, kBinsMax = 4096;

// LDS of a band block: the accumulators, then the scatter's arrays or the
// row transform's (N = 0: no transform).
template <int N, int BINS>
struct MidLds {
  unsigned long long acc[BINS];
  union {
    WalkLds<NT, KB> walk;
    ScanLds<NT, kList> scan;
    RowsLds<N ? N : 8, NT> rows;
  };
};

// The place pass and, beside it in the same launch, the spread of the positions to
// the pins: past kCompactDirectCells the positions and the rest of a net block's
// data no longer fit an XCD's L2 together, and reading them by pin costs more
// than the spread (net blocks of 500k cells, n = 1024: 34 us against 17 us).
template <int NB>
struct PlaceBatch {
  int nblk = 0;
  BandReq r[NB];
  XchReq x[NB];
};
// CB: cells per thread of a place block; CELLS: most cells of a spread block.
template <int NB, int CB, int CELLS>
__global__ void __launch_bounds__(kBandThreads) k_compact_place(PlaceBatch<NB> pb) {
  __shared__ float2 win[CELLS];
  const int b = (int)blockIdx.x - pb.nblk;
  if (b < 0) {
    const BandReq& q = pb.r[blockIdx.y];
    if (q.L.m > 0 && (int)blockIdx.x < q.L.nblk)
      place_block<CB>(q.g, q.L, blockIdx.x, q.x, q.y, q.w, q.h);
    return;
  }
  const XchReq& rq = pb.x[blockIdx.y];
  const int nb = rq.ncb * kXchSpreadSplit;
  if (b < nb)
    spread_part<kBandThreads, CELLS, kXchSpreadSplit>(rq, xcd_order(b, nb), win);
}

// DIRECT: six wavefronts per SIMD, three blocks of 512 threads per CU instead of
// the two that 94 registers leave (27.7 -> 23.9 us at 200k cells).  Spread
// positions: two blocks per CU, every pin staged in one round, and neighbouring net
// blocks on one XCD for the runs they share (30.5 -> 25.4 us at 500k cells, n =
// 1024; the whole evaluation 93.3 -> 87.7).
template <int N, int BINS, bool LSE, bool DIRECT, int NB>
__global__ void __launch_bounds__(NT, DIRECT ? 6 : 4) k_compact_mid(CompactBatch<NB> cb,
                                                    const float2* __restrict__ tw_g,
                                                    const float2* __restrict__ cs_g) {
  // (16 bytes: the scan's list is read and written in float4)
  extern __shared__ __align__(16) float2 smem[];
  static_assert(alignof(MidLds<N, BINS>) <= 16, "as aligned as smem");
  const CompactReq& q = cb.r[blockIdx.y];
  if ((int)blockIdx.x >= cb.nb) {
    const int k = (int)blockIdx.x - cb.nb;
    constexpr int HOLD = DIRECT ? kStageHold : kStageS;
    if (k < q.x.nnb)
      wa_block<kStageS, HOLD, LSE, DIRECT>(q.x, DIRECT ? k : xcd_order(k, q.x.nnb), smem);
    return;
  }
  MidLds<N, BINS>& lds = *reinterpret_cast<MidLds<N, BINS>*>(smem);
  const int t = threadIdx.x;
  const GridF& g = q.g;
  const int n = g.n, R = q.rows, band = xcd_order(blockIdx.x, cb.nb), r0 = band * R;
  const int bins = min(R, n - r0) * n;
  const size_t o = (size_t)r0 * n;
  // fixed charge and capacity of the thread's bins, in flight during the scatter
  constexpr int PA = BINS / NT;
  float bv[PA], cv[PA];
#pragma unroll
  for (int j = 0; j < PA; ++j) bv[j] = q.base ? q.base[o + min(t + j * NT, bins - 1)] : 0.0f;
  if constexpr (N > 0) {
    if (q.cap) {
#pragma unroll
      for (int j = 0; j < PA; ++j) cv[j] = q.cap[o + min(t + j * NT, bins - 1)];
    } else {
#pragma unroll
      for (int j = 0; j < PA; ++j)
        cv[j] = fmaxf(0.0f, g.rho_t - fminf(g.rho_t, bv[j]));
    }
  }
  for (int k = t; k < bins; k += NT) lds.acc[k] = 0ull;
  __syncthreads();
  if (q.nblk > 0)
    band_accumulate<NT, KB, BINS == kBinsPair>(g, q, band, q.x.x, q.x.y, q.w, q.h, lds.acc, lds.walk);
  else
    band_scan<NT, kList>(g, q, band, q.x.x, q.x.y, q.w, q.h, lds.acc, lds.scan);
  __syncthreads();
  float rho[PA];
#pragma unroll
  for (int j = 0; j < PA; ++j) {
    const int k = t + j * NT;
    rho[j] = bv[j] + (float)((double)lds.acc[min(k, bins - 1)] * kAccUnit);
    if (k < bins) q.rho[o + k] = rho[j];
  }
  if constexpr (N > 0) {
    // the row pair's transform: rows of N = 512 lie one sample per thread as
    // they are; shorter rows go back through LDS
    static_assert(N <= NT && PA == 2, "one sample of each row per thread");
    float a1[1], a2[1], b1[1], b2[1], c1[1], c2[1];
    stage_tables<N, NT, false>(lds.rows.tw, tw_g, lds.rows.cs, cs_g, nullptr, nullptr, t);
    if constexpr (N == NT) {
      a1[0] = rho[0];
      a2[0] = rho[1];
      b1[0] = bv[0];
      b2[0] = bv[1];
      c1[0] = cv[0];
      c2[0] = cv[1];
    } else {
      float* f = reinterpret_cast<float*>(lds.acc);
      static_assert(6 * N * sizeof(float) <= sizeof(lds.acc), "three row pairs fit");
      __syncthreads();   // every accumulator is read
#pragma unroll
      for (int j = 0; j < PA; ++j) {
        const int k = t + j * NT;
        if (k < 2 * N) {
          f[k] = rho[j];
          f[2 * N + k] = bv[j];
          f[4 * N + k] = cv[j];
        }
      }
      __syncthreads();
      const int i = min(t, N - 1);
      a1[0] = f[i];
      a2[0] = f[N + i];
      b1[0] = f[2 * N + i];
      b2[0] = f[3 * N + i];
      c1[0] = f[4 * N + i];
      c2[0] = f[5 * N + i];
    }
    rows_dct2<N, NT>(a1, a2, b1, b2, c1, c2, r0, t, lds.rows, q.bT, q.rowsum, q.tau_part);
  }
}

// TC threads, PC cells per thread: (256, 1), (512, 1), (1024, 1), (1024, 2) or (1024, 4), the
// smallest that holds a cell block.  A block of one cell per thread is a short
// chain of loads, and its registers and LDS leave room for several blocks per CU
// (eight designs of up to 62k cells 22.3 -> 17.1 us); the larger blocks, one per
// CU, take 1024 threads for the map reads in flight (500k cells, n = 1024: 25.0 ->
// 20.4 us against (512, 4)).
template <int MODE, int NB, int TC, int PC>
__global__ void __launch_bounds__(TC) k_compact_cells(SumBatch<NB> sb) {
  const SumReq& rq = sb.r[blockIdx.y];
  const int cb = blockIdx.x, t = threadIdx.x;
  const CellGradArgs& a = rq.a;
  if (cb >= rq.ncb) {
    // the block past the design's last cell block sums its scalars
    if (cb == rq.ncb) eval_scalars<TC>(a.fin);
    return;
  }
  constexpr int CELLS = TC * PC;
  __shared__ unsigned long long ax[CELLS], ay[CELLS];
  __shared__ unsigned char bad[CELLS];
  const int m = rq.m, cpb = rq.cpb, c0 = cb * cpb;
  const int a0 = rq.cb_a_ptr[cb], a1 = rq.cb_a_ptr[cb + 1];
  float x[PC], y[PC], w[PC], h[PC];
#pragma unroll
  for (int k = 0; k < PC; ++k) {
    if (k * TC >= cpb) break;
    const int ci = min(c0 + t + k * TC, m - 1);
    x[k] = a.x[ci];
    y[k] = a.y[ci];
    w[k] = a.w[ci];
    h[k] = a.h[ci];
  }
  const float lam = a.dscale ? a.dscale[0] : a.scale;
  PinSums<TC, CELLS> pins;
  pins.prefetch(rq.lc, rq.T, a0, a1);
  for (int c = t; c < cpb; c += TC) {
    ax[c] = 0ull;
    ay[c] = 0ull;
    bad[c] = 0;
  }
  // density part while the accumulators are cleared, of the block's own cells only (in
  // a batch the kernel's block is sized for the largest design: a design of 3000
  // cells 18 bins wide, n = 1024, beside one of 1M held the kernel for 360 us)
  float2 d[PC];
#pragma unroll
  for (int k = 0; k < PC; ++k) {
    if (t + k * TC >= cpb) break;
    const Span sx = cell_span(x[k], w[k], a.g.xl, a.g.inv_bw, a.g.n);
    const Span sy = cell_span(y[k], h[k], a.g.yl, a.g.inv_bh, a.g.n);
    d[k] = density_grad_small<MODE>(a.g, sx, sy, a.exy, a.psi);
  }
  __syncthreads();
  pins.add(rq.fx_scale, ax, ay, bad);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PC; ++k) {
    const int c = t + k * TC, ci = c0 + c;
    if (c >= cpb || ci >= m) break;
    a.gx[ci] = lam * d[k].x + pin_sum(ax[c], bad[c], rq.inv_scale);
    a.gy[ci] = lam * d[k].y + pin_sum(ay[c], bad[c], rq.inv_scale);
  }
}

template <int NB>
hipError_t place_batch(const BandReq* br, const XchReq* xr, int count, hipStream_t s) {
  PlaceBatch<NB> pb;
  static_assert(sizeof(pb) <= 4096, "kernel arguments");
  int max_nblk = 0, max_ncb = 0, max_cpk = 0, max_cpb = 0;
  for (int i = 0; i < count; ++i) {
    pb.r[i] = br[i];
    pb.x[i] = xr[i];
    max_cpk = std::max(max_cpk, br[i].L.cpk);
    max_cpb = std::max(max_cpb, xr[i].cpb);
    if (br[i].L.m > 0) max_nblk = std::max(max_nblk, br[i].L.nblk);
    max_ncb = std::max(max_ncb, xr[i].ncb);
  }
  pb.nblk = max_nblk;
  if (max_cpk > kCellBatch * kBandThreads || max_cpb > kCompactMaxCpb)
    return hipErrorInvalidValue;
  const dim3 grid(max_nblk + max_ncb * kXchSpreadSplit, count), block(kBandThreads);
  if (max_cpk <= 4 * kBandThreads && max_cpb <= 2048)
    hipLaunchKernelGGL((k_compact_place<NB, 4, 2048>), grid, block, 0, s, pb);
  else
    hipLaunchKernelGGL((k_compact_place<NB, kCellBatch, kCompactMaxCpb>), grid, block, 0, s, pb);
  return hipGetLastError();
}

template <int N, int BINS, bool LSE, bool DIRECT, int NB>
hipError_t mid_launch(const Plan& p, const CompactBatch<NB>& cb, int max_nnb, int max_cap,
                      bool scan, hipStream_t s) {
  using L = MidLds<N, BINS>;
  size_t lds = sizeof(L::acc) + std::max(sizeof(L::walk), sizeof(L::rows));
  if (scan) lds = sizeof(L);
  lds = std::max(lds, sizeof(float2) * 2 * (size_t)max_cap);
  hipLaunchKernelGGL((k_compact_mid<N, BINS, LSE, DIRECT, NB>), dim3(cb.nb + max_nnb, cb.count),
                     dim3(NT), lds, s, cb, p.fft_tw, p.dct_cs);
  return hipGetLastError();
}

template <bool LSE, bool DIRECT, int NB>
hipError_t mid_size(const Plan& p, const CompactBatch<NB>& cb, int max_nnb, int max_cap,
                    bool scan, bool fuse_rows, hipStream_t s) {
  constexpr int B = kBinsPair;
  if (p.n > kCompactPairN)
    return mid_launch<0, kBinsMax, LSE, DIRECT, NB>(p, cb, max_nnb, max_cap, scan, s);
  switch (fuse_rows ? p.n : 0) {
    case 64: return mid_launch<64, B, LSE, DIRECT, NB>(p, cb, max_nnb, max_cap, scan, s);
    case 128: return mid_launch<128, B, LSE, DIRECT, NB>(p, cb, max_nnb, max_cap, scan, s);
    case 256: return mid_launch<256, B, LSE, DIRECT, NB>(p, cb, max_nnb, max_cap, scan, s);
    case 512: return mid_launch<512, B, LSE, DIRECT, NB>(p, cb, max_nnb, max_cap, scan, s);
    default: return mid_launch<0, B, LSE, DIRECT, NB>(p, cb, max_nnb, max_cap, scan, s);
  }
}

template <bool LSE, int NB>
hipError_t mid_form(const Plan& p, const CompactBatch<NB>& cb, int max_nnb, int max_cap,
                    bool scan, bool fuse_rows, bool spread, hipStream_t s) {
  return spread ? mid_size<LSE, false, NB>(p, cb, max_nnb, max_cap, scan, fuse_rows, s)
                : mid_size<LSE, true, NB>(p, cb, max_nnb, max_cap, scan, fuse_rows, s);
}

template <int NB>
hipError_t mid_batch(const Plan& p, const CompactReq* reqs, int count, int wl_model,
                     bool fuse_rows, bool spread, hipStream_t s) {
  CompactBatch<NB> cb;
  cb.count = count;
  cb.nb = reqs[0].nb;
  int max_nnb = 0, max_cap = 1;
  bool scan = false;
  for (int i = 0; i < count; ++i) {
    cb.r[i] = reqs[i];
    max_nnb = std::max(max_nnb, reqs[i].x.nnb);
    max_cap = std::max(max_cap, reqs[i].x.cap);
    scan = scan || reqs[i].nblk == 0;
  }
  if (max_cap > kXchPinLds2) return hipErrorInvalidValue;
  return wl_model == FFTPL_WL_LSE
             ? mid_form<true, NB>(p, cb, max_nnb, max_cap, scan, fuse_rows, spread, s)
             : mid_form<false, NB>(p, cb, max_nnb, max_cap, scan, fuse_rows, spread, s);
}

template <int NB, int TC, int PC>
hipError_t cells_launch(const SumBatch<NB>& sb, int max_ncb, int grad_mode, hipStream_t s) {
  const dim3 grid(max_ncb + 1, sb.count), block(TC);
  if (grad_mode == FFTPL_GRAD_EXACT)
    hipLaunchKernelGGL((k_compact_cells<FFTPL_GRAD_EXACT, NB, TC, PC>), grid, block, 0, s, sb);
  else
    hipLaunchKernelGGL((k_compact_cells<FFTPL_GRAD_FIELD, NB, TC, PC>), grid, block, 0, s, sb);
  return hipGetLastError();
}

template <int NB>
hipError_t cells_batch(const SumReq* reqs, int count, int grad_mode, hipStream_t s) {
  SumBatch<NB> sb;
  sb.count = count;
  int max_ncb = 0, max_cpb = 0;
  for (int i = 0; i < count; ++i) {
    sb.r[i] = reqs[i];
    max_ncb = std::max(max_ncb, reqs[i].ncb);
    max_cpb = std::max(max_cpb, reqs[i].cpb);
    if (sum_block_pins(reqs[i]) > kSumBlockPins) max_cpb = std::max(max_cpb, 1024);
  }
  if (max_cpb > kCompactMaxCpb) return hipErrorInvalidValue;
  if (max_cpb <= 256) return cells_launch<NB, 256, 1>(sb, max_ncb, grad_mode, s);
  if (max_cpb <= 512) return cells_launch<NB, 512, 1>(sb, max_ncb, grad_mode, s);
  if (max_cpb <= 1024) return cells_launch<NB, 1024, 1>(sb, max_ncb, grad_mode, s);
  if (max_cpb <= 2048) return cells_launch<NB, 1024, 2>(sb, max_ncb, grad_mode, s);
  return cells_launch<NB, 1024, kCompactMaxCpb / 1024>(sb, max_ncb, grad_mode, s);
}

}  // namespace

// Past n = 512 cells of many bins each are left to the general path: a thread gathers
// its cell's bins from a map larger than an XCD's L2, where the band gather has the
// neighbouring cells' rows in common.  n = 1024, 2500 cells, exact 313 us against 235,
// 4000 225 against 196 (171 against 164 with the fields), 8000 143 against 148 (115
// against 129).
bool compact_design(int n, const XchDims& d) {
  if (n > kCompactPairN && (int64_t)n * n > 128 * (int64_t)d.m) return false;
  return n <= kCompactMaxN && d.m > 0 && d.cpb <= kCompactMaxCpb && d.cap <= kXchPinLds2;
}

// Past n = 512 the row transform is on its own, and few cells are many bins each.
bool compact_scans(int n, int m) { return n <= kCompactPairN && m <= kScanCells; }

bool compact_fuses_rows(const Plan& p) {
  return p.mode == FFTPL_DCT_FFT && p.n >= 64 && p.n <= kCompactPairN;
}

// On every grid: read by pin, 1M cells on n = 256 took 111 us and 140 clustered (75
// and 93 with the spread), on n = 128 117 (83).  Many pins want it too, whose net blocks
// are more than the chip holds at once: 262k cells, n = 512, with 2.2M pins 73 -> 67 us,
// 3.9M 97 -> 81, 7.5M 175 -> 110 (with 1.7M 62 with it, 67 without, but the wirelength
// gradient alone 40.4 and 39.9; with 1.2M 38 and 34).  Positions of up to kScanCells
// cells stay in the L1s (64 KB) and are read by pin in any number (2000 cells, 7.5M
// pins: 520 us, 580 with the spread).
bool compact_spreads(int m, int num_pins) {
  return m > kCompactDirectCells || (m > kScanCells && num_pins > kCompactDirectPins);
}

hipError_t launch_compact_place(const BandReq* br, const XchReq* xr, int count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (count > kMaxBatch) return hipErrorInvalidValue;
  return count == 1 ? place_batch<1>(br, xr, count, s) : place_batch<kMaxBatch>(br, xr, count, s);
}

hipError_t launch_compact_mid(const Plan& p, const CompactReq* reqs, int count, int wl_model,
                              bool fuse_rows, bool spread, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (count > kMaxBatch) return hipErrorInvalidValue;
  return count == 1 ? mid_batch<1>(p, reqs, count, wl_model, fuse_rows, spread, s)
                    : mid_batch<kMaxBatch>(p, reqs, count, wl_model, fuse_rows, spread, s);
}

hipError_t launch_compact_cells(const SumReq* reqs, int count, int grad_mode, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (count > kMaxBatch) return hipErrorInvalidValue;
  return count == 1 ? cells_batch<1>(reqs, count, grad_mode, s)
                    : cells_batch<kMaxBatch>(reqs, count, grad_mode, s);
}

}  // namespace fftpl
