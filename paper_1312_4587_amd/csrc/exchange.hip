// Bucketed pin exchange for the weighted-average wirelength gradient
// (Eq. (3)) and HPWL (Eq. (1)).
//
// Nets pick their cells anywhere in the design, so handing cell positions to
// pins and pin gradients back to cells is a permutation of the pins.  Done
// directly, every pin costs one random 8-byte read and one random 8-byte
// write, each of which moves a whole cache line.  Here the permutation is
// split in two halves that both run through LDS:
//
//   cell blocks: cpb consecutive cells (a multiple of 256, at most kXchCells,
//                about one block per CU);
//   net blocks:  whole nets packed in CSR order, as many as fit in cap =
//                npt - 1 + max_degree <= kXchPinCap pins, so every block but
//                the last holds at least npt pins and there are at most
//                ceil(P / npt) blocks (the trailing ones may be empty);
//   A order:     pins sorted by (cell block, net block);
//   B order:     inside each net block's CSR range, pins sorted by cell block,
//                in the same order as A within each (cell block, net block)
//                segment.
//
//   spread  (one block per cell block): positions of the block's cells into
//           LDS, then T[a] = position of pin a's cell for its A range
//           (coalesced writes, random reads in LDS);
//   wa      (one block per net block): reads T in B order, i.e. runs of the
//           consecutive A positions of each segment, into LDS in CSR order;
//           evaluates every net from LDS (one thread per net of degree <= 8,
//           one wavefront per larger net); writes each pin's gradient back to
//           its own A position of T, again in runs;
//   cellsum (one block per cell block): streams the cell block's A
//           range of T and adds every pin's gradient into its cell's
//           accumulator in LDS (integer fixed point: order-independent),
//           then writes each cell's gradient: lambda times its density
//           gradient (computed per band entry on the density branch) plus
//           that sum.
//
// The index (A/B layout) is built once per netlist by xch_build.
#include <math.h>

#include <algorithm>
#include <atomic>
#include <vector>

#include "xch_device.hpp"

namespace fftpl {

namespace {

constexpr int NT = kXchThreads;
constexpr int NW = kXchWaThreads;
constexpr int kSmall = kXchSmallDeg;
constexpr int kHdrInts = 16;
constexpr int32_t kXchMagic = 0x46584348;   // "FXCH"
constexpr int kMaxDevices = 64;     // device ordinals with a per-device flag
constexpr int kSumThreads = 1024;   // cell sums: one block per cell block

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

int xch_dims(int m, int num_nets, int num_pins, int max_degree, XchDims* d) {
  if (m < 0 || num_nets < 0 || num_pins < 0 || max_degree < 0) return FFTPL_E_INVAL;
  // the largest block that still fits twice in one CU's LDS; failing that
  // (very large nets) one block per CU
  int npt = kXchPinTarget;
  if (npt > kXchPinLds2 + 1 - max_degree) npt = kXchPinLds2 + 1 - max_degree;
  if (npt < kXchMinTarget) {
    npt = kXchPinTarget;
    if (npt > kXchPinCap + 1 - max_degree) npt = kXchPinCap + 1 - max_degree;
  }
  if (npt < kXchMinTarget) return FFTPL_E_UNSUPPORTED;
  // cells per block
  int cpb = kXchCells;
  {
    // (two blocks per CU while a block then holds at most 512 cells, one per
    // thread of the compact cells kernel: 13.4 -> 11.1 us at 200k cells; with
    // more cells the shorter segments cost the net blocks as much)
    const int64_t want = m <= 512 * 2 * kNumCus ? 2 * kNumCus : kNumCus;
    const int64_t per_cu = ((int64_t)m + want - 1) / want;
    const int64_t step = (per_cu + kXchCellStep - 1) / kXchCellStep * kXchCellStep;
    cpb = (int)std::min<int64_t>(kXchCells, std::max<int64_t>(kXchCellStep, step));
  }
  // Netlists that do not fill one block of that size per CU are cut finer: a
  // block's time follows its pins (staging, the nets handed to its eight
  // wavefronts, the write-back), and small blocks share a CU three at a time.
  // Designs whose net blocks read the positions by pin are kept to blocks that
  // stage in one round of four pins per thread (past them the spread's runs want
  // the larger blocks: 500k cells with 2.8M pins at n = 1024 130 -> 119 us).  Net
  // blocks of 30k cells (78k pins) alone: 15.1 us in 20 blocks of 4096 pins, 8.4 us
  // in 153 of 512; eight such designs in one launch prefer 1024 (41.9 -> 35.9 us),
  // one design does not mind.
  {
    const int64_t even = ((int64_t)num_pins + kXchNetBlocks - 1) / kXchNetBlocks;
    npt = (int)std::min<int64_t>(npt, std::max<int64_t>(kXchSmallTarget, even));
    if (!compact_spreads(m, num_pins))
      npt = std::min(npt, std::max(kXchSmallTarget, 4 * kXchWaThreads + 1 - max_degree));
  }
  XchDims r;
  r.m = m;
  r.num_nets = num_nets;
  r.num_pins = num_pins;
  r.max_degree = max_degree;
  r.npt = npt;
  r.cap = max_degree > 0 ? npt - 1 + max_degree : 1;
  r.cpb = cpb;
  r.ncb = (m + r.cpb - 1) / r.cpb;
  r.nnb = num_pins > 0 ? (num_pins + npt - 1) / npt : 1;
  size_t off = 0;
  r.o_hdr = off;
  off = align256(off + sizeof(int32_t) * kHdrInts);
  r.o_cb = off;
  off = align256(off + sizeof(int32_t) * ((size_t)r.ncb + 1));
  r.o_nb = off;
  off = align256(off + sizeof(int32_t) * ((size_t)r.nnb + 1));
  r.o_ab = off;
  off = align256(off + sizeof(int32_t) * (size_t)num_pins);
  r.o_lcsr = off;
  off = align256(off + sizeof(uint16_t) * (size_t)num_pins);
  r.o_lc = off;
  off = align256(off + sizeof(uint16_t) * (size_t)num_pins);
  r.o_ns = off;
  off = align256(off + sizeof(uint32_t) * (size_t)num_nets);
  r.index_bytes = off;
  // build workspace: counts / cursors, A starts, transposed counts, B starts,
  // scan block sums, flag and scan totals
  const size_t seg = (size_t)r.ncb * r.nnb;
  r.work_bytes = align256(sizeof(int32_t) * seg) * 4 +
                 align256(sizeof(int32_t) * ((seg + 1023) / 1024 + 1)) +
                 align256(sizeof(int32_t) * 4);
  *d = r;
  return FFTPL_OK;
}

XchIndex xch_index(const XchDims& d, const void* index) {
  XchIndex X;
  const char* b = static_cast<const char*>(index);
  X.cb_a_ptr = reinterpret_cast<const int32_t*>(b + d.o_cb);
  X.nb_net_ptr = reinterpret_cast<const int32_t*>(b + d.o_nb);
  X.a_of_b = reinterpret_cast<const int32_t*>(b + d.o_ab);
  X.lcsr = reinterpret_cast<const uint16_t*>(b + d.o_lcsr);
  X.lc = reinterpret_cast<const uint16_t*>(b + d.o_lc);
  X.nmeta = reinterpret_cast<const uint32_t*>(b + d.o_ns);
  return X;
}

// ---------------------------------------------------------------------------
// Index build
// ---------------------------------------------------------------------------
namespace {

// Checks the CSR (net_ptr[0] = 0, net_ptr[E] = P, monotone, degrees <=
// max_degree, pin cells in range) and, with PLACE = false, counts the pins of
// every (cell block, net block) segment; with PLACE = true, hands each pin its
// A and B positions (the same rank inside the segment on both sides).
template <bool PLACE>
__global__ void __launch_bounds__(256)
    k_xi_pins(int num_nets, const int32_t* __restrict__ net_ptr, int num_pins,
              const int32_t* __restrict__ pin_cell, int m, int cpb, int max_degree, int ncb,
              int nnb, int32_t* __restrict__ cnt, const int32_t* __restrict__ seg_a,
              const int32_t* __restrict__ seg_bt, const int32_t* __restrict__ nb_net_ptr,
              int32_t* __restrict__ a_of_b, uint16_t* __restrict__ lcsr,
              uint16_t* __restrict__ lc, int32_t* __restrict__ flag) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (!PLACE && e == 0 && (net_ptr[0] != 0 || net_ptr[num_nets] != num_pins))
    atomicOr(flag, 1);
  // placing is only safe when the count saw a valid CSR covering every pin
  // once: then every A and B position stays below num_pins
  if (PLACE && (flag[0] != 0 || flag[1] != num_pins)) return;
  if (e >= num_nets) return;
  const int p0 = net_ptr[e], p1 = net_ptr[e + 1];
  if (p0 < 0 || p1 < p0 || p1 > num_pins || p1 - p0 > max_degree) {
    if (!PLACE) atomicOr(flag, 2);
    return;
  }
  if (p1 == p0) return;
  // the net block holding net e: the last k with nb_net_ptr[k] <= e
  int lo = 0, hi = nnb - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (nb_net_ptr[mid] <= e)
      lo = mid;
    else
      hi = mid - 1;
  }
  const int k = lo;
  if (e >= nb_net_ptr[k + 1]) {
    if (!PLACE) atomicOr(flag, 4);
    return;
  }
  const int base = PLACE ? net_ptr[nb_net_ptr[k]] : 0;
  for (int p = p0; p < p1; ++p) {
    const int c = pin_cell[p];
    if (c < 0 || c >= m) {
      if (!PLACE) atomicOr(flag, 8);
      continue;
    }
    const int cb = c / cpb;
    const size_t idx = (size_t)cb * nnb + k;
    if (!PLACE) {
      atomicAdd(&cnt[idx], 1);
    } else {
      const int r = atomicAdd(&cnt[idx], 1);
      const int a = seg_a[idx] + r;
      const int b = seg_bt[(size_t)k * ncb + cb] + r;
      a_of_b[b] = a;
      lcsr[b] = (uint16_t)(p - base);
      lc[a] = (uint16_t)(c - cb * cpb);
    }
  }
}

// Degree class of the net order: the degree itself up to kSmall, then one
// class per power of two (9-16, 17-32, ..., the last one open-ended).
__device__ __forceinline__ int degree_class(int deg) {
  if (deg <= kSmall) return deg;
  const int c = kSmall + 1 + (31 - __clz(deg - 1)) - 3;
  return c < kXchBuckets - 1 ? c : kXchBuckets - 1;
}

// Per net block, its nets in increasing degree class, each as (first pin -
// the block's first pin) << 16 | degree; the order inside a class is
// arbitrary.  A wavefront walking this order from the front sees small nets
// of equal degree together (its loops over pins run the length of the
// degree); walking it from the back it meets the largest nets first.  The
// kernel reads each net's extent from here with one coalesced load.
__global__ void __launch_bounds__(256)
    k_xi_netsort(const int32_t* __restrict__ net_ptr, const int32_t* __restrict__ nb_net_ptr,
                 uint32_t* __restrict__ nmeta) {
  __shared__ int cnt[kXchBuckets], cur[kXchBuckets];
  const int k = blockIdx.x, t = threadIdx.x;
  const int e0 = nb_net_ptr[k], e1 = nb_net_ptr[k + 1];
  const int p0 = net_ptr[e0];
  if (t < kXchBuckets) cnt[t] = 0;
  __syncthreads();
  for (int e = e0 + t; e < e1; e += blockDim.x)
    atomicAdd(&cnt[degree_class(net_ptr[e + 1] - net_ptr[e])], 1);
  __syncthreads();
  if (t == 0) {
    int run = 0;
    for (int b = 0; b < kXchBuckets; ++b) {
      cur[b] = run;
      run += cnt[b];
    }
  }
  __syncthreads();
  for (int e = e0 + t; e < e1; e += blockDim.x) {
    const int q0 = net_ptr[e], deg = net_ptr[e + 1] - q0;
    nmeta[e0 + atomicAdd(&cur[degree_class(deg)], 1)] =
        ((uint32_t)(q0 - p0) << 16) | (uint32_t)deg;
  }
}

__global__ void k_xi_transpose(int ncb, int nnb, const int32_t* __restrict__ cnt,
                               int32_t* __restrict__ cnt_t) {
  const size_t total = (size_t)ncb * nnb;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total;
       i += (size_t)gridDim.x * blockDim.x) {
    const size_t cb = i / nnb, k = i % nnb;
    cnt_t[k * ncb + cb] = cnt[i];
  }
}

__global__ void k_xi_finish(int ncb, int nnb, int num_pins, const int32_t* __restrict__ seg_a,
                            int32_t* __restrict__ cb_a_ptr, int32_t* __restrict__ hdr,
                            int m, int num_nets, int max_degree, int npt, int cpb) {
  const int cb = blockIdx.x * blockDim.x + threadIdx.x;
  if (cb < ncb) cb_a_ptr[cb] = seg_a[(size_t)cb * nnb];
  if (cb == ncb) cb_a_ptr[cb] = num_pins;
  if (cb == 0) {
    hdr[0] = kXchMagic;
    hdr[1] = m;
    hdr[2] = num_nets;
    hdr[3] = num_pins;
    hdr[4] = max_degree;
    hdr[5] = npt;
    hdr[6] = ncb;
    hdr[7] = nnb;
    hdr[8] = cpb;
  }
}

}  // namespace

int pack_net_blocks(const int32_t* ptr, int E, int P, int max_degree, int cap, int nnb,
                    int32_t* first) {
  if (E < 0 || nnb < 1 || cap < 1) return FFTPL_E_INVAL;
  if (ptr[0] != 0 || ptr[E] != P) return FFTPL_E_INVAL;
  for (int k = 0; k <= nnb; ++k) first[k] = E;
  int k = 0;
  int64_t cur = 0;
  first[0] = 0;
  for (int en = 0; en < E; ++en) {
    const int64_t deg = (int64_t)ptr[(size_t)en + 1] - ptr[en];
    if (deg < 0 || deg > max_degree) return FFTPL_E_INVAL;
    if (cur + deg > cap) {
      if (++k >= nnb) return FFTPL_E_INVAL;   // cannot happen for a valid CSR
      first[k] = en;
      cur = 0;
    }
    cur += deg;
  }
  return FFTPL_OK;
}

int xch_build(const XchDims& d, const int32_t* net_ptr, const int32_t* pin_cell, void* index,
              void* work, hipStream_t s) {
  const size_t seg = (size_t)d.ncb * d.nnb;
  if (seg > (size_t)INT32_MAX) return FFTPL_E_UNSUPPORTED;
  char* w = static_cast<char*>(work);
  int32_t* cnt = reinterpret_cast<int32_t*>(w);
  w += align256(sizeof(int32_t) * seg);
  int32_t* seg_a = reinterpret_cast<int32_t*>(w);
  w += align256(sizeof(int32_t) * seg);
  int32_t* cnt_t = reinterpret_cast<int32_t*>(w);
  w += align256(sizeof(int32_t) * seg);
  int32_t* seg_bt = reinterpret_cast<int32_t*>(w);
  w += align256(sizeof(int32_t) * seg);
  int32_t* sums = reinterpret_cast<int32_t*>(w);
  w += align256(sizeof(int32_t) * ((seg + 1023) / 1024 + 1));
  int32_t* flag = reinterpret_cast<int32_t*>(w);   // [0] error bits, [1] [2] scan totals

  char* ib = static_cast<char*>(index);
  int32_t* hdr = reinterpret_cast<int32_t*>(ib + d.o_hdr);
  int32_t* cb_a_ptr = reinterpret_cast<int32_t*>(ib + d.o_cb);
  int32_t* nb_net_ptr = reinterpret_cast<int32_t*>(ib + d.o_nb);
  int32_t* a_of_b = reinterpret_cast<int32_t*>(ib + d.o_ab);
  uint16_t* lcsr = reinterpret_cast<uint16_t*>(ib + d.o_lcsr);
  uint16_t* lc = reinterpret_cast<uint16_t*>(ib + d.o_lc);

  const int E = d.num_nets, P = d.num_pins;
  const dim3 net_grid((E + 255) / 256 > 0 ? (E + 255) / 256 : 1);
  // Net blocks, packed greedily on the host from the CSR (a sequential scan
  // of the net sizes, once per netlist): a block is closed when the next net
  // does not fit in cap pins.  Packing instead of cutting at fixed pin counts
  // fills the blocks (the LDS is sized for cap) rather than reserving room
  // for a largest net at every block end.
  {
    std::vector<int32_t> hptr((size_t)E + 1), hnb((size_t)d.nnb + 1, E);
    if (hipMemcpyAsync(hptr.data(), net_ptr, sizeof(int32_t) * ((size_t)E + 1),
                       hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return FFTPL_E_DEVICE;
    const int st = pack_net_blocks(hptr.data(), E, P, d.max_degree, d.cap, d.nnb, hnb.data());
    if (st != FFTPL_OK) return st;
    if (hipMemcpyAsync(nb_net_ptr, hnb.data(), sizeof(int32_t) * hnb.size(),
                       hipMemcpyHostToDevice, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return FFTPL_E_DEVICE;
  }
  hipError_t e = launch_zero_i32(cnt, (int64_t)seg, s);
  if (e == hipSuccess) e = launch_zero_i32(flag, 4, s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL((k_xi_pins<false>), net_grid, dim3(256), 0, s, E, net_ptr, P, pin_cell,
                       d.m, d.cpb, d.max_degree, d.ncb, d.nnb, cnt, nullptr, nullptr, nb_net_ptr,
                       nullptr, nullptr, nullptr, flag);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = launch_exclusive_scan(cnt, (int)seg, seg_a, sums, flag + 1, s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_xi_transpose, dim3(1024), dim3(256), 0, s, d.ncb, d.nnb, cnt, cnt_t);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = launch_exclusive_scan(cnt_t, (int)seg, seg_bt, sums, flag + 2, s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_xi_finish, dim3((d.ncb + 256) / 256), dim3(256), 0, s, d.ncb, d.nnb,
                       P, seg_a, cb_a_ptr, hdr, d.m, E, d.max_degree, d.npt, d.cpb);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return FFTPL_E_DEVICE;
  // the netlist is valid (every pin counted once, cells in range) before
  // anything indexes by it
  int32_t hflag[3] = {0, 0, 0};
  if (hipMemcpyAsync(hflag, flag, sizeof(hflag), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return FFTPL_E_DEVICE;
  if (hflag[0] != 0 || hflag[1] != P || hflag[2] != P) return FFTPL_E_INVAL;
  e = launch_zero_i32(cnt, (int64_t)seg, s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL((k_xi_pins<true>), net_grid, dim3(256), 0, s, E, net_ptr, P, pin_cell,
                       d.m, d.cpb, d.max_degree, d.ncb, d.nnb, cnt, seg_a, seg_bt, nb_net_ptr,
                       a_of_b, lcsr, lc, flag);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    uint32_t* nmeta = reinterpret_cast<uint32_t*>(ib + d.o_ns);
    hipLaunchKernelGGL(k_xi_netsort, dim3(d.nnb), dim3(256), 0, s, net_ptr, nb_net_ptr, nmeta);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  return e == hipSuccess ? FFTPL_OK : FFTPL_E_DEVICE;
}

// ---------------------------------------------------------------------------
// Evaluation kernels
// ---------------------------------------------------------------------------
namespace {

template <int NB>
__global__ void __launch_bounds__(NT) k_xch_spread(XchBatch<NB> xb) {
  // design blockIdx.y of the batch; blocks past its cell blocks idle
  const XchReq& rq = xb.r[blockIdx.y];
  const int nb = rq.ncb * kXchSpreadSplit;
  if ((int)blockIdx.x >= nb) return;
  __shared__ float2 win[kXchCells];
  spread_part<NT, kXchCells, kXchSpreadSplit>(rq, xcd_order(blockIdx.x, nb), win);
}

template <int STAGE, bool LSE, int NB, bool DIRECT>
__global__ void __launch_bounds__(NW) k_xch_wa(XchBatch<NB> xb) {
  extern __shared__ float2 smem[];
  const XchReq& rq = xb.r[blockIdx.y];
  if ((int)blockIdx.x >= rq.nnb) return;
  wa_block<STAGE, DIRECT ? kStageHold : STAGE, LSE, DIRECT>(rq, xcd_order(blockIdx.x, rq.nnb), smem);
}

// The gradient of every cell (CellGradArgs): its density part plus the sum
// of the gradients in T of its pins.  One block per cell
// block: the block streams the cell block's A range of T together with the
// cell-local index lc (both coalesced) and adds each pin into per-cell
// accumulators in LDS.  The adds are 64-bit integer adds of the gradients in
// fixed point (units of 2^-S), so the sums come out the same whatever order
// the atomics land in (LDS float atomics would not, and run several times
// slower).  One pin's gradient component is bounded by 1.15 + ln(largest
// degree) (its softmax weight times one plus its distance to the weighted
// mean, and that distance is at most ln(degree) in units of gamma), so S is
// the largest scale that keeps every pin within a 32-bit conversion; the
// 64-bit sums then hold any number of pins.  A non-finite pin gradient makes
// its cell's sum NaN.
// NTS threads, at most CELLS cells per block: (1024, kXchCells), 153 KB of LDS
// and one block per CU, or (256, kXchSmallCells) for designs cut into blocks
// of up to 1024 cells, whose fixed work (clearing the accumulators, waiting at
// the barriers) is that of 256 threads and 17 KB, several blocks per CU.
template <int MODE, bool DENS, int NB, int NTS, int CELLS>
__global__ void __launch_bounds__(NTS) k_xch_cellsum(SumBatch<NB> sb) {
  const SumReq& rq = sb.r[blockIdx.y];
  const int cb = blockIdx.x, t = threadIdx.x;
  if (cb >= rq.ncb) return;
  const int m = rq.m, cpb = rq.cpb;
  const int32_t* __restrict__ cb_a_ptr = rq.cb_a_ptr;
  const uint16_t* __restrict__ lc = rq.lc;
  const float2* __restrict__ T = rq.T;
  const float scale = rq.fx_scale;
  const double inv_scale = rq.inv_scale;
  const CellGradArgs& a = rq.a;
  __shared__ unsigned long long ax[CELLS], ay[CELLS];
  __shared__ unsigned char bad[CELLS];
  // the block's A range, then the first-band entry of each of the thread's
  // cells and its first group of pins: all in flight while LDS is cleared
  const int a0 = cb_a_ptr[cb], a1 = cb_a_ptr[cb + 1];
  constexpr int PC = CELLS / NTS;
  const int c0 = cb * cpb;
  int ep[PC];
  if (DENS) {
#pragma unroll
    for (int k = 0; k < PC; ++k) ep[k] = a.epos[min(c0 + t + k * NTS, m - 1)];
  }
  PinSums<NTS, CELLS> pins;
  pins.prefetch(lc, T, a0, a1);
  for (int c = t; c < CELLS; c += NTS) {
    ax[c] = 0ull;
    ay[c] = 0ull;
    bad[c] = 0;
  }
  __syncthreads();
  pins.add(scale, ax, ay, bad);
  __syncthreads();
  // each cell's gradient: its density part from its first-band entry (one
  // 8-byte read; all of a thread's reads issued together) or, for a cell
  // without one, from the maps; plus its wirelength sum (DENS = false: the
  // wirelength sum alone, written or added to the gradient)
  float2 d[PC];
  const float lam = DENS && a.dscale ? a.dscale[0] : a.scale;
  if (DENS) {
#pragma unroll
    for (int k = 0; k < PC; ++k) d[k] = a.egrad[max(ep[k], 0)];
  } else if (a.accumulate) {
#pragma unroll
    for (int k = 0; k < PC; ++k) {
      const int ci = min(c0 + t + k * NTS, m - 1);
      d[k] = make_float2(a.gx[ci], a.gy[ci]);
    }
  }
#pragma unroll
  for (int k = 0; k < PC; ++k) {
    const int c = t + k * NTS, ci = c0 + c;
    if (c >= cpb || ci >= m) break;
    if (DENS && ep[k] < 0)
      d[k] = cell_density_grad<MODE, true>(a.g, a.x[ci], a.y[ci], a.w[ci], a.h[ci], nullptr,
                                           nullptr, a.exy, a.psi);
    const float sx = pin_sum(ax[c], bad[c], inv_scale), sy = pin_sum(ay[c], bad[c], inv_scale);
    if (DENS) {
      a.gx[ci] = lam * d[k].x + sx;
      a.gy[ci] = lam * d[k].y + sy;
    } else if (a.accumulate) {
      a.gx[ci] = d[k].x + sx;
      a.gy[ci] = d[k].y + sy;
    } else {
      a.gx[ci] = sx;
      a.gy[ci] = sy;
    }
  }
  if (cb == a.fin_block) {
    __syncthreads();
    eval_scalars<NTS>(a.fin);
  }
}

}  // namespace

// Fixed-point scale 2^S of the cell sums: the largest S <= 26 with
// bound * 2^S <= 2^30 for the largest pin gradient component bound.
static int cellsum_shift(int max_degree) {
  const double bound = 1.15 + log((double)(max_degree > 2 ? max_degree : 2));
  int S = 26;
  while (S > 0 && bound * ldexp(1.0, S) > ldexp(1.0, 30)) --S;
  return S;
}

SumReq sum_req(const XchDims& d, const XchIndex& X, const float2* T, const CellGradArgs& a) {
  SumReq q;
  q.m = d.m;
  q.cpb = d.cpb;
  q.ncb = d.ncb;
  q.num_pins = d.num_pins;
  q.cb_a_ptr = X.cb_a_ptr;
  q.lc = X.lc;
  q.T = T;
  const int S = cellsum_shift(d.max_degree);
  q.fx_scale = (float)ldexp(1.0, S);
  q.inv_scale = ldexp(1.0, -S);
  q.a = a;
  return q;
}

template <int NB, int NTS, int CELLS>
static hipError_t cellsum_nb(const SumBatch<NB>& sb, int max_ncb, int grad_mode, bool dens,
                             hipStream_t s) {
  const dim3 grid(max_ncb, sb.count), block(NTS);
  if (!dens)
    hipLaunchKernelGGL((k_xch_cellsum<FFTPL_GRAD_FIELD, false, NB, NTS, CELLS>), grid, block, 0,
                       s, sb);
  else if (grad_mode == FFTPL_GRAD_EXACT)
    hipLaunchKernelGGL((k_xch_cellsum<FFTPL_GRAD_EXACT, true, NB, NTS, CELLS>), grid, block, 0,
                       s, sb);
  else
    hipLaunchKernelGGL((k_xch_cellsum<FFTPL_GRAD_FIELD, true, NB, NTS, CELLS>), grid, block, 0,
                       s, sb);
  return hipGetLastError();
}

template <int NB>
static hipError_t cellsum_size(const SumBatch<NB>& sb, int max_ncb, int max_cpb, int grad_mode,
                               bool dens, hipStream_t s) {
  if (max_cpb <= kXchSmallCells)
    return cellsum_nb<NB, 256, kXchSmallCells>(sb, max_ncb, grad_mode, dens, s);
  return cellsum_nb<NB, kSumThreads, kXchCells>(sb, max_ncb, grad_mode, dens, s);
}

hipError_t launch_xch_cellsum_batch(const SumReq* reqs, int count, int grad_mode, bool dens,
                                    hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (count > kMaxBatch) return hipErrorInvalidValue;
  int max_ncb = 0, max_cpb = 0;
  for (int i = 0; i < count; ++i) {
    if (reqs[i].m > 0) max_ncb = std::max(max_ncb, reqs[i].ncb);
    max_cpb = std::max(max_cpb, reqs[i].cpb);
    if (sum_block_pins(reqs[i]) > kSumBlockPins) max_cpb = kXchCells;
  }
  if (max_ncb == 0) return hipSuccess;
  if (count == 1) {
    SumBatch<1> sb;
    sb.count = 1;
    sb.r[0] = reqs[0];
    return cellsum_size(sb, max_ncb, max_cpb, grad_mode, dens, s);
  }
  SumBatch<kMaxBatch> sb;
  sb.count = count;
  for (int i = 0; i < count; ++i) sb.r[i] = reqs[i];
  return cellsum_size(sb, max_ncb, max_cpb, grad_mode, dens, s);
}

XchReq xch_req(const XchDims& d, const XchIndex& X, const float* x, const float* y, float2* T,
               const int32_t* net_ptr, const int32_t* pin_cell, const float* pin_dx,
               const float* pin_dy, float gamma, double* part) {
  XchReq q;
  q.pin_cell = pin_cell;
  q.m = d.m;
  q.cpb = d.cpb;
  q.ncb = d.ncb;
  q.cb_a_ptr = X.cb_a_ptr;
  q.lc = X.lc;
  q.x = x;
  q.y = y;
  q.T = T;
  q.num_pins = d.num_pins;
  q.cap = d.cap;
  q.nnb = d.nnb;
  q.net_ptr = net_ptr;
  q.nb_net_ptr = X.nb_net_ptr;
  q.nmeta = X.nmeta;
  q.a_of_b = X.a_of_b;
  q.lcsr = X.lcsr;
  q.pin_dx = pin_dx;
  q.pin_dy = pin_dy;
  q.gamma = gamma;
  q.inv_gamma = 1.0f / gamma;
  q.part = part;
  return q;
}

template <int NB>
static hipError_t spread_nb(const XchBatch<NB>& xb, int max_ncb, hipStream_t s) {
  hipLaunchKernelGGL((k_xch_spread<NB>), dim3(max_ncb * kXchSpreadSplit, xb.count), dim3(NT),
                     0, s, xb);
  return hipGetLastError();
}

hipError_t launch_xch_spread_batch(const XchReq* reqs, int count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (count > kMaxBatch) return hipErrorInvalidValue;
  int max_ncb = 0;
  for (int i = 0; i < count; ++i) max_ncb = std::max(max_ncb, reqs[i].ncb);
  if (max_ncb == 0) return hipSuccess;
  if (count == 1) {
    XchBatch<1> xb;
    xb.count = 1;
    xb.r[0] = reqs[0];
    return spread_nb(xb, max_ncb, s);
  }
  XchBatch<kMaxBatch> xb;
  xb.count = count;
  for (int i = 0; i < count; ++i) xb.r[i] = reqs[i];
  return spread_nb(xb, max_ncb, s);
}

// The largest net blocks' LDS (up to 152 KiB) is asked for explicitly, once per device
// and kernel instantiation (twice from racing threads is harmless).  The runtime takes
// what fits a CU without it too, and the 76 KiB of the other net blocks rely on that.
template <typename K>
static hipError_t allow_big_lds(K* kernel, std::atomic<bool>* flags) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  if (!flags[dev].load(std::memory_order_acquire)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)(sizeof(float2) * 2 * kXchPinCap));
    if (e != hipSuccess) return e;
    flags[dev].store(true, std::memory_order_release);
  }
  return hipSuccess;
}

template <bool LSE, int NB>
static hipError_t wa_nb(const XchBatch<NB>& xb, int max_nnb, int max_cap, bool direct,
                        hipStream_t s) {
  const size_t lds = sizeof(float2) * 2 * (size_t)max_cap;
  const dim3 grid(max_nnb, xb.count);
  if (direct) {
    hipLaunchKernelGGL((k_xch_wa<kStageS, LSE, NB, true>), grid, dim3(NW), lds, s, xb);
  } else if (max_cap <= kXchPinLds2) {
    hipLaunchKernelGGL((k_xch_wa<kStageS, LSE, NB, false>), grid, dim3(NW), lds, s, xb);
  } else {
    static std::atomic<bool> attr[kMaxDevices];
    const hipError_t e = allow_big_lds(&k_xch_wa<kStageL, LSE, NB, false>, attr);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_xch_wa<kStageL, LSE, NB, false>), grid, dim3(NW), lds, s, xb);
  }
  return hipGetLastError();
}

template <bool LSE>
static hipError_t wa_model(const XchReq* reqs, int count, bool direct, hipStream_t s) {
  int max_nnb = 0, max_cap = 1;
  for (int i = 0; i < count; ++i) {
    max_nnb = std::max(max_nnb, reqs[i].nnb);
    max_cap = std::max(max_cap, reqs[i].cap);
  }
  if (max_nnb == 0) return hipSuccess;
  if (direct && max_cap > kXchPinLds2) return hipErrorInvalidValue;
  if (count == 1) {
    XchBatch<1> xb;
    xb.count = 1;
    xb.r[0] = reqs[0];
    return wa_nb<LSE, 1>(xb, max_nnb, max_cap, direct, s);
  }
  XchBatch<kMaxBatch> xb;
  xb.count = count;
  for (int i = 0; i < count; ++i) xb.r[i] = reqs[i];
  return wa_nb<LSE, kMaxBatch>(xb, max_nnb, max_cap, direct, s);
}

hipError_t launch_xch_wa_batch(const XchReq* reqs, int count, int wl_model, hipStream_t s,
                               bool direct) {
  if (count <= 0) return hipSuccess;
  if (count > kMaxBatch) return hipErrorInvalidValue;
  return wl_model == FFTPL_WL_LSE ? wa_model<true>(reqs, count, direct, s)
                                  : wa_model<false>(reqs, count, direct, s);
}

}  // namespace fftpl
