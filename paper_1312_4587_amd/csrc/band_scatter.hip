// Banded density scatter (Eq. (2), Section III-B) without float atomics in
// global memory, which retire at roughly 20 G/s on the whole chip whatever
// their scope:
//   place: each block of cpk cells histograms the bands its cells
//          touch in LDS (plus one slot for cells too tall to list per band),
//          scans the histogram, and writes each cell's edges (bin units)
//          into every band it touches, in a region of its own sliced by band
//          (LDS-atomic ranks inside each slice); per band, each block's slice
//          offset and count go out band-major;
//   accum: one block per band walks the band's slices of every region and
//          adds its entries into an LDS copy of its rows, then writes
//          rho = base + rows once.  The LDS adds are 64-bit integer adds of
//          the overlaps in fixed point (every overlap lies in [0, 1], units
//          of 2^-31): they retire many times faster than LDS float atomics,
//          and the sums do not depend on the order of the entries, so rho is
//          the same on every run;
//   gather (after the solve): one block per band walks the same slices and
//          computes the density gradient of every cell whose first band it
//          is, from the band's field rows staged in LDS.
// Every thread issues the loads of its cells (or entries) before it uses any
// of them, so each block keeps many misses in flight.
#include <algorithm>
#include <mutex>

#include "band_device.hpp"

namespace fftpl {

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

BandLayout band_shape(int n, int m, bool pairs) {
  BandLayout L;
  L.n = n;
  // As few rows as leave at most 256 bands, at most 4 for n <= 1024: rows * n <=
  // 4096 bins, the last band short.  pairs: two rows at least, which is what a
  // band block of the compact evaluation transforms; on grids of up to 256 that
  // is half the blocks, each with twice the cells (the map alone, 1M cells, n = 64:
  // 98 us in pairs, 51 us in single rows; crowded cells, n = 256, 446 and 231).
  L.rows = pairs && n <= kCompactPairN ? 2 : (n + 255) / 256;
  L.nb = (n + L.rows - 1) / L.rows;
  L.m = m;
  // Cells per counting block: the fewest (512 threads times 1, 2, 4 or 8
  // cells) that need no more blocks than there are CUs, else 8.  A block is a
  // chain of load, count, scan and store whose length follows its cells:
  // k_band_place at 200k cells 11.4 us in 49 blocks of 4096 cells, 7.6 us in
  // 196 of 1024; at 123k cells 10.6 us, 6.9 us in 242 of 512; 2.1M cells keep
  // 4096.
  int cb = 1;
  while (cb < kCellBatch && (int64_t)kBandThreads * cb * kNumCus < m) cb *= 2;
  L.cpk = kBandThreads * cb;
  L.region = kMaxBands * L.cpk;
  L.nblk = m > 0 ? (m + L.cpk - 1) / L.cpk : 1;
  return L;
}

// Entries of blk_off and of blk_cnt: as many as any design of up to m cells takes
// on this grid, in bands of either shape (a design just past a step of cpk has fewer
// counting blocks than the last one before it), so that the memory of a design
// holds every smaller one.
static size_t blk_entries(const BandLayout& L) {
  const int most = std::min(kNumCus, (L.m + kBandThreads - 1) / kBandThreads);
  const int bands = std::max(L.nb, std::min(L.n, kMaxBandCount));
  return (size_t)std::max(L.nblk, most) * (bands + 1);
}

BandLayout band_layout(int n, int m, int num_nets, int num_pins, void* work,
                       size_t* bytes_out, bool pairs) {
  BandLayout L = band_shape(n, m, pairs);
  L.nwa = (num_nets + 255) / 256;
  // wirelength partials: 4 per 256 nets (slot path) or 2 per net block of at
  // least kXchSmallTarget pins (exchange path)
  size_t nwp = 4 * (size_t)L.nwa;
  const size_t nxp = 2 * (((size_t)num_pins + kXchSmallTarget - 1) / kXchSmallTarget + 1);
  if (nwp < nxp) nwp = nxp;
  size_t off = 0;
  const size_t o_wp = off;
  off = align256(off + sizeof(double) * nwp);
  const size_t o_xy = off;
  off = align256(off + sizeof(float2) * (size_t)m);
  const size_t o_pg = off;
  off = align256(off + sizeof(float2) * (size_t)num_pins);
  const size_t nreg = (size_t)L.nblk * L.region;   // entries of all regions
  const size_t o_en = off;
  off = align256(off + sizeof(float4) * nreg);
  const size_t o_big = off;
  off = align256(off + sizeof(int32_t) * (size_t)L.nblk * L.cpk);
  const size_t o_ep = off;
  off = align256(off + sizeof(int32_t) * (size_t)m);
  const size_t o_eg = off;
  off = align256(off + sizeof(float2) * nreg);
  const size_t o_bo = off;
  off = align256(off + sizeof(int32_t) * blk_entries(L));
  const size_t o_bc = off;
  off = align256(off + sizeof(int32_t) * blk_entries(L));
  if (bytes_out) *bytes_out = off;
  if (work) {
    char* b = static_cast<char*>(work);
    L.wa_part = reinterpret_cast<double*>(b + o_wp);
    L.xy = reinterpret_cast<float2*>(b + o_xy);
    L.pin_grad = reinterpret_cast<float2*>(b + o_pg);
    L.entries = reinterpret_cast<float4*>(b + o_en);
    L.big = reinterpret_cast<int32_t*>(b + o_big);
    L.epos = reinterpret_cast<int32_t*>(b + o_ep);
    L.egrad = reinterpret_cast<float2*>(b + o_eg);
    L.blk_off = reinterpret_cast<int32_t*>(b + o_bo);
    L.blk_cnt = reinterpret_cast<int32_t*>(b + o_bc);
  }
  return L;
}

namespace {

constexpr int NT = kBandThreads;
constexpr int B = kCellBatch;   // entries a thread of a band walk takes together

}  // namespace

// CB: the most cells per thread among the batch's designs (a design with fewer
// per block leaves the rest of its threads' slots empty).
template <int NB, int CB>
__global__ void __launch_bounds__(kBandThreads) k_band_place(BandBatch<NB> bb) {
  // design blockIdx.y of the batch; blocks past its count of cell blocks idle
  const BandReq& q = bb.r[blockIdx.y];
  if (q.L.m <= 0 || (int)blockIdx.x >= q.L.nblk) return;
  place_block<CB>(q.g, q.L, blockIdx.x, q.x, q.y, q.w, q.h);
}

// NTA threads taking KB entries each, at most BINS bins per band: (1024, 8,
// 4096), or (512, 4, 1024) for batches with n <= 512 and up to 1024 cells per band on
// average.  Such a band holds a few hundred entries, less than the larger
// block's fixed work (owner map, scan over the threads, clears), and the smaller
// block leaves room for four per CU: a batch of eight designs at n = 256 takes
// 14.5 us instead of 53.2.  One design has at most one block per CU and nothing
// to share it with: the larger block takes as long where the cells are spread (200k
// cells, n = 512, 7.8 us against 8.2) and less where they crowd into a few bands
// (123k cells in a dozen bands 56 us, the whole map, against 74).
template <int NB, int NTA, int KB, int BINS>
__global__ void __launch_bounds__(NTA) k_band_accum(BandBatch<NB> bb) {
  const BandReq& q = bb.r[blockIdx.y];
  const GridF g = q.g;
  const BandLayout L = q.L;
  const float* __restrict__ base = q.base;
  float* __restrict__ rho = q.rho;
  __shared__ unsigned long long acc[BINS];
  __shared__ WalkLds<NTA, KB> lds;
  const int t = threadIdx.x;
  const int n = g.n, R = L.rows, band = xcd_order(blockIdx.x, gridDim.x), r0 = band * R;
  const int cells = min(R, n - r0) * n;
  for (int k = t; k < cells; k += NTA) acc[k] = 0ull;
  __syncthreads();
  band_accumulate<NTA, KB, BINS == 1024>(g, L, band, q.x, q.y, q.w, q.h, acc, lds);
  __syncthreads();
  // rho = base + rows: all of a thread's base loads issued before any store
  constexpr int PA = BINS / NTA;
  const size_t o = (size_t)r0 * n;
  float bv[PA];
#pragma unroll
  for (int j = 0; j < PA; ++j) bv[j] = base ? base[o + min(t + j * NTA, cells - 1)] : 0.0f;
#pragma unroll
  for (int j = 0; j < PA; ++j) {
    const int k = t + j * NTA;
    if (k < cells) rho[o + k] = bv[j] + (float)((double)acc[k] * kAccUnit);
  }
}

// The density map of a small design in one launch: each band's block reads every
// cell, so there are no band lists and no memory to hold them.  Up to
// kScanCells cells the reads cost less than the place pass and the launch they
// replace: the stateless map of 1000 to 8192 cells, n = 32 to 128, 25 -> 9.6 us
// (n = 512, 8192 cells 23.6 -> 12.9).  On larger grids so few cells are many bins
// each and the blocks' adds outweigh it (n = 1024, 8192 cells 24.7 -> 34.9 us).
// Where the lists would have to be allocated for the call the line lies at
// kScanCellsAlloc for n <= 256: n = 64, 16384 cells 30 -> 11.1 us, 20k 30 -> 23.
// Past n = 256 a few large cells, each added by one thread, are enough to lose it
// (n = 300, 12288 cells, one in a hundred 30 bins wide: 33 us, through lists 26).
// There is at most one block per CU: 1024 threads, for cells that crowd into a few
// bands (16384 cells, n = 256: 17.7 us, with 512 threads on row pairs 30.9, by way
// of the lists 24.8).
bool density_scans(int n, int m, bool alloc) {
  return n <= 512 && m <= (alloc && n <= 256 ? kScanCellsAlloc : kScanCells);
}

constexpr int kScanThreads = 1024;
__global__ void __launch_bounds__(kScanThreads) k_band_scan(BandReq q) {
  constexpr int NTS = kScanThreads, LIST = 2048, BINS = 1024;   // bins of a band
  __shared__ unsigned long long acc[BINS];
  __shared__ ScanLds<NTS, LIST> lds;
  const int t = threadIdx.x, n = q.g.n, R = q.L.rows;
  const int band = xcd_order(blockIdx.x, gridDim.x), r0 = band * R;
  const int cells = min(R, n - r0) * n;
  const size_t o = (size_t)r0 * n;
  static_assert(BINS == NTS, "one bin per thread");
  const float bv = q.base ? q.base[o + min(t, cells - 1)] : 0.0f;
  if (t < cells) acc[t] = 0ull;
  __syncthreads();
  band_scan<NTS, LIST>(q.g, q.L, band, q.x, q.y, q.w, q.h, acc, lds);
  __syncthreads();
  if (t < cells) q.rho[o + t] = bv + (float)((double)acc[t] * kAccUnit);
}

// Density gradient of every cell listed in band b with b its first band,
// from the cell's entry (its edges), into egrad at the entry's position.  A
// band's cells read the field rows of that band and the next, so the map
// reads of one block stay within a few tens of KiB (staged in LDS), where a
// per-cell gather in cell order reads the whole map at random.
constexpr int NTG = 1024;   // threads of a band-gather block
template <int MODE, int NB>
__global__ void __launch_bounds__(NTG) k_band_gather(BandBatch<NB> bb) {
  const BandReq& q = bb.r[blockIdx.y];
  const GridF g = q.g;
  const BandLayout L = q.L;
  const float2* __restrict__ exy = q.exy;
  const float* __restrict__ psi = q.psi;
  // the band's field rows and the next one (cells of up to two rows whose
  // first row is in the band read only these) staged in LDS
  __shared__ float2 rows[5 * kBandMaxN];
  __shared__ int pre[NTG];
  __shared__ int64_t start[NTG];
  __shared__ __align__(16) unsigned short owner[NTG * B];
  const int t = threadIdx.x;
  const int n = g.n, R = L.rows, band = xcd_order(blockIdx.x, gridDim.x);
  const int r0 = band * R, nr = min(R + 1, n - r0);
  if (MODE == FFTPL_GRAD_FIELD) {
    // all of a thread's loads issued before its LDS stores
    constexpr int PS = (5 * kBandMaxN + NTG - 1) / NTG;
    const int cnt = nr * n;
    float2 v[PS];
#pragma unroll
    for (int j = 0; j < PS; ++j) v[j] = exy[(int64_t)r0 * n + min(t + j * NTG, cnt - 1)];
#pragma unroll
    for (int j = 0; j < PS; ++j)
      if (t + j * NTG < cnt) rows[t + j * NTG] = v[j];
  }
  // (the walk's first scan synchronises the block after the staging)
  walk_band<NTG, B>(L, band, L.region, pre, start, owner, [&](const int64_t (&idx)[B]) {
    float4 q[B];
#pragma unroll
    for (int j = 0; j < B; ++j) q[j] = L.entries[idx[j] >= 0 ? idx[j] : 0];
#pragma unroll
    for (int j = 0; j < B; ++j) {
      if (idx[j] < 0) continue;
      const Span sx = span_from_edges(q[j].x, q[j].y, n);
      const Span sy = span_from_edges(q[j].z, q[j].w, n);
      if (sy.i0 / R != band) continue;   // listed again below its first band
      if (MODE == FFTPL_GRAD_FIELD && sy.i1 < r0 + nr) {
        // the same sum as the per-cell gather, from the staged rows
        float ax = 0.0f, ay = 0.0f;
        for (int iy = sy.i0; iy <= sy.i1; ++iy) {
          const float oy = span_overlap(sy, iy);
          const float2* row = rows + (iy - r0) * n;
          for (int ix = sx.i0; ix <= sx.i1; ++ix) {
            const float ov = span_overlap(sx, ix) * oy;
            const float2 f = row[ix];
            ax += ov * f.x;
            ay += ov * f.y;
          }
        }
        L.egrad[idx[j]] = make_float2(ax * -g.inv_bw, ay * -g.inv_bh);
      } else {
        // (EXACT: the maps are not staged; straight-line loads in place of the loops,
        // 2.1M cells, n = 1024, whole evaluation 191.7 -> 188.3 us, clustered 226.8 ->
        // 214.1; FIELD comes here for tall cells alone)
        L.egrad[idx[j]] = MODE == FFTPL_GRAD_EXACT
                              ? density_grad_small<MODE>(g, sx, sy, exy, psi)
                              : density_grad_spans<MODE, true>(g, sx, sy, nullptr, nullptr, exy,
                                                               psi);
      }
    }
  });
}

template <int NB>
static hipError_t band_gather_nb(const BandBatch<NB>& bb, int nb, int grad_mode,
                                 hipStream_t s) {
  const dim3 grid(nb, bb.count);
  if (grad_mode == FFTPL_GRAD_EXACT)
    hipLaunchKernelGGL((k_band_gather<FFTPL_GRAD_EXACT, NB>), grid, dim3(NTG), 0, s, bb);
  else
    hipLaunchKernelGGL((k_band_gather<FFTPL_GRAD_FIELD, NB>), grid, dim3(NTG), 0, s, bb);
  return hipGetLastError();
}

hipError_t launch_band_gather_batch(const BandReq* reqs, int count, int grad_mode,
                                    hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (count > kMaxBatch) return hipErrorInvalidValue;
  const int nb = reqs[0].L.nb;
  if (count == 1) {
    BandBatch<1> bb;
    bb.count = 1;
    bb.r[0] = reqs[0];
    return band_gather_nb(bb, nb, grad_mode, s);
  }
  BandBatch<kMaxBatch> bb;
  bb.count = count;
  for (int i = 0; i < count; ++i) bb.r[i] = reqs[i];
  return band_gather_nb(bb, nb, grad_mode, s);
}

// xy[i] = (x[i], y[i]): the wirelength pass then gathers one float2 per pin.
__global__ void __launch_bounds__(256)
    k_interleave(int m, const float* __restrict__ x, const float* __restrict__ y,
                 float2* __restrict__ xy) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gridDim.x * blockDim.x)
    xy[i] = make_float2(x[i], y[i]);
}

hipError_t launch_interleave(int m, const float* x, const float* y, float2* xy,
                             hipStream_t s) {
  if (m <= 0) return hipSuccess;
  int blocks = (m + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_interleave, dim3(blocks), dim3(256), 0, s, m, x, y, xy);
  return hipGetLastError();
}

template <int NB>
static hipError_t band_place_nb(const BandBatch<NB>& bb, int max_nblk, int cpk, hipStream_t s) {
  const dim3 grid(max_nblk, bb.count), block(NT);
  if (cpk <= NT)
    hipLaunchKernelGGL((k_band_place<NB, 1>), grid, block, 0, s, bb);
  else if (cpk <= 2 * NT)
    hipLaunchKernelGGL((k_band_place<NB, 2>), grid, block, 0, s, bb);
  else if (cpk <= 4 * NT)
    hipLaunchKernelGGL((k_band_place<NB, 4>), grid, block, 0, s, bb);
  else
    hipLaunchKernelGGL((k_band_place<NB, kCellBatch>), grid, block, 0, s, bb);
  return hipGetLastError();
}

template <int NB>
static hipError_t band_scatter_nb(const BandBatch<NB>& bb, int max_nblk, int max_cpk, int max_m,
                                  hipStream_t s, Plan* tp) {
  hipError_t e = hipSuccess;
  if (max_m > 0) {
    if ((e = band_place_nb<NB>(bb, max_nblk, max_cpk, s)) != hipSuccess) return e;
    if (tp) plan_mark(*tp, "k_band_place", s);
  }
  const int n = bb.r[0].L.n, nb = bb.r[0].L.nb;
  if (bb.count > 1 && n <= 512 && max_m <= 1024 * (int64_t)nb)
    hipLaunchKernelGGL((k_band_accum<NB, 512, 4, 1024>), dim3(nb, bb.count), dim3(512), 0, s, bb);
  else
    hipLaunchKernelGGL((k_band_accum<NB, 1024, B, 4096>), dim3(nb, bb.count), dim3(1024), 0, s, bb);
  e = hipGetLastError();
  if (tp) plan_mark(*tp, "k_band_accum", s);
  return e;
}

hipError_t launch_band_place_batch(const BandReq* reqs, int count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (count > kMaxBatch) return hipErrorInvalidValue;
  int max_nblk = 0, max_cpk = 0;
  for (int i = 0; i < count; ++i) {
    if (reqs[i].L.m <= 0) continue;
    max_nblk = std::max(max_nblk, reqs[i].L.nblk);
    max_cpk = std::max(max_cpk, reqs[i].L.cpk);
  }
  if (max_nblk == 0) return hipSuccess;
  if (count == 1) {
    BandBatch<1> bb;
    bb.count = 1;
    bb.r[0] = reqs[0];
    return band_place_nb(bb, max_nblk, max_cpk, s);
  }
  BandBatch<kMaxBatch> bb;
  bb.count = count;
  for (int i = 0; i < count; ++i) bb.r[i] = reqs[i];
  return band_place_nb(bb, max_nblk, max_cpk, s);
}

hipError_t launch_band_scatter_batch(const BandReq* reqs, int count, hipStream_t s,
                                     Plan* tp) {
  if (count <= 0) return hipSuccess;
  if (count > kMaxBatch) return hipErrorInvalidValue;
  int max_nblk = 1, max_cpk = 0, max_m = 0;
  for (int i = 0; i < count; ++i) {
    if (reqs[i].L.m > 0) {
      max_m = std::max(max_m, reqs[i].L.m);
      max_cpk = std::max(max_cpk, reqs[i].L.cpk);
      max_nblk = std::max(max_nblk, reqs[i].L.nblk);
    } else {
      // no cells: one empty region
      hipError_t e = launch_zero_i32(reqs[i].L.blk_cnt,
                                     (int64_t)reqs[i].L.nblk * (reqs[i].L.nb + 1), s);
      if (e != hipSuccess) return e;
    }
  }
  if (count == 1) {
    BandBatch<1> bb;
    bb.count = 1;
    bb.r[0] = reqs[0];
    return band_scatter_nb(bb, max_nblk, max_cpk, max_m, s, tp);
  }
  BandBatch<kMaxBatch> bb;
  bb.count = count;
  for (int i = 0; i < count; ++i) bb.r[i] = reqs[i];
  return band_scatter_nb(bb, max_nblk, max_cpk, max_m, s, tp);
}

// ---- the density map without allocation -----------------------------------
// A file-scope device array holds the band lists for callers that cannot
// allocate (see fftpl_density_map_noalloc).  Host code never passes the
// array's name to a kernel: its device address, looked up once per device,
// is what the launches get.
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevicesNoalloc] = {};
}  // namespace

// Band lists of the density scatter alone (no wirelength or gather arrays).
BandLayout band_layout_density(int n, int m, void* work, size_t* bytes_out) {
  BandLayout L = band_shape(n, m, false);
  size_t off = 0;
  const size_t o_en = off;
  off = align256(off + sizeof(float4) * (size_t)L.nblk * L.region);
  const size_t o_big = off;
  off = align256(off + sizeof(int32_t) * (size_t)L.nblk * L.cpk);
  const size_t o_ep = off;
  off = align256(off + sizeof(int32_t) * (size_t)m);
  const size_t o_bo = off;
  off = align256(off + sizeof(int32_t) * blk_entries(L));
  const size_t o_bc = off;
  off = align256(off + sizeof(int32_t) * blk_entries(L));
  if (bytes_out) *bytes_out = off;
  if (work) {
    char* b = static_cast<char*>(work);
    L.entries = reinterpret_cast<float4*>(b + o_en);
    L.big = reinterpret_cast<int32_t*>(b + o_big);
    L.epos = reinterpret_cast<int32_t*>(b + o_ep);
    L.blk_off = reinterpret_cast<int32_t*>(b + o_bo);
    L.blk_cnt = reinterpret_cast<int32_t*>(b + o_bc);
  }
  return L;
}

hipError_t noalloc_scratch(void** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevicesNoalloc) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_band_scan(const GridF& g, const BandLayout& L, const float* x,
                            const float* y, const float* w, const float* h, const float* base,
                            float* rho, hipStream_t s, Plan* tp) {
  BandReq q;
  q.g = g;
  q.L = L;
  q.x = x;
  q.y = y;
  q.w = w;
  q.h = h;
  q.base = base;
  q.rho = rho;
  hipLaunchKernelGGL(k_band_scan, dim3(L.nb), dim3(kScanThreads), 0, s, q);
  if (tp) plan_mark(*tp, "k_band_scan", s);
  return hipGetLastError();
}

hipError_t launch_band_scatter(const GridF& g, const BandLayout& L, const float* x,
                               const float* y, const float* w, const float* h,
                               const float* base, float* rho, hipStream_t s, Plan* tp) {
  if (density_scans(g.n, L.m, false))
    return launch_band_scan(g, L, x, y, w, h, base, rho, s, tp);
  BandReq q;
  q.g = g;
  q.L = L;
  q.L.xy = nullptr;   // no interleaved copy of the positions
  q.x = x;
  q.y = y;
  q.w = w;
  q.h = h;
  q.base = base;
  q.rho = rho;
  return launch_band_scatter_batch(&q, 1, s, tp);
}

}  // namespace fftpl
