// Device code of the banded density scatter shared by its own kernels and the
// compact evaluation kernels: the walk over a band's entries and their
// fixed-point accumulation in LDS.
#pragma once

#include "fftpl_internal.hpp"

namespace fftpl {

template <int CB>
struct CellBatch {
  float x[CB], y[CB], w[CB], h[CB];
};

template <int CB>
__device__ __forceinline__ void load_batch(CellBatch<CB>& c, int base, int m,
                                           const float* __restrict__ x,
                                           const float* __restrict__ y,
                                           const float* __restrict__ w,
                                           const float* __restrict__ h) {
  // unconditional (index clamped, m >= 1) so the whole batch is in flight
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    const int i = min(base + j * kBandThreads + (int)threadIdx.x, m - 1);
    c.x[j] = x[i];
    c.y[j] = y[i];
    c.w[j] = w[i];
    c.h[j] = h[i];
  }
}

// Counting block k of the scatter: sorts its cells' edges by band into its own
// region.  LT: BandLayout, or a request with its fields.
template <int CB, typename LT>
__device__ __forceinline__ void place_block(const GridF& g, const LT& L, int k,
                                            const float* __restrict__ x,
                                            const float* __restrict__ y,
                                            const float* __restrict__ w,
                                            const float* __restrict__ h) {
  constexpr int NT = kBandThreads;
  const int t = threadIdx.x;
  __shared__ int hist[257], cur[257];   // the bands, then the tall cells
  for (int b = t; b <= L.nb; b += NT) hist[b] = 0;
  __syncthreads();
  const int c0 = k * L.cpk, c1 = min(L.m, c0 + L.cpk);   // one batch of cells per thread
  CellBatch<CB> c;
  load_batch(c, c0, L.m, x, y, w, h);
  float4 e[CB];
  int b0[CB], nbd[CB];   // first band, bands listed (0: none, -1: tall)
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    const int i = c0 + j * NT + t;
    nbd[j] = 0;
    b0[j] = 0;
    if (i >= c1) continue;
    if (L.xy) L.xy[i] = make_float2(c.x[j], c.y[j]);
    const Span sx = cell_span(c.x[j], c.w[j], g.xl, g.inv_bw, g.n);
    const Span sy = cell_span(c.y[j], c.h[j], g.yl, g.inv_bh, g.n);
    if (sx.i0 > sx.i1 || sy.i0 > sy.i1) continue;
    b0[j] = sy.i0 / L.rows;
    const int b1 = sy.i1 / L.rows;
    e[j] = make_float4(sx.lo, sx.hi, sy.lo, sy.hi);
    if (b1 - b0[j] >= kMaxBands) {
      nbd[j] = -1;
      atomicAdd(&hist[L.nb], 1);
    } else {
      nbd[j] = b1 - b0[j] + 1;
      for (int b = b0[j]; b <= b1; ++b) atomicAdd(&hist[b], 1);
    }
  }
  __syncthreads();
  int tot;
  const int ex = block_exclusive_scan<NT>(t < L.nb ? hist[t] : 0, &tot);
  if (t <= L.nb) {
    const int off = t < L.nb ? ex : 0;   // the tall cells have a list of their own
    L.blk_off[(size_t)t * L.nblk + k] = off;
    L.blk_cnt[(size_t)t * L.nblk + k] = hist[t];
    cur[t] = off;
  }
  __syncthreads();
  const int64_t rbase = (int64_t)k * L.region;
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    const int i = c0 + j * NT + t;
    if (i >= c1) continue;
    int first = -1;   // the cell's entry in its first band, if listed
    if (nbd[j] > 0) {
      for (int b = b0[j]; b < b0[j] + nbd[j]; ++b) {
        const int q = atomicAdd(&cur[b], 1);
        L.entries[rbase + q] = e[j];
        if (b == b0[j]) first = (int)(rbase + q);
      }
    } else if (nbd[j] < 0) {
      L.big[(int64_t)k * L.cpk + atomicAdd(&cur[L.nb], 1)] = i;
    }
    if (L.epos) L.epos[i] = first;
  }
}

// owner[a .. e - 1] = t for the window positions of every thread t's slice
// (ascending over t, together all of the window's).  Short slices (`longs` unset)
// are written by their own threads.  Otherwise each writes its first position and
// a running maximum over the positions, KB per thread, fills in the rest: a
// crowded band's slices are long, and writing them one after another took most
// of its walk (a wavefront per slice: 37 of the 78 us of 123k cells crowded into
// 12 bands of n = 512).  Every thread must call it; ends with a barrier.
constexpr int kOwnFill = 32;   // most entries of a short slice
template <int NTB, int KB>
__device__ __forceinline__ void fill_owner(unsigned short* owner, int a, int e, bool longs) {
  typedef unsigned short Chunk __attribute__((ext_vector_type(KB > 1 ? KB : 2)));
  const int t = threadIdx.x;
  if (!longs) {
    for (int v = a; v < e; ++v) owner[v] = (unsigned short)t;
    __syncthreads();
    return;
  }
  __shared__ unsigned short wmax[NTB / kWave];
  const int lane = t & (kWave - 1), w = t / kWave;
  Chunk o = 0;
  if constexpr (KB > 1)
    reinterpret_cast<Chunk*>(owner)[t] = o;
  else
    owner[t] = 0;
  __syncthreads();
  if (a < e) owner[a] = (unsigned short)t;
  __syncthreads();
  if constexpr (KB > 1)
    o = reinterpret_cast<Chunk*>(owner)[t];
  else
    o[0] = owner[t];
#pragma unroll
  for (int j = 1; j < KB; ++j) o[j] = max(o[j], o[j - 1]);
  int m = o[KB - 1];
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int u = __shfl_up(m, off, kWave);
    if (lane >= off) m = max(m, u);
  }
  if (lane == kWave - 1) wmax[w] = (unsigned short)m;
  int before = __shfl_up(m, 1, kWave);   // of the wavefront's lower lanes
  if (lane == 0) before = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NTB / kWave; ++k)
    if (k < w) before = max(before, (int)wmax[k]);
#pragma unroll
  for (int j = 0; j < KB; ++j) o[j] = max(o[j], (unsigned short)before);
  if constexpr (KB > 1)
    reinterpret_cast<Chunk*>(owner)[t] = o;
  else
    owner[t] = o[0];
  __syncthreads();
}

// The entries of band `band` (band = nb: the tall cells) lie in one slice per
// region: slice k holds blk_cnt[band][k] entries from index
// k * stride + blk_off[band][k].  A block of NTB threads walks them in chunks
// of NTB slices: the chunk's counts are scanned, and the chunk's entries are
// taken in windows of NTB * KB.  For each window every slice enters its own
// number into an LDS owner map at the window positions it covers, so a
// thread finds the slice of its entry with one LDS read (a binary search over
// the scan, ten dependent LDS reads per entry, cost the walk more than its
// loads).  Thread t takes window entries t, t + NTB, ...: KB of them, whose
// indices are all known before f(index) uses any, so the caller can issue
// their loads together.  Every thread of the block must call it; `owner`
// holds NTB * KB entries, 16-byte aligned.  LT: BandLayout, or a request with its fields.
template <int NTB, int KB, typename LT, typename F>
__device__ __forceinline__ void walk_band(const LT& L, int band, int64_t stride,
                                          int* pre, int64_t* start, unsigned short* owner,
                                          F f) {
  static_assert(NTB <= 65536, "slice numbers are u16");
  constexpr int W = NTB * KB;
  const int t = threadIdx.x;
  for (int k0 = 0; k0 < L.nblk; k0 += NTB) {
    const int k = k0 + t;
    const int c = k < L.nblk ? L.blk_cnt[(size_t)band * L.nblk + k] : 0;
    const int o = k < L.nblk ? L.blk_off[(size_t)band * L.nblk + k] : 0;
    int tot;
    bool longs;   // any slice longer than kOwnFill
    const int ex = block_exclusive_scan<NTB>(c, &tot, c > kOwnFill, &longs);
    pre[t] = ex;
    start[t] = (int64_t)k * stride + o;
    for (int w0 = 0; w0 < tot; w0 += W) {
      fill_owner<NTB, KB>(owner, max(ex, w0) - w0, min(ex + c, w0 + W) - w0, longs);
      int64_t idx[KB];
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        const int v = w0 + j * NTB + t;
        idx[j] = -1;
        if (v < tot) {
          const int sl = owner[v - w0];
          idx[j] = start[sl] + (v - pre[sl]);
        }
      }
      f(idx);
      __syncthreads();   // owner, pre and start are rewritten next
    }
  }
}

// Fixed-point LDS add of an overlap v in [0, 1] (units of 2^-31; a sum of
// up to 2^32 entries stays inside 64 bits).
constexpr double kAccUnit = 1.0 / 2147483648.0;
__device__ __forceinline__ void add_fixed(unsigned long long* a, float v) {
  atomicAdd(a, (unsigned long long)__float2uint_rn(v * 2147483648.0f));
}

// The overlaps of one cell with rows r0 .. r0 + R - 1.
__device__ __forceinline__ void add_span_rows(const Span& sx, const Span& sy, int r0, int R, int n,
                                         unsigned long long* acc) {
  const int ya = max(sy.i0, r0), yb = min(sy.i1, r0 + R - 1);
  for (int iy = ya; iy <= yb; ++iy) {
    const float oy = span_overlap(sy, iy);
    unsigned long long* row = acc + (iy - r0) * n;
    for (int ix = sx.i0; ix <= sx.i1; ++ix) add_fixed(&row[ix], span_overlap(sx, ix) * oy);
  }
}

// Adds the entries of band `band` as long as every slice is short (at most
// kSliceMax entries per lane): each slice is taken by the same few lanes, which
// need its count and offset and nothing from the other slices, where walk_band
// scans the counts and fills the owner map first.  Returns false, having
// added nothing, when a slice is longer (cells crowded into few bands) or there
// are more slices than threads.  Every thread of the block must call it.
constexpr int kSliceMax = 8;
template <int NTB, typename LT>
__device__ __forceinline__ bool add_short_slices(const LT& L, int band, int r0, int n,
                                                 unsigned long long* acc) {
  if (L.nblk > NTB) return false;
  const int lanes = NTB / L.nblk;   // >= 1, per slice
  const int k = (int)threadIdx.x / lanes, l = (int)threadIdx.x - k * lanes;
  int c = 0, o = 0;
  if (k < L.nblk) {
    c = L.blk_cnt[(size_t)band * L.nblk + k];
    o = L.blk_off[(size_t)band * L.nblk + k];
  }
  if (__syncthreads_or(c > kSliceMax * lanes)) return false;
  const float4* e = L.entries + (int64_t)k * L.region + o;
#pragma unroll
  for (int j0 = 0; j0 < kSliceMax; j0 += 4) {
    if (!__any(l + j0 * lanes < c)) break;
    float4 q[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int v = l + (j0 + j) * lanes;
      if (v < c) q[j] = e[v];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (l + (j0 + j) * lanes < c)
        add_span_rows(span_from_edges(q[j].x, q[j].y, n), span_from_edges(q[j].z, q[j].w, n), r0,
                 L.rows, n, acc);
  }
  return true;
}

// LDS of a band walk by NTB threads taking KB entries each.
template <int NTB, int KB>
struct WalkLds {
  int64_t start[NTB];
  int pre[NTB];
  alignas(16) unsigned short owner[NTB * KB];
};

// Adds the cells of band `band` (rows r0 .. r0 + R - 1) into acc (R rows of n
// fixed-point bins, cleared by the caller): the band's entries, then the
// cells too tall to be listed per band, a thread per cell.
// SHORT: try the short slices' form first.
template <int NTB, int KB, bool SHORT, typename LT>
__device__ __forceinline__ void band_accumulate(const GridF& g, const LT& L, int band,
                                                const float* __restrict__ x,
                                                const float* __restrict__ y,
                                                const float* __restrict__ w,
                                                const float* __restrict__ h,
                                                unsigned long long* acc, WalkLds<NTB, KB>& lds) {
  const int n = g.n, R = L.rows, r0 = band * R;
  if (!SHORT || !add_short_slices<NTB>(L, band, r0, n, acc))
    walk_band<NTB, KB>(L, band, L.region, lds.pre, lds.start, lds.owner,
                       [&](const int64_t (&idx)[KB]) {
    float4 q[KB];
#pragma unroll
    for (int j = 0; j < KB; ++j) q[j] = L.entries[idx[j] >= 0 ? idx[j] : 0];
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      if (idx[j] < 0) continue;
      const Span sx = span_from_edges(q[j].x, q[j].y, n);
      const Span sy = span_from_edges(q[j].z, q[j].w, n);
      add_span_rows(sx, sy, r0, R, n, acc);
    }
  });
  if constexpr (NTB >= 1024) {
    walk_band<NTB, 1>(L, L.nb, L.cpk, lds.pre, lds.start, lds.owner, [&](const int64_t (&idx)[1]) {
      if (idx[0] < 0) return;
      const int i = L.big[idx[0]];
      add_span_rows(cell_span(x[i], w[i], g.xl, g.inv_bw, n),
                    cell_span(y[i], h[i], g.yl, g.inv_bh, n), r0, R, n, acc);
    });
  } else {
    // several per thread, as every window of the list costs its barriers: 200k cells,
    // one in ten 30 bins high, the evaluation 403 -> 368 us (with 1024 threads the
    // window is long enough, and the extra slots cost 1 us)
    walk_band<NTB, KB>(L, L.nb, L.cpk, lds.pre, lds.start, lds.owner,
                       [&](const int64_t (&idx)[KB]) {
      int c[KB];
      float cy[KB], ch[KB];
#pragma unroll
      for (int j = 0; j < KB; ++j) c[j] = idx[j] >= 0 ? L.big[idx[j]] : -1;
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        cy[j] = y[max(c[j], 0)];
        ch[j] = h[max(c[j], 0)];
      }
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        if (c[j] < 0) continue;
        const Span sy = cell_span(cy[j], ch[j], g.yl, g.inv_bh, n);
        if (sy.i1 < r0 || sy.i0 >= r0 + R) continue;
        add_span_rows(cell_span(x[c[j]], w[c[j]], g.xl, g.inv_bw, n), sy, r0, R, n, acc);
      }
    });
  }
}

// The same; the usual cell, at most three bins wide in at most two of the
// band's rows, takes straight-line code (the same products in the same order).
__device__ __forceinline__ void add_span(const Span& sx, const Span& sy, int r0, int R, int n,
                                         unsigned long long* acc) {
  const int ya = max(sy.i0, r0), yb = min(sy.i1, r0 + R - 1);
  const int nx = sx.i1 - sx.i0 + 1, ny = yb - ya + 1;
  if (nx <= 0 || ny <= 0) return;
  if (nx <= 3 && ny <= 2) {
    const float o0 = span_overlap(sx, sx.i0), o1 = span_overlap(sx, sx.i0 + 1),
                o2 = span_overlap(sx, sx.i0 + 2);
    unsigned long long* row = acc + (ya - r0) * n + sx.i0;
    float oy = span_overlap(sy, ya);
    add_fixed(row, o0 * oy);
    if (nx > 1) add_fixed(row + 1, o1 * oy);
    if (nx > 2) add_fixed(row + 2, o2 * oy);
    if (ny > 1) {
      oy = span_overlap(sy, ya + 1);
      row += n;
      add_fixed(row, o0 * oy);
      if (nx > 1) add_fixed(row + 1, o1 * oy);
      if (nx > 2) add_fixed(row + 2, o2 * oy);
    }
    return;
  }
  add_span_rows(sx, sy, r0, R, n, acc);
}

// LDS of a band block of NTB threads that reads a small design's cells itself:
// the cells that meet the band go to a list, which all threads drain together.
// Few cells meet a band (90 of 2000 at n = 64); handled where they are found,
// each would hold up its wavefront alone.  k_compact_mid at 2k cells 9.4 ->
// 7.7 us.
template <int NTB, int CAP>
struct ScanLds {
  float4 list[CAP];
  int count;
};

// Adds a small design's cells straight from their arrays (no entries).
template <int NTB, int CAP, typename LT>
__device__ __forceinline__ void band_scan(const GridF& g, const LT& L, int band,
                                          const float* __restrict__ x,
                                          const float* __restrict__ y,
                                          const float* __restrict__ w,
                                          const float* __restrict__ h, unsigned long long* acc,
                                          ScanLds<NTB, CAP>& lds) {
  constexpr int U = CAP / NTB;
  const int n = g.n, R = L.rows, r0 = band * R, t = threadIdx.x, m = L.m;
#pragma unroll 1
  for (int i0 = 0; i0 < m; i0 += CAP) {
    float cx[U], cy[U], cw[U], ch[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + t + u * NTB, m - 1);
      cx[u] = x[i];
      cy[u] = y[i];
      cw[u] = w[i];
      ch[u] = h[i];
    }
    if (t == 0) lds.count = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + t + u * NTB >= m) continue;
      const Span sy = cell_span(cy[u], ch[u], g.yl, g.inv_bh, n);
      if (sy.i1 < r0 || sy.i0 >= r0 + R || sy.i0 > sy.i1) continue;
      const Span sx = cell_span(cx[u], cw[u], g.xl, g.inv_bw, n);
      lds.list[atomicAdd(&lds.count, 1)] = make_float4(sx.lo, sx.hi, sy.lo, sy.hi);
    }
    __syncthreads();
    const int count = lds.count;
#pragma unroll 1
    for (int i = t; i < count; i += NTB) {
      const float4 q = lds.list[i];
      add_span(span_from_edges(q.x, q.y, n), span_from_edges(q.z, q.w, n), r0, R, n, acc);
    }
    __syncthreads();
  }
}

}  // namespace fftpl
