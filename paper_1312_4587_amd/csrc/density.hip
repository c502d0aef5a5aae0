// Bin-grid kernels: map fill, fixed-charge rasterisation, the movable-cell
// density scatter (Eq. (2), Section III-B) and the field gather that turns
// E or psi back into per-cell density gradients (Section III-C).
#include "fftpl_internal.hpp"

namespace fftpl {

GridF make_gridf(const fftpl_grid& g) {
  GridF f;
  f.n = g.n;
  f.xl = (float)g.xl;
  f.yl = (float)g.yl;
  f.inv_bw = (float)(1.0 / g.bin_w);
  f.inv_bh = (float)(1.0 / g.bin_h);
  f.bin_w = (float)g.bin_w;
  f.bin_h = (float)g.bin_h;
  f.rho_t = (float)g.target_density;
  return f;
}

// dst[i] = src ? src[i] : value
__global__ void k_fill(float* __restrict__ dst, const float* __restrict__ src,
                       float value, int64_t count) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < count; i += stride) dst[i] = src ? src[i] : value;
}

__global__ void k_fill_f64(double* __restrict__ dst, double value, int count) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = value;
}

hipError_t launch_fill(float* dst, const float* src, float value, int64_t count,
                       hipStream_t s) {
  if (count <= 0) return hipSuccess;
  int64_t blocks = (count + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_fill, dim3((unsigned)blocks), dim3(256), 0, s, dst, src, value,
                     count);
  return hipGetLastError();
}

hipError_t launch_fill_f64(double* dst, double value, int count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_f64, dim3((count + 63) / 64), dim3(64), 0, s, dst, value,
                     count);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fixed charge: one block per rectangle accumulates its overlap f_b, then a
// pointwise pass scales by rho_t and derives the movable capacity.
// ---------------------------------------------------------------------------
__global__ void k_fixed_cover(GridF g, const float* __restrict__ fx,
                              const float* __restrict__ fy, const float* __restrict__ fw,
                              const float* __restrict__ fh, float* __restrict__ cover) {
  const int i = blockIdx.x;
  const Span sx = cell_span(fx[i], fw[i], g.xl, g.inv_bw, g.n);
  const Span sy = cell_span(fy[i], fh[i], g.yl, g.inv_bh, g.n);
  if (sx.i0 > sx.i1 || sy.i0 > sy.i1) return;
  const int nx = sx.i1 - sx.i0 + 1;
  const int ny = sy.i1 - sy.i0 + 1;
  const int64_t total = (int64_t)nx * ny;
  for (int64_t t = threadIdx.x; t < total; t += blockDim.x) {
    const int ix = sx.i0 + (int)(t % nx);
    const int iy = sy.i0 + (int)(t / nx);
    const float ov = span_overlap(sx, ix) * span_overlap(sy, iy);
    atomicAdd(&cover[(int64_t)iy * g.n + ix], ov);
  }
}

__global__ void k_fixed_finalize(float* __restrict__ base, float* __restrict__ cap,
                                 float rho_t, int64_t count) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float f = base[i];
  base[i] = rho_t * f;
  if (cap) cap[i] = rho_t * fmaxf(0.0f, 1.0f - fminf(1.0f, f));
}

hipError_t launch_fixed_map(const GridF& g, int num_fixed, const float* fx,
                            const float* fy, const float* fw, const float* fh,
                            float* base, float* cap, hipStream_t s) {
  const int64_t nn = (int64_t)g.n * g.n;
  hipError_t e = launch_fill(base, nullptr, 0.0f, nn, s);
  if (e != hipSuccess) return e;
  if (num_fixed > 0) {
    hipLaunchKernelGGL(k_fixed_cover, dim3(num_fixed), dim3(256), 0, s, g, fx, fy, fw,
                       fh, base);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_fixed_finalize, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0,
                     s, base, cap, g.rho_t, nn);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Movable-cell scatter: one thread per cell adds ox*oy into every bin of its
// span with float atomics on the n*n map (4 MB at n = 1024, cache resident).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_scatter(GridF g, int m, const float* __restrict__ x,
                                                 const float* __restrict__ y,
                                                 const float* __restrict__ w,
                                                 const float* __restrict__ h,
                                                 float* __restrict__ rho) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  const Span sx = cell_span(x[i], w[i], g.xl, g.inv_bw, g.n);
  const Span sy = cell_span(y[i], h[i], g.yl, g.inv_bh, g.n);
  for (int iy = sy.i0; iy <= sy.i1; ++iy) {
    const float oy = span_overlap(sy, iy);
    float* row = rho + (int64_t)iy * g.n;
    for (int ix = sx.i0; ix <= sx.i1; ++ix) {
      unsafeAtomicAdd(&row[ix], span_overlap(sx, ix) * oy);
    }
  }
}

hipError_t launch_scatter(const GridF& g, int m, const float* x, const float* y,
                          const float* w, const float* h, float* rho, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter, dim3((m + 255) / 256), dim3(256), 0, s, g, m, x, y, w, h,
                     rho);
  return hipGetLastError();
}

// Zero the per-evaluation scalars and the band counters in one launch.
__global__ void k_init_eval(double* __restrict__ out4, int32_t* __restrict__ counters,
                            int ncount) {
  const int t = threadIdx.x;
  if (t < 4) out4[t] = 0.0;
  if (counters)
    for (int k = t; k < ncount; k += blockDim.x) counters[k] = 0;
}

hipError_t launch_init_eval(double* out4, int32_t* counters, int ncount, hipStream_t s) {
  hipLaunchKernelGGL(k_init_eval, dim3(1), dim3(256), 0, s, out4, counters, ncount);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Field gather.  FIELD: g = -scale/bin * sum ov * E (E separate or
// interleaved).  EXACT: g = 2*scale/bin * sum_other-axis ov *
// [psi at right edge - psi at left edge] for edges strictly inside (0, n).
// ---------------------------------------------------------------------------
// PINS: 0 density gradient only; 1 plus the sum of the cell's contiguous pin
// slots (cell_ptr, pin_grad).
// Random reads of the maps bound it: a cell touches one or two 128-byte lines of
// a map row for 24 bytes of it.  density_grad_small and density_grad_maps
// read a cell's bins of one row in one or two loads; 2.1M cells at n = 1024 in
// random order: EXACT 59.9 -> 24.7 us, FIELD 77.3 -> 72.5 us.
constexpr int kGatherThreads = 256;

template <int MODE, bool INTERLEAVED, int PINS>
__global__ void __launch_bounds__(kGatherThreads)
    k_gather(GridF g, int m, const float* __restrict__ x, const float* __restrict__ y,
             const float* __restrict__ w, const float* __restrict__ h,
             const float* __restrict__ ex, const float* __restrict__ ey,
             const float2* __restrict__ exy, const float* __restrict__ psi, float scale,
             int accumulate, const int32_t* __restrict__ cell_ptr,
             const float2* __restrict__ pin_grad, float* __restrict__ gx,
             float* __restrict__ gy) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) {
    // the cell's own loads go out together, before the map reads that
    // depend on them
    const float xi = x[i], yi = y[i], wi = w[i], hi = h[i];
    const Span sx = cell_span(xi, wi, g.xl, g.inv_bw, g.n);
    const Span sy = cell_span(yi, hi, g.yl, g.inv_bh, g.n);
    const float2 d = INTERLEAVED ? density_grad_small<MODE>(g, sx, sy, exy, psi)
                                 : density_grad_maps<MODE>(g, sx, sy, ex, ey, psi);
    float ax = scale * d.x, ay = scale * d.y;
    if (PINS == 1) {
      // the cell's wirelength gradient: its pins' slots are contiguous
      const int k1 = cell_ptr[i + 1];
      for (int k = cell_ptr[i]; k < k1; ++k) {
        const float2 q = pin_grad[k];
        ax += q.x;
        ay += q.y;
      }
    }
    if (accumulate) {
      gx[i] += ax;
      gy[i] += ay;
    } else {
      gx[i] = ax;
      gy[i] = ay;
    }
  }
}

// FIELD from two maps that together are larger than an XCD's L2 (4 MB).  The two
// are read one after the other: a block keeps its cells in LDS (each lane its
// own), gathers Ex for all of them and then Ey, and as the blocks of the grid
// run in step, most of the chip works on one map at a time.  Results pass the
// caches by (non-temporal; the cells too made clustered ones slower, 37 -> 42 us).
// m = 2.1M, n = 1024, random order: 72.5 -> 60 us (L2 misses bound both); m = 1M:
// 41.4 -> 30; n = 2048: 155 -> 134.
// Blocks of four or five cells per lane drift apart and measured the same at
// 2.1M; one launch half per map (cells read twice) 54 us, but 24.9 in place of
// 19.3 us when the cells are ordered by position.
// A large cell's bins are shared out over its wavefront, in the first pass and for
// both maps: by its own lane, 2.1M cells with one in a hundred 30 bins wide took
// 1140 us (585 where one pass summed both maps), now 103.
// Smaller maps (n = 512: 2 MB both) stay in the L2 together, 27.5 us in one pass
// against 34.8 in two; fewer cells than the chip has lanes (8 blocks of 256 on
// each of 256 compute units) are one cell per lane in flight at once, and gain
// nothing (n = 1024: 20.9 against 19.7 us at 262k, 18.1 against 23.9 at 123k; at
// 524k 26.3 against 23.5).  All cells in one place, both maps in the L1, is what it
// loses (2.1M 13.0 -> 17.6).
constexpr int kGatherPhaseCells = 2;
constexpr int kTwoMapsMinN = 1024;
constexpr int kTwoMapsMinCells = 524288;

__global__ void __launch_bounds__(kGatherThreads, 8)
    k_gather_two_maps(GridF g, int m, const float* __restrict__ x,
                      const float* __restrict__ y, const float* __restrict__ w,
                      const float* __restrict__ h, const float* __restrict__ ex,
                      const float* __restrict__ ey, float scale, int accumulate,
                      float* __restrict__ gx, float* __restrict__ gy) {
  __shared__ float4 cell[kGatherPhaseCells][kGatherThreads];
  const int n = g.n, t = threadIdx.x;
  const int64_t i0 = (int64_t)blockIdx.x * kGatherThreads + t;
  const int64_t step = (int64_t)gridDim.x * kGatherThreads;
  const int lane = t & (kWave - 1);
#pragma unroll
  for (int c = 0; c < kGatherPhaseCells; ++c) {
    const int64_t i = min(i0 + c * step, (int64_t)m - 1);
    cell[c][t] = make_float4(x[i], y[i], w[i], h[i]);
  }
  unsigned done = 0;   // the lane's large cells, both sums taken in the first pass
#pragma unroll 1
  for (int p = 0; p < 2; ++p) {
    const float* __restrict__ e = p ? ey : ex;
    float* __restrict__ out = p ? gy : gx;
    const float inv = p ? g.inv_bh : g.inv_bw;
#pragma unroll 1
    for (int c = 0; c < kGatherPhaseCells; ++c) {
      const int64_t i = i0 + c * step;
      const float4 q = cell[c][t];
      const Span sx = cell_span(q.x, q.z, g.xl, g.inv_bw, n);
      const Span sy = cell_span(q.y, q.w, g.yl, g.inv_bh, n);
      if (p == 0) {
        // large cells: each by the whole wavefront, eight columns of eight rows at a time
        const bool large = i < m && sx.i0 <= sx.i1 && sy.i0 <= sy.i1 && !WideRows::fits(sx, sy, n);
        for (unsigned long long bm = __ballot(large); bm; bm &= bm - 1) {
          const int l = __ffsll((long long)bm) - 1;
          const Span bx = span_from_edges(__shfl(sx.lo, l), __shfl(sx.hi, l), n);
          const Span by = span_from_edges(__shfl(sy.lo, l), __shfl(sy.hi, l), n);
          float ax = 0.0f, ay = 0.0f;
          for (int iy = by.i0 + (lane >> 3); iy <= by.i1; iy += 8) {
            const float oy = span_overlap(by, iy);
            for (int ix = bx.i0 + (lane & 7); ix <= bx.i1; ix += 8) {
              const float ov = span_overlap(bx, ix) * oy;
              ax += ov * ex[(int64_t)iy * n + ix];
              ay += ov * ey[(int64_t)iy * n + ix];
            }
          }
          ax = scale * (-g.inv_bw * wave_sum_dpp(ax));
          ay = scale * (-g.inv_bh * wave_sum_dpp(ay));
          if (lane == l) {
            gx[i] = accumulate ? gx[i] + ax : ax;
            gy[i] = accumulate ? gy[i] + ay : ay;
            done |= 1u << c;
          }
        }
      }
      if (i >= m || (done >> c & 1)) continue;
      const float a = scale * (-inv * span_map_sum(n, sx, sy, e));
      if (accumulate)
        out[i] += a;
      else
        __builtin_nontemporal_store(a, out + i);
    }
  }
}

hipError_t launch_gather(const GridF& g, int m, const float* x, const float* y,
                         const float* w, const float* h, const float* ex,
                         const float* ey, const float* exy, const float* psi,
                         int grad_mode, float scale, int accumulate, float* gx,
                         float* gy, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  dim3 grid((m + kGatherThreads - 1) / kGatherThreads), block(kGatherThreads);
  const float2* e2 = reinterpret_cast<const float2*>(exy);
  if (grad_mode == FFTPL_GRAD_EXACT && exy) {
    // difference maps (Dx, Dy) in exy, psi for cells at the border
    hipLaunchKernelGGL((k_gather<FFTPL_GRAD_EXACT, true, 0>), grid, block, 0, s, g, m, x, y,
                       w, h, ex, ey, e2, psi, scale, accumulate, nullptr, nullptr, gx, gy);
  } else if (grad_mode == FFTPL_GRAD_EXACT) {
    hipLaunchKernelGGL((k_gather<FFTPL_GRAD_EXACT, false, 0>), grid, block, 0, s, g, m, x, y,
                       w, h, ex, ey, e2, psi, scale, accumulate, nullptr, nullptr, gx, gy);
  } else if (exy) {
    hipLaunchKernelGGL((k_gather<FFTPL_GRAD_FIELD, true, 0>), grid, block, 0, s, g, m, x, y,
                       w, h, ex, ey, e2, psi, scale, accumulate, nullptr, nullptr, gx, gy);
  } else if (g.n >= kTwoMapsMinN && m >= kTwoMapsMinCells) {
    const int per = kGatherThreads * kGatherPhaseCells;
    hipLaunchKernelGGL(k_gather_two_maps, dim3((unsigned)((m + (int64_t)per - 1) / per)), block,
                       0, s, g, m, x, y, w, h, ex, ey, scale, accumulate, gx, gy);
  } else {
    hipLaunchKernelGGL((k_gather<FFTPL_GRAD_FIELD, false, 0>), grid, block, 0, s, g, m, x, y,
                       w, h, ex, ey, e2, psi, scale, accumulate, nullptr, nullptr, gx, gy);
  }
  return hipGetLastError();
}

hipError_t launch_gather_pins(const GridF& g, int m, const float* x, const float* y,
                              const float* w, const float* h, const float* exy,
                              const float* psi, int grad_mode, float scale,
                              const int32_t* cell_ptr, const float2* pin_grad, float* gx,
                              float* gy, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  dim3 grid((m + kGatherThreads - 1) / kGatherThreads), block(kGatherThreads);
  const float2* e2 = reinterpret_cast<const float2*>(exy);
  if (grad_mode == FFTPL_GRAD_EXACT) {
    hipLaunchKernelGGL((k_gather<FFTPL_GRAD_EXACT, true, 1>), grid, block, 0, s, g, m, x,
                       y, w, h, nullptr, nullptr, e2, psi, scale, 0, cell_ptr, pin_grad, gx, gy);
  } else {
    hipLaunchKernelGGL((k_gather<FFTPL_GRAD_FIELD, true, 1>), grid, block, 0, s, g, m, x,
                       y, w, h, nullptr, nullptr, e2, psi, scale, 0, cell_ptr, pin_grad, gx, gy);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Test export: the integer span of every cell.
// ---------------------------------------------------------------------------
__global__ void k_cell_bins(GridF g, int m, const float* __restrict__ x,
                            const float* __restrict__ y, const float* __restrict__ w,
                            const float* __restrict__ h, int32_t* __restrict__ ranges) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  const Span sx = cell_span(x[i], w[i], g.xl, g.inv_bw, g.n);
  const Span sy = cell_span(y[i], h[i], g.yl, g.inv_bh, g.n);
  int32_t* r = ranges + 4 * (int64_t)i;
  r[0] = sx.i0;
  r[1] = sx.i1;
  r[2] = sy.i0;
  r[3] = sy.i1;
}

hipError_t launch_cell_bins(const GridF& g, int m, const float* x, const float* y,
                            const float* w, const float* h, int32_t* ranges,
                            hipStream_t s) {
  if (m <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_cell_bins, dim3((m + 255) / 256), dim3(256), 0, s, g, m, x, y, w, h,
                     ranges);
  return hipGetLastError();
}

}  // namespace fftpl
