// LBE time step: fused pull streaming + collision (Sec. II.B evolution
// equation; BGK or MRT collision), two cells of a row per thread in FP64
// (one 16-byte access per population; one cell if n is odd), one in FP32.
//
// Data layout: 19 population arrays of `stride` elements each (SoA), cell
// index x fastest.  A wavefront covers 64 consecutive runs, so each of the
// 19 gathers and 19 stores is one contiguous access (the pull of a
// population moving in +-x is shifted by one element, still one run; the
// lanes where a two-cell run wraps around the periodic row fix one element
// up).
//
// Phase: the buffer holds post-collision populations.  Thread (cell x)
// gathers g_q(x) = f*_q(x - xi_q), which is the pre-collision state of the
// next time level, takes its moments, collides, and stores f*_q(x).  The
// moments of the new level are reduced per block into `partials` for the
// global FP64 sums.
#include <cstring>

#include "collision.hpp"

namespace dhit {

// Cells a thread updates.  FP64: two consecutive cells of a row, so that
// each population moves as one 16-byte access per lane (measured 0.962
// against 0.980 ms per 256^3 MRT step with one cell); boxes with odd n run
// one cell per thread.  FP32: one cell (runs of 2 or 4 cells measured 15%
// slower: the registers of several cells' collisions cost occupancy that the
// wider accesses do not win back).
// BGK boxes of more than kBgkRunMaxCells cells run one cell per thread in FP64
// too: two BGK collisions take 176 registers (MRT 136), two waves per SIMD,
// which does not keep enough accesses in flight once the populations come
// from HBM (us per step with two cells and with one: 256^3 971 and 930, 128^3
// 135 and 122, 96^3 62.2 and 57.1; 64^3, in the caches, 19.0 and 19.5).
// At 256^3 in FP64 the MRT step takes 0.927 ms; plain copies of 19 arrays of its
// layout took 0.902 (64-thread blocks) to 0.960 ms over access widths and block
// sizes.
template <typename Real>
constexpr int kRunCells = sizeof(Real) == 8 ? 2 : 1;
constexpr int64_t kBgkRunMaxCells = 512000;

// A small box stepped alone runs one cell per thread in blocks of
// kSmallBlock threads, up to kSmallCells<Real> cells: its launch lasts as long
// as one thread's chain of loads, collision and stores, and two cells in a
// row, or fewer and larger blocks, only lengthen it.  Step of a 32^3 box, us
// (with its finalisation launch), against kRunCells in blocks of kBlock:
// FP64 MRT 6.8 (11.8), 48^3 12.6 (15.1), 52^3 14.8 (16.2), but 56^3 17.4
// (16.6); FP32 7.0 (7.3), 36^3 8.1 (7.9).  Blocks of 64 threads: 32^3 7.0,
// 48^3 12.7, 52^3 15.7.  (Batches keep blocks of kBlock threads: a small box's
// populations are the same bits there, its step sums are grouped otherwise and
// agree to rounding.)
constexpr int kSmallBlock = 128;
template <typename Real>
constexpr int64_t kSmallCells = sizeof(Real) == 8 ? 150000 : 32768;

template <typename Real, int C>
struct Run {
  Real v[C];
};

// Values of one population at the C cells x - SX .. x - SX + C - 1 of a row
// (periodic in x; x is a multiple of C, SX = xi_x of the population), where
// `row` points at element 0 of the source row.  One vector access per lane;
// the lanes at the row's ends, where the run wraps, fix one element up with
// an extra scalar load.
template <int SX, int C, typename Real>
__device__ __forceinline__ Run<Real, C> load_run(const global_t<Real> *row, int x, int n) {
  Run<Real, C> r;
  if constexpr (C == 1) {
    int s = x - SX;
    s = s < 0 ? s + n : (s >= n ? s - n : s);
    r.v[0] = row[s];
  } else if constexpr (SX == 0) {
    __builtin_memcpy(&r, row + x, sizeof(r));
  } else {
    // a wrapping run starts at x (SX = +1, x = 0) or ends at n - 1 (SX = -1)
    const bool wrap = SX > 0 ? x == 0 : x + C == n;
    Run<Real, C> a;
    __builtin_memcpy(&a, row + (wrap ? x : x - SX), sizeof(a));
    if (wrap) {
      const Real e = SX > 0 ? row[n - 1] : row[0];
#pragma unroll
      for (int k = 0; k < C; ++k) {
        if constexpr (SX > 0)
          r.v[k] = k == 0 ? e : a.v[k - 1];
        else
          r.v[k] = k == C - 1 ? e : a.v[k + 1];
      }
    } else {
      r = a;
    }
  }
  return r;
}

// Pull of the C cells starting at `cell` (same row): f[k][q] = the value that
// streams into cell + k along xi_q.
template <int C, typename Real>
__device__ __forceinline__ void pull(const global_t<Real> *__restrict__ src, int n, int64_t stride, int cell,
                                     Real (&f)[C][kQ]) {
  const int x = cell % n;
  const int t = cell / n;
  const int y = t % n;
  const int z = t / n;
  const int row = cell - x;
  const AxisOff oy = axis_offsets(y, n, n), oz = axis_offsets(z, n, n * n);
  static_for<kQ>([&](auto q) {
    // source row of the cells - xi_q
    int off = row;
    if constexpr (kCy[q] == 1) off += oy.dn;
    if constexpr (kCy[q] == -1) off += oy.up;
    if constexpr (kCz[q] == 1) off += oz.dn;
    if constexpr (kCz[q] == -1) off += oz.up;
    const Run<Real, C> r = load_run<kCx[q], C>(src + (int64_t)q * stride + off, x, n);
#pragma unroll
    for (int k = 0; k < C; ++k) f[k][q] = r.v[k];
  });
}

// Update of the C cells starting at `cell` (same row); adds their moments
// to the block's sums v.
template <int K, int C, typename Real>
__device__ __forceinline__ void lbe_run(const global_t<Real> *__restrict__ src, global_t<Real> *__restrict__ dst,
                                        const StepParams &p, int cell, double (&v)[kNumSums]) {
  Real f[C][kQ];
  pull<C, Real>(src, p.n, p.stride, cell, f);
#pragma unroll
  for (int k = 0; k < C; ++k) {
    Real drho, jx, jy, jz;
    cell_moments<Real>(f[k], drho, jx, jy, jz);
    sums_of_cell<Real>(drho, jx, jy, jz, p.inv_rho0, v);
    collide<K, Real>(f[k], drho, jx, jy, jz, p);
  }
  // the new state is read only by the next step: stream it past the caches
  static_for<kQ>([&](auto q) {
    global_t<Real> *d = dst + (int64_t)q * p.stride + cell;
    if constexpr (C == 1) {
      __builtin_nontemporal_store(f[0][q], d);
    } else {
      typedef Real Vec __attribute__((ext_vector_type(C)));
      Vec w;
#pragma unroll
      for (int k = 0; k < C; ++k) w[k] = f[k][q];
      __builtin_nontemporal_store(w, reinterpret_cast<global_t<Vec> *>(d));
    }
  });
}

// One pass of the initial-state iteration of an LBE box (Sec. IV.A: the
// kinetic schemes start from the density fluctuation and non-equilibrium
// part that belong to the initial velocity, found by running the scheme
// with the velocity held at its initial value): a time step from src, then
// every cell's momentum put back to rho0 u while its density and its
// non-equilibrium part are kept, f += E(drho, rho0 u) - E(drho, j), with E
// the state init_kernel builds, into dst.  Both collisions conserve drho and j
// and relax only f - E, so the update gives the same result on the
// post-collision state as on the pre-collision one.
// drho_out (optional) receives drho; with drho_prev and block_max given,
// block b stores the largest |drho - drho_prev| of its cells in block_max[b].
// Bound by memory: one pass reads and writes the state once (as a step and a
// pass of its own, with the sums nobody asked for, 34 us at 64^3 in FP64;
// now 17).
template <int K, typename Real>
__global__ __launch_bounds__(kBlock) void lbe_hold_kernel(const Real *__restrict__ src, Real *__restrict__ dst,
                                                          const double *__restrict__ u, double *__restrict__ drho_out,
                                                          const double *__restrict__ drho_prev,
                                                          double *__restrict__ block_max, StepParams p, int ncell) {
  __shared__ double wave_max[kWaves];
  const int cell = blockIdx.x * kBlock + threadIdx.x;
  double dev = 0.0;
  if (cell < ncell) {
    Real g[1][kQ];
    pull<1, Real>(to_global(src), p.n, p.stride, cell, g);
    Real (&f)[kQ] = g[0];
    Real r, jx, jy, jz;
    cell_moments<Real>(f, r, jx, jy, jz);
    collide<K, Real>(f, r, jx, jy, jz, p);
    cell_moments<Real>(f, r, jx, jy, jz);
    const Real hx = Real(p.rho0 * u[cell]);
    const Real hy = Real(p.rho0 * u[(int64_t)ncell + cell]);
    const Real hz = Real(p.rho0 * u[2 * (int64_t)ncell + cell]);
    Real held[kQ], now[kQ];
    if constexpr (K == kMRT) {
      mrt_equilibrium_populations<Real>(r, hx, hy, hz, p, held);
      mrt_equilibrium_populations<Real>(r, jx, jy, jz, p, now);
    } else {
      equilibrium<Real>(r, hx, hy, hz, Real(p.rho0), Real(p.inv_rho0), held);
      equilibrium<Real>(r, jx, jy, jz, Real(p.rho0), Real(p.inv_rho0), now);
    }
    static_for<kQ>([&](auto q) {
      __builtin_nontemporal_store(f[q] + (held[q] - now[q]), to_global(dst) + (int64_t)q * p.stride + cell);
    });
    if (drho_out) drho_out[cell] = (double)r;
    if (drho_prev) {
      dev = fabs((double)r - drho_prev[cell]);
      if (!(dev < INFINITY)) dev = INFINITY;  // a NaN must survive the fmax reduction
    }
  }
  if (!block_max) return;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) dev = fmax(dev, __shfl_down(dev, off, 64));
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = dev;
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = wave_max[0];
    for (int w = 1; w < kWaves; ++w) m = fmax(m, wave_max[w]);
    block_max[blockIdx.x] = m;
  }
}

template <typename Real>
static void hold_launch(dhit_box &b, const void *src, void *dst, const double *d_u, double *d_drho_out,
                        const double *d_drho_prev, double *d_block_max) {
  const Real *s = static_cast<const Real *>(src);
  Real *d = static_cast<Real *>(dst);
  const int blocks = cell_blocks(b.ncell), n = (int)b.ncell;
  if (b.p.method == DHIT_LBE_MRT)
    hipLaunchKernelGGL((lbe_hold_kernel<kMRT, Real>), dim3(blocks), dim3(kBlock), 0, b.stream, s, d, d_u, d_drho_out,
                       d_drho_prev, d_block_max, b.sp, n);
  else
    hipLaunchKernelGGL((lbe_hold_kernel<kBGK, Real>), dim3(blocks), dim3(kBlock), 0, b.stream, s, d, d_u, d_drho_out,
                       d_drho_prev, d_block_max, b.sp, n);
}

void launch_lbe_hold(dhit_box &b, const void *src, void *dst, const double *d_u, double *d_drho_out,
                     const double *d_drho_prev, double *d_block_max) {
  TimedLaunch t(b, DHIT_K_LBE);
  if (b.p.precision == DHIT_FP64)
    hold_launch<double>(b, src, dst, d_u, d_drho_out, d_drho_prev, d_block_max);
  else
    hold_launch<float>(b, src, dst, d_u, d_drho_out, d_drho_prev, d_block_max);
  DHIT_HIP(hipGetLastError());
  t.done();
}

// One launch advances one or many boxes: work item = a run of B * C cells of
// one box of the device table `boxes` (sorted by item_begin), where C, 1 or
// kRunCells<Real>, and the block size B are the same for the whole launch.  A
// single box is a table of one entry.  The per-item partial sums are laid out
// as a block launch's would be.  With prev the launch has one more block, which
// adds up the partials of the step before (see launch_lbe_step).
template <int K, typename Real, int C, int B>
__global__ __launch_bounds__(B) void lbe_kernel(const BatchBox *__restrict__ boxes, int nbox, int total_items,
                                                PendingSums prev) {
  __shared__ double smem[kPendingMax / 64][kNumSums];
  // the extra block is the first: it starts with the others and has ended
  // before they do
  const int extra = prev.nblocks > 0, G = gridDim.x - extra, block = blockIdx.x - extra;
  if (block < 0) {
    add_pending<B / 64>(prev.partials, prev.nblocks, prev.out, smem);
    return;
  }
  for (int it = block; it < total_items; it += G) {
    const int b = find_batch_box(boxes, nbox, it);
    const BatchBox &d = boxes[b];
    const int local = it - d.item_begin;
    const int cell = (local * B + threadIdx.x) * C;
    double v[kNumSums] = {0, 0, 0, 0, 0};
    if (cell < d.ncell)
      lbe_run<K, C, Real>(to_global(static_cast<const Real *>(d.f[d.cur])), to_global(static_cast<Real *>(d.f[d.cur ^ 1])),
                          d.sp, cell, v);
    write_block_partials<B / 64>(v, d.partials, d.items, local, smem);
    __syncthreads();
  }
}

// Work split of a box stepped alone.
LbeSplit lbe_split(int n, int method, int precision) {
  const int64_t ncell = (int64_t)n * n * n;
  if (ncell <= (precision == DHIT_FP64 ? kSmallCells<double> : kSmallCells<float>)) return {1, kSmallBlock};
  return {lbe_cells_per_thread(n, method, precision), kBlock};
}

int lbe_cells_per_thread(int n, int method, int precision) {
  int c = precision == DHIT_FP64 ? kRunCells<double> : kRunCells<float>;
  if (method == DHIT_LBE_BGK && (int64_t)n * n * n > kBgkRunMaxCells) c = 1;
  return n % c == 0 ? c : 1;
}

int lbe_items(int64_t ncell, const LbeSplit &s) {
  return (int)((ncell / s.cells + s.threads - 1) / s.threads);
}

template <typename Real, int C, int B>
static void lbe_launch_typed(hipStream_t s, int method, const BatchBox *d_boxes, int nbox, int total_items, int grid,
                             const PendingSums &prev) {
  if (method == DHIT_LBE_BGK)
    hipLaunchKernelGGL((lbe_kernel<kBGK, Real, C, B>), dim3(grid + (prev.nblocks > 0)), dim3(B), 0, s, d_boxes, nbox,
                       total_items, prev);
  else
    hipLaunchKernelGGL((lbe_kernel<kMRT, Real, C, B>), dim3(grid + (prev.nblocks > 0)), dim3(B), 0, s, d_boxes, nbox,
                       total_items, prev);
}

template <typename Real>
static void lbe_launch_split(hipStream_t s, int method, const LbeSplit &w, const BatchBox *d_boxes, int nbox,
                             int total_items, int grid, const PendingSums &prev) {
  if (w.threads == kSmallBlock && w.cells == 1)
    lbe_launch_typed<Real, 1, kSmallBlock>(s, method, d_boxes, nbox, total_items, grid, prev);
  else if (w.threads == kBlock && w.cells == kRunCells<Real>)
    lbe_launch_typed<Real, kRunCells<Real>, kBlock>(s, method, d_boxes, nbox, total_items, grid, prev);
  else if (w.threads == kBlock && w.cells == 1)
    lbe_launch_typed<Real, 1, kBlock>(s, method, d_boxes, nbox, total_items, grid, prev);
  else
    throw Error(DHIT_EINVAL, "no LBE kernel for this work split");
}

void launch_lbe_batch(hipStream_t s, int method, int precision, const LbeSplit &w, const BatchBox *d_boxes, int nbox,
                      int total_items, int grid, const PendingSums &prev) {
  if (precision == DHIT_FP64)
    lbe_launch_split<double>(s, method, w, d_boxes, nbox, total_items, grid, prev);
  else
    lbe_launch_split<float>(s, method, w, d_boxes, nbox, total_items, grid, prev);
  DHIT_HIP(hipGetLastError());
}

// The two one-box tables of an LBE box (entry c steps from f[c] to f[1 - c]).
void lbe_table_entries(const dhit_box &b, BatchBox (&e)[2]) {
  const LbeSplit w = lbe_split(b.n, b.p.method, b.p.precision);
  for (int c = 0; c < 2; ++c) {
    std::memset(&e[c], 0, sizeof(BatchBox));
    e[c].f[0] = b.f[0];
    e[c].f[1] = b.f[1];
    e[c].sp = b.sp;
    e[c].ncell = (int)b.ncell;
    e[c].item_begin = 0;
    e[c].items = lbe_items(b.ncell, w);
    e[c].partials = b.partials + (size_t)c * 5 * b.max_blocks;
    e[c].hist = b.hist;
    e[c].cur = c;
  }
}

void launch_lbe_step(dhit_box &b, const void *src, void *dst, double *sums_out, bool defer, PendingSums *pend) {
  if (!b.step_table) throw Error(DHIT_EINVAL, "box has no step table");
  int entry;
  if (src == b.f[0] && dst == b.f[1]) entry = 0;
  else if (src == b.f[1] && dst == b.f[0]) entry = 1;
  else throw Error(DHIT_EINVAL, "LBE step between buffers that are not the box's");
  const LbeSplit w = lbe_split(b.n, b.p.method, b.p.precision);
  const int items = lbe_items(b.ncell, w);
  {
    TimedLaunch t(b, DHIT_K_LBE);
    launch_lbe_batch(b.stream, b.p.method, b.p.precision, w, b.step_table + entry, 1, items, items,
                     pend ? *pend : PendingSums{});
    t.done();
  }
  finish_step(b, b.partials + (size_t)entry * 5 * b.max_blocks, items, sums_out, defer, pend);
}

}  // namespace dhit
