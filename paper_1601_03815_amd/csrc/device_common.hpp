// Device helpers shared by the LBE, DUGKS and diagnostics kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "lattice.hpp"
#include "runtime.hpp"

namespace dhit {

constexpr int kBlock = 256;            // threads per block of the streaming kernels
constexpr int kWaves = kBlock / 64;    // 64-wide wavefronts per block
constexpr int kNumSums = 5;            // sum drho, sum jx, sum jy, sum jz, 1/2 sum |u|^2

// Compensated summation (Kahan): s carries the running sum and c the
// rounding error of the last addition (with its sign reversed), which is
// fed back into the next term, so that the error of a sum of m terms is
// about 2 eps sum |x_i| instead of (m - 1) eps sum |x_i|.  Used for the
// per-cell moment sums of FP32 boxes.
template <typename Real>
struct CompSum {
  Real s = Real(0), c = Real(0);
  __device__ __forceinline__ void add(Real x) {
    const Real y = x - c;
    const Real t = s + y;
    c = (t - s) - y;
    s = t;
  }
  __device__ __forceinline__ void sub(Real x) { add(-x); }
  __device__ __forceinline__ Real value() const { return s - c; }
};

// Moments of one cell: drho = sum f, j = sum xi f (Sec. II.A / II.B).
// Double: plain sums.  Float: compensated sums.
template <typename Real>
__device__ __forceinline__ void cell_moments(const Real (&f)[kQ], Real &drho, Real &jx, Real &jy, Real &jz) {
  if constexpr (std::is_same<Real, double>::value) {
    double r = 0, ax = 0, ay = 0, az = 0;
    static_for<kQ>([&](auto q) {
      r += f[q];
      if constexpr (kCx[q] == 1) ax += f[q];
      if constexpr (kCx[q] == -1) ax -= f[q];
      if constexpr (kCy[q] == 1) ay += f[q];
      if constexpr (kCy[q] == -1) ay -= f[q];
      if constexpr (kCz[q] == 1) az += f[q];
      if constexpr (kCz[q] == -1) az -= f[q];
    });
    drho = r; jx = ax; jy = ay; jz = az;
  } else {
    CompSum<Real> r, ax, ay, az;
    static_for<kQ>([&](auto q) {
      r.add(f[q]);
      if constexpr (kCx[q] == 1) ax.add(f[q]);
      if constexpr (kCx[q] == -1) ax.sub(f[q]);
      if constexpr (kCy[q] == 1) ay.add(f[q]);
      if constexpr (kCy[q] == -1) ay.sub(f[q]);
      if constexpr (kCz[q] == 1) az.add(f[q]);
      if constexpr (kCz[q] == -1) az.sub(f[q]);
    });
    drho = r.value(); jx = ax.value(); jy = ay.value(); jz = az.value();
  }
}

// Discrete incompressible equilibrium of Sec. II.A with RT = 1/3:
// f_q^eq = W_q [drho + rho0 (3 xi.u + 9/2 (xi.u)^2 - 3/2 |u|^2)], u = j/rho0,
// evaluated as W_q (base + 9/2 rho0 (xi.u)^2) + L_q rho0 xi.u with
// base = drho - 3/2 rho0 |u|^2 and L_q = 3 W_q (1/6 on the axes, 1/12 on the
// diagonals).  The momentum of the linear term is u sum_q L_q xi_qx^2 =
// u (2 L_axis + 8 L_diag); with 3 W_q rounded to the working precision that
// factor is 1 + d (d = 7e-9 in FP32), and a BGK or DUGKS collision then adds
// a fixed fraction of d j to the momentum at every step (a steady energy
// drift, 3e-8 per DUGKS step in FP32).  L_diag is rounded and L_axis taken as
// (1 - 8 L_diag)/2, which is exact, so that the factor is exactly 1.
template <typename Real>
constexpr Real kLinDiag = Real(1.0 / 12.0);
template <typename Real>
constexpr Real kLinAxis = (Real(1) - Real(8) * kLinDiag<Real>) / Real(2);

// xi_q . u
template <int Q, typename Real>
__device__ __forceinline__ Real xi_dot(Real ux, Real uy, Real uz) {
  Real xu = Real(0);
  if constexpr (kCx[Q] == 1) xu += ux;
  if constexpr (kCx[Q] == -1) xu -= ux;
  if constexpr (kCy[Q] == 1) xu += uy;
  if constexpr (kCy[Q] == -1) xu -= uy;
  if constexpr (kCz[Q] == 1) xu += uz;
  if constexpr (kCz[Q] == -1) xu -= uz;
  return xu;
}

// f_Q^eq from base and xu = xi_Q . u (see above).
template <int Q, typename Real>
__device__ __forceinline__ Real equilibrium_q(Real base, Real xu, Real rho0) {
  constexpr Real w = Real(kWeight(Q));
  constexpr Real l = speed2(Q) == 0 ? Real(0) : (speed2(Q) == 1 ? kLinAxis<Real> : kLinDiag<Real>);
  const Real even = w * (base + Real(4.5) * rho0 * xu * xu);
  if constexpr (Q == 0)
    return even;
  else
    return even + l * rho0 * xu;
}

template <typename Real>
__device__ __forceinline__ void equilibrium(Real drho, Real jx, Real jy, Real jz, Real rho0, Real inv_rho0,
                                            Real (&feq)[kQ]) {
  const Real ux = jx * inv_rho0, uy = jy * inv_rho0, uz = jz * inv_rho0;
  const Real uu = ux * ux + uy * uy + uz * uz;
  const Real base = drho - Real(1.5) * rho0 * uu;
  static_for<kQ>([&](auto q) { feq[q] = equilibrium_q<q, Real>(base, xi_dot<q>(ux, uy, uz), rho0); });
}

// Value of the lane `Off` lanes above (lanes without one get some value): the
// permlane swaps exchange half-wavefronts and 16-lane rows, DPP shifts within a
// row; no LDS traffic, unlike a shuffle.
template <int Off>
__device__ __forceinline__ unsigned lane_above(unsigned v) {
  if constexpr (Off == 32)
    return __builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
  else if constexpr (Off == 16)
    return __builtin_amdgcn_permlane16_swap(v, v, false, false)[1];
  else
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x100 + Off, 0xf, 0xf, true);
}
template <int Off>
__device__ __forceinline__ double lane_above(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = lane_above<Off>((unsigned)b), hi = lane_above<Off>((unsigned)(b >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// Sum over the wavefront in lane 0, by halving (l takes l + 32, then l + 16, ...).
__device__ __forceinline__ double wave_sum(double v) {
  v += lane_above<32>(v);
  v += lane_above<16>(v);
  v += lane_above<8>(v);
  v += lane_above<4>(v);
  v += lane_above<2>(v);
  v += lane_above<1>(v);
  return v;
}

// Sums of five doubles over a block of NW wavefronts: thread i < 5 returns
// the total of v[i].  Deterministic: a fixed tree inside each wavefront, then
// the wavefront totals in the order of `wave`, the wavefront's place in the sum
// (a kernel that gives its wavefronts changing roles passes the role, so that
// the order does not change with them).
template <int NW>
__device__ __forceinline__ double block_sum5(double (&v)[kNumSums], double (*smem)[kNumSums], int wave) {
  static_for<kNumSums>([&](auto i) { v[i] = wave_sum(v[i]); });
  const int lane = threadIdx.x & 63;
  if (lane == 0) {
    static_for<kNumSums>([&](auto i) { smem[wave][i] = v[i]; });
  }
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x < kNumSums) {
    s = smem[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += smem[w][threadIdx.x];
  }
  return s;
}
template <int NW>
__device__ __forceinline__ double block_sum5(double (&v)[kNumSums], double (*smem)[kNumSums]) {
  return block_sum5<NW>(v, smem, threadIdx.x >> 6);
}

// Per-cell contributions to the five global sums, accumulated in FP64 from
// the stored values (exact for FP32 populations, which double represents).
template <typename Real>
__device__ __forceinline__ void sums_of_populations(const Real (&f)[kQ], double inv_rho0, double (&v)[kNumSums]) {
  double r = 0, ax = 0, ay = 0, az = 0;
  static_for<kQ>([&](auto q) {
    const double x = (double)f[q];
    r += x;
    if constexpr (kCx[q] == 1) ax += x;
    if constexpr (kCx[q] == -1) ax -= x;
    if constexpr (kCy[q] == 1) ay += x;
    if constexpr (kCy[q] == -1) ay -= x;
    if constexpr (kCz[q] == 1) az += x;
    if constexpr (kCz[q] == -1) az -= x;
  });
  v[0] += r;
  v[1] += ax;
  v[2] += ay;
  v[3] += az;
  v[4] += 0.5 * (ax * ax + ay * ay + az * az) * inv_rho0 * inv_rho0;
}

// Per-cell contributions to the five global sums.
template <typename Real>
__device__ __forceinline__ void sums_of_cell(Real drho, Real jx, Real jy, Real jz, double inv_rho0,
                                             double (&v)[kNumSums]) {
  const double x = (double)jx, y = (double)jy, z = (double)jz;
  v[0] += (double)drho;
  v[1] += x;
  v[2] += y;
  v[3] += z;
  v[4] += 0.5 * (x * x + y * y + z * z) * inv_rho0 * inv_rho0;
}

// Pointer into global memory.  The device functions that stream population
// fields take these, so that their accesses compile to global instructions
// also where a kernel reads the field pointers from a device table (through
// a generic pointer they would compile to flat instructions, which count
// against the LDS counter as well: every LDS wait would also wait for memory).
template <typename T>
using global_t = __attribute__((address_space(1))) T;
template <typename T>
__device__ __forceinline__ global_t<T> *to_global(T *p) {
  return (global_t<T> *)p;
}

// Writes the block's five sums to partials laid out [5][nblocks], using
// smem (at least one row of five doubles per wavefront of the block) for
// the reduction (wave as in block_sum5).
template <int NW>
__device__ __forceinline__ void write_block_partials(double (&v)[kNumSums], double *partials, int nblocks, int block,
                                                     double (*smem)[kNumSums], int wave) {
  const double t = block_sum5<NW>(v, smem, wave);
  if (threadIdx.x < kNumSums) to_global(partials)[(int64_t)threadIdx.x * nblocks + block] = t;
}
template <int NW>
__device__ __forceinline__ void write_block_partials(double (&v)[kNumSums], double *partials, int nblocks, int block,
                                                     double (*smem)[kNumSums]) {
  write_block_partials<NW>(v, partials, nblocks, block, smem, threadIdx.x >> 6);
}
template <int NW = kWaves>
__device__ __forceinline__ void write_block_partials(double (&v)[kNumSums], double *partials, int nblocks,
                                                     int block) {
  __shared__ double smem[NW][kNumSums];
  write_block_partials<NW>(v, partials, nblocks, block, smem);
}

// Adds up the partials of the step before (at most kPendingMax), by one block
// of NW wavefronts in the order of a 1024-thread finalisation launch: its
// wavefronts' trees in turn, then their totals in order.  smem: 16 rows.
template <int NW>
__device__ __forceinline__ void add_pending(const double *partials, int nblocks, double *out, double (*smem)[kNumSums]) {
  constexpr int kTurns = kPendingMax / 64 / NW;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = (nblocks + 63) / 64;
  double v[kTurns][kNumSums];  // all turns' loads in flight together
  static_for<kTurns>([&](auto k) {
    const int b = (k * NW + wave) * 64 + lane;
    static_for<kNumSums>([&](auto i) { v[k][i] = b < nblocks ? to_global(partials)[i * nblocks + b] : 0.0; });
  });
  static_for<kTurns>([&](auto k) {
    if (k * NW + wave < waves)
      static_for<kNumSums>([&](auto i) {
        const double t = wave_sum(v[k][i]);
        if (lane == 0) smem[k * NW + wave][i] = t;
      });
  });
  __syncthreads();
  if (threadIdx.x < kNumSums) {
    double t = smem[0][threadIdx.x];
    for (int w = 1; w < waves; ++w) t += smem[w][threadIdx.x];
    to_global(out)[threadIdx.x] = t;
  }
}

// Flat-index offsets of the +-1 neighbours along one axis with periodic
// wrap: up = offset of coordinate+1, dn = offset of coordinate-1.
struct AxisOff {
  int up, dn;
};
__device__ __forceinline__ AxisOff axis_offsets(int c, int n, int unit) {
  AxisOff o;
  o.up = (c == n - 1) ? -(n - 1) * unit : unit;
  o.dn = (c == 0) ? (n - 1) * unit : -unit;
  return o;
}

}  // namespace dhit
