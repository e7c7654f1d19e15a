// DUGKS time step in one kernel (Sec. II.A), marching in z with one plane
// of cell data in LDS at a time.
//
// Arithmetic.  With B = fbar+ (the cell transform of f~), h = dt/2 and the
// face distribution f_face = alpha fbar_face + beta f^eq_face, the update
//   f~(t+dt) = f~+ - dt sum_d xi_d (f_face(+d) - f_face(-d))
// splits, because fbar_face is linear in B, into
//   f~(t+dt)_q = f~+_q - dt [alpha L_q + beta E_q]
//   L_q = sum_d xi_qd (fbar_face,q(+d) - fbar_face,q(-d))   a fixed stencil of B_q
//   E_q = sum_d xi_qd (f^eq_q(face +d) - f^eq_q(face -d)).
// With the face value (B_L + B_R)/2 - h [xi_d (B_R - B_L) + sum_{t != d}
// xi_t (G_t(L) + G_t(R))/4] and G_t(c) = B(c+e_t) - B(c-e_t):
//   axis population along d, sign s:
//     L = s/2 (B(+d) - B(-d)) - h (B(+d) - 2 B(0) + B(-d))
//   diagonal population in (d1, d2), signs s1, s2:
//     L = s1/2 (B(+d1) - B(-d1)) + s2/2 (B(+d2) - B(-d2))
//         - h (B(+d1) + B(-d1) + B(+d2) + B(-d2) - 4 B(0))
//         - h/2 s1 s2 (B(+d1+d2) - B(+d1-d2) - B(-d1+d2) + B(-d1-d2)).
// The face moments (drho_b = sum fbar_face, j_b = sum xi fbar_face) are the
// same linear reconstruction applied to the cell moment fields of B:
//   R0 = sum B = drho, J = sum xi B = j, P = sum xi xi B
//      = a Pi(f~) + b (drho/3 I + j j / rho0),
// so only 10 moment fields (not 19 populations) are read per face.
//
// Plane-by-plane evaluation.  Every term above is a sum of pieces that each
// involve one z-plane only (a plane's own cell and its in-plane
// neighbours).  When plane p is in LDS, each thread adds the pieces of
// plane p to the three centres that use it:
//   centre p-1 (p is its z+1 plane): the z+1 terms of the z-moving
//     populations and the upper half of the face between p-1 and p;
//   centre p: the in-plane terms of the populations and the lower half of
//     the face between p and p+1;
//   centre p+1 (p is its z-1 plane): the z-1 terms of the z-moving
//     populations.
// The x- and y-faces of centre p-1 are formed in the same iteration from
// the moment fields of planes p-2, p-1 and p, after which centre p-1 is
// complete and stored.  The moments of an x-face are joined from a half of each
// of its two cells (face_halves), which are neighbouring lanes; in 32-wide tiles
// the wavefront that holds the two halo rows, and has no centres of its own, does
// that for the others' columns (and in the FP32 march forms their z-faces'
// moments too) and leaves the moments in LDS.  A y-face's ten terms are formed by
// its lower cell and applied by the upper one after the barrier that ends the
// iteration (FP32), or its moments are joined from the two cells' halves in LDS
// by every thread that needs them (FP64).  Between planes a thread carries the running
// results of centres p and p+1 in registers.  LDS holds the populations of
// plane p only, the in-plane moment fields (R0, Jx, Jy, Pxx, Pxy, Pyy) of
// planes p-1 and p, and the fields the x/y-faces differentiate in z (Jz,
// Pxz, Pyz, Pzz) of planes p-2, p-1 and p: 16 + 12 + 12 values per column.
//
// Two marches implement this.  fused_tile (FP32): one thread per column,
// 58 values of LDS per column (59 KB for a 32 x 8 tile, two blocks per
// compute unit).  split_tile (FP64): two threads per column, one in each of
// two groups that hold about half of the populations each (see below), so
// that a thread's registers fit two waves per SIMD; 68 values per column.
// LDS reads are gathered (see gathered()) so that each chunk of work waits
// for LDS once.
//
// Tiling.  A block owns W x 8 (x, y) columns, of which the inner (W-2) x 6
// are updated and the outer ring is the halo, and marches over a chunk of
// z.  HBM traffic per updated cell: 19 loads + 19 stores, plus the halo
// ring (loads only).  Blocks are numbered so that the tiles one XCD (one L2)
// works on at a time are neighbours, whose halo columns then come from that
// L2.

// Rounding.  From here to the split march, multiply-adds are contracted within
// one expression only (in the included device functions too): left to the
// optimiser, which of two products of a sum goes into the multiply-add depends
// on the code around it, and the FP32 march is inlined several times in a
// kernel (two planes per turn, the halo wavefront's part) and in two tile widths
// that share the work differently.  So every copy rounds alike by construction,
// whatever the z-chunk and the tile width (before, FP32 boxes on unit cells
// differed in the last bits between the widths).  Alone this cost the FP32 march
// 1-2% (128^3 3.60 -> 3.64 ms for 30 steps); with pair_equilibrium() the two
// together: 128^3 3.58 ms, 97^3 on a mesh 1.30 -> 1.27 ms for 20 steps, 256^3 0.822
// -> 0.832 ms a step.
#pragma clang fp contract(on)
#include <array>
#include <cstring>
#include <map>
#include <mutex>

#include "collision.hpp"

namespace dhit {
namespace fused {

// Column tile of a block: W x 8 columns, the inner (W-2) x 6 updated.
template <int W>
struct Tile {
  static constexpr int TX = W, TY = 8, NT = TX * TY, IX = TX - 2, IY = TY - 2;
};

// Field ids: 0..18 populations of B; moment fields after them.
enum : int { kR0 = 19, kJx, kJy, kJz, kPxx, kPxy, kPxz, kPyy, kPyz, kPzz };

// LDS buffers: populations (one plane) other than 0, 5, 6 (the rest
// population has no stencil, q5 and q6 only use their own column); the
// in-plane moment fields (two planes); the fields differentiated in z
// across x/y-faces (three planes).
constexpr int kNPop = 16, kNQ = 6, kNZ = 4;
constexpr int kLdsValues = kNPop + 2 * kNQ + 3 * kNZ;  // per column
// The one-thread march adds the ten face-equilibrium terms of the y-face
// between each column and the next row (read back by the column above as
// its lower y-face), and the moments of the column's x+ face and of the
// z-face below the plane (formed by the halo rows' wavefront).
constexpr int kFusedValues = kLdsValues + 18;
constexpr int pop_index(int id) { return (id >= 1 && id <= 4) ? id - 1 : ((id >= 7 && id <= 18) ? id - 3 : -1); }
constexpr int q_index(int id) {
  switch (id) {
    case kR0: return 0;
    case kJx: return 1;
    case kJy: return 2;
    case kPxx: return 3;
    case kPxy: return 4;
    case kPyy: return 5;
  }
  return -1;
}
constexpr int z_index(int id) {
  switch (id) {
    case kJz: return 0;
    case kPxz: return 1;
    case kPyz: return 2;
    case kPzz: return 3;
  }
  return -1;
}
constexpr int jid(int a) { return kJx + a; }
constexpr int pid(int a, int b) {
  const int lo = a < b ? a : b, hi = a < b ? b : a;
  return lo == 0 ? (hi == 0 ? kPxx : (hi == 1 ? kPxy : kPxz)) : (lo == 1 ? (hi == 1 ? kPyy : kPyz) : kPzz);
}
// Position of a z-moving population among the ten (q5, q6, q11..q18).
constexpr int zslot(int q) { return q == 5 ? 0 : (q == 6 ? 1 : q - 9); }
constexpr bool is_diag_z(int q) { return q >= 11; }

// Column of the tile (row-major, ty * W + tx) that thread t of a march
// handles.  In the 32-wide tile a wavefront covers two rows; the two rows
// made only of halo columns (0 and 7) are put together in the last
// wavefront, so that the work of the updated cells (stencils, faces,
// stores), which halo rows skip, runs on three wavefronts instead of four:
// wavefronts 0..2 take rows (1, 2), (3, 4), (5, 6) and wavefront 3 rows 0
// and 7.  A row stays 32 consecutive lanes, as the x-face lane shift needs.
// Other widths keep row-major order.
template <int W>
__device__ __forceinline__ int tile_column(int t) {
  if constexpr (W == 32) {
    const int w = t >> 6, half = (t >> 5) & 1, tx = t & 31;
    const int ty = w < 3 ? 2 * w + 1 + half : (half ? 7 : 0);
    return ty * 32 + tx;
  } else {
    return t;
  }
}

// Compiler-only memory fence between the phases of a plane's work: LDS
// values are re-read after it instead of being kept live in registers
// across phases, which bounds register pressure.  No instruction is emitted.
__device__ __forceinline__ void phase() { asm volatile("" ::: "memory"); }

template <int T>
struct Unit {
  static constexpr int x = T == 0, y = T == 1, z = T == 2;
};

// Value of the previous / next lane of the wavefront (lane 0 / 63 gets 0): a
// DPP whole-wavefront shift by one lane, one move per 32 bits.
template <int Ctrl>
__device__ __forceinline__ int lane_shift(int v) { return __builtin_amdgcn_update_dpp(0, v, Ctrl, 0xf, 0xf, true); }
template <int Ctrl>
__device__ __forceinline__ float lane_shift(float v) {
  return __builtin_bit_cast(float, lane_shift<Ctrl>(__builtin_bit_cast(int, v)));
}
template <int Ctrl>
__device__ __forceinline__ double lane_shift(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = lane_shift<Ctrl>((int)b), hi = lane_shift<Ctrl>((int)(b >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}
template <typename T>
__device__ __forceinline__ T from_previous_lane(T v) { return lane_shift<0x138>(v); }
template <typename T>
__device__ __forceinline__ T from_next_lane(T v) { return lane_shift<0x130>(v); }
// Whether the corner neighbours (x+-1, y+-1) of an in-plane diagonal population
// come as lane shifts of the (x, y+-1) values (a tile row is consecutive
// lanes) instead of LDS reads.  FP64: a plane's LDS traffic and its vector work
// take about as long as each other and add up, and a shift costs two of a
// SIMD's moves against a 512-byte read of the LDS all four SIMDs share; with
// the trimmed exchanges of the split march 256^3 1.72 -> 1.70 ms, 128^3
// 224 us either way, 64^3 43.6 -> 41.9 us.  FP32 is bound by vector issue:
// 1-3% slower with the shifts.
template <typename Real>
constexpr bool kLaneCorners = sizeof(Real) == 8;

// Reads of one plane: populations from P, in-plane moment fields from Q,
// z-differentiated fields from Z (each offset to the thread's column; a
// plane whose populations or Q fields are no longer held has null there).
template <typename Real, int W>
struct Plane {
  const Real *P;
  const Real *Q;
  const Real *Z;
  template <int ID, int DX, int DY>
  __device__ __forceinline__ Real at() const {
    constexpr int NT = Tile<W>::NT, off = DY * W + DX;
    constexpr int ip = pop_index(ID), iq = q_index(ID), iz = z_index(ID);
    static_assert(ip >= 0 || iq >= 0 || iz >= 0, "field not in LDS");
    if constexpr (ip >= 0)
      return P[ip * NT + off];
    else if constexpr (iq >= 0)
      return Q[iq * NT + off];
    else
      return Z[iz * NT + off];
  }
};

// In-plane central difference of field ID along in-plane axis t (0 or 1)
// at the column offset (DX, DY).
template <int ID, int T, int DX, int DY, class P>
__device__ __forceinline__ auto dif(const P &c) {
  return c.template at<ID, DX + Unit<T>::x, DY + Unit<T>::y>() - c.template at<ID, DX - Unit<T>::x, DY - Unit<T>::y>();
}

// Reads gathered ahead of their use.  A computation written against a
// plane is run twice: once on a Load view, which issues every LDS read the
// computation makes (its arithmetic is discarded), then on a Use view, which
// replays it on the gathered values.  All reads of a chunk of work are thus
// in flight together and their latencies overlap, instead of one read being
// waited for before the next is issued.
constexpr int kNumIds = 29;
template <typename Real>
struct Gathered {
  Real v[kNumIds][3][3];  // field id, dy + 1, dx + 1
};
template <typename Real, int W, bool kLoad>
struct GView {
  static constexpr bool use = !kLoad;
  const Plane<Real, W> &src;
  Gathered<Real> &g;
  template <int ID, int DX, int DY>
  __device__ __forceinline__ Real at() const {
    if constexpr (kLoad) {
      g.v[ID][DY + 1][DX + 1] = src.template at<ID, DX, DY>();
      return Real(0);
    } else {
      return g.v[ID][DY + 1][DX + 1];
    }
  }
};
// f(view0, view1) with views of planes c0 and c1; f must change state only
// when view0.use is true.
template <typename Real, int W, class F>
__device__ __forceinline__ void gathered(const Plane<Real, W> &c0, const Plane<Real, W> &c1, F &&f) {
  Gathered<Real> g0, g1;
  f(GView<Real, W, true>{c0, g0}, GView<Real, W, true>{c1, g1});
  __builtin_amdgcn_sched_barrier(0);
  f(GView<Real, W, false>{c0, g0}, GView<Real, W, false>{c1, g1});
  phase();
}

// In-plane part of the moments of the y-face between the column (L) and the one
// above it (R) in the current plane: everything but the z-tangential gradients.
// Face moment of field pair (value field V, normal-flux field N, in-plane
// tangential field T):
//   V_L + (V_R - V_L)/2 - h [(N_R - N_L) + (T(L+e_x) - T(L-e_x) + T(R+e_x) - T(R-e_x))/4]
template <typename Real, class P>
__device__ __forceinline__ void yface_inplane(const P &c, Real h, Real (&m)[4]) {
  {
    const Real tang = dif<kJx, 0, 0, 0>(c) + dif<kJx, 0, 0, 1>(c);
    const Real vl = c.template at<kR0, 0, 0>(), vr = c.template at<kR0, 0, 1>();
    const Real nl = c.template at<kJy, 0, 0>(), nr = c.template at<kJy, 0, 1>();
    m[0] = (vl + Real(0.5) * (vr - vl)) - h * ((nr - nl) + Real(0.25) * tang);
  }
  static_for<3>([&](auto a) {
    constexpr int PN = pid(a, 1), PT = pid(a, 0);
    const Real tang = dif<PT, 0, 0, 0>(c) + dif<PT, 0, 0, 1>(c);
    const Real vl = c.template at<jid(a), 0, 0>(), vr = c.template at<jid(a), 0, 1>();
    const Real nl = c.template at<PN, 0, 0>(), nr = c.template at<PN, 0, 1>();
    m[1 + a] = (vl + Real(0.5) * (vr - vl)) - h * ((nr - nl) + Real(0.25) * tang);
  });
}

// z-tangential part of that face: the fields (Jz, Pxz, Pyz, Pzz) summed over L
// and R.
template <typename Real, class P>
__device__ __forceinline__ void yface_zsum(const P &c, Real (&s)[4]) {
  s[0] = c.template at<kJz, 0, 0>() + c.template at<kJz, 0, 1>();
  s[1] = c.template at<kPxz, 0, 0>() + c.template at<kPxz, 0, 1>();
  s[2] = c.template at<kPyz, 0, 0>() + c.template at<kPyz, 0, 1>();
  s[3] = c.template at<kPzz, 0, 0>() + c.template at<kPzz, 0, 1>();
}

// Half of the moments of a z-face that comes from one plane (the cell of
// the column and its in-plane neighbours).  For the plane below the face
// (S = +1) and the plane above it (S = -1):
//   R0/2 + S h Jz - h/4 (dJx/dx + dJy/dy) and, for component a,
//   J_a/2 + S h P_az - h/4 (dP_ax/dx + dP_ay/dy)   (central differences).
template <int S, typename Real, class P>
__device__ __forceinline__ void zface_half(const P &c, Real h, Real (&m)[4]) {
  {
    const Real tang = dif<kJx, 0, 0, 0>(c) + dif<kJy, 1, 0, 0>(c);
    m[0] = Real(0.5) * c.template at<kR0, 0, 0>() + Real(S) * h * c.template at<kJz, 0, 0>() - Real(0.25) * h * tang;
  }
  static_for<3>([&](auto a) {
    const Real tang = dif<pid(a, 0), 0, 0, 0>(c) + dif<pid(a, 1), 1, 0, 0>(c);
    m[1 + a] = Real(0.5) * c.template at<jid(a), 0, 0>() + Real(S) * h * c.template at<pid(a, 2), 0, 0>() -
               Real(0.25) * h * tang;
  });
}

// ---------------------------------------------------------------------------
// Stretched mesh (set_mesh).  With cell widths w that vary along each axis
// the reconstruction reads, at the face between L = i and R = i+1 of an axis
// (lam = w_L/(w_L + w_R), g = 1/(c_R - c_L), s_t = 1/(c_{k+1} - c_{k-1}) of
// the tangential axis t),
//   fbar = B_L + lam (B_R - B_L) - h [xi_d g (B_R - B_L)
//          + sum_t xi_t s_t (G_t(L) + lam (G_t(R) - G_t(L)))],
// and each axis's flux difference is divided by the cell's width, so that
// with A = lam_i/w_i, E = (1 - lam_{i-1})/w_i, b = h g_i/w_i,
// f = h g_{i-1}/w_i of the centre i along an axis
//   axis part, sign s:  U (B(+) - B(0)) + V (B(0) - B(-)),  U = s A - b, V = s E + f
//   mixed part of a diagonal population in (d1, d2):
//     - h s1 s2 { s_2 [A_1 (G_2(+) - G_2(0)) + E_1 (G_2(0) - G_2(-))]
//               + s_1 [A_2 (G_1(+) - G_1(0)) + E_2 (G_1(0) - G_1(-))] }
// (unit widths give the stencils above).  The pieces of a plane go to the
// same three centres as on unit cells, with the coefficients of the centre
// they go to: those of x and y are per column (a table in LDS, read in each
// phase: held in registers, or hoisted there, they would not fit), those of z
// are uniform over the block (scalar loads).
//
// The tables hold one row of n values per coefficient and axis (MarchCoef,
// runtime.hpp), already multiplied by dt alpha (U, V, A, E) and by h.
//
// Like the march on unit cells it is bound by the latency its two waves per
// SIMD cannot cover (FP64) and by vector issue (FP32): 15-20% more
// instructions than there.  It took
// the place of a transform pass and a face pass that rebuilt six faces of 19
// populations per cell from some 700 cached loads: 128^3 FP64 1.04 -> 0.237 ms
// a step, 97^3 FP32 0.132 -> 0.069 ms (unit cells: 0.215 ms at 128^3).
template <typename T>
using constant_t = __attribute__((address_space(4))) T;
template <typename Real, int W>
struct MeshMarch {
  const constant_t<Real> *zc;  // the z axis's rows
  const Real *X, *Y;           // LDS: the column's x and y coefficients
  int n;
  __device__ __forceinline__ Real z(int k, int plane) const {
    const int i = plane < 0 ? plane + n : (plane >= n ? plane - n : plane);
    return zc[k * n + i];
  }
  template <int D>
  __device__ __forceinline__ Real col(int k) const {
    return D == 0 ? X[k * W] : Y[k * 8];
  }
};
// Values of the x/y coefficient table in LDS of a tile.
template <int W>
constexpr int kMeshValues = kMarchCoefs * (W + 8);

// Fills the block's x/y coefficient table for tile (x0, y0).
template <typename Real, int W>
__device__ __forceinline__ void load_mesh_columns(const Real *coef, int n, int x0, int y0, Real *L) {
  for (int i = threadIdx.x; i < kMeshValues<W>; i += blockDim.x) {
    const bool isx = i < kMarchCoefs * W;
    const int j = isx ? i : i - kMarchCoefs * W;
    const int k = isx ? j / W : j / 8, c = (isx ? x0 + j % W : y0 + j % 8) - 1;
    const int cell = c < 0 ? c + n : c % n;
    L[i] = to_global(coef)[((isx ? 0 : kMarchCoefs) + k) * n + cell];
  }
}

// In-plane part of a y-face's moments on the mesh (see yface_inplane): the
// value v of cell L and the rest m, which is small beside it (added to v once,
// so that in FP32 a moment is rounded at the scale of v once).
template <typename Real, class P>
__device__ __forceinline__ void yface_inplane_mesh(const P &c, Real lam, Real hg, Real hs, Real (&v)[4], Real (&m)[4]) {
  auto moment = [&](auto i, auto V, auto N, auto T) {
    const Real vl = c.template at<V, 0, 0>(), vr = c.template at<V, 0, 1>();
    const Real tl = dif<T, 0, 0, 0>(c), tr = dif<T, 0, 0, 1>(c);
    v[i] = vl;
    m[i] = lam * ((vr - vl) - hs * (tr - tl)) - (hs * tl + hg * (c.template at<N, 0, 1>() - c.template at<N, 0, 0>()));
  };
  using std::integral_constant;
  moment(integral_constant<int, 0>{}, integral_constant<int, kR0>{}, integral_constant<int, kJy>{},
         integral_constant<int, kJx>{});
  static_for<3>([&](auto a) {
    moment(integral_constant<int, 1 + a>{}, integral_constant<int, jid(a)>{}, integral_constant<int, pid(a, 1)>{},
           integral_constant<int, pid(a, 0)>{});
  });
}

// The z-differentiated fields at that face (see yface_zsum).
template <typename Real, class P>
__device__ __forceinline__ void yface_zvalue_mesh(const P &c, Real lam, Real (&s)[4]) {
  constexpr int ids[4] = {kJz, kPxz, kPyz, kPzz};
  static_for<4>([&](auto i) {
    const Real l = c.template at<ids[i], 0, 0>(), r = c.template at<ids[i], 0, 1>();
    s[i] = l + lam * (r - l);
  });
}

// What a plane gives to its z-faces' moments on the mesh: the value with the
// tangential gradients taken off (w) and the normal-flux field (nf); between
// planes L and R the moments are w_L + lam (w_R - w_L) - hg (nf_R - nf_L).
template <typename Real, class P>
__device__ __forceinline__ void zface_parts_mesh(const P &c, Real hsx, Real hsy, Real (&w)[4], Real (&nf)[4]) {
  w[0] = c.template at<kR0, 0, 0>() - (hsx * dif<kJx, 0, 0, 0>(c) + hsy * dif<kJy, 1, 0, 0>(c));
  nf[0] = c.template at<kJz, 0, 0>();
  static_for<3>([&](auto a) {
    w[1 + a] = c.template at<jid(a), 0, 0>() - (hsx * dif<pid(a, 0), 0, 0, 0>(c) + hsy * dif<pid(a, 1), 1, 0, 0>(c));
    nf[1 + a] = c.template at<pid(a, 2), 0, 0>();
  });
}

// Index of the population with velocity (x, y, z).
constexpr int pop_of(int x, int y, int z) {
  for (int q = 0; q < kQ; ++q)
    if (kCx[q] == x && kCy[q] == y && kCz[q] == z) return q;
  return -1;
}

// Face-equilibrium terms of a D-face: calls put(q, k, t) for the ten
// populations crossing it, k t = dt beta xi_qD f^eq_q(face) (two factors: a
// caller that adds the product has one multiply-add).  With u = j_b/rho0 and
// f^eq_q = W_q [rho_b - 3/2 rho0 |u|^2 + 3 rho0 (xi.u) + 9/2 rho0 (xi.u)^2],
// opposite velocities share the even part and flip the odd part, so each pair
// is formed from one even and one odd term.
template <int D, typename Real, class Put>
__device__ __forceinline__ void face_equilibrium(const Real (&m)[4], const StepParams &p, Real dtbe, Put &&put) {
  const Real rho0 = Real(p.rho0), ir = Real(p.inv_rho0);
  const Real u[3] = {m[1] * ir, m[2] * ir, m[3] * ir};
  const Real base = m[0] - Real(1.5) * rho0 * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
  const Real c3 = Real(3) * rho0, c45 = Real(4.5) * rho0;
  const Real k1 = dtbe * Real(1.0 / 18.0), k2 = dtbe * Real(1.0 / 36.0);
  const Real ud = u[D];
  {
    const Real ev = base + c45 * ud * ud;
    put(std::integral_constant<int, pop_of(Unit<D>::x, Unit<D>::y, Unit<D>::z)>{}, k1, ev + c3 * ud);
    put(std::integral_constant<int, pop_of(-Unit<D>::x, -Unit<D>::y, -Unit<D>::z)>{}, k1, c3 * ud - ev);
  }
  static_for<3>([&](auto t) {
    if constexpr (t != D) {
      const Real ut = u[t];
      const Real up = ud + ut, um = ud - ut;
      const Real ep = base + c45 * up * up;
      const Real em = base + c45 * um * um;
      constexpr int x = Unit<D>::x, y = Unit<D>::y, z = Unit<D>::z;
      constexpr int tx = Unit<t>::x, ty = Unit<t>::y, tz = Unit<t>::z;
      put(std::integral_constant<int, pop_of(x + tx, y + ty, z + tz)>{}, k2, ep + c3 * up);      // xi.u = ud + ut
      put(std::integral_constant<int, pop_of(x - tx, y - ty, z - tz)>{}, k2, em + c3 * um);      // xi.u = ud - ut
      put(std::integral_constant<int, pop_of(-x + tx, -y + ty, -z + tz)>{}, k2, c3 * um - em);  // -(ud - ut)
      put(std::integral_constant<int, pop_of(-x - tx, -y - ty, -z - tz)>{}, k2, c3 * up - ep);  // -(ud + ut)
    }
  });
}

// Slot of population q among the ten that cross a D-face (increasing q).
template <int D>
constexpr int cross_slot(int q) {
  int k = 0;
  for (int r = 0; r < q; ++r) k += cdir(r, D) != 0;
  return k;
}

// The ten face-equilibrium terms of a D-face, v[cross_slot<D>(q)] =
// dt beta xi_qD f^eq_q(face) (face_equilibrium), formed once for both of the
// face's cells.
template <int D, typename Real>
__device__ __forceinline__ void face_terms(const Real (&m)[4], const StepParams &p, Real dtbe, Real (&v)[10]) {
  face_equilibrium<D, Real>(m, p, dtbe, [&](auto q, Real k, Real t) { v[cross_slot<D>(q)] = k * t; });
}

// acc_q -= S v_q for the face terms of a D-face (S = +1: the centre's upper
// face, -1: its lower face).
template <int D, int S, typename Real>
__device__ __forceinline__ void apply_terms(const Real (&v)[10], Real (&acc)[kQ]) {
  static_for<kQ>([&](auto q) {
    if constexpr (cdir(q, D) != 0) {
      if constexpr (S > 0)
        acc[q] -= v[cross_slot<D>(q)];
      else
        acc[q] += v[cross_slot<D>(q)];
    }
  });
}
// The same on the mesh: divided by the cell's width along the axis.
template <int D, int S, typename Real>
__device__ __forceinline__ void apply_terms(const Real (&v)[10], Real iw, Real (&acc)[kQ]) {
  static_for<kQ>([&](auto q) {
    if constexpr (cdir(q, D) != 0) acc[q] -= (S > 0 ? iw : -iw) * v[cross_slot<D>(q)];
  });
}

// Cell idx of the population array that starts at qbase.  With O32 the
// byte offset is formed in 32 bits (every population array of the box is
// below 4 GB), so that the access can go through the array's uniform base
// in scalar registers with a 32-bit lane offset, with no 64-bit address
// arithmetic per access.
template <bool O32, typename T>
__device__ __forceinline__ T *at_cell(T *qbase, int idx) {
  if constexpr (O32) {
    using Byte = std::conditional_t<std::is_const<T>::value, const global_t<char>, global_t<char>>;
    return reinterpret_cast<T *>(reinterpret_cast<Byte *>(qbase) + (uint32_t)idx * (uint32_t)sizeof(T));
  } else {
    return qbase + idx;
  }
}

// Issues the loads of the 19 f~ of the column's cell in plane `plane`
// (periodic in z).
template <typename Real, bool O32>
__device__ __forceinline__ void load_raw(const global_t<Real> *__restrict__ ft, int64_t stride, int n, int col, int plane,
                                         Real (&f)[kQ]) {
  const int z = plane < 0 ? plane + n : (plane >= n ? plane - n : plane);
  const int idx = z * n * n + col;
  static_for<kQ>([&](auto q) { f[q] = *at_cell<O32>(ft + (int64_t)q * stride, idx); });
}

// The ten moments drho, j, Pi of a cell (or of the populations get(q)
// yields for q in a set closed under q -> -q), formed from opposite-velocity
// pairs: with s = f_q + f_-q and d = f_q - f_-q over the pairs (q < -q),
//   drho = f_0 + sum s,  j = sum xi_q d,  Pi_ab = sum xi_qa xi_qb s.
// drho and j are summed in double also for FP32 populations and rounded
// once: double additions issue at the rate of FP32 ones, so that this takes
// 39 vector instructions fewer per cell than FP32 sums with compensation, the
// same time, and is more accurate (errors against double after 30 steps at
// 128^3 2.9e-7 instead of 3.2e-7; on a 97^3 mesh after 20 steps 2.7e-7
// instead of 3.0e-7).
// m = {drho, jx, jy, jz, Pxx, Pyy, Pzz, Pxy, Pxz, Pyz}.
template <typename Real, class Has, class Get>
__device__ __forceinline__ void pair_moments(Has has, Get get, Real (&m)[10]) {
  double r = 0, ax = 0, ay = 0, az = 0;
  Real pxx = 0, pyy = 0, pzz = 0, pxy = 0, pxz = 0, pyz = 0;
  if constexpr (has(0)) r += (double)get(std::integral_constant<int, 0>{});
  static_for<kQ>([&](auto q) {
    constexpr int qb = opposite(q);
    if constexpr (q != 0 && q < qb && has(q)) {
      const Real fq = get(q), fb = get(std::integral_constant<int, qb>{});
      const double sd = (double)fq + (double)fb, df = (double)fq - (double)fb;
      const Real sm = std::is_same<Real, double>::value ? Real(sd) : fq + fb;
      constexpr int x = kCx[q], y = kCy[q], z = kCz[q];
      r += sd;
      if constexpr (x != 0) ax += x > 0 ? df : -df;
      if constexpr (y != 0) ay += y > 0 ? df : -df;
      if constexpr (z != 0) az += z > 0 ? df : -df;
      if constexpr (x != 0) pxx += sm;
      if constexpr (y != 0) pyy += sm;
      if constexpr (z != 0) pzz += sm;
      if constexpr (x * y == 1) pxy += sm;
      if constexpr (x * y == -1) pxy -= sm;
      if constexpr (x * z == 1) pxz += sm;
      if constexpr (x * z == -1) pxz -= sm;
      if constexpr (y * z == 1) pyz += sm;
      if constexpr (y * z == -1) pyz -= sm;
    }
  });
  m[0] = Real(r); m[1] = Real(ax); m[2] = Real(ay); m[3] = Real(az);
  m[4] = pxx; m[5] = pyy; m[6] = pzz; m[7] = pxy; m[8] = pxz; m[9] = pyz;
}

// f^eq of the populations with has(q) (a set closed under q -> -q), as in
// equilibrium_q(): calls put(q, f^eq_q).  Opposite velocities are formed
// together: they share the even part and flip the odd one, 5% fewer vector
// instructions per plane of the one-thread march, which makes good what
// contraction within expressions costs (top of this file): 128^3 FP32 121.2 ->
// 119.2 us a step, 97^3 on a mesh 64.9 -> 63.5; FP64 32^3 14.4 -> 14.2 us, 256^3
// 1.541 -> 1.532 ms.
template <typename Real, class Has, class Put>
__device__ __forceinline__ void pair_equilibrium(Has has, Real drho, const Real (&u)[3], Real rho0, Put &&put) {
  const Real base = drho - Real(1.5) * rho0 * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
  const Real c45 = Real(4.5) * rho0;
  if constexpr (has(0)) put(std::integral_constant<int, 0>{}, Real(kWeight(0)) * base);
  static_for<kQ>([&](auto q) {
    constexpr int qb = opposite(q);
    if constexpr (q != 0 && q < qb && has(q)) {
      constexpr Real w = Real(kWeight(q)), l = speed2(q) == 1 ? kLinAxis<Real> : kLinDiag<Real>;
      constexpr int d1 = kCx[q] != 0 ? 0 : (kCy[q] != 0 ? 1 : 2), d2 = kCz[q] != 0 ? 2 : 1;
      static_assert(speed2(q) == 1 ? cdir(q, d1) == 1 : cdir(q, d2) == 1);
      Real xu = u[d1];
      if constexpr (speed2(q) == 2) xu = cdir(q, d1) > 0 ? u[d2] + u[d1] : u[d2] - u[d1];
      const Real even = w * (base + c45 * xu * xu);
      put(q, even + l * rho0 * xu);
      put(std::integral_constant<int, qb>{}, even - l * rho0 * xu);
    }
  });
}

// From the 19 f~ of a cell: moments, B = a f~ + b f^eq and f~+ =
// 4/3 B - 1/3 f~, and the moment fields of B; writes the fields other
// columns read to the plane's LDS buffers P, Q, Z (offset to the thread's
// column) and hands each population's (B, f~+) to
// use(q, B_q, f~+_q) as soon as it is formed.
template <typename Real, int W, class Use>
__device__ __forceinline__ void publish_cell(const Real (&f)[kQ], Real *P, Real *Q, Real *Z, const StepParams &p,
                                             Use &&use) {
  constexpr int NT = Tile<W>::NT;
  Real mom[10];
  pair_moments<Real>([](int) constexpr { return true; }, [&](auto q) { return f[q]; }, mom);
  const Real drho = mom[0], jx = mom[1], jy = mom[2], jz = mom[3];
  const Real pxx = mom[4], pyy = mom[5], pzz = mom[6], pxy = mom[7], pxz = mom[8], pyz = mom[9];
  const Real rho0 = Real(p.rho0), ir = Real(p.inv_rho0);
  const Real a = Real(p.a_bp);
  const Real d3 = drho * Real(1.0 / 3.0);
  // P = a Pi(f~) + b Pi(f^eq), Pi(f^eq) = drho/3 I + j j / rho0, formed as
  // Pi(f^eq) + a (Pi(f~) - Pi(f^eq)) (see below)
  {
    const Real exx = d3 + jx * jx * ir, eyy = d3 + jy * jy * ir, ezz = d3 + jz * jz * ir;
    const Real exy = jx * jy * ir, exz = jx * jz * ir, eyz = jy * jz * ir;
    Q[q_index(kR0) * NT] = drho;
    Q[q_index(kJx) * NT] = jx;
    Q[q_index(kJy) * NT] = jy;
    Q[q_index(kPxx) * NT] = exx + a * (pxx - exx);
    Q[q_index(kPxy) * NT] = exy + a * (pxy - exy);
    Q[q_index(kPyy) * NT] = eyy + a * (pyy - eyy);
    Z[z_index(kJz) * NT] = jz;
    Z[z_index(kPxz) * NT] = exz + a * (pxz - exz);
    Z[z_index(kPyz) * NT] = eyz + a * (pyz - eyz);
    Z[z_index(kPzz) * NT] = ezz + a * (pzz - ezz);
  }
  // B = a f~ + b f^eq with a + b = 1 is formed as f^eq + a (f~ - f^eq) and
  // f~+ = 4/3 B - 1/3 f~ as B + (B - f~)/3, so that an equilibrium cell maps
  // to itself exactly in any precision (rounded 4/3 and 1/3, or a and b,
  // would otherwise scale the state by 1 + O(ulp) every step).  f^eq is the
  // equilibrium of Sec. II.A.
  const Real u[3] = {jx * ir, jy * ir, jz * ir};
  pair_equilibrium<Real>([](int) constexpr { return true; }, drho, u, rho0, [&](auto q, Real feq) {
    const Real b = feq + a * (f[q] - feq);
    if constexpr (pop_index(q) >= 0) P[pop_index(q) * NT] = b;
    use(q, b, b + (b - f[q]) * Real(1.0 / 3.0));
  });
}

// The mesh coefficients each phase of the marches reads, with the terms they
// make (on unit cells stubs that no code calls).  Plane p is the one being worked on: p_.
template <typename Real, int W, bool Mesh>
struct OwnCoef {
  __device__ __forceinline__ OwnCoef(const MeshMarch<Real, W> &, int) {}
  template <int S> __device__ __forceinline__ void add(Real, Real &, Real &, Real &) const {}
};
// The column's own B of plane p along z: to centre p-1 (its z+1 value), to
// centre p (its own value, -U + V) and to centre p+1 (its z-1 value).  U and
// V enter centre p with the same rounded values as they do its neighbours.
template <typename Real, int W>
struct OwnCoef<Real, W, true> {
  Real u[2], v[2], ua[2], vb[2];  // by sign (+, -): of centre p, U of centre p-1, V of centre p+1
  __device__ __forceinline__ OwnCoef(const MeshMarch<Real, W> &m, int p) {
    static_for<2>([&](auto s) {
      u[s] = m.z(kMarchUp + s, p);
      v[s] = m.z(kMarchVp + s, p);
      ua[s] = m.z(kMarchUp + s, p - 1);
      vb[s] = m.z(kMarchVp + s, p + 1);
    });
  }
  template <int S>
  __device__ __forceinline__ void add(Real b, Real &acc_c, Real &r, Real &nxt) const {
    constexpr int i = S > 0 ? 0 : 1;
    acc_c -= ua[i] * b;
    r += nxt - v[i] * b;
    r += u[i] * b;
    nxt = vb[i] * b;
  }
};

// The z-face between planes p-1 and p.
template <typename Real, int W, bool Mesh>
struct ZFaceCoef {
  static constexpr Real iw_c = 1, iw_p = 1;
  __device__ __forceinline__ ZFaceCoef(const MeshMarch<Real, W> &, int) {}
  template <class G> __device__ __forceinline__ void face(const G &, Real (&)[4], Real (&)[4], Real (&)[4]) const {}
};
template <typename Real, int W>
struct ZFaceCoef<Real, W, true> {
  Real hsx, hsy, lam, hg, iw_c, iw_p;
  __device__ __forceinline__ ZFaceCoef(const MeshMarch<Real, W> &m, int p)
      : hsx(m.template col<0>(kMarchHs)), hsy(m.template col<1>(kMarchHs)), lam(m.z(kMarchLam, p - 1)),
        hg(m.z(kMarchHg, p - 1)), iw_c(m.z(kMarchIw, p - 1)), iw_p(m.z(kMarchIw, p)) {}
  // moments of the face between the plane below (wl, nl) and this one, whose
  // parts then replace the plane below's
  template <class G>
  __device__ __forceinline__ void face(const G &g, Real (&wl)[4], Real (&nl)[4], Real (&m)[4]) const {
    Real w[4], nf[4];
    zface_parts_mesh(g, hsx, hsy, w, nf);
    if constexpr (G::use)
      static_for<4>([&](auto i) {
        m[i] = wl[i] + (lam * (w[i] - wl[i]) - hg * (nf[i] - nl[i]));
        wl[i] = w[i];
        nl[i] = nf[i];
      });
  }
};

// The diagonal z-moving populations' in-plane neighbours in plane p: with
// D = B(+) - B(-) and X = A (B(+) - B(0)) + E (B(0) - B(-)) along the
// in-plane axis, the mixed terms of centres p-1, p and p+1 and the in-plane
// axis part of centre p.
template <typename Real, int W, bool Mesh>
struct DiagZCoef {
  __device__ __forceinline__ DiagZCoef(const MeshMarch<Real, W> &, int) {}
  template <int Q, class G> __device__ __forceinline__ void add(const G &, Real &, Real &, Real &) const {}
};
template <typename Real, int W>
struct DiagZCoef<Real, W, true> {
  Real a[2], e[2], hs[2], u[2][2], v[2][2];  // per in-plane axis
  Real hsz_c, az_c, eaz_p, hsz_n, ez_n;      // of centres p-1, p, p+1
  __device__ __forceinline__ DiagZCoef(const MeshMarch<Real, W> &m, int p) {
    static_for<2>([&](auto d) {
      a[d] = m.template col<d>(kMarchA);
      e[d] = m.template col<d>(kMarchE);
      hs[d] = m.template col<d>(kMarchHs);
      static_for<2>([&](auto s) {
        u[d][s] = m.template col<d>(kMarchUp + s);
        v[d][s] = m.template col<d>(kMarchVp + s);
      });
    });
    hsz_c = m.z(kMarchHs, p - 1);
    az_c = m.z(kMarchA, p - 1);
    eaz_p = m.z(kMarchE, p) - m.z(kMarchA, p);
    hsz_n = m.z(kMarchHs, p + 1);
    ez_n = m.z(kMarchE, p + 1);
  }
  template <int Q, class G>
  __device__ __forceinline__ void add(const G &g, Real &acc_c, Real &acc_p, Real &nxt) const {
    constexpr int d = kCx[Q] != 0 ? 0 : 1, s = kCx[Q] + kCy[Q], i = s > 0 ? 0 : 1;
    const Real bp = g.template at<Q, Unit<d>::x, Unit<d>::y>();
    const Real b0 = g.template at<Q, 0, 0>();
    const Real bm = g.template at<Q, -Unit<d>::x, -Unit<d>::y>();
    if constexpr (G::use) {
      const Real dp = bp - b0, dm = b0 - bm;
      const Real x = a[d] * dp + e[d] * dm;
      const Real y = hs[d] * (bp - bm);
      const Real up = hsz_c * x + az_c * y, dn = hsz_n * x + ez_n * y;
      const Real in = u[d][i] * dp + v[d][i] * dm;
      if constexpr (s * kCz[Q] > 0) {
        acc_c += up;
        acc_p += eaz_p * y - in;
        nxt -= dn;
      } else {
        acc_c -= up;
        acc_p -= eaz_p * y + in;
        nxt += dn;
      }
    }
  }
};

// In-plane neighbours of the populations that move in the plane, as
// differences from the column's own B (in FP32 they round at the scale of
// the differences and not of B).
template <typename Real, int W, bool Mesh>
struct InPlaneCoef {
  __device__ __forceinline__ InPlaneCoef(const MeshMarch<Real, W> &) {}
  template <int Q, class G> __device__ __forceinline__ void axis(const G &, Real &) const {}
  template <int Q, class G> __device__ __forceinline__ void diag(const G &, Real &) const {}
};
template <typename Real, int W>
struct InPlaneCoef<Real, W, true> {
  Real a[2], e[2], hs[2], u[2][2], v[2][2];
  __device__ __forceinline__ InPlaneCoef(const MeshMarch<Real, W> &m) {
    static_for<2>([&](auto d) {
      a[d] = m.template col<d>(kMarchA);
      e[d] = m.template col<d>(kMarchE);
      hs[d] = m.template col<d>(kMarchHs);
      static_for<2>([&](auto s) {
        u[d][s] = m.template col<d>(kMarchUp + s);
        v[d][s] = m.template col<d>(kMarchVp + s);
      });
    });
  }
  template <int Q, class G>
  __device__ __forceinline__ void axis(const G &g, Real &acc) const {
    constexpr int d = kCx[Q] != 0 ? 0 : 1, i = kCx[Q] + kCy[Q] > 0 ? 0 : 1;
    const Real bp = g.template at<Q, Unit<d>::x, Unit<d>::y>(), bm = g.template at<Q, -Unit<d>::x, -Unit<d>::y>();
    const Real b0 = g.template at<Q, 0, 0>();
    if constexpr (G::use) acc -= u[d][i] * (bp - b0) + v[d][i] * (b0 - bm);
  }
  template <int Q, class G>
  __device__ __forceinline__ void diag(const G &g, Real &acc) const {
    constexpr int i = kCx[Q] > 0 ? 0 : 1, j = kCy[Q] > 0 ? 0 : 1;
    const Real p1 = g.template at<Q, 1, 0>(), m1 = g.template at<Q, -1, 0>();
    const Real p2 = g.template at<Q, 0, 1>(), m2 = g.template at<Q, 0, -1>();
    const Real b0 = g.template at<Q, 0, 0>();
    Real pp, pm, mp, mm;
    if constexpr (kLaneCorners<Real>) {
      if constexpr (G::use) {
        pp = from_next_lane(p2), pm = from_next_lane(m2);
        mp = from_previous_lane(p2), mm = from_previous_lane(m2);
      }
    } else {
      pp = g.template at<Q, 1, 1>(), pm = g.template at<Q, 1, -1>();
      mp = g.template at<Q, -1, 1>(), mm = g.template at<Q, -1, -1>();
    }
    if constexpr (G::use) {
      const Real y0 = p2 - m2, x0 = p1 - m1;
      const Real mix = hs[1] * (a[0] * ((pp - pm) - y0) + e[0] * (y0 - (mp - mm))) +
                       hs[0] * (a[1] * ((pp - mp) - x0) + e[1] * (x0 - (pm - mm)));
      const Real in = (u[0][i] * (p1 - b0) + v[0][i] * (b0 - m1)) + (u[1][j] * (p2 - b0) + v[1][j] * (b0 - m2));
      if constexpr (kCx[Q] * kCy[Q] > 0)
        acc += mix - in;
      else
        acc -= mix + in;
    }
  }
};

// A cell's halves of the moments of its two D-faces (D = 0 or 1) at centre
// plane p-1 (planes p, p-1, p-2): with w the value less the tangential
// gradients and n the normal-flux field, the face between L and R has
//   unit cells: (w_L/2 + h n_L) + (w_R/2 - h n_R),
//   mesh:       ((1 - lam_L) w_L + hg_L n_L) + (lam_L w_R - hg_L n_R),
// so a cell forms up (as L of its upper face) and dn (as R of its lower one)
// from its own column's fields and their differences across D, and a face
// takes one half from each side: 23 field values instead of the 46 of the two
// cells' reads, and each gradient is formed once.
template <int D, bool Mesh, typename Real, int W>
__device__ __forceinline__ void face_halves(const MeshMarch<Real, W> &mc, int p, Real h, const Plane<Real, W> &c,
                                            const Plane<Real, W> &c1, const Plane<Real, W> &c2, Real (&up)[4],
                                            Real (&dn)[4]) {
  constexpr int t = 1 - D;
  using std::integral_constant;
  Real lam = Real(0), hg = Real(0), lam_m = Real(0), hg_m = Real(0), hst = Real(0.25) * h, hsz = hst;
  if constexpr (Mesh) {
    lam = mc.template col<D>(kMarchLam), hg = mc.template col<D>(kMarchHg);
    // of the lower face: the cell below's (column 0 of the tile, whose lower
    // half nobody reads, gets another entry of the table)
    lam_m = D == 0 ? mc.X[kMarchLam * W - 1] : mc.Y[kMarchLam * 8 - 1];
    hg_m = D == 0 ? mc.X[kMarchHg * W - 1] : mc.Y[kMarchHg * 8 - 1];
    hst = mc.template col<t>(kMarchHs), hsz = mc.z(kMarchHs, p - 1);
  }
  Real zd[4];
  gathered<Real, W>(c, c2, [&](const auto &g, const auto &g2) {
    constexpr int ids[4] = {kJz, kPxz, kPyz, kPzz};
    static_for<4>([&](auto i) {
      const Real a = g.template at<ids[i], 0, 0>(), b = g2.template at<ids[i], 0, 0>();
      if constexpr (std::decay_t<decltype(g)>::use) zd[i] = a - b;
    });
  });
  gathered<Real, W>(c1, c1, [&](const auto &g, const auto &) {
    auto half = [&](auto i, auto V, auto N, auto T) {
      const Real v = g.template at<V, 0, 0>(), nf = g.template at<N, 0, 0>(), d = dif<T, t, 0, 0>(g);
      if constexpr (std::decay_t<decltype(g)>::use) {
        if constexpr (Mesh) {
          const Real w = v - (hst * d + hsz * zd[i]);
          up[i] = (w - lam * w) + hg * nf;
          dn[i] = lam_m * w - hg_m * nf;
        } else {
          const Real w = Real(0.5) * v - hst * (d + zd[i]);
          up[i] = w + h * nf;
          dn[i] = w - h * nf;
        }
      }
    };
    half(integral_constant<int, 0>{}, integral_constant<int, kR0>{}, integral_constant<int, jid(D)>{},
         integral_constant<int, jid(t)>{});
    static_for<3>([&](auto a) {
      half(integral_constant<int, 1 + a>{}, integral_constant<int, jid(a)>{}, integral_constant<int, pid(a, D)>{},
           integral_constant<int, pid(a, t)>{});
    });
  });
}

// Moments of the y-face between the column and its upper neighbour at centre
// plane p-1, on the mesh (planes p, p-1, p-2).
template <typename Real, int W>
__device__ __forceinline__ void yface_moments_mesh(const MeshMarch<Real, W> &mc, int p, const Plane<Real, W> &c,
                                                  const Plane<Real, W> &c1, const Plane<Real, W> &c2, Real (&m)[4]) {
  const Real lam = mc.template col<1>(kMarchLam), hg = mc.template col<1>(kMarchHg);
  const Real hs = mc.template col<0>(kMarchHs), hsz = mc.z(kMarchHs, p - 1);
  Real vl[4], s1[4];
  gathered<Real, W>(c1, c1, [&](const auto &g, const auto &) {
    Real v[4], t[4];
    yface_inplane_mesh(g, lam, hg, hs, v, t);
    if constexpr (std::decay_t<decltype(g)>::use) static_for<4>([&](auto i) { vl[i] = v[i]; m[i] = t[i]; });
  });
  gathered<Real, W>(c, c2, [&](const auto &g, const auto &g2) {
    Real a[4], b[4];
    yface_zvalue_mesh(g, lam, a);
    yface_zvalue_mesh(g2, lam, b);
    if constexpr (std::decay_t<decltype(g)>::use) static_for<4>([&](auto i) { s1[i] = a[i] - b[i]; });
  });
  static_for<4>([&](auto i) { m[i] = vl[i] + (m[i] - hsz * s1[i]); });
}

// Thread number of the one-thread march: a 32-wide tile's wavefronts rotated so
// that the one with the halo rows is the first of its block, or the third in
// blocks whose number has an odd multiple of 256 (8 XCDs x 32 compute units: the
// two blocks a unit starts with).  A block's wavefronts go to the unit's four
// SIMDs in turn, so the halo wavefronts of its two blocks fall on different
// SIMDs, where as the last of every block both shared one.  FP32 160^3
// 228 -> 222 us, 256^3 0.846 -> 0.832 ms.
template <int W>
__device__ __forceinline__ int fused_thread() {
  return W == 32 ? (threadIdx.x + ((blockIdx.x >> 8) & 1 ? 64 : 192)) & 255 : threadIdx.x;
}

// The z-march of one tile (bx, by) over the planes [z0, z1) of a box; adds
// the moments of the updated cells to v.  L is the block's LDS, kFusedValues
// values per column: P [kNPop][NT], Q [2][kNQ][NT], Z [3][kNZ][NT].
// Mesh: on a stretched mesh with the tables coef (x, y, z rows of
// MarchCoef) and width (the cell widths, the weights of the sums); the x/y
// coefficients follow the plane data in L (kMeshValues).
// Halo: the code of the wavefront that holds the two halo rows of a 32-wide
// tile (tile_column).  It has no centres of its own and forms the moments of
// the interior wavefronts' x- and z-faces for them (lane l takes the columns of
// lane l of each in turn): the march is bound by the interior wavefronts'
// vector issue, and this one had a third of their work.  128^3 129.5 -> 124.2
// us, 256^3 0.868 -> 0.846 ms.
// In the second phase of a plane, after the barrier that follows the
// publishing, the interior wavefronts issue before a halo one on the same SIMD,
// which has less to do; up to that barrier, which all wait for, all are alike
// (and above another block's second phase).  256^3 0.843 -> 0.818 ms, 160^3
// 225 -> 219 us, 128^3 121.7 -> 119.8 us; the halo ones first, 0.832 ms.
template <typename Real, int W, bool O32, bool Mesh, bool Halo>
__device__ __forceinline__ void fused_tile(const global_t<Real> *__restrict__ ft, global_t<Real> *__restrict__ out, const StepParams &p,
                                           int bx, int by, int z0, int z1, Real *L, double (&v)[kNumSums],
                                           const Real *coef, const double *width) {
  constexpr int TX = Tile<W>::TX, TY = Tile<W>::TY, IX = Tile<W>::IX, IY = Tile<W>::IY, NT = Tile<W>::NT;
  const int n = p.n;
  const int64_t stride = p.stride;
  const int tid = tile_column<W>(fused_thread<W>());  // column of the tile
  const int tx = tid % TX, ty = tid / TX;
  const int x0 = bx * IX, y0 = by * IY;
  int gx = x0 - 1 + tx, gy = y0 - 1 + ty;
  gx = gx < 0 ? gx + n : (gx >= n ? gx % n : gx);
  gy = gy < 0 ? gy + n : (gy >= n ? gy % n : gy);
  const int col = gy * n + gx;
  constexpr bool kHelp = W == 32;                              // the halo rows have a wavefront of their own
  const bool rows = kHelp ? !Halo : ty >= 1 && ty <= TY - 2;   // interior rows, halo columns too
  const bool inner = rows && tx >= 1 && tx <= TX - 2 && (x0 + tx - 1) < n && (y0 + ty - 1) < n;
  const bool yface = tx >= 1 && tx <= TX - 2 && ty <= TY - 2;  // forms the y+ face
  const Real h = Real(p.h), dt = Real(p.dt);
  const Real dtal = dt * Real(p.alpha), dtbe = dt * Real(p.beta);
  Real *const LP = L + tid;
  Real *const LQ = L + kNPop * NT + tid;
  Real *const LZ = L + (kNPop + 2 * kNQ) * NT + tid;
  Real *const LY = L + kLdsValues * NT + tid;
  Real *const FX = L + (kLdsValues + 10) * NT + tid;
  Real *const RZ = L + (kLdsValues + 14) * NT + tid;
  MeshMarch<Real, W> mc{};
  const constant_t<double> *wz = nullptr;
  double wxy = 1.0;
  if constexpr (Mesh) {
    Real *const LM = L + kFusedValues * NT;
    load_mesh_columns<Real, W>(coef, n, x0, y0, LM);
    mc = {(const constant_t<Real> *)(coef + 2 * kMarchCoefs * n), LM + tx, LM + kMarchCoefs * W + ty, n};
    wz = (const constant_t<double> *)(width + 2 * n);
    wxy = to_global(width)[gx] * to_global(width)[n + gy];
    __syncthreads();
  }

  Real pf[kQ];        // f~ of the plane being published (loaded one plane ahead)
  // A centre's result is f~+ plus the stencil and face terms, which are
  // small beside it: they are summed apart (acc) and f~+ (fp) is added once,
  // when the centre is stored, so that the result is rounded at the scale of
  // f~ once instead of at every term (in FP32 this more than halves the
  // rounding noise the march adds per step).
  // Two centres at a time: p-1, completed in plane p's iteration, and p.
  Real acc_0[kQ], fp_0[kQ], acc_1[kQ], fp_1[kQ];
  Real nxt[10];       // z-1 terms of the z-moving populations of centre p+1
  // lower half of the z-face above the previous plane (mesh: its w, and nf in
  // zn), of the own column or of each helped one
  constexpr int kZ = kHelp ? 3 : 1;
  Real zl[kZ][4], zn[kZ][4];
  static_for<kQ>([&](auto q) { acc_0[q] = acc_1[q] = fp_0[q] = fp_1[q] = Real(0); });
  static_for<10>([&](auto i) { nxt[i] = Real(0); });
  static_for<kZ>([&](auto j) { static_for<4>([&](auto i) { zl[j][i] = Real(0); zn[j][i] = Real(0); }); });

  // With the faces formed at plane P: the z-face between P-1 and P to the
  // centres P-1 (acc_c, fp_c) and P (acc_p), then the x-faces and the lower
  // y-face (from the slot of the column W before) of centre P-1, its store and
  // its sums.  Runs after the barrier that ends plane P's iteration, in every
  // lane of an interior row (the x- terms are the previous lane's x+ terms).
  auto finish = [&](int P, Real (&acc_c)[kQ], const Real (&fp_c)[kQ], Real (&acc_p)[kQ]) {
    const int plane = P - 1;
    if (inner) {
      Real m[4];
      static_for<4>([&](auto i) { m[i] = RZ[i * NT]; });
      Real iw_c = Real(1), iw_p = Real(1);
      if constexpr (Mesh) iw_c = mc.z(kMarchIw, P - 1), iw_p = mc.z(kMarchIw, P);
      face_equilibrium<2, Real>(m, p, dtbe, [&](auto q, Real k, Real t) {
        if constexpr (Mesh) {
          acc_c[q] -= iw_c * (k * t);
          acc_p[q] += iw_p * (k * t);
        } else {
          acc_c[q] -= k * t;
          acc_p[q] += k * t;
        }
      });
    }
    if (P <= z0) return;
    Real mx[4], fxp[10], fxm[10];
    static_for<4>([&](auto i) { mx[i] = FX[i * NT]; });
    face_terms<0>(mx, p, dtbe, fxp);
    static_for<10>([&](auto k) { fxm[k] = from_previous_lane(fxp[k]); });
    if (!inner) return;
    Real fym[10];
    static_for<10>([&](auto k) { fym[k] = LY[k * NT - W]; });
    if constexpr (Mesh) {
      const Real iw = mc.template col<0>(kMarchIw);
      apply_terms<0, 1>(fxp, iw, acc_c);
      apply_terms<0, -1>(fxm, iw, acc_c);
      apply_terms<1, -1>(fym, mc.template col<1>(kMarchIw), acc_c);
    } else {
      apply_terms<0, 1>(fxp, acc_c);
      apply_terms<0, -1>(fxm, acc_c);
      apply_terms<1, -1>(fym, acc_c);
    }
    const int cell = plane * n * n + col;
    // plain (L2-allocating) stores: a tile row's 30 updated cells do not
    // fill whole 128-byte lines, and L2 merges them with the neighbouring
    // tiles' rows before they are written back
    Real res[kQ];
    static_for<kQ>([&](auto q) {
      res[q] = fp_c[q] + acc_c[q];
      *at_cell<O32>(out + (int64_t)q * stride, cell) = res[q];
    });
    if constexpr (Mesh) {
      double s[kNumSums] = {0, 0, 0, 0, 0};
      sums_of_populations<Real>(res, p.inv_rho0, s);
      const double vol = wxy * wz[plane];
      static_for<kNumSums>([&](auto i) { v[i] += vol * s[i]; });
    } else {
      sums_of_populations<Real>(res, p.inv_rho0, v);
    }
  };

  load_raw<Real, O32>(ft, stride, n, col, z0 - 1, pf);
  int q2 = 0, q3 = 0;  // Q slot and Z slot of plane p
  // Plane p_ of the march: acc_c, fp_c hold centre p-1; acc_p, fp_p hold the
  // centre the last iteration formed (p-2, finished here) and then centre p.
  // One iteration past the chunk's end only finishes its last centre (and
  // returns false), so that every centre is completed by the same code (and
  // rounds the same whatever the chunk length).
  auto iteration = [&](int p_, Real (&acc_c)[kQ], const Real (&fp_c)[kQ], Real (&acc_p)[kQ], Real (&fp_p)[kQ]) {
    if (p_ > z0 && rows) finish(p_ - 1, acc_p, fp_p, acc_c);
    if (p_ > z1) return false;
    const bool has_prev = p_ > z0;          // centre p-1 is in the chunk
    const bool has_cur = p_ >= z0 && p_ < z1;
    const int q2m = q2 ^ 1, q3m = q3 == 0 ? 2 : q3 - 1, q3mm = q3 == 2 ? 0 : q3 + 1;
    const Plane<Real, W> c{LP, LQ + q2 * (kNQ * NT), LZ + q3 * (kNZ * NT)};        // plane p
    const Plane<Real, W> c1{nullptr, LQ + q2m * (kNQ * NT), LZ + q3m * (kNZ * NT)};  // plane p-1
    const Plane<Real, W> c2{nullptr, nullptr, LZ + q3mm * (kNZ * NT)};              // plane p-2

    // own-column pieces of plane p: z+1 terms of centre p-1, the centre
    // terms and initial value of centre p, z-1 terms of centre p+1 (formed
    // by halo columns too, which never store them)
    const OwnCoef<Real, W, Mesh> own(mc, p_);
    publish_cell<Real, W>(pf, LP, LQ + q2 * (kNQ * NT), LZ + q3 * (kNZ * NT), p, [&](auto q, Real bq, Real ftq) {
      if constexpr (Mesh) {
        Real r = Real(0);
        if constexpr (kCz[q] != 0) own.template add<kCz[q]>(bq, acc_c[q], r, nxt[zslot(q)]);
        acc_p[q] = r;
        fp_p[q] = ftq;
        return;
      }
      if constexpr (kCz[q] != 0) acc_c[q] -= dtal * ((Real(0.5 * kCz[q]) - h) * bq);
      Real r = Real(0);
      if constexpr (kCz[q] != 0) r = nxt[zslot(q)];
      if constexpr (q != 0) r -= dtal * (Real(speed2(q) == 1 ? 2 : 4) * h * bq);
      acc_p[q] = r;
      fp_p[q] = ftq;
      if constexpr (kCz[q] != 0) nxt[zslot(q)] = -(dtal * ((Real(-0.5 * kCz[q]) - h) * bq));
    });
    __syncthreads();
    __builtin_amdgcn_s_setprio(Halo ? 0 : 2);

    // face between p-1 and p of a column (upper half from plane p, lower half
    // carried from plane p-1), and the lower half of the next one
    auto face_below = [&](const Plane<Real, W> &pl, const MeshMarch<Real, W> &cf, Real *rz, Real (&zl)[4], Real (&zn)[4]) {
      const ZFaceCoef<Real, W, Mesh> zf(cf, p_);
      gathered<Real, W>(pl, pl, [&](const auto &g, const auto &) {
        Real m[4], lo[4];
        if constexpr (Mesh) {
          zf.face(g, zl, zn, m);
        } else {
          zface_half<-1>(g, h, m);
          zface_half<1>(g, h, lo);
        }
        if constexpr (std::decay_t<decltype(g)>::use) {
          static_for<4>([&](auto i) { rz[i * NT] = Mesh ? m[i] : m[i] + zl[i]; });
          if constexpr (!Mesh) static_for<4>([&](auto i) { zl[i] = lo[i]; });
        }
      });
    };
    // x+ face of a column: its upper half and the next lane's lower one
    auto face_right = [&](const Plane<Real, W> &a, const Plane<Real, W> &b, const Plane<Real, W> &e,
                          const MeshMarch<Real, W> &cf, Real *f) {
      Real up[4], dn[4];
      face_halves<0, Mesh>(cf, p_, h, a, b, e, up, dn);
      static_for<4>([&](auto i) { f[i * NT] = up[i] + from_next_lane(dn[i]); });
    };
    if constexpr (Halo) {
      static_for<3>([&](auto j) {
        const int d = tile_column<W>(j * 64 + (threadIdx.x & 63)) - tid;
        MeshMarch<Real, W> cf = mc;
        if constexpr (Mesh) cf.Y += d / W;  // the same x, d / W rows further
        const Plane<Real, W> a{nullptr, c.Q + d, c.Z + d}, b{nullptr, c1.Q + d, c1.Z + d}, e{nullptr, nullptr, c2.Z + d};
        face_below(a, cf, RZ + d, zl[j], zn[j]);
        if (has_prev) face_right(a, b, e, cf, FX + d);
      });
    } else if constexpr (!kHelp) {
      if (inner) face_below(c, mc, RZ, zl[0], zn[0]);
      if (has_prev && rows) face_right(c, c1, c2, mc, FX);
    }
    if (inner) {
      // diagonal z-moving populations: the in-plane differences D = B(+d1)
      // - B(-d1) and sums S = B(+d1) + B(-d1) of plane p enter centre p-1
      // (z+1 mixed term), centre p (in-plane terms) and centre p+1 (z-1
      // mixed term)
      const DiagZCoef<Real, W, Mesh> dz(mc, p_);
      gathered<Real, W>(c, c, [&](const auto &g, const auto &) {
        static_for<kQ>([&](auto q) {
          if constexpr (is_diag_z(q) && Mesh) {
            dz.template add<q>(g, acc_c[q], acc_p[q], nxt[zslot(q)]);
          } else if constexpr (is_diag_z(q)) {
            constexpr int d1 = kCx[q] != 0 ? 0 : 1, s1 = kCx[q] + kCy[q];
            constexpr Real k = Real(0.5 * s1 * kCz[q]);
            const Real bp_ = g.template at<q, Unit<d1>::x, Unit<d1>::y>();
            const Real bm_ = g.template at<q, -Unit<d1>::x, -Unit<d1>::y>();
            if constexpr (std::decay_t<decltype(g)>::use) {
              const Real dd = bp_ - bm_;
              acc_c[q] += dtal * (k * h * dd);
              acc_p[q] -= dtal * (Real(0.5 * s1) * dd - h * (bp_ + bm_));
              nxt[zslot(q)] -= dtal * (k * h * dd);
            }
          }
        });
      });
    }
    if (has_prev) {
      // y-faces of centre p-1: in-plane part from plane p-1, the z-tangential
      // gradients -h/4 [(M_L + M_R)(p) - (M_L + M_R)(p-2)]
      const Real hq = Real(0.25) * h;
      auto yface_moments = [&](Real (&m)[4]) {
        if constexpr (Mesh) {
          yface_moments_mesh(mc, p_, c, c1, c2, m);
          return;
        }
        gathered<Real, W>(c1, c1, [&](const auto &g, const auto &) {
          Real t[4];
          yface_inplane(g, h, t);
          if constexpr (std::decay_t<decltype(g)>::use) static_for<4>([&](auto i) { m[i] = t[i]; });
        });
        gathered<Real, W>(c, c2, [&](const auto &g, const auto &g2) {
          Real s1[4], s0[4];
          yface_zsum(g, s1);
          yface_zsum(g2, s0);
          if constexpr (std::decay_t<decltype(g)>::use) static_for<4>([&](auto i) { m[i] -= hq * (s1[i] - s0[i]); });
        });
      };
      // The y-face between the column and the next row is formed once, by
      // every interior column of every row but the last (halo row 0 too); its
      // ten terms are left in LY for the column above, which applies them as
      // its lower face in finish().
      if (yface) {
        Real my[4], fy[10];
        yface_moments(my);
        face_terms<1>(my, p, dtbe, fy);
        static_for<10>([&](auto k) { LY[k * NT] = fy[k]; });
        if (inner) {
          if constexpr (Mesh)
            apply_terms<1, 1>(fy, mc.template col<1>(kMarchIw), acc_c);
          else
            apply_terms<1, 1>(fy, acc_c);    // y+
        }
      }
    }

    phase();
    // the next plane's loads overlap the rest of this one (issued right
    // after publishing they took the same time and fetched 33% more bytes
    // from HBM)
    if (p_ < z1) load_raw<Real, O32>(ft, stride, n, col, p_ + 1, pf);

    if (inner && has_cur) {
      // in-plane terms of the in-plane populations of centre p (the centre
      // value was added before)
      //   axis: L = s/2 (B(+d) - B(-d)) - h (B(+d) + B(-d))
      const InPlaneCoef<Real, W, Mesh> xy(mc);
      gathered<Real, W>(c, c, [&](const auto &g, const auto &) {
        static_for<5>([&](auto q) {
          if constexpr (q >= 1 && Mesh) {
            xy.template axis<q>(g, acc_p[q]);
          } else if constexpr (q >= 1) {
            constexpr int d = kCx[q] != 0 ? 0 : 1, s = kCx[q] + kCy[q];
            const Real bp_ = g.template at<q, Unit<d>::x, Unit<d>::y>();
            const Real bm_ = g.template at<q, -Unit<d>::x, -Unit<d>::y>();
            if constexpr (std::decay_t<decltype(g)>::use)
              acc_p[q] -= dtal * (Real(0.5 * s) * (bp_ - bm_) - h * (bp_ + bm_));
          }
        });
      });
      //   diagonal in the plane, in the (x, y) frame of its own signs
      auto diag_xy = [&](auto q, const auto &g) {
        if constexpr (Mesh) {
          xy.template diag<q>(g, acc_p[q]);
          return;
        }
        constexpr int sx = kCx[q], sy = kCy[q];
        const Real p1 = g.template at<q, 1, 0>(), m1 = g.template at<q, -1, 0>();
        const Real p2 = g.template at<q, 0, 1>(), m2 = g.template at<q, 0, -1>();
        const Real pp = g.template at<q, sx, sy>(), pm = g.template at<q, sx, -sy>();
        const Real mp = g.template at<q, -sx, sy>(), mm = g.template at<q, -sx, -sy>();
        if constexpr (std::decay_t<decltype(g)>::use) {
          const Real a1 = sx > 0 ? (p1 - m1) : (m1 - p1);
          const Real a2 = sy > 0 ? (p2 - m2) : (m2 - p2);
          acc_p[q] -= dtal * ((Real(0.5) * a1 + Real(0.5) * a2) - h * ((p1 + m1) + (p2 + m2)) -
                              Real(0.5) * h * (((pp - pm) - mp) + mm));
        }
      };
      gathered<Real, W>(c, c, [&](const auto &g, const auto &) {
        diag_xy(std::integral_constant<int, 7>{}, g);
        diag_xy(std::integral_constant<int, 8>{}, g);
      });
      gathered<Real, W>(c, c, [&](const auto &g, const auto &) {
        diag_xy(std::integral_constant<int, 9>{}, g);
        diag_xy(std::integral_constant<int, 10>{}, g);
      });
    }
    q2 ^= 1;
    q3 = q3 == 2 ? 0 : q3 + 1;
    __syncthreads();
    __builtin_amdgcn_s_setprio(3);
    return true;
  };
  // two planes per turn, the two centres' arrays changing places: as one
  // iteration with a copy from one to the other, 38 of its ~1200 vector
  // instructions were that copy (both copies of the code round alike, see the
  // top of this file)
  for (int p_ = z0 - 1;; p_ += 2) {
    if (!iteration(p_, acc_0, fp_0, acc_1, fp_1)) break;
    if (!iteration(p_ + 1, acc_1, fp_1, acc_0, fp_0)) break;
  }
}

// Register budget of the one-thread march: in FP32, 256 registers, two
// waves per SIMD.  (Without the separate f~+ of two centres it fits 168
// registers and three waves, 10% faster, but its rounding noise then puts
// the FP32 spectrum's weakest resolved shells at ~1e-4 of FP64.)  FP64
// tiles use the split march.
template <typename Real>
constexpr int kWavesPerSimd = sizeof(Real) == 4 ? 2 : 1;

// Tile and planes of work item `local` of a box.  Items are tile z-chunks,
// numbered by tile (x fastest, then y), then by chunk.  With tail_split =
// m > 1 (a box launched alone, one block per item, blocks dealt to the 8
// XCDs in turn): the first tail_from chunk items fill whole rounds of the
// device; each of the t chunks left over is cut in z into m parts of
// ceil(chunk planes / m) planes (the last parts may be short or empty),
// numbered part by part so that the parts of neighbouring tiles run side by
// side.  The work of each XCD (a contiguous eighth of the items, see
// xcd_tile) is its eighth of the whole chunks followed by its eighth of the
// parts (slots past the last part are empty), so that every XCD's last
// round is made of parts and fills its compute units for a fraction of a
// chunk's time.
// (Host and device code: the library's work-split query runs it on the host.)
__host__ __device__ constexpr int imin(int a, int b) { return a < b ? a : b; }
struct ItemPlanes {
  int tile, z0, left;
  __host__ __device__ __forceinline__ ItemPlanes(const BatchBox &d, int local) {
    const int n = d.sp.n, c = d.nz_chunk, tiles = d.tiles_x * d.tiles_y;
    int item = local, part = 0, parts = 1;
    if (d.tail_split > 1) {
      const int t = tiles * ((n + c - 1) / c) - d.tail_from;
      const int pieces = t * d.tail_split;
      const int fx = d.tail_from / 8, px = (pieces + 7) / 8;
      const int x = local / (fx + px), j = local - x * (fx + px);
      if (j < fx) {
        item = x * fx + j;
      } else {
        const int piece = x * px + (j - fx);
        if (piece >= pieces) {  // an empty slot of the last XCD
          tile = z0 = left = 0;
          return;
        }
        part = piece / t;
        item = d.tail_from + (piece - part * t);
        parts = d.tail_split;
      }
    }
    tile = item % tiles;
    const int zc = item / tiles * c, zc1 = imin(zc + c, n);
    const int len = (zc1 - zc + parts - 1) / parts;
    z0 = imin(zc1, zc + part * len);
    left = imin(zc1, z0 + len) - z0;
  }
};

// Tile of a block, numbered so that the blocks one XCD runs (blocks are
// dealt to the eight XCDs in turn) take consecutive tiles: block b of a
// launch of `padded` blocks (a multiple of 8) takes tile
// (b mod 8) * padded/8 + b/8.
__device__ __forceinline__ int xcd_tile(int b, int padded) { return (b & 7) * (padded >> 3) + (b >> 3); }

// One launch advances one or many boxes: work item = one tile z-chunk of
// one box of the device table `boxes` (sorted by item_begin), numbered as
// the tiles of that box's own launch.  Round r of the grid takes items
// [r G, (r+1) G), dealt to the XCDs in contiguous eighths.  A single box is
// a table of one entry, so a box stepped alone and the same box stepped in
// a batch of its tile width run the same machine code; other tile widths and
// offsets round alike too, so the populations are the same bits.
template <typename Real, int W, bool O32, bool Mesh>
__global__ __launch_bounds__(Tile<W>::NT, kWavesPerSimd<Real>) void dugks_fused_kernel(const BatchBox *__restrict__ boxes, int nbox,
                                                                  int total_items, PendingSums prev) {
  __shared__ Real L[kFusedValues * Tile<W>::NT + (Mesh ? kMeshValues<W> : 0)];
  // the extra block (see launch_lbe_step) is the first; the others keep their
  // distribution over the XCDs, one further on
  const int extra = prev.nblocks > 0, G = gridDim.x - extra, block = blockIdx.x - extra;
  if (block < 0) {
    add_pending<Tile<W>::NT / 64>(prev.partials, prev.nblocks, prev.out, reinterpret_cast<double (*)[kNumSums]>(L));
    return;
  }
  for (int base = 0; base < total_items; base += G) {
    const int it = base + xcd_tile(block, G);
    if (it >= total_items) continue;
    const int b = find_batch_box(boxes, nbox, it);
    const BatchBox &d = boxes[b];
    const int local = it - d.item_begin;
    double v[kNumSums] = {0, 0, 0, 0, 0};
    const global_t<Real> *src = to_global(static_cast<const Real *>(d.f[d.cur]));
    global_t<Real> *dst = to_global(static_cast<Real *>(d.f[d.cur ^ 1]));
    const ItemPlanes ip(d, local);
    if (ip.left > 0) {
      auto march = [&](auto halo) {
        fused_tile<Real, W, O32, Mesh, halo>(src, dst, d.sp, ip.tile % d.tiles_x, ip.tile / d.tiles_x, ip.z0,
                                             ip.z0 + ip.left, L, v, static_cast<const Real *>(d.mesh_coef), d.mesh_width);
      };
      if (W != 32 || fused_thread<W>() < Tile<W>::NT - 64)
        march(std::false_type{});
      else if constexpr (W == 32)
        march(std::true_type{});
    }
    // After the march's last barrier, finish() reads the face terms and moments
    // and the mesh coefficients; the reduction's rows lie in the populations'
    // part of L, which it does not read.
    static_assert(sizeof(double) * kNumSums * (Tile<W>::NT / 64) <= sizeof(Real) * kNPop * Tile<W>::NT);
    // summed in the order of the wavefronts' rows: which wavefront has which rows
    // depends on the block's number, which the extra block shifts
    write_block_partials<Tile<W>::NT / 64>(v, d.partials, d.items, local, reinterpret_cast<double (*)[kNumSums]>(L),
                                           fused_thread<W>() >> 6);
    __syncthreads();
  }
}


// The FP64 march is one copy of the code per kernel, so that the z-chunk cannot
// change its rounding; with contraction left to the optimiser a 32^3 box is 2%
// faster (1.46 -> 1.43 ms for 100 steps).  The two tile widths give the same bits
// (tests).
#pragma clang fp contract(fast)
// ---------------------------------------------------------------------------
// Split-population march.  Two thread groups share each column of the
// tile: group A (the first NT threads) holds the ten z-moving populations
// (5, 6, 11..18), group B the other nine.  Each step is done by one group:
// A the z-moving stencils and the x-face moments, B the in-plane stencils,
// the z-face and y-face moments and the global sums; each applies the face
// equilibria to its own populations.  The groups exchange the partial
// moment sums of each published cell, the face moments and A's part of the
// stored cells' sums through LDS.  A thread carries the state of about half
// a column, so each compute unit holds twice the waves of the
// one-thread-per-column march.
constexpr int kPopsA[10] = {5, 6, 11, 12, 13, 14, 15, 16, 17, 18};
constexpr int kPopsB[9] = {0, 1, 2, 3, 4, 7, 8, 9, 10};
template <int G>
struct Group {
  static constexpr int N = G == 0 ? 10 : 9;
  static constexpr int pop(int i) { return G == 0 ? kPopsA[i] : kPopsB[i]; }
};
constexpr int group_of(int q) { return (q == 5 || q == 6 || q >= 11) ? 0 : 1; }
constexpr int local_of(int q) {
  for (int i = 0; i < 10; ++i)
    if (kPopsA[i] == q) return i;
  for (int i = 0; i < 9; ++i)
    if (kPopsB[i] == q) return i;
  return -1;
}
// The partial moments the groups exchange (indices of pair_moments): B needs
// A's part of drho, j, Pi_xx and Pi_yy (A's populations have no Pi_xy), A needs
// B's part of drho, jx and jy (B's have no jz, Pi_zz, Pi_xz, Pi_yz).
constexpr int kToB = 6, kToA = 3;
constexpr int kForB[kToB] = {0, 1, 2, 3, 4, 5};
constexpr int kForA[kToA] = {0, 1, 2};
// LDS per column after the plane buffers:
//   RA [6]:  A's partial moments (read by B after the first barrier of an
//            iteration);
//   RB [3]:  B's partial moments;
//   RZ [4]:  the moments of the z-face below plane p, formed by B in the third
//            phase, read by A after the third barrier;
//   FX [4]:  those of the x-face between the column and the next one, formed by
//            A, read by B of both columns;
//   RU, RD [4]: the column's halves of the moments of its upper and lower
//            y-faces (face_halves), formed by B, read by A of the column and by
//            both threads of the columns above and below;
//   SA [3]:  A's part of the momentum of its last stored cell (read by B in the
//            next iteration).
// RA, RB and SA are written in the first or last phase of an iteration and
// read after the barrier that follows; RZ, FX, RU, RD are written in the third
// phase, and next written after the second barrier of the next iteration.
constexpr int kRA = kNPop + 2 * kNQ + 3 * kNZ, kRB = kRA + kToB, kRZ = kRB + kToA, kFX = kRZ + 4, kRU = kFX + 4,
              kRD = kRU + 4, kSA = kRD + 4;
constexpr int kSplitValues = kSA + 3;

// Loads of the group's populations of the column's cell in plane `plane`.
template <typename Real, int G, bool O32>
__device__ __forceinline__ void load_group(const global_t<Real> *__restrict__ ft, int64_t stride, int n, int col, int plane,
                                           Real (&f)[Group<G>::N]) {
  const int z = plane < 0 ? plane + n : (plane >= n ? plane - n : plane);
  const int idx = z * n * n + col;
  static_for<Group<G>::N>([&](auto i) { f[i] = *at_cell<O32>(ft + (int64_t)Group<G>::pop(i) * stride, idx); });
}

// Partial moment sums over the group's populations (both groups' sets are
// closed under q -> -q): drho, jx, jy, jz, Pi_xx, Pi_yy, Pi_zz, Pi_xy,
// Pi_xz, Pi_yz, formed as in pair_moments().
template <typename Real, int G>
__device__ __forceinline__ void partial_moments(const Real (&f)[Group<G>::N], Real (&m)[10]) {
  pair_moments<Real>([](int q) constexpr { return group_of(q) == G; }, [&](auto q) { return f[local_of(q)]; }, m);
}

// The rest of publishing a cell, from its full moment sums m: B and f~+ of
// the group's populations (handed to use(q, B_q, f~+_q)), their LDS
// entries, and the group's moment fields (A: Jz, Pxz, Pyz, Pzz; B: R0, Jx,
// Jy, Pxx, Pxy, Pyy), in the equilibrium-exact forms of publish_cell().
template <typename Real, int W, int G, class Use>
__device__ __forceinline__ void publish_group(const Real (&f)[Group<G>::N], const Real (&m)[10], Real *P, Real *Q,
                                              Real *Z, const StepParams &p, Use &&use) {
  constexpr int NT = Tile<W>::NT;
  const Real drho = m[0], jx = m[1], jy = m[2], jz = m[3];
  const Real rho0 = Real(p.rho0), ir = Real(p.inv_rho0);
  const Real a = Real(p.a_bp);
  const Real d3 = drho * Real(1.0 / 3.0);
  if constexpr (G == 0) {
    const Real ezz = d3 + jz * jz * ir, exz = jx * jz * ir, eyz = jy * jz * ir;
    Z[z_index(kJz) * NT] = jz;
    Z[z_index(kPxz) * NT] = exz + a * (m[8] - exz);
    Z[z_index(kPyz) * NT] = eyz + a * (m[9] - eyz);
    Z[z_index(kPzz) * NT] = ezz + a * (m[6] - ezz);
  } else {
    const Real exx = d3 + jx * jx * ir, eyy = d3 + jy * jy * ir, exy = jx * jy * ir;
    Q[q_index(kR0) * NT] = drho;
    Q[q_index(kJx) * NT] = jx;
    Q[q_index(kJy) * NT] = jy;
    Q[q_index(kPxx) * NT] = exx + a * (m[4] - exx);
    Q[q_index(kPxy) * NT] = exy + a * (m[7] - exy);
    Q[q_index(kPyy) * NT] = eyy + a * (m[5] - eyy);
  }
  const Real u[3] = {jx * ir, jy * ir, jz * ir};
  pair_equilibrium<Real>([](int q) constexpr { return group_of(q) == G; }, drho, u, rho0, [&](auto q, Real feq) {
    constexpr int i = local_of(q);
    const Real b = feq + a * (f[i] - feq);
    if constexpr (pop_index(q) >= 0) P[pop_index(q) * NT] = b;
    use(q, b, b + (b - f[i]) * Real(1.0 / 3.0));
  });
}

// The z-march of group G of a tile over the planes [z0, z1) (see above).
// L: the block's LDS, kSplitValues values per column.
// Mesh: as in fused_tile.
// Halo: the code of the wavefront of a group that holds the two halo rows of a
// 32-wide tile.  It has no centres of its own; A's forms the x-faces of the
// group's three interior wavefronts (lane l takes the columns of lane l of
// each in turn).  A's is its group's last wavefront and B's its first: the
// wavefronts of a block go to the compute unit's four SIMDs in turn, so the
// halo wavefronts are on different SIMDs, each beside an interior one, where
// together on one they left it idle while the others worked.  256^3 1.665 ms
// with both last, 1.610 ms apart, 1.535 ms with the x-faces handed over
// (128^3 217, 216, 214 us; 64^3 40.9, 39.3, 39.8 us); the z-faces handed to B's
// halo wavefront 1.55 ms at 256^3 but 220 us at 128^3.
// The interior wavefronts issue before a halo one on the same SIMD: 256^3 1.541
// -> 1.515 ms, 64^3 37.6 -> 37.2 us (the halo ones first 1.590 ms; group B before
// A 1.648 ms, A before B as without).
template <typename Real, int W, int G, bool O32, bool Mesh, bool Halo>
__device__ __forceinline__ void split_tile(const global_t<Real> *__restrict__ ft, global_t<Real> *__restrict__ out, const StepParams &p,
                                           int bx, int by, int z0, int z1, Real *L, double (&v)[kNumSums],
                                           const Real *coef, const double *width) {
  constexpr int TX = Tile<W>::TX, TY = Tile<W>::TY, IX = Tile<W>::IX, IY = Tile<W>::IY, NT = Tile<W>::NT;
  constexpr int NG = Group<G>::N;
  const int n = p.n;
  const int64_t stride = p.stride;
  // column of the tile; B's wavefronts of a 32-wide tile are rotated by one, its
  // halo wavefront first
  const int c = tile_column<W>(G == 0 ? threadIdx.x : (threadIdx.x - (W == 32 ? 64 : 0)) % NT);
  __builtin_amdgcn_s_setprio(Halo ? 0 : 2);
  const int tx = c % TX, ty = c / TX;
  const int x0 = bx * IX, y0 = by * IY;
  int gx = x0 - 1 + tx, gy = y0 - 1 + ty;
  gx = gx < 0 ? gx + n : (gx >= n ? gx % n : gx);
  gy = gy < 0 ? gy + n : (gy >= n ? gy % n : gy);
  const int col = gy * n + gx;
  constexpr bool kHelp = W == 32;  // the halo rows have a wavefront of their own
  const bool rows = kHelp ? !Halo : ty >= 1 && ty <= TY - 2;  // interior rows, halo columns too
  const bool inner = rows && tx >= 1 && tx <= TX - 2 && (x0 + tx - 1) < n && (y0 + ty - 1) < n;
  // Halo: distance (columns, rows) to the columns of interior wavefront j
  auto helped = [&](int j) { return tile_column<W>(j * 64 + (threadIdx.x & 63)) - c; };
  const Real h = Real(p.h), dt = Real(p.dt);
  const Real dtal = dt * Real(p.alpha), dtbe = dt * Real(p.beta);
  const double ir = p.inv_rho0;
  Real *const LP = L + c;
  Real *const LQ = L + kNPop * NT + c;
  Real *const LZ = L + (kNPop + 2 * kNQ) * NT + c;
  Real *const RA = L + kRA * NT + c;
  Real *const RB = L + kRB * NT + c;
  Real *const RZ = L + kRZ * NT + c;
  Real *const FX = L + kFX * NT + c;
  Real *const RU = L + kRU * NT + c;
  Real *const RD = L + kRD * NT + c;
  Real *const SA = L + kSA * NT + c;
  MeshMarch<Real, W> mc{};
  const constant_t<double> *wz = nullptr;
  double wxy = 1.0;
  if constexpr (Mesh) {  // filled by both groups; first read after the first barrier of the march
    Real *const LM = L + kSplitValues * NT;
    load_mesh_columns<Real, W>(coef, n, x0, y0, LM);
    mc = {(const constant_t<Real> *)(coef + 2 * kMarchCoefs * n), LM + tx, LM + kMarchCoefs * W + ty, n};
    wz = (const constant_t<double> *)(width + 2 * n);
    wxy = to_global(width)[gx] * to_global(width)[n + gy];
  }
  // adds the group's part of a stored cell's sums, weighted by the cell volume
  // on the mesh
  auto add_sums = [&](int plane, double r, double x, double y, double z) {
    if constexpr (Mesh) {
      const double vol = wxy * wz[plane];
      v[0] += vol * r; v[1] += vol * x; v[2] += vol * y; v[3] += vol * z;
    } else {
      v[0] += r; v[1] += x; v[2] += y; v[3] += z;
    }
  };

  Real pf[NG];            // the group's f~ of the plane being published
  Real acc_c[NG];         // centre p-1
  Real acc_p[NG];         // centre p
  Real nxt[10];           // A: z-1 terms of centre p+1 (all of A's populations move in z)
  // B: lower half of the z-face above the previous plane (mesh: its w, and nf in zn)
  Real zl[4], zn[4];
  double jb[3] = {0, 0, 0};  // B: its part of the momentum of the last stored cell
  // B: the kinetic energy of the last stored cell, in plane `plane`
  auto add_energy = [&](int plane) {
    const double x = jb[0] + (double)SA[0], y = jb[1] + (double)SA[NT], z = jb[2] + (double)SA[2 * NT];
    const double ke = 0.5 * (x * x + y * y + z * z) * ir * ir;
    if constexpr (Mesh)
      v[4] += wxy * wz[plane] * ke;
    else
      v[4] += ke;
  };
  static_for<NG>([&](auto i) { acc_p[i] = Real(0); });
  static_for<10>([&](auto i) { nxt[i] = Real(0); });
  static_for<4>([&](auto i) { zl[i] = Real(0); zn[i] = Real(0); });

  load_group<Real, G, O32>(ft, stride, n, col, z0 - 1, pf);
  int q2 = 0, q3 = 0;
  for (int p_ = z0 - 1; p_ <= z1; ++p_) {
    const bool has_prev = p_ > z0;
    const bool has_cur = p_ >= z0 && p_ < z1;
    const bool stored_last = p_ - 1 > z0;  // a cell was stored in the previous iteration
    const int q2m = q2 ^ 1, q3m = q3 == 0 ? 2 : q3 - 1, q3mm = q3 == 2 ? 0 : q3 + 1;
    const Plane<Real, W> pc{LP, LQ + q2 * (kNQ * NT), LZ + q3 * (kNZ * NT)};
    const Plane<Real, W> pc1{nullptr, LQ + q2m * (kNQ * NT), LZ + q3m * (kNZ * NT)};
    const Plane<Real, W> pc2{nullptr, nullptr, LZ + q3mm * (kNZ * NT)};

    static_for<NG>([&](auto i) { acc_c[i] = acc_p[i]; });
    // partial moments of this group's populations, exchanged with the other group
    Real m[10];
    partial_moments<Real, G>(pf, m);
    if constexpr (G == 0)
      static_for<kToB>([&](auto k) { RA[k * NT] = m[kForB[k]]; });
    else
      static_for<kToA>([&](auto k) { RB[k * NT] = m[kForA[k]]; });
    __syncthreads();
    if constexpr (G == 0)
      static_for<kToA>([&](auto k) { m[kForA[k]] = m[kForA[k]] + RB[k * NT]; });
    else
      static_for<kToB>([&](auto k) { m[kForB[k]] = RA[k * NT] + m[kForB[k]]; });
    if constexpr (G == 1) {
      if (inner && stored_last) {
        add_energy(p_ - 2);
      }
    }
    // own-column pieces of plane p (see fused_tile)
    const OwnCoef<Real, W, Mesh> own(mc, p_);
    publish_group<Real, W, G>(pf, m, LP, LQ + q2 * (kNQ * NT), LZ + q3 * (kNZ * NT), p, [&](auto q, Real bq, Real ftq) {
      constexpr int i = local_of(q);
      if constexpr (Mesh) {
        Real r = ftq;
        if constexpr (kCz[q] != 0) own.template add<kCz[q]>(bq, acc_c[i], r, nxt[i]);
        acc_p[i] = r;
        return;
      }
      if constexpr (kCz[q] != 0) acc_c[i] -= dtal * ((Real(0.5 * kCz[q]) - h) * bq);
      Real r = ftq;
      if constexpr (kCz[q] != 0) r += nxt[i];
      if constexpr (q != 0) r -= dtal * (Real(speed2(q) == 1 ? 2 : 4) * h * bq);
      acc_p[i] = r;
      if constexpr (kCz[q] != 0) nxt[i] = -(dtal * ((Real(-0.5 * kCz[q]) - h) * bq));
    });
    __syncthreads();

    Real fx[2][4];  // A: the x+ and x- faces; B: its halves of the y+ and y- faces, then the faces
    // B: face between p-1 and p (upper half from plane p, lower half carried
    // from plane p-1) for A, and the lower half of the next one
    auto face_below = [&]() {
      const ZFaceCoef<Real, W, Mesh> zf(mc, p_);
      gathered<Real, W>(pc, pc, [&](const auto &g, const auto &) {
        Real mm[4], lo[4];
        if constexpr (Mesh) {
          zf.face(g, zl, zn, mm);
        } else {
          zface_half<-1>(g, h, mm);
          zface_half<1>(g, h, lo);
        }
        if constexpr (std::decay_t<decltype(g)>::use) {
          static_for<4>([&](auto i) { RZ[i * NT] = Mesh ? mm[i] : mm[i] + zl[i]; });
          if constexpr (!Mesh) static_for<4>([&](auto i) { zl[i] = lo[i]; });
        }
      });
    };
    // A: x-faces of a column: its halves and those of the lanes beside
    auto x_faces = [&](const Plane<Real, W> &a, const Plane<Real, W> &b, const Plane<Real, W> &e,
                       const MeshMarch<Real, W> &m, Real *f, Real (&xp)[4], Real (&xm)[4]) {
      Real up[4], dn[4];
      face_halves<0, Mesh>(m, p_, h, a, b, e, up, dn);
      static_for<4>([&](auto i) {
        xp[i] = up[i] + from_next_lane(dn[i]);
        xm[i] = from_previous_lane(up[i]) + dn[i];
        f[i * NT] = xp[i];
      });
    };
    if constexpr (Halo && G == 0) {
      if (has_prev)
        static_for<3>([&](auto j) {
          const int d = helped(j);
          MeshMarch<Real, W> m = mc;
          if constexpr (Mesh) m.Y += d / W;  // the same x, d / W rows further
          const Plane<Real, W> a{nullptr, nullptr, pc.Z + d}, b{nullptr, pc1.Q + d, pc1.Z + d}, e{nullptr, nullptr, pc2.Z + d};
          Real xp[4], xm[4];
          x_faces(a, b, e, m, FX + d, xp, xm);
        });
    }
    if (inner) {
      if constexpr (G == 0) {
        // diagonal z-moving populations: in-plane differences D = B(+d1) -
        // B(-d1) and sums S = B(+d1) + B(-d1) of plane p enter centre p-1
        // (z+1 mixed term), centre p (in-plane terms), centre p+1 (z-1 mixed term)
        const DiagZCoef<Real, W, Mesh> dz(mc, p_);
        gathered<Real, W>(pc, pc, [&](const auto &g, const auto &) {
          static_for<kQ>([&](auto q) {
            if constexpr (is_diag_z(q) && Mesh) {
              constexpr int i = local_of(q);
              dz.template add<q>(g, acc_c[i], acc_p[i], nxt[i]);
            } else if constexpr (is_diag_z(q)) {
              constexpr int d1 = kCx[q] != 0 ? 0 : 1, s1 = kCx[q] + kCy[q];
              constexpr Real k = Real(0.5 * s1 * kCz[q]);
              constexpr int i = local_of(q);
              const Real bp_ = g.template at<q, Unit<d1>::x, Unit<d1>::y>();
              const Real bm_ = g.template at<q, -Unit<d1>::x, -Unit<d1>::y>();
              if constexpr (std::decay_t<decltype(g)>::use) {
                const Real dd = bp_ - bm_;
                acc_c[i] += dtal * (k * h * dd);
                acc_p[i] -= dtal * (Real(0.5 * s1) * dd - h * (bp_ + bm_));
                nxt[i] -= dtal * (k * h * dd);
              }
            }
          });
        });
      } else {
        face_below();
      }
    }
    if constexpr (G == 1) {
      // (every lane of an interior row: the corners come from the lanes beside)
      if (rows && has_cur) {
        const InPlaneCoef<Real, W, Mesh> xy(mc);
        gathered<Real, W>(pc, pc, [&](const auto &g, const auto &) {
          static_for<5>([&](auto q) {
            if constexpr (q >= 1 && Mesh) {
              xy.template axis<q>(g, acc_p[local_of(q)]);
            } else if constexpr (q >= 1) {
              constexpr int d = kCx[q] != 0 ? 0 : 1, s = kCx[q] + kCy[q];
              const Real bp_ = g.template at<q, Unit<d>::x, Unit<d>::y>();
              const Real bm_ = g.template at<q, -Unit<d>::x, -Unit<d>::y>();
              if constexpr (std::decay_t<decltype(g)>::use)
                acc_p[local_of(q)] -= dtal * (Real(0.5 * s) * (bp_ - bm_) - h * (bp_ + bm_));
            }
          });
        });
        auto diag_xy = [&](auto q, const auto &g) {
          if constexpr (Mesh) {
            xy.template diag<q>(g, acc_p[local_of(q)]);
            return;
          }
          constexpr int sx = kCx[q], sy = kCy[q];
          const Real p1 = g.template at<q, 1, 0>(), m1 = g.template at<q, -1, 0>();
          const Real p2 = g.template at<q, 0, 1>(), m2 = g.template at<q, 0, -1>();
          if constexpr (std::decay_t<decltype(g)>::use) {
            // the corners' mixed difference: the y-differences of the next and
            // the previous column, which are the lanes beside this one
            const Real gx = p1 - m1, gy = p2 - m2;
            const Real mix = from_next_lane(gy) - from_previous_lane(gy);
            constexpr Real hx = Real(0.5 * sx), hy = Real(0.5 * sy), hm = Real(0.5 * sx * sy);
            acc_p[local_of(q)] -= dtal * ((hx * gx + hy * gy) - h * ((p1 + m1) + (p2 + m2)) - hm * (h * mix));
          }
        };
        gathered<Real, W>(pc, pc, [&](const auto &g, const auto &) {
          diag_xy(std::integral_constant<int, 7>{}, g);
          diag_xy(std::integral_constant<int, 8>{}, g);
        });
        gathered<Real, W>(pc, pc, [&](const auto &g, const auto &) {
          diag_xy(std::integral_constant<int, 9>{}, g);
          diag_xy(std::integral_constant<int, 10>{}, g);
        });
      }
    }
    if (has_prev) {
      // the group's faces of centre p-1
      if constexpr (G == 0) {
        if constexpr (!kHelp) {
          if (rows) x_faces(pc, pc1, pc2, mc, FX, fx[0], fx[1]);
        }
      } else {
        // y-faces: halves of every row (halo rows too), joined after the barrier
        face_halves<1, Mesh>(mc, p_, h, pc, pc1, pc2, fx[0], fx[1]);
        static_for<4>([&](auto i) { RU[i * NT] = fx[0][i]; RD[i * NT] = fx[1][i]; });
      }
    }
    phase();
    if (p_ < z1) load_group<Real, G, O32>(ft, stride, n, col, p_ + 1, pf);
    if (p_ >= z0) {
      __syncthreads();
      if (inner) {
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        Real iw[2] = {Real(1), Real(1)};
        if constexpr (Mesh) static_for<2>([&](auto d) { iw[d] = mc.template col<d>(kMarchIw); });
        auto put_face = [&](const Real (&fm)[4], auto D, auto S) {
          face_equilibrium<D, Real>(fm, p, dtbe, [&](auto q, Real k, Real t) {
            if constexpr (group_of(q) == G) {
              if constexpr (Mesh)
                acc_c[local_of(q)] -= (S > 0 ? iw[D] : -iw[D]) * (k * t);
              else if constexpr (S > 0)
                acc_c[local_of(q)] -= k * t;
              else
                acc_c[local_of(q)] += k * t;
            }
          });
        };
        if constexpr (G == 0) {
          // the z-face between p-1 and p: upper face of centre p-1, lower of centre p
          Real zf[4];
          static_for<4>([&](auto i) { zf[i] = RZ[i * NT]; });
          Real iwc = Real(1), iwp = Real(1);
          if constexpr (Mesh) {
            iwc = mc.z(kMarchIw, p_ - 1);
            iwp = mc.z(kMarchIw, p_);
          }
          face_equilibrium<2, Real>(zf, p, dtbe, [&](auto q, Real k, Real t) {
            if constexpr (Mesh) {
              acc_c[local_of(q)] -= iwc * (k * t);
              acc_p[local_of(q)] += iwp * (k * t);
            } else {
              acc_c[local_of(q)] -= k * t;
              acc_p[local_of(q)] += k * t;
            }
          });
        }
        if (has_prev) {
          // equilibrium parts of the four x/y-faces of centre p-1 for this
          // group's populations: its own two faces and the other group's
          Real fo[2][4];
          if constexpr (G == 0) {
            static_for<4>([&](auto i) {
              fo[0][i] = RU[i * NT] + RD[i * NT + W];
              fo[1][i] = RU[i * NT - W] + RD[i * NT];
            });
            if constexpr (kHelp) static_for<4>([&](auto i) { fx[0][i] = FX[i * NT]; fx[1][i] = FX[i * NT - 1]; });
          } else {
            static_for<4>([&](auto i) { fo[0][i] = FX[i * NT]; fo[1][i] = FX[i * NT - 1]; });
            static_for<4>([&](auto i) {
              fx[0][i] += RD[i * NT + W];
              fx[1][i] = RU[i * NT - W] + fx[1][i];
            });
          }
          using Ip = std::integral_constant<int, 1>;
          using Im = std::integral_constant<int, -1>;
          if constexpr (G == 0) {
            put_face(fx[0], I0{}, Ip{}); put_face(fx[1], I0{}, Im{});
            put_face(fo[0], I1{}, Ip{}); put_face(fo[1], I1{}, Im{});
          } else {
            put_face(fo[0], I0{}, Ip{}); put_face(fo[1], I0{}, Im{});
            put_face(fx[0], I1{}, Ip{}); put_face(fx[1], I1{}, Im{});
          }
          const int cell = (p_ - 1) * n * n + col;
          double r = 0, ax = 0, ay = 0, az = 0;
          static_for<NG>([&](auto i) {
            constexpr int q = Group<G>::pop(i);
            *at_cell<O32>(out + (int64_t)q * stride, cell) = acc_c[i];  // plain stores, as in fused_tile
            const double x = (double)acc_c[i];
            r += x;
            if constexpr (kCx[q] != 0) ax += kCx[q] * x;
            if constexpr (kCy[q] != 0) ay += kCy[q] * x;
            if constexpr (kCz[q] != 0) az += kCz[q] * x;
          });
          add_sums(p_ - 1, r, ax, ay, az);
          if constexpr (G == 0) {
            SA[0] = Real(ax); SA[NT] = Real(ay); SA[2 * NT] = Real(az);
          } else {
            jb[0] = ax; jb[1] = ay; jb[2] = az;
          }
        }
      }
    }
    q2 ^= 1;
    q3 = q3 == 2 ? 0 : q3 + 1;
  }
  // A's part of the sums of the last stored cell
  __syncthreads();
  if constexpr (G == 1) {
    if (inner) {
      add_energy(z1 - 1);
    }
  }
  __syncthreads();
}

// Work-list kernel of the split march (see dugks_fused_kernel).
template <typename Real, int W, bool O32, bool Mesh>
__global__ __launch_bounds__(2 * Tile<W>::NT) void dugks_split_kernel(const BatchBox *__restrict__ boxes, int nbox,
                                                                      int total_items, PendingSums prev) {
  __shared__ Real L[kSplitValues * Tile<W>::NT + (Mesh ? kMeshValues<W> : 0)];
  // the extra block (see launch_lbe_step) is the first; the others keep their
  // distribution over the XCDs, one further on
  const int extra = prev.nblocks > 0, G = gridDim.x - extra, block = blockIdx.x - extra;
  if (block < 0) {
    add_pending<2 * Tile<W>::NT / 64>(prev.partials, prev.nblocks, prev.out, reinterpret_cast<double (*)[kNumSums]>(L));
    return;
  }
  for (int base = 0; base < total_items; base += G) {
    const int it = base + xcd_tile(block, G);
    if (it >= total_items) continue;
    const int b = find_batch_box(boxes, nbox, it);
    const BatchBox &d = boxes[b];
    const int local = it - d.item_begin;
    double v[kNumSums] = {0, 0, 0, 0, 0};
    const global_t<Real> *src = to_global(static_cast<const Real *>(d.f[d.cur]));
    global_t<Real> *dst = to_global(static_cast<Real *>(d.f[d.cur ^ 1]));
    const ItemPlanes ip(d, local);
    if (ip.left > 0) {
      const int bx = ip.tile % d.tiles_x, by = ip.tile / d.tiles_x, z1 = ip.z0 + ip.left;
      const Real *coef = static_cast<const Real *>(d.mesh_coef);
      auto march = [&](auto G, auto halo) {
        split_tile<Real, W, G, O32, Mesh, halo>(src, dst, d.sp, bx, by, ip.z0, z1, L, v, coef, d.mesh_width);
      };
      using std::integral_constant;
      constexpr int NT = Tile<W>::NT;
      const int t = threadIdx.x;
      const int halo_from = W == 32 ? NT - 64 : NT;
      if (t < halo_from)
        march(integral_constant<int, 0>{}, std::false_type{});
      else if (W == 32 ? t >= NT + 64 : t >= NT)
        march(integral_constant<int, 1>{}, std::false_type{});
      else if constexpr (W == 32) {
        if (t < NT)
          march(integral_constant<int, 0>{}, std::true_type{});
        else
          march(integral_constant<int, 1>{}, std::true_type{});
      }
    }
    write_block_partials<2 * Tile<W>::NT / 64>(v, d.partials, d.items, local, reinterpret_cast<double (*)[kNumSums]>(L));
    __syncthreads();
  }
}

// Writes table entries given by value (the launch carries them in its
// arguments), for callers that must not copy from host memory.
__global__ void store_table_kernel(BatchBox e0, BatchBox e1, BatchBox *__restrict__ dst) {
  if (threadIdx.x == 0) {
    dst[0] = e0;
    dst[1] = e1;
  }
}

}  // namespace fused

// Default tile: 32 x 8 columns in both precisions (rows of 256 B in FP64).
// FP64 (split march, 512 threads): 136 KB of LDS, one block per compute
// unit; FP32 (256 threads): 59 KB of LDS, two blocks per compute unit
// (two waves per SIMD).  The choice does not look at n: 16-wide tiles lose from
// 80^3 on (us a step, 32- and 16-wide: FP64 128^3 213 and 237, 80^3 49.8 and 50.7;
// FP32 128^3 120 and 139, 80^3 31.7 and 34.5) and below win at some sizes only (FP64
// 16^3 9.9 and 8.7, 40^3 17.1 and 14.6, 64^3 37.5 and 32.8, but 32^3 13.9 and 14.0,
// 48^3 17.4 and 18.0; FP32 40^3 14.9 and 12.2, 64^3 24.7 and 23.5, but 32^3 10.8 and
// 11.2, 48^3 15.0 and 15.8).  tile_width lets the caller choose; the populations
// are the same bits.
constexpr int fused_tile_width(int) { return 32; }

int fused_default_chunk(int n) { return n >= 128 ? 32 : (n >= 32 ? 16 : n); }

// Chunk items of a box (tiles x z-chunks) at tile width w and z-chunk
// `chunk` planes, and its tiling.
int fused_dugks_items(int n, int w, int chunk, int *tiles_x, int *tiles_y) {
  const int ix = w - 2, iy = 8 - 2;
  const int tx = (n + ix - 1) / ix;
  const int ty = (n + iy - 1) / iy;
  if (tiles_x) *tiles_x = tx;
  if (tiles_y) *tiles_y = ty;
  return tx * ty * ((n + chunk - 1) / chunk);
}

// Shortest z-chunk the balanced choice below takes for a launch that fills
// the device (shorter chunks re-read the two halo planes too often), and the
// most items a launch of shorter chunks has.
constexpr int kMinAutoChunk = 8;
constexpr int kMaxShortItems = 1024;

// Parts each chunk of a launch's last round is cut into: `chunks` items of
// `chunk` planes run in rounds of `slots` blocks; when at least one round
// is full and the t items left over fill at most half a round, each is cut
// into parts of ceil(chunk / min(slots / t, chunk)) planes, as many as that
// length needs (1: no cut).
static int tail_parts(int chunks, int slots, int chunk) {
  const int full = chunks / slots, t = chunks - full * slots;
  if (full < 1 || t == 0) return 1;
  const int m = std::min(slots / t, chunk);
  if (m < 2) return 1;
  const int len = (chunk + m - 1) / m;
  return (chunk + len - 1) / len;
}

static int fused_slots(int precision, int w);

FusedPlan fused_plan_for(const dhit_params &p, int slots) {
  FusedPlan f{};
  const int n = p.n;
  f.width = p.tile_width ? p.tile_width : fused_tile_width(p.precision);
  // an unresolved setting (0) is taken as kMinAutoChunk planes
  f.chunk = p.z_chunk > 0 ? p.z_chunk : (p.z_chunk < 0 ? -p.z_chunk : std::min(n, kMinAutoChunk));
  const int chunks = fused_dugks_items(n, f.width, f.chunk, &f.tiles_x, &f.tiles_y);
  f.items = f.tail_from = f.grid = chunks;
  f.tail_split = 1;
  if (p.z_chunk < 0 && slots > 0) {
    const int m = tail_parts(chunks, slots, f.chunk);
    if (m > 1 && slots % 8 == 0) {
      f.tail_from = chunks / slots * slots;
      f.tail_split = m;
      // per XCD: its eighth of the whole chunks, then its eighth of the parts
      const int pieces = (chunks - f.tail_from) * m;
      f.items = f.grid = 8 * (f.tail_from / 8 + (pieces + 7) / 8);
    }
  }
  return f;
}

FusedPlan fused_plan(const dhit_params &p) {
  return fused_plan_for(p, p.z_chunk < 0 ? fused_slots(p.precision, p.tile_width ? p.tile_width : fused_tile_width(p.precision)) : 0);
}

void fused_item_planes(const FusedPlan &f, int n, int item, int *tile, int *z0, int *planes) {
  BatchBox d;
  std::memset(&d, 0, sizeof(d));
  d.sp.n = n;
  d.tiles_x = f.tiles_x;
  d.tiles_y = f.tiles_y;
  d.nz_chunk = f.chunk;
  d.tail_from = f.tail_from;
  d.tail_split = f.tail_split;
  const fused::ItemPlanes ip(d, item);
  *tile = ip.tile;
  *z0 = ip.z0;
  *planes = ip.left;
}

// Work items of a box's fused launch (and its tiling).  With z_chunk = 0
// (not yet resolved) an upper bound for sizing buffers: twice the items of
// an automatic chunk of kMinAutoChunk planes and 8 (a cut last round adds at
// most a round's items, rounded up to a multiple of 8, to at least one full
// round), or what shorter chunks may have (kMaxShortItems, at most one item
// per tile-plane).
int fused_dugks_blocks(const dhit_params &p, int *width, int *tiles_x, int *tiles_y, int *nz_chunk) {
  const FusedPlan f = fused_plan(p);
  if (width) *width = f.width;
  if (tiles_x) *tiles_x = f.tiles_x;
  if (tiles_y) *tiles_y = f.tiles_y;
  if (nz_chunk) *nz_chunk = f.chunk;
  if (p.z_chunk != 0) return f.items;
  return std::max(2 * f.items + 8, std::min(f.tiles_x * f.tiles_y * p.n, kMaxShortItems));
}

// FP64 tiles use the split-population march (two thread groups per
// column), FP32 tiles one thread per column.
template <typename Real>
constexpr bool kSplit = sizeof(Real) == 8;

template <typename Real, int W, bool O32, bool Mesh>
static void list_launch(hipStream_t s, const BatchBox *d_boxes, int nbox, int total_items, int grid,
                        const PendingSums &prev) {
  grid = (grid + 7) / 8 * 8;  // the XCD numbering of work items needs a multiple of 8
  if constexpr (kSplit<Real>)
    hipLaunchKernelGGL((fused::dugks_split_kernel<Real, W, O32, Mesh>), dim3(grid + (prev.nblocks > 0)), dim3(2 * fused::Tile<W>::NT), 0, s,
                       d_boxes, nbox, total_items, prev);
  else
    hipLaunchKernelGGL((fused::dugks_fused_kernel<Real, W, O32, Mesh>), dim3(grid + (prev.nblocks > 0)), dim3(fused::Tile<W>::NT), 0, s,
                       d_boxes, nbox, total_items, prev);
}

// Whether 32-bit byte offsets reach every cell of one population array of
// an n^3 box (n^3 elements of `elem` bytes below 4 GB).
static bool offsets32(int max_n, int precision) {
  const uint64_t elem = precision == DHIT_FP64 ? 8 : 4;
  return (uint64_t)max_n * max_n * max_n * elem < (uint64_t(1) << 32);
}

template <typename Real, bool Mesh>
static void list_launch(hipStream_t s, int w, bool o32, const BatchBox *d_boxes, int nbox, int total_items, int grid,
                        const PendingSums &prev) {
  if (w == 16)
    o32 ? list_launch<Real, 16, true, Mesh>(s, d_boxes, nbox, total_items, grid, prev)
        : list_launch<Real, 16, false, Mesh>(s, d_boxes, nbox, total_items, grid, prev);
  else
    o32 ? list_launch<Real, 32, true, Mesh>(s, d_boxes, nbox, total_items, grid, prev)
        : list_launch<Real, 32, false, Mesh>(s, d_boxes, nbox, total_items, grid, prev);
}

void launch_dugks_batch(hipStream_t s, int precision, int w, int max_n, const BatchBox *d_boxes, int nbox,
                        int total_items, int grid, bool mesh, const PendingSums &prev) {
  if (w != 16 && w != 32) throw Error(DHIT_EINVAL, "fused DUGKS tile width must be 16 or 32");
  const bool o32 = offsets32(max_n, precision);
  if (precision == DHIT_FP64)
    mesh ? list_launch<double, true>(s, w, o32, d_boxes, nbox, total_items, grid, prev)
         : list_launch<double, false>(s, w, o32, d_boxes, nbox, total_items, grid, prev);
  else
    mesh ? list_launch<float, true>(s, w, o32, d_boxes, nbox, total_items, grid, prev)
         : list_launch<float, false>(s, w, o32, d_boxes, nbox, total_items, grid, prev);
  DHIT_HIP(hipGetLastError());
}

// The two one-box tables of a box: entry c steps from f[c] to f[1 - c].
void fused_table_entries(const dhit_box &b, BatchBox (&e)[2]) {
  const FusedPlan f = fused_plan(b.p);
  for (int c = 0; c < 2; ++c) {
    std::memset(&e[c], 0, sizeof(BatchBox));
    e[c].f[0] = b.f[0];
    e[c].f[1] = b.f[1];
    e[c].sp = b.sp;
    e[c].ncell = (int)b.ncell;
    e[c].item_begin = 0;
    e[c].items = f.items;
    e[c].tiles_x = f.tiles_x;
    e[c].tiles_y = f.tiles_y;
    e[c].nz_chunk = f.chunk;
    e[c].tail_from = f.tail_from;
    e[c].tail_split = f.tail_split;
    e[c].partials = b.partials + (size_t)c * 5 * b.max_blocks;
    e[c].hist = b.hist;
    e[c].cur = c;
    e[c].mesh_width = b.mesh;
    e[c].mesh_coef = b.mesh ? b.mesh + 3 * b.n : nullptr;
  }
}

void launch_store_table(hipStream_t s, const BatchBox (&e)[2], BatchBox *dst) {
  hipLaunchKernelGGL(fused::store_table_kernel, dim3(1), dim3(64), 0, s, e[0], e[1], dst);
  DHIT_HIP(hipGetLastError());
}

static void fused_step(dhit_box &b, const void *src, void *dst, double *sums_out, bool defer, PendingSums *pend) {
  if (!b.step_table) throw Error(DHIT_EINVAL, "box has no fused-step table");
  int entry;
  if (src == b.f[0] && dst == b.f[1]) entry = 0;
  else if (src == b.f[1] && dst == b.f[0]) entry = 1;
  else throw Error(DHIT_EINVAL, "fused DUGKS step between buffers that are not the box's");
  const FusedPlan f = fused_plan(b.p);
  {
    TimedLaunch t(b, DHIT_K_DUGKS_FUSED);
    launch_dugks_batch(b.stream, b.p.precision, f.width, b.n, b.step_table + entry, 1, f.items, f.grid,
                       b.mesh != nullptr, pend ? *pend : PendingSums{});
    t.done();
  }
  finish_step(b, b.partials + (size_t)entry * 5 * b.max_blocks, f.items, sums_out, defer, pend);
}

int fused_tile_width_of(int precision) { return fused_tile_width(precision); }

// Blocks of the fused kernel of this precision and tile width that one
// compute unit holds at once (registers and LDS decide: one for the FP64
// split march, two for FP32 at width 32).
static int fused_resident_blocks(int precision, int w) {
  int nb = 0;
  hipError_t e;
  if (precision == DHIT_FP64)
    e = w == 16 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                      &nb, reinterpret_cast<const void *>(&fused::dugks_split_kernel<double, 16, true, false>), 2 * fused::Tile<16>::NT, 0)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                      &nb, reinterpret_cast<const void *>(&fused::dugks_split_kernel<double, 32, true, false>), 2 * fused::Tile<32>::NT, 0);
  else
    e = w == 16 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                      &nb, reinterpret_cast<const void *>(&fused::dugks_fused_kernel<float, 16, true, false>), fused::Tile<16>::NT, 0)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                      &nb, reinterpret_cast<const void *>(&fused::dugks_fused_kernel<float, 32, true, false>), fused::Tile<32>::NT, 0);
  return e == hipSuccess && nb > 0 ? nb : 1;
}

int fused_resident_blocks_of(int precision, int w) { return fused_resident_blocks(precision, w); }

// Blocks of the fused kernel that the current device holds at once
// (compute units x resident blocks), kept per device.
static int fused_slots(int precision, int w) {
  int dev = 0;
  DHIT_HIP(hipGetDevice(&dev));
  static std::mutex mu;
  static std::map<std::array<int, 3>, int> known;
  std::lock_guard<std::mutex> lock(mu);
  const std::array<int, 3> key{dev, precision, w};
  const auto it = known.find(key);
  if (it != known.end()) return it->second;
  int cus = 0;
  DHIT_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const int slots = std::max(cus, 1) * fused_resident_blocks(precision, w);
  known[key] = slots;
  return slots;
}

// z-chunk that balances a launch.  Its blocks run in rounds of `slots`
// (compute units x resident blocks); a block marching c planes costs about
// c + 2 plane iterations (the two halo planes), so a launch of K chunk items
// costs about ceil(K / slots) (c + 2); with its last, partly filled round
// cut into m parts per chunk (tail_parts) it costs floor(K / slots) (c + 2)
// + ceil(c / m) + 2.  Among the chunks ceil(n / k) of at least kMinAutoChunk
// planes (or n, if smaller), each with and without the cut, the cheapest is
// taken (the cut one is returned as -c), the longest and the uncut of equal
// ones.  At 256^3 in FP64 (1 block per unit, 387 column tiles): chunks of
// 37 planes cost 11 rounds of 39 iterations (the last round 58% full: 429);
// chunks of 128 planes, 3 full rounds of 130 and 6 chunks left over that
// are cut into 32 parts of 4 planes, 396.
// A small box does not fill one round even with chunks of kMinAutoChunk
// planes; its launch lasts as long as one block's march, so the shorter
// chunks whose items still fit one round are taken into the choice: at 32^3
// (12 column tiles) FP64 chunks of 2 planes (192 items) ran 22.6 us a step
// (13.8 with the march's later changes) against 44.6 with 8 planes (48 items), at 48^3 3 planes (256 items) 26.9
// against 42.6, at 64^3 in FP32 (512 slots) 6 planes 37.0 against 42.9.  Two
// rounds of the shortest chunks lose again (32^3, 1 plane, 384 items: 30.7).
int fused_balanced_chunk(int n, int tiles_xy, int slots) {
  const int cmin = std::min(n, kMinAutoChunk);
  const int one_round = std::min(slots, kMaxShortItems);
  int best = n;
  int64_t best_cost = INT64_MAX;
  for (int c = n; c >= 1; --c) {
    const int k = (n + c - 1) / c;
    if ((n + k - 1) / k != c) continue;  // k chunks can be shorter
    const int64_t blocks = (int64_t)tiles_xy * k;
    if (c < cmin && blocks > one_round) break;
    const int64_t cost = (blocks + slots - 1) / slots * (c + 2);
    if (cost < best_cost) {
      best_cost = cost;
      best = c;
    }
    if (blocks <= INT32_MAX) {
      const int m = tail_parts((int)blocks, slots, c);
      const int64_t cut = blocks / slots * (c + 2) + (c + m - 1) / m + 2;
      if (m > 1 && cut < best_cost) {
        best_cost = cut;
        best = -c;
      }
    }
  }
  return best;
}

// Default z-chunk of a box on the current device.
int fused_auto_chunk(const dhit_params &p) {
  dhit_params q = p;
  q.z_chunk = 0;
  const FusedPlan f = fused_plan(q);
  return fused_balanced_chunk(p.n, f.tiles_x * f.tiles_y, fused_slots(p.precision, f.width));
}

void launch_dugks_fused(dhit_box &b, const void *src, void *dst, double *sums_out, bool defer, PendingSums *pend) {
  fused_step(b, src, dst, sums_out, defer, pend);
}

}  // namespace dhit
