// Energy spectrum and velocity-derivative statistics of a box (Sec. III):
//   u = j/rho0 -> u_hat = DFT(u)/n^3 (hipFFT, real-to-complex, batch of 3)
//   -> shell binning of 1/2 |u_hat|^2 and of |kappa|^2 1/2 |u_hat|^2
//      (exact integer sums, so E(k) is the same bits on every run)
//   -> spectral derivatives i kappa_a u_hat_a (inverse transforms)
//   -> <(d_a u_a)^m>, m = 2, 3, 4 -> K, eps, S, F.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "device_common.hpp"
#include "runtime.hpp"

namespace dhit {

struct SpectrumWork {
  int n = 0;
  int nshell = 0;
  int64_t nhalf = 0;  // modes of one real-to-complex transform, n*n*(n/2+1)
  double *u = nullptr;                   // three fields (room for three half spectra, see gradient_compute)
  hipfftDoubleComplex *uh = nullptr;     // their transforms
  hipfftDoubleComplex *tmp = nullptr;    // one more half spectrum (pressure; made when first needed)
  // what energy_spectrum brings to the host, in one piece: the shells' digit
  // sums [2][kShellParts][nshell] of E and kappa^2-weighted E, the power sums
  // of the three derivatives [3][5] (doubles), and a word that is set when a
  // shell term is out of range or not finite
  unsigned long long *result = nullptr;
  double *partials = nullptr;  // [3][5][kPowerBlocks]
  // real-to-complex and complex-to-real of three fields, for everything done
  // here (with a plan of its own for one field, the first spectrum after a
  // pressure took 2.4 instead of 0.12 ms at 64^3), and the work area they share: a
  // box's transforms run one after the other (with an area each, and one more
  // plan, odd sizes took 280 instead of 152 bytes per cell)
  hipfftHandle fwd = 0, inv = 0;
  void *area = nullptr;
};
constexpr int kPowerBlocks = 1024;

#define DHIT_FFT(expr)                                                                               \
  do {                                                                                               \
    hipfftResult r_ = (expr);                                                                        \
    if (r_ != HIPFFT_SUCCESS) throw ::dhit::Error(DHIT_EDEVICE, std::string(#expr " failed, code ") + std::to_string((int)r_)); \
  } while (0)

// Signed integer wavenumber of FFT index i (numpy fftfreq order).
__device__ __forceinline__ int signed_k(int i, int n) { return (i <= (n - 1) / 2) ? i : i - n; }

// Shell sums are accumulated exactly, so that E(k) does not depend on the
// order in which threads add their modes: a term e (>= 0) is taken as the
// integer floor(e 2^kShellFrac), split into three kShellDigit-bit digits,
// and each digit is summed with integer atomic adds (associative, so the
// order does not matter).  The host joins the digits in 128-bit integers
// and rounds once.  Terms below 2^-kShellFrac (3e-27) in absolute value are
// truncated; a term of 2^8 or more (or not finite; velocities of order one
// in lattice units already mean a blown-up run) raises the overflow flag.
// With 34-bit digits a digit sum stays below 2^64, and the joined value
// below 2^126, for up to 2^30 modes (n <= 1024).
constexpr int kShellFrac = 88, kShellDigit = 34, kShellParts = 3;

__device__ __forceinline__ void shell_digits(double e, unsigned long long (&d)[kShellParts], bool &over) {
  if (!(e >= 0.0 && e < 256.0)) {
    over = true;
    d[0] = d[1] = d[2] = 0;
    return;
  }
  const double x = e * 0x1p88;                 // exact: a power of two, x < 2^96
  const double hi = floor(x * 0x1p-68);        // < 2^28
  const double r = x - hi * 0x1p68;            // exact: a multiple of ulp(x) below 2^68
  const double mid = floor(r * 0x1p-34);       // < 2^34
  const double lo = floor(r - mid * 0x1p34);   // < 2^34; drops bits below 2^-88 of e
  d[2] = (unsigned long long)hi;
  d[1] = (unsigned long long)mid;
  d[0] = (unsigned long long)lo;
}

// Wavenumber of a derivative: the Nyquist component is dropped.
__device__ __forceinline__ int derivative_k(int k, int n) { return (2 * k == n || 2 * k == -n) ? 0 : k; }

// One thread per mode of the half spectrum; block histogram of the digits
// in LDS, then one integer atomic add per digit, shell and block.  Modes
// 0 < kx < n/2 stand for their Hermitian partners too (weight 2).
// shells: [2][kShellParts][nshell] digit sums of E and of kappa^2 E.  The modes
// are then replaced by those of d_a u_a (i kappa_a u_hat_a, each thread its
// own), so that the three derivatives go back in one batched transform
// (three passes of deriv, transform and sums took 160 us of a 128^3
// spectrum's 330).
__global__ __launch_bounds__(256) void bin_kernel(hipfftDoubleComplex *__restrict__ uh, int n, int64_t nhalf,
                                                  int nshell, double inv_n6, unsigned long long *__restrict__ shells,
                                                  unsigned long long *__restrict__ overflow) {
  extern __shared__ unsigned long long hist[];  // [2][kShellParts][nshell]
  const int nh = 2 * kShellParts * nshell;
  for (int i = threadIdx.x; i < nh; i += blockDim.x) hist[i] = 0ull;
  __syncthreads();
  const int nxh = n / 2 + 1;
  const double kfac = 2.0 * M_PI / n;
  bool over = false;
  for (int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; m < nhalf; m += (int64_t)gridDim.x * blockDim.x) {
    const int kxh = (int)(m % nxh);
    const int64_t r = m / nxh;
    const int iy = (int)(r % n), iz = (int)(r / n);
    const int kx = kxh, ky = signed_k(iy, n), kz = signed_k(iz, n);
    const int kd[3] = {derivative_k(kx, n), derivative_k(ky, n), derivative_k(kz, n)};
    double e = 0.0;
    static_for<3>([&](auto c) {
      const hipfftDoubleComplex v = uh[(int64_t)c * nhalf + m];
      e += v.x * v.x + v.y * v.y;
      const double kap = kfac * kd[c];
      uh[(int64_t)c * nhalf + m] = make_double2(-kap * v.y, kap * v.x);
    });
    const bool self = (kx == 0) || (2 * kx == n);
    e *= 0.5 * inv_n6 * (self ? 1.0 : 2.0);
    const int k2 = kx * kx + ky * ky + kz * kz;
    const int s = (int)rint(sqrt((double)k2));
    unsigned long long d[kShellParts], dk[kShellParts];
    shell_digits(e, d, over);
    shell_digits(kfac * kfac * (double)k2 * e, dk, over);
    for (int j = 0; j < kShellParts; ++j) {
      if (d[j]) atomicAdd(&hist[j * nshell + s], d[j]);
      if (dk[j]) atomicAdd(&hist[(kShellParts + j) * nshell + s], dk[j]);
    }
  }
  if (over) atomicOr(overflow, 1ull);
  __syncthreads();
  for (int i = threadIdx.x; i < nh; i += blockDim.x)
    if (hist[i] != 0ull) atomicAdd(&shells[i], hist[i]);
}

// u_hat -> spectrum of the vorticity, in place and scaled by `scale`:
// component a becomes scale i (kappa_b u_hat_c - kappa_c u_hat_b), (a, b, c)
// cyclic, the Nyquist wavenumber of each derivative direction dropped.
__global__ __launch_bounds__(256) void curl_kernel(hipfftDoubleComplex *__restrict__ uh, int n, int64_t nhalf,
                                                   double scale) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= nhalf) return;
  const int nxh = n / 2 + 1;
  const int64_t r = m / nxh;
  const double kfac = 2.0 * M_PI / n;
  const double k[3] = {kfac * derivative_k((int)(m % nxh), n), kfac * derivative_k(signed_k((int)(r % n), n), n),
                       kfac * derivative_k(signed_k((int)(r / n), n), n)};
  hipfftDoubleComplex v[3];
  static_for<3>([&](auto c) { v[c] = uh[(int64_t)c * nhalf + m]; });
  static_for<3>([&](auto a) {
    constexpr int b = (a + 1) % 3, c = (a + 2) % 3;
    const double re = k[b] * v[c].x - k[c] * v[b].x, im = k[b] * v[c].y - k[c] * v[b].y;
    uh[(int64_t)a * nhalf + m] = make_double2(-im * scale, re * scale);
  });
}

// Spectrum of the velocity-gradient component d_a u_b, scaled by `scale`:
// out = scale i kappa_a u_hat_b on the half spectrum, the Nyquist
// wavenumber of the derivative direction set to zero.
__global__ __launch_bounds__(256) void gradient_kernel(const hipfftDoubleComplex *__restrict__ uhb,
                                                       hipfftDoubleComplex *__restrict__ out, int n, int64_t nhalf,
                                                       int a, double scale) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= nhalf) return;
  const int nxh = n / 2 + 1;
  const int64_t r = m / nxh;
  const int k = a == 0 ? (int)(m % nxh) : (a == 1 ? signed_k((int)(r % n), n) : signed_k((int)(r / n), n));
  const double kap = 2.0 * M_PI / n * derivative_k(k, n) * scale;
  const hipfftDoubleComplex v = uhb[m];
  hipfftDoubleComplex o;
  o.x = -kap * v.y;
  o.y = kap * v.x;
  out[m] = o;
}

// Products of velocity components for the pressure source: set 0 gives
// (u u, v v, w w), set 1 gives (u v, v w, w u), into three fields of out.
__global__ __launch_bounds__(256) void products_kernel(const double *__restrict__ u, double *__restrict__ out,
                                                       int64_t ncell, int set) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ncell) return;
  const double a = u[i], b = u[ncell + i], c = u[2 * ncell + i];
  if (set == 0) {
    out[i] = a * a;
    out[ncell + i] = b * b;
    out[2 * ncell + i] = c * c;
  } else {
    out[i] = a * b;
    out[ncell + i] = b * c;
    out[2 * ncell + i] = c * a;
  }
}

// acc (half spectrum) (=, set 0) or (+=, set 1) sum over the three
// transformed products ph of their weights: set 0 k_a^2 for (aa),
// set 1 2 k_a k_b for (ab) = (xy, yz, zx); k the integer wavevector with the
// Nyquist component of each derivative factor dropped.
__global__ __launch_bounds__(256) void pressure_source_kernel(const hipfftDoubleComplex *__restrict__ ph,
                                                              hipfftDoubleComplex *__restrict__ acc, int n,
                                                              int64_t nhalf, int set) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= nhalf) return;
  const int nxh = n / 2 + 1;
  const int64_t r = m / nxh;
  const int k[3] = {derivative_k((int)(m % nxh), n), derivative_k(signed_k((int)(r % n), n), n),
                    derivative_k(signed_k((int)(r / n), n), n)};
  double re = 0.0, im = 0.0;
  for (int c = 0; c < 3; ++c) {
    const double w = set == 0 ? (double)k[c] * k[c] : 2.0 * (double)k[c] * k[(c + 1) % 3];
    const hipfftDoubleComplex v = ph[(int64_t)c * nhalf + m];
    re += w * v.x;
    im += w * v.y;
  }
  if (set == 0) {
    acc[m].x = re;
    acc[m].y = im;
  } else {
    acc[m].x += re;
    acc[m].y += im;
  }
}

// out = scale acc / |k|^2 (full integer |k|^2; the k = 0 mode set to 0).
__global__ __launch_bounds__(256) void inverse_laplacian_kernel(const hipfftDoubleComplex *__restrict__ acc,
                                                                hipfftDoubleComplex *__restrict__ out, int n,
                                                                int64_t nhalf, double scale) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= nhalf) return;
  const int nxh = n / 2 + 1;
  const int64_t r = m / nxh;
  const int kx = (int)(m % nxh), ky = signed_k((int)(r % n), n), kz = signed_k((int)(r / n), n);
  const int k2 = kx * kx + ky * ky + kz * kz;
  const double f = k2 == 0 ? 0.0 : scale / (double)k2;
  out[m] = make_double2(acc[m].x * f, acc[m].y * f);
}

// Sums of d^2, d^3, d^4 of three real fields scaled by `scale` (field
// blockIdx.y): partials [3][5][gridDim.x].
__global__ __launch_bounds__(kBlock) void power_sums_kernel(const double *__restrict__ d, int64_t ncell, double scale,
                                                            double *__restrict__ partials) {
  double v[kNumSums] = {0, 0, 0, 0, 0};
  d += (int64_t)blockIdx.y * ncell;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < ncell; i += (int64_t)gridDim.x * kBlock) {
    const double x = d[i] * scale;
    const double x2 = x * x;
    v[0] += x2;
    v[1] += x2 * x;
    v[2] += x2 * x2;
  }
  write_block_partials(v, partials + (int64_t)blockIdx.y * kNumSums * gridDim.x, gridDim.x, blockIdx.x);
}
// Adds them up: block a the partials of field a, into out[a][5].
__global__ __launch_bounds__(kBlock) void power_totals_kernel(const double *__restrict__ partials, int nblocks,
                                                              double *__restrict__ out) {
  __shared__ double smem[kWaves][kNumSums];
  double v[kNumSums] = {0, 0, 0, 0, 0};
  const double *p = partials + (int64_t)blockIdx.x * kNumSums * nblocks;
  for (int b = threadIdx.x; b < nblocks; b += kBlock)
    static_for<kNumSums>([&](auto i) { v[i] += p[(int64_t)i * nblocks + b]; });
  const double t = block_sum5<kWaves>(v, smem);
  if (threadIdx.x < kNumSums) out[blockIdx.x * kNumSums + threadIdx.x] = t;
}

// Words of SpectrumWork::result.
static size_t shell_words(int nshell) { return 2 * kShellParts * (size_t)nshell; }
static size_t result_words(int nshell) { return shell_words(nshell) + 15 + 1; }

// Makes one of the two plans without a work area; *need = the bytes it needs.
static void make_plan(hipfftHandle *h, int n, bool forward, size_t *need) {
  int dims[3] = {n, n, n};
  const int ncell = n * n * n, nhalf = n * n * (n / 2 + 1);
  hipfftHandle p = 0;
  DHIT_FFT(hipfftCreate(&p));
  *h = p;
  DHIT_FFT(hipfftSetAutoAllocation(p, 0));
  DHIT_FFT(forward ? hipfftMakePlanMany(p, 3, dims, nullptr, 1, ncell, nullptr, 1, nhalf, HIPFFT_D2Z, 3, need)
                   : hipfftMakePlanMany(p, 3, dims, nullptr, 1, nhalf, nullptr, 1, ncell, HIPFFT_Z2D, 3, need));
}

static void work_free(SpectrumWork *w) {
  if (w->fwd) hipfftDestroy(w->fwd);
  if (w->inv) hipfftDestroy(w->inv);
  if (w->area) (void)hipFree(w->area);
  if (w->u) (void)hipFree(w->u);
  if (w->uh) (void)hipFree(w->uh);
  if (w->tmp) (void)hipFree(w->tmp);
  if (w->result) (void)hipFree(w->result);
  if (w->partials) (void)hipFree(w->partials);
  delete w;
}

template <typename T>
static void allocate(T **p, size_t bytes) {
  if (hipMalloc(p, bytes) == hipSuccess) return;
  *p = nullptr;
  throw Error(DHIT_ENOMEM, "cannot allocate spectrum work space");
}

static int shells_of(int n) { return (int)std::floor(std::sqrt(3.0) * (n / 2 + 1)) + 2; }

static void ensure_work(dhit_box &b) {
  if (!b.spec) {
    SpectrumWork *w = new SpectrumWork();
    try {
      const int n = b.n;
      w->n = n;
      w->nhalf = (int64_t)n * n * (n / 2 + 1);
      w->nshell = shells_of(n);
      const size_t three = 3 * (size_t)w->nhalf * sizeof(hipfftDoubleComplex);
      allocate(&w->u, three);
      allocate(&w->uh, three);
      allocate(&w->result, result_words(w->nshell) * sizeof(unsigned long long));
      allocate(&w->partials, 3 * 5 * kPowerBlocks * sizeof(double));
      size_t need_f = 0, need_i = 0;
      make_plan(&w->fwd, n, true, &need_f);
      make_plan(&w->inv, n, false, &need_i);
      const size_t need = std::max(need_f, need_i);
      if (need > 0) {
        allocate(&w->area, need);
        DHIT_FFT(hipfftSetWorkArea(w->fwd, w->area));
        DHIT_FFT(hipfftSetWorkArea(w->inv, w->area));
      }
    } catch (...) {
      work_free(w);
      throw;
    }
    b.spec = w;
  }
  DHIT_FFT(hipfftSetStream(b.spec->fwd, b.stream));
  DHIT_FFT(hipfftSetStream(b.spec->inv, b.stream));
}

// Device bytes of the spectrum work space of an n^3 box: the arrays of
// ensure_work and pressure_compute and the plans' work area (the plans are made
// here to ask; nothing is allocated).
int64_t spectrum_work_bytes(int n) {
  const int64_t nhalf = (int64_t)n * n * (n / 2 + 1);
  size_t need[2] = {0, 0};
  for (int forward = 0; forward < 2; ++forward) {
    hipfftHandle h = 0;
    try {
      make_plan(&h, n, forward != 0, &need[forward]);
    } catch (...) {
      if (h) hipfftDestroy(h);
      throw;
    }
    hipfftDestroy(h);
  }
  return 7 * nhalf * (int64_t)sizeof(hipfftDoubleComplex) +
         (int64_t)(result_words(shells_of(n)) * sizeof(unsigned long long)) +
         3 * 5 * kPowerBlocks * (int64_t)sizeof(double) + (int64_t)std::max(need[0], need[1]);
}

void spectrum_free(dhit_box &b) {
  if (b.spec) work_free(b.spec);
  b.spec = nullptr;
}

void spectrum_compute(dhit_box &b, double *E_host, int kmax, double *stats_host) {
  ensure_work(b);
  SpectrumWork &w = *b.spec;
  const int n = b.n;
  launch_velocity(b, b.f[b.cur], w.u);
  DHIT_FFT(hipfftExecD2Z(w.fwd, w.u, w.uh));
  const size_t shells = shell_words(w.nshell), words = result_words(w.nshell);
  double *dstats = reinterpret_cast<double *>(w.result + shells);
  DHIT_HIP(hipMemsetAsync(w.result, 0, words * sizeof(unsigned long long), b.stream));
  const double inv_n3 = 1.0 / ((double)n * n * n);
  {
    const int blocks = (int)std::min<int64_t>((w.nhalf + 255) / 256, 2048);
    hipLaunchKernelGGL(bin_kernel, dim3(blocks), dim3(256), shells * sizeof(unsigned long long), b.stream, w.uh, n,
                       w.nhalf, w.nshell, inv_n3 * inv_n3, w.result, w.result + words - 1);
    DHIT_HIP(hipGetLastError());
  }
  DHIT_FFT(hipfftExecZ2D(w.inv, w.uh, w.u));
  const int rb = (int)std::min<int64_t>((b.ncell + kBlock - 1) / kBlock, kPowerBlocks);
  hipLaunchKernelGGL(power_sums_kernel, dim3(rb, 3), dim3(kBlock), 0, b.stream, w.u, b.ncell, inv_n3, w.partials);
  DHIT_HIP(hipGetLastError());
  {
    TimedLaunch t(b, DHIT_K_FINALIZE);
    hipLaunchKernelGGL(power_totals_kernel, dim3(3), dim3(kBlock), 0, b.stream, w.partials, rb, dstats);
    DHIT_HIP(hipGetLastError());
    t.done();
  }
  std::vector<unsigned long long> dig(words);
  DHIT_HIP(hipMemcpyAsync(dig.data(), w.result, words * sizeof(unsigned long long), hipMemcpyDeviceToHost, b.stream));
  DHIT_HIP(hipStreamSynchronize(b.stream));
  double ds[15];
  std::memcpy(ds, dig.data() + shells, sizeof(ds));
  if (dig[words - 1]) throw Error(DHIT_ENONFINITE, "velocity field is not finite (or a spectral term exceeds 2^8)");
  // join the digits of each shell: sum_j digit_j 2^(34 j), then times 2^-88
  std::vector<double> sh(2 * w.nshell);
  for (int q = 0; q < 2; ++q)
    for (int k = 0; k < w.nshell; ++k) {
      unsigned __int128 v = 0;
      for (int j = kShellParts - 1; j >= 0; --j)
        v = (v << kShellDigit) + (unsigned __int128)dig[((size_t)q * kShellParts + j) * w.nshell + k];
      sh[(size_t)q * w.nshell + k] = std::ldexp((double)v, -kShellFrac);
    }
  for (int k = 0; k <= kmax; ++k) E_host[k] = k < w.nshell ? sh[k] : 0.0;
  if (stats_host) {
    double K = 0, D = 0;
    for (int k = 0; k < w.nshell; ++k) {
      K += sh[k];
      D += sh[w.nshell + k];
    }
    double num3 = 0, den3 = 0, num4 = 0, den4 = 0;
    for (int a = 0; a < 3; ++a) {
      const double m2 = ds[5 * a + 0] * inv_n3, m3 = ds[5 * a + 1] * inv_n3, m4 = ds[5 * a + 2] * inv_n3;
      num3 += m3;
      num4 += m4;
      den3 += std::pow(m2, 1.5);
      den4 += m2 * m2;
    }
    stats_host[0] = K;
    stats_host[1] = 2.0 * b.p.nu * D;
    stats_host[2] = den3 > 0 ? num3 / den3 : 0.0;
    stats_host[3] = den4 > 0 ? num4 / den4 : 0.0;
  }
  for (int i = 0; i < 15; ++i)
    if (!std::isfinite(ds[i])) throw Error(DHIT_ENONFINITE, "velocity field is not finite");
}

void pressure_compute(dhit_box &b, const double *u_host, double *drho_host) {
  ensure_work(b);
  SpectrumWork &w = *b.spec;
  const int n = b.n;
  if (!w.tmp) allocate(&w.tmp, w.nhalf * sizeof(hipfftDoubleComplex));
  double *du = nullptr;
  if (hipMalloc(&du, 3 * b.ncell * sizeof(double)) != hipSuccess)
    throw Error(DHIT_ENOMEM, "cannot allocate the velocity upload buffer");
  try {
    DHIT_HIP(hipMemcpyAsync(du, u_host, 3 * b.ncell * sizeof(double), hipMemcpyHostToDevice, b.stream));
    const int cb = (int)((b.ncell + 255) / 256), mb = (int)((w.nhalf + 255) / 256);
    for (int set = 0; set < 2; ++set) {
      hipLaunchKernelGGL(products_kernel, dim3(cb), dim3(256), 0, b.stream, du, w.u, (int64_t)b.ncell, set);
      DHIT_HIP(hipGetLastError());
      DHIT_FFT(hipfftExecD2Z(w.fwd, w.u, w.uh));
      hipLaunchKernelGGL(pressure_source_kernel, dim3(mb), dim3(256), 0, b.stream, w.uh, w.tmp, n, w.nhalf, set);
      DHIT_HIP(hipGetLastError());
    }
    // p_hat = -rho0 rhs / |k|^2; drho = 3 p; both transforms are unnormalised
    const double scale = -3.0 * b.p.rho0 / ((double)n * n * n);
    hipLaunchKernelGGL(inverse_laplacian_kernel, dim3(mb), dim3(256), 0, b.stream, w.tmp, w.uh, n, w.nhalf, scale);
    DHIT_HIP(hipGetLastError());
    // the first of the three fields; the other two are what is left in uh (their
    // transforms take 1% of the call's time)
    DHIT_FFT(hipfftExecZ2D(w.inv, w.uh, w.u));
    copy_to_host({{drho_host, w.u, b.ncell * sizeof(double)}}, b.stream);
  } catch (...) {
    (void)hipStreamSynchronize(b.stream);
    (void)hipFree(du);
    throw;
  }
  (void)hipFree(du);
}

void gradient_compute(dhit_box &b, const double *d_u, double *d_grad) {
  ensure_work(b);
  SpectrumWork &w = *b.spec;
  const int n = b.n;
  DHIT_HIP(hipMemcpyAsync(w.u, d_u, 3 * b.ncell * sizeof(double), hipMemcpyDeviceToDevice, b.stream));
  DHIT_FFT(hipfftExecD2Z(w.fwd, w.u, w.uh));
  const double inv_n3 = 1.0 / ((double)n * n * n);  // both transforms are unnormalised
  const int blocks = (int)((w.nhalf + 255) / 256);
  // the three components' derivatives along a at a time: their spectra take the
  // place of u, which has been transformed
  hipfftDoubleComplex *du = reinterpret_cast<hipfftDoubleComplex *>(w.u);
  for (int a = 0; a < 3; ++a) {
    for (int c = 0; c < 3; ++c) {
      hipLaunchKernelGGL(gradient_kernel, dim3(blocks), dim3(256), 0, b.stream, w.uh + (int64_t)c * w.nhalf,
                         du + (int64_t)c * w.nhalf, n, w.nhalf, a, inv_n3);
      DHIT_HIP(hipGetLastError());
    }
    DHIT_FFT(hipfftExecZ2D(w.inv, du, d_grad + (int64_t)3 * a * b.ncell));
  }
}

void vorticity_compute(dhit_box &b, double *omega_host) {
  ensure_work(b);
  SpectrumWork &w = *b.spec;
  const int n = b.n;
  launch_velocity(b, b.f[b.cur], w.u);
  DHIT_FFT(hipfftExecD2Z(w.fwd, w.u, w.uh));
  const double inv_n3 = 1.0 / ((double)n * n * n);  // both transforms are unnormalised
  const int blocks = (int)((w.nhalf + 255) / 256);
  hipLaunchKernelGGL(curl_kernel, dim3(blocks), dim3(256), 0, b.stream, w.uh, n, w.nhalf, inv_n3);
  DHIT_HIP(hipGetLastError());
  DHIT_FFT(hipfftExecZ2D(w.inv, w.uh, w.u));
  copy_to_host({{omega_host, w.u, 3 * b.ncell * sizeof(double)}}, b.stream);
}

}  // namespace dhit
