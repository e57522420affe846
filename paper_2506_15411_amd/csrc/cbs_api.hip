// C ABI of the CBS solver: plans, setup kernels, the iteration loop,
// adjoint source, gradient and the Green's-operator entry point.
//
// The operation each entry point performs is specified in include/cbs.h.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <chrono>
#include <climits>
#include <complex>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/cbs.h"
#include "kernels.hpp"
#include "pace.hpp"
#include "scpml.hpp"

namespace cbs {

const SizeOps* sizes_small(int* count);
const SizeOps* sizes_mid(int* count);
const SizeOps* sizes_large(int* count);

const SizeOps* find_size(int n) {
  const SizeOps* (*tables[])(int*) = {sizes_small, sizes_mid, sizes_large};
  for (auto tab : tables) {
    int cnt = 0;
    const SizeOps* t = tab(&cnt);
    for (int i = 0; i < cnt; ++i)
      if (t[i].n == n) return &t[i];
  }
  return nullptr;
}

// ---------------------------------------------------------------------------
// errors
// ---------------------------------------------------------------------------
static thread_local std::string g_err;

static int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

#define HIP_TRY(call)                                                               \
  do {                                                                              \
    hipError_t e_ = (call);                                                         \
    if (e_ != hipSuccess) return fail(CBS_E_HIP, "%s: %s", #call, hipGetErrorString(e_)); \
  } while (0)

#define HIP_LAUNCHED()                                                              \
  do {                                                                              \
    hipError_t e_ = hipGetLastError();                                              \
    if (e_ != hipSuccess) return fail(CBS_E_HIP, "kernel launch: %s", hipGetErrorString(e_)); \
  } while (0)

// ---------------------------------------------------------------------------
// setup and small kernels
// ---------------------------------------------------------------------------
constexpr int kSetupBlocks = 1024;
constexpr int kSetupThreads = 256;

struct SetupArgs {
  int nx, ny, nz, px, py, pz, order, dtype;
  double sigma_max, k0d2, kbd2, nb2;
  float nb2f;
  const void* eps;
  float2* V0;
  double* part;  // 2 per block: max|V0|, flags
};

__device__ __forceinline__ double layer_depth(int i, int n, int p) {
  if (p <= 0) return 0.0;
  if (i < p) return double(p - i) / double(p);
  if (i >= n - p) return double(i - (n - p - 1)) / double(p);
  return 0.0;
}

__device__ __forceinline__ double ipow(double u, int m) {
  double r = 1.0;
  for (int k = 0; k < m; ++k) r *= u;
  return r;
}

// sigma, V0 = k0^2 (eps_r - n_bg^2) + i kb^2 sigma (times d^2), max|V0| in
// FP64 and input validation flags (1 non-finite, 2 gain, 4 layer != n_bg^2)
__global__ void __launch_bounds__(kSetupThreads) k_setup(SetupArgs a) {
  __shared__ double smx[kSetupThreads / 64];
  __shared__ unsigned sfl[kSetupThreads / 64];
  const unsigned N = (unsigned)a.nx * a.ny * a.nz;   // below 2^29: 32-bit index arithmetic
  double mx = 0.0;
  unsigned fl = 0;
  for (unsigned i = blockIdx.x * kSetupThreads + threadIdx.x; i < N; i += gridDim.x * kSetupThreads) {
    const unsigned r = i / (unsigned)a.nx;
    const int x = (int)(i - r * a.nx), y = (int)(r % (unsigned)a.ny), z = (int)(r / (unsigned)a.ny);
    float er, ei;
    if (a.dtype == CBS_F32) {
      er = static_cast<const float*>(a.eps)[i];
      ei = 0.f;
    } else {
      const float2 e = static_cast<const float2*>(a.eps)[i];
      er = e.x;
      ei = e.y;
    }
    if (!isfinite(er) || !isfinite(ei)) fl |= 1u;
    if (ei < 0.f) fl |= 2u;
    const bool layer = x < a.px || x >= a.nx - a.px || y < a.py || y >= a.ny - a.py ||
                       z < a.pz || z >= a.nz - a.pz;
    if (layer && (er != a.nb2f || ei != 0.f)) fl |= 4u;
    const double su = ipow(layer_depth(x, a.nx, a.px), a.order) +
                      ipow(layer_depth(y, a.ny, a.py), a.order) +
                      ipow(layer_depth(z, a.nz, a.pz), a.order);
    const double sigma = a.sigma_max * (su < 1.0 ? su : 1.0);
    const double vr = a.k0d2 * ((double)er - a.nb2);
    const double vi = a.k0d2 * (double)ei + a.kbd2 * sigma;
    const double m = sqrt(vr * vr + vi * vi);
    mx = m > mx ? m : mx;
    a.V0[i] = make_float2((float)vr, (float)vi);
  }
  for (int o = 32; o > 0; o >>= 1) {
    const double om = __shfl_xor(mx, o, 64);
    mx = om > mx ? om : mx;
    fl |= (unsigned)__shfl_xor((int)fl, o, 64);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) {
    smx[wv] = mx;
    sfl[wv] = fl;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kSetupThreads / 64; ++w) {
      mx = smx[w] > smx[0] ? smx[w] : smx[0];
      smx[0] = mx;
      sfl[0] |= sfl[w];
    }
    a.part[2 * blockIdx.x] = smx[0];
    a.part[2 * blockIdx.x + 1] = (double)sfl[0];
  }
}

__global__ void k_state_init(DevState* st, double tol, int max_iter, int record) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    st->done = 0;
    st->iter = 0;
    st->status = 0;
    st->max_iter = max_iter;
    st->tol = tol;
    st->eta = INFINITY;
    st->record = record;
    st->pending = 0;
  }
}

// w[0, n) = 0
__global__ void k_clear_words(unsigned* w, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) w[i] = 0u;
}

// point-source amplitude: conj(E(r0)) * scale (from_field) or given * scale
__global__ void k_point_amp(DevState* st, const float2* E, long long idx, long long sE,
                            int from_field, float scale, float2 g0, float2 g1, float2 g2) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    if (from_field) {
      for (int c = 0; c < 3; ++c) {
        const float2 e = E[c * sE + idx];
        st->amp[c] = make_float2(e.x * scale, -e.y * scale);
      }
    } else {
      st->amp[0] = make_float2(g0.x * scale, g0.y * scale);
      st->amp[1] = make_float2(g1.x * scale, g1.y * scale);
      st->amp[2] = make_float2(g2.x * scale, g2.y * scale);
    }
  }
}

// eta = sqrt(sum |dE|^2 / sum |E|^2) over the K1 block partials (fixed order);
// a separate launch when the x-pass does not fold it in
constexpr int kResThreads = 256;
__global__ void __launch_bounds__(kResThreads)
k_residual(const double* part, int per_b, int nb, DevState* st, double* hist) {
  __shared__ double red[2 * kResStreams];
  if (st->done || !st->pending) return;
  residual_finish<kResThreads>(part, per_b, nb, st, hist, red);
  if (threadIdx.x == 0) st->pending = 0;
}

// E_b += sign * pol_b exp(i k_b . r) for every illumination b of a solve
// (the incident plane waves; normal incidence: pol exp(i kb z)).  Components the
// polarisation leaves at zero are not touched: an x-polarised wave reads and
// writes 16 bytes a voxel instead of 48 (275 x 275 x 315: 200 -> 62 us).
__global__ void k_incident(CbsArgs a, float sign) {
  const unsigned N = (unsigned)a.nx * a.ny * a.nz;   // below 2^29: 32-bit index arithmetic
  for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) {
    const unsigned l = i / (unsigned)a.nx;
    const int x = (int)(i - l * a.nx), y = (int)(l % (unsigned)a.ny), z = (int)(l / (unsigned)a.ny);
    for (int b = 0; b < a.nb; ++b) {
      const float2 pxy = a.oblique ? cmul(a.phy[b * a.ny + y], a.phx[b * a.nx + x])
                                   : make_float2(1.f, 0.f);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (!((a.pol_mask >> (3 * b + c)) & 1u)) continue;
        const float2 pz = a.phase[(b * 3 + c) * a.nz + z];
        const float2 inc = a.oblique ? cmul(pz, pxy) : pz;
        float2* ep = a.E + b * a.sEb + c * a.sE + i;
        float2 e = *ep;
        e.x += sign * inc.x;
        e.y += sign * inc.y;
        *ep = e;
      }
    }
  }
}

// Plane-wave tables of the illuminations of a solve, in FP64 rounded to FP32:
// phx[b][x] = exp(i kx_b d x), phy[b][y] = exp(i ky_b d y) and
// phz[b][c][z] = pol_{b,c} exp(i kz_b d z); phase zero at the voxel (0, 0, 0).
struct Kvec {
  int nb;
  double kd[kMaxIllum][3];       // (kx, ky, kz) d of each illumination
  double pol[kMaxIllum][3][2];   // polarisation (re, im)
};
__global__ void k_phase_tables(float2* phx, float2* phy, float2* phz, int nx, int ny, int nz,
                               Kvec kv) {
  const int per = nx + ny + 3 * nz;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kv.nb * per; i += gridDim.x * blockDim.x) {
    const int b = i / per, j = i - b * per;
    double sn, cs;
    if (j < nx) {
      sincos(kv.kd[b][0] * (double)j, &sn, &cs);
      phx[b * nx + j] = make_float2((float)cs, (float)sn);
    } else if (j < nx + ny) {
      const int k = j - nx;
      sincos(kv.kd[b][1] * (double)k, &sn, &cs);
      phy[b * ny + k] = make_float2((float)cs, (float)sn);
    } else {
      const int m = j - nx - ny, c = m / nz, k = m - c * nz;
      sincos(kv.kd[b][2] * (double)k, &sn, &cs);
      const double pr = kv.pol[b][c][0], pi = kv.pol[b][c][1];
      phz[(b * 3 + c) * nz + k] = make_float2((float)(pr * cs - pi * sn), (float)(pr * sn + pi * cs));
    }
  }
}

// grad[z][y][x] = scale * Re(sum_c Ea_c E_c) over the box (FP64 accumulate)
__global__ void k_gradient(const float2* E, const float2* Ea, long long sE, int nx, int ny,
                           int x0, int y0, int z0, int bx, int by, int bz, double scale,
                           float* grad) {
  const unsigned NB = (unsigned)bx * by * bz;   // below 2^29: 32-bit index arithmetic
  for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < NB; i += gridDim.x * blockDim.x) {
    const unsigned r = i / (unsigned)bx;
    const int xi = (int)(i - r * bx), yi = (int)(r % (unsigned)by), zi = (int)(r / (unsigned)by);
    const long long idx = ((long long)(z0 + zi) * ny + (y0 + yi)) * nx + (x0 + xi);
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float2 e = E[c * sE + idx], ea = Ea[c * sE + idx];
      s += (double)ea.x * (double)e.x - (double)ea.y * (double)e.y;
    }
    grad[i] = (float)(scale * s);
  }
}

// ---------------------------------------------------------------------------
// lens metrics: focus search, line profiles, disc power (FP64 reductions)
// ---------------------------------------------------------------------------
constexpr int kMetricBlocks = 1024;
constexpr int kMetricThreads = 256;

__device__ __forceinline__ double intensity(const float2* E, long long sE, long long idx) {
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float2 e = E[c * sE + idx];
    s += (double)e.x * (double)e.x + (double)e.y * (double)e.y;
  }
  return s;
}

// Per-block maximum of |E|^2 over a box with its linear voxel index; ties go
// to the smaller index, so the result does not depend on the launch shape.
__global__ void __launch_bounds__(kMetricThreads)
k_argmax_intensity(const float2* E, long long sE, int nx, int ny, int x0, int y0, int z0, int bx,
                   int by, int bz, double* part) {
  __shared__ double sv[kMetricThreads];
  __shared__ long long si[kMetricThreads];
  double best = -1.0;
  long long bi = 0x7fffffffffffffffLL;
  const unsigned NB = (unsigned)bx * by * bz;   // a grid holds fewer than 2^31 voxels
  for (unsigned i = blockIdx.x * kMetricThreads + threadIdx.x; i < NB; i += gridDim.x * kMetricThreads) {
    const unsigned r = i / (unsigned)bx, xi = i - r * bx;
    const unsigned zi = r / (unsigned)by, yi = r - zi * by;
    const long long idx = ((long long)(z0 + zi) * ny + (y0 + yi)) * nx + (x0 + xi);
    const double s = intensity(E, sE, idx);
    if (s > best || (s == best && idx < bi)) {
      best = s;
      bi = idx;
    }
  }
  sv[threadIdx.x] = best;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int o = kMetricThreads / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      const double v = sv[threadIdx.x + o];
      const long long j = si[threadIdx.x + o];
      if (v > sv[threadIdx.x] || (v == sv[threadIdx.x] && j < si[threadIdx.x])) {
        sv[threadIdx.x] = v;
        si[threadIdx.x] = j;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = sv[0];
    part[2 * blockIdx.x + 1] = (double)si[0];
  }
}

// The maximum of the per-block maxima of k_argmax_intensity (same tie rule):
// focus[0] = |E|^2, focus[1] = linear voxel index.  One work-group, one wave.
__global__ void k_argmax_finish(const double* part, int nb, double* focus) {
  double best = -1.0, bi = 1e300;
  for (int b = threadIdx.x; b < nb; b += 64) {
    const double v = part[2 * b], j = part[2 * b + 1];
    if (v > best || (v == best && j < bi)) {
      best = v;
      bi = j;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const double v = __shfl_xor(best, o, 64), j = __shfl_xor(bi, o, 64);
    if (v > best || (v == best && j < bi)) {
      best = v;
      bi = j;
    }
  }
  if (threadIdx.x == 0) {   // no finite |E|^2 in the box: -1 at voxel 0
    focus[0] = best;
    focus[1] = best < 0.0 ? 0.0 : bi;
  }
}

// |E|^2 along the x, y and z lines through the focus: out[0, nx) then
// out[nx, nx + ny) then out[nx + ny, nx + ny + nz).
__global__ void k_line_intensity(const float2* E, long long sE, int nx, int ny, int nz,
                                 const double* focus, double* out) {
  const long long bi = (long long)focus[1];
  const int fx = (int)(bi % nx), fy = (int)((bi / nx) % ny), fz = (int)(bi / ((long long)nx * ny));
  const int n = nx + ny + nz;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    int x = fx, y = fy, z = fz;
    if (i < nx) x = i;
    else if (i < nx + ny) y = i - nx;
    else z = i - nx - ny;
    out[i] = intensity(E, sE, ((long long)z * ny + y) * nx + x);
  }
}

// The transverse field of the focal plane in FP64: ex, ey [ny][nx].
__global__ void k_plane_extract(const float2* E, long long sE, int nx, int ny,
                                const double* focus, double2* ex, double2* ey) {
  const long long NP = (long long)nx * ny;
  const long long fz = (long long)focus[1] / NP;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < NP;
       i += (long long)gridDim.x * blockDim.x) {
    const float2 a = E[fz * NP + i], b = E[sE + fz * NP + i];
    ex[i] = make_double2(a.x, a.y);
    ey[i] = make_double2(b.x, b.y);
  }
}

// One pass of plane DFTs in FP64, in place: the lines of the [ny][nx] planes that
// follow each other (blockIdx.y), along x (axis 0) or y (axis 1), out[k] = sum_j
// in[j] w^(sign j k), w = tw[m] = exp(-2 pi i m / n) (sign -1: forward, +1:
// inverse, unscaled).  A work-group holds kDftLines lines and the table in LDS;
// n = n1 n2 is summed in the two levels of the passes, n1 + n2 terms an output
// (direct sums of n terms from global memory took 84 us a 275 x 275 plane and
// axis, from LDS for four planes at once 42; now 14 for the four).
constexpr int kDftLines = 2;
constexpr int kDftThreads = 512;
__global__ void __launch_bounds__(kDftThreads)
k_plane_dft(double2* planes, int nx, int ny, int axis, int sign, int n1, int n2,
            const double2* tw) {
  extern __shared__ double2 sh[];   // lines, their level-A results, the table
  const int n = axis == 0 ? nx : ny, lines = axis == 0 ? ny : nx;
  const long long ls = axis == 0 ? nx : 1, es = axis == 0 ? 1 : nx;
  const int l0 = blockIdx.x * kDftLines, tasks = kDftLines * n;
  double2* f = planes + (long long)blockIdx.y * nx * ny + l0 * ls;
  double2 *mid = sh + tasks, *t = mid + tasks;
  for (int i = threadIdx.x; i < tasks; i += kDftThreads) {
    // consecutive threads along the contiguous direction
    const int r = axis == 0 ? i / n : i % kDftLines, j = axis == 0 ? i % n : i / kDftLines;
    sh[r * n + j] = l0 + r < lines ? f[r * ls + j * es] : make_double2(0.0, 0.0);
  }
  for (int i = threadIdx.x; i < n; i += kDftThreads) {
    const double2 w = tw[i];
    t[i] = make_double2(w.x, sign < 0 ? w.y : -w.y);
  }
  __syncthreads();
  // level A: mid[j2 n1 + k1] = w^(j2 k1) sum_j1 in[j2 + n2 j1] w^(n2 j1 k1)
  for (int i = threadIdx.x; i < tasks; i += kDftThreads) {
    const int r = i / n, q = i - r * n, j2 = q / n1, k1 = q - j2 * n1;
    const double2* v = sh + r * n + j2;
    double2 s = make_double2(0.0, 0.0);
    int m = 0;   // j1 k1 mod n1
    for (int j1 = 0; j1 < n1; ++j1) {
      s = zadd(s, zmul(v[n2 * j1], t[m * n2]));
      m += k1;
      m -= m >= n1 ? n1 : 0;
    }
    mid[i] = zmul(s, t[j2 * k1]);
  }
  __syncthreads();
  // level B: out[k1 + n1 k2] = sum_j2 mid[j2 n1 + k1] w^(n1 j2 k2)
  for (int i = threadIdx.x; i < tasks; i += kDftThreads) {
    const int r = axis == 0 ? i / n : i % kDftLines, k = axis == 0 ? i - r * n : i / kDftLines;
    const int k2 = k / n1, k1 = k - k2 * n1;
    const double2* v = mid + r * n + k1;
    double2 s = make_double2(0.0, 0.0);
    int m = 0;   // j2 k2 mod n2
    for (int j2 = 0; j2 < n2; ++j2) {
      s = zadd(s, zmul(v[j2 * n1], t[m * n1]));
      m += k2;
      m -= m >= n2 ? n2 : 0;
    }
    if (l0 + r < lines) f[r * ls + k * es] = s;
  }
}

// Angular spectrum of the transverse field -> propagating part of E and the
// magnetic field in units where a plane wave has H = z x E:
//   kz = sqrt(k^2 - kx^2 - ky^2) (evanescent components dropped),
//   Ez = -(kx Ex + ky Ey) / kz,  H = k_vec x E / k.
__global__ void k_angular_h(double2* ax, double2* ay, double2* hx, double2* hy, int nx, int ny,
                            double dkx, double dky, double k) {
  const long long NP = (long long)nx * ny;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < NP;
       i += (long long)gridDim.x * blockDim.x) {
    const int ix = (int)(i % nx), iy = (int)(i / nx);
    const double kx = dkx * (ix < (nx + 1) / 2 ? ix : ix - nx);
    const double ky = dky * (iy < (ny + 1) / 2 ? iy : iy - ny);
    const double kz2 = k * k - kx * kx - ky * ky;
    if (kz2 <= 0.0) {
      ax[i] = ay[i] = hx[i] = hy[i] = make_double2(0.0, 0.0);
      continue;
    }
    const double kz = sqrt(kz2);
    const double2 ex = ax[i], ey = ay[i];
    const double2 ez = make_double2(-(kx * ex.x + ky * ey.x) / kz, -(kx * ex.y + ky * ey.y) / kz);
    hx[i] = make_double2((ky * ez.x - kz * ey.x) / k, (ky * ez.y - kz * ey.y) / k);
    hy[i] = make_double2((kz * ex.x - kx * ez.x) / k, (kz * ex.y - kx * ez.y) / k);
  }
}

// Per-block sums of S_z = Re(Ex conj(Hy) - Ey conj(Hx)) (times scale) over the
// voxels of the plane whose centres lie within sqrt(r2) voxels of (cx, cy).
__global__ void __launch_bounds__(kMetricThreads)
k_disc_flux(const double2* ex, const double2* ey, const double2* hx, const double2* hy, int nx,
            int ny, double cx, double cy, double r2, double scale, double* part) {
  __shared__ double sh[kMetricThreads];
  double acc = 0.0;
  const long long NP = (long long)nx * ny;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < NP;
       i += (long long)gridDim.x * blockDim.x) {
    const int x = (int)(i % nx), y = (int)(i / nx);
    const double dx = x - cx, dy = y - cy;
    if (dx * dx + dy * dy <= r2) {
      const double2 a = ex[i], b = ey[i], u = hx[i], v = hy[i];
      acc += (a.x * v.x + a.y * v.y) - (b.x * u.x + b.y * u.y);
    }
  }
  sh[threadIdx.x] = acc * scale;
  __syncthreads();
  for (int o = kMetricThreads / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// ---------------------------------------------------------------------------
// total-field / scattered-field source: S = (L - K_bg)(chi E_inc)
// ---------------------------------------------------------------------------
// chi is the indicator of a box and E_inc = q exp(i k.r), so chi E_inc = q u
// with u = fx(x) fy(y) fz(z), f_a(i) = chi_a(i) exp(i k_a d i), and every term
// of L (q u) = F^-1 [ |p|^2 q u^ - pt (pt . q) u^ ] is a product of 1D
// transforms of the f_a.  Per axis the tables hold (FP64, n_a entries each,
// axes one after the other):
//   tab[0] = f,  tab[1] = F f (spectrum),  tab[2] = F^-1[p^2 F f],
//   tab[3] = F^-1[pt F f],  tab[4] = F^-1[pt^2 F f]   (p in 1/m; pt = p except
// 0 at the Nyquist bin of an even axis), by direct O(n^2) sums.
struct TfsfArgs {
  int n[3], lo[3], hi[3], off[3];   // axis lengths, box, table offsets
  int ntot;                         // n[0] + n[1] + n[2]
  double kd[3];                     // (kx, ky, kz) d of the plane wave
  double pitch;
  double2* tab;                     // 5 ntot entries
};

__device__ __forceinline__ int tfsf_axis(const TfsfArgs& t, int j, int& i) {
  const int a = j < t.n[0] ? 0 : (j < t.n[0] + t.n[1] ? 1 : 2);
  i = j - t.off[a];
  return a;
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// f and its DFT: one wave per axis entry, its lanes share the sum (one thread per
// entry, a serial chain of two sincos per term, took 80 us on 192 x 192 x 256)
__global__ void __launch_bounds__(64) k_tfsf_forward(TfsfArgs t) {
  const int j = blockIdx.x, lane = threadIdx.x;
  int m;
  const int a = tfsf_axis(t, j, m);
  const int n = t.n[a];
  double re = 0.0, im = 0.0;
  for (int i = t.lo[a] + lane; i < t.hi[a]; i += 64) {   // f vanishes outside the box
    double sf, cf, sw, cw;
    sincos(t.kd[a] * (double)i, &sf, &cf);
    sincos(-2.0 * M_PI * (double)((m * i) % n) / (double)n, &sw, &cw);
    re += cf * cw - sf * sw;
    im += cf * sw + sf * cw;
  }
  re = wave_sum(re);
  im = wave_sum(im);
  if (lane != 0) return;
  t.tab[t.ntot + j] = make_double2(re, im);
  double sf = 0.0, cf = 0.0;
  if (m >= t.lo[a] && m < t.hi[a]) sincos(t.kd[a] * (double)m, &sf, &cf);
  t.tab[j] = make_double2(cf, sf);
}

// the three filtered inverse transforms, one wave per axis entry
__global__ void __launch_bounds__(64) k_tfsf_inverse(TfsfArgs t) {
  const int j = blockIdx.x, lane = threadIdx.x;
  int i;
  const int a = tfsf_axis(t, j, i);
  const int n = t.n[a];
  double r2 = 0.0, i2 = 0.0, r1 = 0.0, i1 = 0.0, rt = 0.0, it = 0.0;
  for (int m = lane; m < n; m += 64) {
    const double2 F = t.tab[t.ntot + t.off[a] + m];
    const int mm = (m < (n + 1) / 2) ? m : m - n;
    const double pm = 2.0 * M_PI * (double)mm / ((double)n * t.pitch);
    const double ptm = ((n & 1) == 0 && 2 * m == n) ? 0.0 : pm;
    double sw, cw;
    sincos(2.0 * M_PI * (double)((m * i) % n) / (double)n, &sw, &cw);
    const double gr = F.x * cw - F.y * sw, gi = F.x * sw + F.y * cw;   // F(m) e^{+2 pi i m i/n}
    r2 += pm * pm * gr;
    i2 += pm * pm * gi;
    r1 += ptm * gr;
    i1 += ptm * gi;
    rt += ptm * ptm * gr;
    it += ptm * ptm * gi;
  }
  const double inv = 1.0 / (double)n;
  r2 = wave_sum(r2) * inv;
  i2 = wave_sum(i2) * inv;
  r1 = wave_sum(r1) * inv;
  i1 = wave_sum(i1) * inv;
  rt = wave_sum(rt) * inv;
  it = wave_sum(it) * inv;
  if (lane != 0) return;
  t.tab[2 * t.ntot + j] = make_double2(r2, i2);
  t.tab[3 * t.ntot + j] = make_double2(r1, i1);
  t.tab[4 * t.ntot + j] = make_double2(rt, it);
}

// zmul: complex FP64 product (scpml.hpp)
__device__ __forceinline__ double2 zmul3(double2 a, double2 b, double2 c) {
  return zmul(zmul(a, b), c);
}

struct TfsfAssemble {
  TfsfArgs t;
  int nx, ny, nz, px, py, pz, order;
  double sigma_max, kb2;
  double2 q[3];          // polarisation
  float2* S;             // [3][nz][ny][nx]
};

// S_c = q_c (D2x fy fz + fx D2y fz + fx fy D2z - kb^2 (1 + i sigma) u)
//       - sum_b q_b T_c T_b u   (T_c T_b u = (T1 f)(T1 f)(f) for c != b, (T2 f)(f)(f) for c = b)
__global__ void k_tfsf_assemble(TfsfAssemble A) {
  const TfsfArgs& t = A.t;
  const unsigned N = (unsigned)A.nx * A.ny * A.nz;   // below 2^29: 32-bit index arithmetic
  const double2* f = t.tab;
  const double2* d2 = t.tab + 2 * t.ntot;
  const double2* t1 = t.tab + 3 * t.ntot;
  const double2* t2 = t.tab + 4 * t.ntot;
  for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) {
    const unsigned l = i / (unsigned)A.nx;
    const int x = (int)(i - l * A.nx), y = (int)(l % (unsigned)A.ny), z = (int)(l / (unsigned)A.ny);
    const int ix = t.off[0] + x, iy = t.off[1] + y, iz = t.off[2] + z;
    const double2 u = zmul3(f[ix], f[iy], f[iz]);
    const double su = ipow(layer_depth(x, A.nx, A.px), A.order) +
                      ipow(layer_depth(y, A.ny, A.py), A.order) +
                      ipow(layer_depth(z, A.nz, A.pz), A.order);
    const double sigma = A.sigma_max * (su < 1.0 ? su : 1.0);
    const double2 kbg = make_double2(A.kb2, A.kb2 * sigma);
    const double2 lap = make_double2(
        zmul3(d2[ix], f[iy], f[iz]).x + zmul3(f[ix], d2[iy], f[iz]).x + zmul3(f[ix], f[iy], d2[iz]).x,
        zmul3(d2[ix], f[iy], f[iz]).y + zmul3(f[ix], d2[iy], f[iz]).y + zmul3(f[ix], f[iy], d2[iz]).y);
    const double2 diag = make_double2(lap.x - zmul(kbg, u).x, lap.y - zmul(kbg, u).y);
    // T_c T_b u for the 3 x 3 pairs
    const int idx[3] = {ix, iy, iz};
    double2 tt[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        double2 v;
        if (c == b) {
          v = t2[idx[c]];
        } else {
          v = zmul(t1[idx[c]], t1[idx[b]]);
        }
        const int o = 3 - c - b;   // the remaining axis when c != b
        if (c == b) {
          const int o1 = (c + 1) % 3, o2 = (c + 2) % 3;
          v = zmul3(v, f[idx[o1]], f[idx[o2]]);
        } else {
          v = zmul(v, f[idx[o]]);
        }
        tt[c][b] = v;
      }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      double2 sc = zmul(A.q[c], diag);
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const double2 w = zmul(A.q[b], tt[c][b]);
        sc.x -= w.x;
        sc.y -= w.y;
      }
      A.S[(size_t)c * N + i] = make_float2((float)sc.x, (float)sc.y);
    }
  }
}

// streaming copy: one float4 per thread over a grid that covers the buffer
// (the fastest plain copy form measured on this part)
constexpr int kCopyThreads = 256;
__global__ void __launch_bounds__(kCopyThreads)
k_copy(const float4* __restrict__ src, float4* __restrict__ dst, long long n4) {
  const long long i = (long long)blockIdx.x * kCopyThreads + threadIdx.x;
  if (i < n4) dst[i] = src[i];
}

}  // namespace cbs

using namespace cbs;

// ---------------------------------------------------------------------------
// plan
// ---------------------------------------------------------------------------
struct cbs_plan_s {
  int nx, ny, nz, nxp;
  int pml[3];
  double pitch, lambda0, n_bg, k0, kb;
  int order;
  double sigma_max;
  double shift_factor;
  const SizeOps *ox, *oy, *oz;
  int k1_blocks;
  hipStream_t stream;
  // workspace carve-up
  float2 *W, *V0, *twx, *twy, *twz, *phase, *phx, *phy;
  double *partials, *setup_part, *hist, *metrics;
  unsigned char* rows;   // zero rows of a field source (CbsArgs::rows)
  DevState* state;
  bool have_eps;
  double eps;  // 1/m^2
  int hist_len;
  hipEvent_t ev0, ev1;
  hipEvent_t evp[5];
  // asynchronous solve in progress (cbs_solve_begin .. cbs_solve_end)
  struct Active {
    bool on;        // begun and not ended
    bool stopped;   // device reported the stop; later launches are no-ops
    bool plane;     // plane-wave source: E_inc is added at the end
    unsigned flags;
    int max_iter;
    double tol;
    int enqueued;   // iterations enqueued so far
    int head, count;  // ring of outstanding quanta
    float ms;       // device time from begin to the quantum that stopped
    CbsArgs args;
  } act;
  static constexpr int kRing = 4;
  hipEvent_t evq[kRing];
  DevState* mirror;  // pinned host copies of the device state, one per quantum slot
  DevState last;     // state read at the last completed quantum
};

// The workspace of cbs_solve_static: one plan's scratch in a static device
// array, held by each GPU the library runs on until the process ends.  In host
// code cbs_scratch names a host-side stand-in; its device address comes from
// hipGetSymbolAddress, once per device (static_scratch below), and only that
// address is ever passed to a kernel or a copy.
static __device__ __align__(256) unsigned char cbs_scratch[CBS_STATIC_SCRATCH_BYTES];

namespace {

struct Layout {
  size_t W, V0, twx, twy, twz, phase, phx, phy, partials, setup, hist, metrics, rows, state, total;
};

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

int padded_pitch(int nx) { return (nx + kBrick - 1) / kBrick * kBrick; }

bool layout_of(int nx, int ny, int nz, Layout& L) {
  const SizeOps* ox = find_size(nx);
  if (!ox) return false;
  const long long N = (long long)nx * ny * nz;
  const long long k1b = 3LL * ((ny + ox->k1_rows - 1) / ox->k1_rows) * nz;   // x-pass blocks
  const size_t c8 = sizeof(float2);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  L.W = take((size_t)3 * nz * ny * padded_pitch(nx) * c8);
  L.V0 = take((size_t)N * c8);
  L.twx = take((size_t)nx * c8);
  L.twy = take((size_t)ny * c8);
  L.twz = take((size_t)nz * c8);
  L.phase = take((size_t)3 * nz * c8);
  L.phx = take((size_t)nx * c8);
  L.phy = take((size_t)ny * c8);
  L.partials = take((size_t)2 * k1b * sizeof(double));
  L.setup = take((size_t)2 * kSetupBlocks * sizeof(double));
  L.hist = take((size_t)kHistCap * sizeof(double));
  L.metrics = take((size_t)(2 * kMetricBlocks + 2 + nx + ny + nz + 1) * sizeof(double) +
                   (size_t)(nx + ny + 5 * N / nz) * sizeof(double2));
  L.rows = take((size_t)3 * nz * ny);
  L.state = take(sizeof(DevState));
  L.total = off;
  return true;
}

// Twiddles of a two-level split n = n1 n2: t[j2 n1 + k1] = exp(-2 pi i j2 k1 / n),
// j2 < n2, k1 < n1 (FP64 on the host, rounded to FP32).  j2 k1 < n, so the
// angle needs no reduction, and the same table read at [k][t] serves the
// transposed split.  t holds n entries.
void fill_twiddles(float2* t, int n1, int n2) {
  const int n = n1 * n2;
  for (int j2 = 0; j2 < n2; ++j2)
    for (int k1 = 0; k1 < n1; ++k1) {
      const double ang = -2.0 * M_PI * double(j2 * k1) / double(n);
      t[j2 * n1 + k1] = make_float2((float)std::cos(ang), (float)std::sin(ang));
    }
}

// Longest registered axis: the host staging arrays of the tables are this long.
constexpr int kMaxAxis = 1024;

// Argument checks of a grid and its optics (cbs_plan_create's contract).
int check_grid(int nx, int ny, int nz, double pitch_m, double lambda0_m, double n_bg,
               const int pml[3], int pm[3]) {
  if (nx < 2 || ny < 2 || nz < 2) return fail(CBS_E_INVALID, "grid %dx%dx%d: each axis must be >= 2", nx, ny, nz);
  const int dims[3] = {nx, ny, nz};
  for (int a = 0; a < 3; ++a)
    if (!cbs_axis_supported(a, dims[a]) || dims[a] > kMaxAxis)
      return fail(CBS_E_INVALID, "axis %d length %d has no FFT specialisation", a, dims[a]);
  if (!(pitch_m > 0) || !std::isfinite(pitch_m)) return fail(CBS_E_INVALID, "pitch must be > 0");
  if (!(lambda0_m > 0) || !std::isfinite(lambda0_m)) return fail(CBS_E_INVALID, "lambda0 must be > 0");
  if (!(n_bg > 0) || !std::isfinite(n_bg)) return fail(CBS_E_INVALID, "n_bg must be > 0");
  pm[0] = pm[1] = pm[2] = 0;
  if (pml)
    for (int a = 0; a < 3; ++a) {
      pm[a] = pml[a];
      if (pm[a] < 0 || 2 * pm[a] >= dims[a])
        return fail(CBS_E_INVALID, "pml[%d]=%d must satisfy 0 <= 2 pml < %d", a, pm[a], dims[a]);
    }
  return CBS_OK;
}

// Fill a plan's grid, optics and workspace carve-up (no HIP calls).
void init_plan(cbs_plan_s* p, int nx, int ny, int nz, double pitch_m, double lambda0_m,
               double n_bg, const int pm[3], void* workspace, hipStream_t stream) {
  Layout L;
  layout_of(nx, ny, nz, L);
  p->nx = nx;
  p->ny = ny;
  p->nz = nz;
  p->nxp = padded_pitch(nx);
  for (int a = 0; a < 3; ++a) p->pml[a] = pm[a];
  p->pitch = pitch_m;
  p->lambda0 = lambda0_m;
  p->n_bg = n_bg;
  p->k0 = 2.0 * M_PI / lambda0_m;
  p->kb = p->k0 * n_bg;
  p->order = 2;
  p->sigma_max = 1.0;
  p->shift_factor = 1.1;
  p->ox = find_size(nx);
  p->oy = find_size(ny);
  p->oz = find_size(nz);
  p->k1_blocks = (int)(3LL * ((ny + p->ox->k1_rows - 1) / p->ox->k1_rows) * nz);
  p->stream = stream;
  char* base = static_cast<char*>(workspace);
  p->W = reinterpret_cast<float2*>(base + L.W);
  p->V0 = reinterpret_cast<float2*>(base + L.V0);
  p->twx = reinterpret_cast<float2*>(base + L.twx);
  p->twy = reinterpret_cast<float2*>(base + L.twy);
  p->twz = reinterpret_cast<float2*>(base + L.twz);
  p->phase = reinterpret_cast<float2*>(base + L.phase);
  p->phx = reinterpret_cast<float2*>(base + L.phx);
  p->phy = reinterpret_cast<float2*>(base + L.phy);
  p->partials = reinterpret_cast<double*>(base + L.partials);
  p->setup_part = reinterpret_cast<double*>(base + L.setup);
  p->hist = reinterpret_cast<double*>(base + L.hist);
  p->metrics = reinterpret_cast<double*>(base + L.metrics);
  p->rows = reinterpret_cast<unsigned char*>(base + L.rows);
  p->state = reinterpret_cast<DevState*>(base + L.state);
  p->have_eps = false;
  p->eps = -1.0;
  p->hist_len = 0;
}

// Enqueue the twiddle tables (FP64 on the host, rounded to FP32) from host
// staging arrays that live until the stream has consumed them (the caller
// synchronises before they go out of scope).  The plane-wave phase tables are
// built on the device when a solve starts (k_phase_tables).
struct Tables {
  float2 tx[kMaxAxis], ty[kMaxAxis], tz[kMaxAxis];
};
hipError_t upload_tables(cbs_plan_s* p, Tables& t) {
  fill_twiddles(t.tx, p->ox->n1, p->ox->n2);
  fill_twiddles(t.ty, p->oy->n1, p->oy->n2);
  fill_twiddles(t.tz, p->oz->z1, p->oz->z2);
  hipError_t e = hipMemcpyAsync(p->twx, t.tx, p->nx * sizeof(float2), hipMemcpyHostToDevice, p->stream);
  e = e == hipSuccess ? hipMemcpyAsync(p->twy, t.ty, p->ny * sizeof(float2), hipMemcpyHostToDevice, p->stream) : e;
  e = e == hipSuccess ? hipMemcpyAsync(p->twz, t.tz, p->nz * sizeof(float2), hipMemcpyHostToDevice, p->stream) : e;
  return e;
}

// The potential V0, the shift eps and the validity checks of a medium
// (cbs_set_permittivity's contract).  Synchronises the plan's stream.
int set_permittivity_impl(cbs_plan_s* p, const void* eps_r, int dtype) {
  if (!eps_r) return fail(CBS_E_INVALID, "eps_r is NULL");
  if (dtype != CBS_F32 && dtype != CBS_C64) return fail(CBS_E_INVALID, "dtype must be CBS_F32 or CBS_C64");
  p->have_eps = false;
  SetupArgs s;
  s.nx = p->nx;
  s.ny = p->ny;
  s.nz = p->nz;
  s.px = p->pml[0];
  s.py = p->pml[1];
  s.pz = p->pml[2];
  s.order = p->order;
  s.dtype = dtype;
  s.sigma_max = p->sigma_max;
  const double d2 = p->pitch * p->pitch;
  s.k0d2 = p->k0 * p->k0 * d2;
  s.kbd2 = p->kb * p->kb * d2;
  s.nb2 = p->n_bg * p->n_bg;
  s.nb2f = (float)(p->n_bg * p->n_bg);
  s.eps = eps_r;
  s.V0 = p->V0;
  s.part = p->setup_part;
  hipLaunchKernelGGL(k_setup, dim3(kSetupBlocks), dim3(kSetupThreads), 0, p->stream, s);
  HIP_LAUNCHED();
  double part[2 * kSetupBlocks];
  HIP_TRY(hipMemcpyAsync(part, p->setup_part, sizeof(part), hipMemcpyDeviceToHost, p->stream));
  HIP_TRY(hipStreamSynchronize(p->stream));
  double mx = 0.0;
  unsigned fl = 0;
  for (int b = 0; b < kSetupBlocks; ++b) {
    mx = part[2 * b] > mx ? part[2 * b] : mx;
    fl |= (unsigned)part[2 * b + 1];
  }
  if (fl & 1u) return fail(CBS_E_INVALID, "eps_r has non-finite values");
  if (fl & 2u) return fail(CBS_E_INVALID, "gain medium (Im eps_r < 0) is not admissible");
  if (fl & 4u) return fail(CBS_E_INVALID, "eps_r must equal n_bg^2 inside the absorbing layer");
  const double floor_ = 1e-3 * p->kb * p->kb * d2;
  const double eps_d2 = p->shift_factor * (mx > floor_ ? mx : floor_);
  // the iteration forms (V0 - i eps) E in FP32: keep the shift far inside its range
  if (!(eps_d2 < 1e30))
    return fail(CBS_E_INVALID, "eps_r contrast too large for the FP32 iteration (shift %g)", eps_d2);
  p->eps = eps_d2 / d2;
  p->have_eps = true;
  return CBS_OK;
}

// Whether the fused plane pass runs instead of the three passes of a plane:
// square planes that fit in LDS, enough of them to occupy the CUs.  A plane's
// time does not depend on how many there are until every CU has one, the three
// passes' does: up to 64 x 64 the fused pass wins from 12 planes on (64 x 64 x 4:
// 12.5 us an iteration against 15.2), above that from about N^2 / 192 planes
// (96^2: 36 planes 21.4 against 21.3 us; 121^2: 60 planes 38.6 against 35.4, 72
// planes 40.0 against 39.1; 128^2: 60 planes 34.4 against 35.0).  The number of
// illuminations does not enter, so a batch takes the path of its single solves.
bool plane_fused(const cbs_plan_s* p) {
  const int n = p->nx;
  return n == p->ny && p->ox->kxy && (n <= 64 || 3LL * p->nz * 192 >= (long long)n * n);
}

// the number of illuminations and what follows from it
void set_illuminations(const cbs_plan_s* p, CbsArgs& a, int nb) {
  a.nb = nb;
  a.fused = plane_fused(p) ? 1 : 0;
  a.k1_blocks = a.fused ? 3 * p->nz : p->k1_blocks;
}

// Grids whose x and y passes look at the stop flag before they load anything: on the
// others the flag's latency costs more than a stopped solve's few remaining launches,
// which read the volume for nothing.  Iteration in us, flag late -> first: 121 x 189 x
// 100 105.0 -> 105.6, 189 x 189 x 121 180.7 -> 181.7; 192 x 192 x 256 solved to 1e-4,
// 179.3 -> 178.1 ms.
bool large_grid(const cbs_plan_s* p) {
  return (long long)p->nx * p->ny * p->nz > 6LL << 20;
}

// Iterations longer than the 20 us of a host's reading, so that a solve's last ones are
// worth a reading each: a stopped iteration of 275 x 275 x 315 still takes 140 us (a
// solve of 160 iterations in quanta of 20 left 0.7 ms behind it with quarter quanta at
// the end, 0.33 with single iterations).  96^3 takes 46 us, a stopped one 9.
bool long_iteration(const cbs_plan_s* p) {
  return (long long)p->nx * p->ny * p->nz > 1LL << 20;
}

CbsArgs base_args(cbs_plan_s* p) {
  CbsArgs a;
  std::memset(&a, 0, sizeof(a));
  a.nx = p->nx;
  a.ny = p->ny;
  a.nz = p->nz;
  a.nxp = p->nxp;
  a.gx = p->nxp / kBrick;
  a.gy = (p->ny + p->ox->k1_rows - 1) / p->ox->k1_rows;
  a.px = p->pml[0];
  a.py = p->pml[1];
  a.pz = p->pml[2];
  a.sW = (long long)p->nz * p->ny * p->nxp;
  a.sE = (long long)p->nz * p->ny * p->nx;
  a.W = p->W;
  a.V0 = p->V0;
  a.twx = p->twx;
  a.twy = p->twy;
  a.twz = p->twz;
  a.phase = p->phase;
  a.partials = p->partials;
  set_illuminations(p, a, 1);
  a.sWb = 3 * a.sW;
  a.sEb = 3 * a.sE;
  a.phx = p->phx;
  a.phy = p->phy;
  a.oblique = 0;
  a.hist = p->hist;
  a.st = p->state;
  const double d2 = p->pitch * p->pitch;
  a.eps = (float)(p->eps * d2);
  a.inv_eps = (float)(1.0 / (p->eps * d2));
  a.kb2 = (float)(p->kb * p->kb * d2);
  a.pfx = (float)(2.0 * M_PI / p->nx);
  a.pfy = (float)(2.0 * M_PI / p->ny);
  a.pfz = (float)(2.0 * M_PI / p->nz);
  a.invN = (float)(1.0 / ((double)p->nx * p->ny * p->nz));
  a.src_scale = (float)d2;
  a.flag_first = large_grid(p) ? 1 : 0;
  return a;
}

int check_plan(cbs_plan_t p, bool need_eps) {
  if (!p) return fail(CBS_E_INVALID, "null plan");
  if (need_eps && !p->have_eps)
    return fail(CBS_E_STATE, "cbs_set_permittivity must be called before solving");
  return CBS_OK;
}

int check_opts(const cbs_opts* o) {
  if (!o) return fail(CBS_E_INVALID, "opts is NULL");
  if (o->max_iter < 1) return fail(CBS_E_INVALID, "max_iter must be >= 1 (got %d)", o->max_iter);
  if (o->check_every < 1) return fail(CBS_E_INVALID, "check_every must be >= 1");
  if (!(o->tol >= 0.0)) return fail(CBS_E_INVALID, "tol must be >= 0");
  return CBS_OK;
}

// prologue of a loop of iterations: W = V E + S (mode K1_FWD), x and y forward
void enqueue_prologue(cbs_plan_s* p, const CbsArgs& a) {
  if (a.fused) {
    p->ox->kxy(a, K1_FWD, p->stream);
    return;
  }
  p->ox->k1(a, K1_FWD, p->stream);
  p->oy->ky(a, -1, p->stream);
}

// one CBS iteration on W's x and y spectra: z forward + Green + z inverse, y
// inverse, x inverse + update + next forward x, and the next forward y unless
// no iteration follows (last); the plane's three in one launch where fused
int enqueue_iteration(cbs_plan_s* p, const CbsArgs& a, bool last) {
  p->oz->kz(a, p->stream);            // also reduces the iteration before's residual
  if (a.fused) {
    p->ox->kxy(a, K1_ITER, p->stream);
    HIP_LAUNCHED();
    return CBS_OK;
  }
  p->oy->ky(a, +1, p->stream);
  p->ox->k1(a, K1_ITER, p->stream);
  if (!last) p->oy->ky(a, -1, p->stream);
  HIP_LAUNCHED();
  return CBS_OK;
}

// reduce the residual of the last enqueued iteration (a no-op when nothing is
// pending), so the state copied to the host is current
int enqueue_residual(cbs_plan_s* p, const CbsArgs& a) {
  hipLaunchKernelGGL(k_residual, dim3(1), dim3(kResThreads), 0, p->stream, a.partials,
                     a.k1_blocks, a.nb, p->state, p->hist);
  HIP_LAUNCHED();
  return CBS_OK;
}

// Start a solve: device state, point-source amplitude, optional warm-start
// conversion to the scattered field, and the prologue (W = V E + S, forward x).
// Device state, point-source amplitude and warm-start conversion of a solve.
int enqueue_solve_start(cbs_plan_s* p, CbsArgs& a, const cbs_opts* o, const cbs_source* src,
                        const void* E_fwd, const Kvec& kv) {
  if (a.src == SRC_PLANE) {
    // the incident plane waves' phase tables (built before anything reads them)
    const int n = kv.nb * (p->nx + p->ny + 3 * p->nz);
    hipLaunchKernelGGL(k_phase_tables, dim3((n + 255) / 256), dim3(256), 0, p->stream,
                       const_cast<float2*>(a.phx), const_cast<float2*>(a.phy),
                       const_cast<float2*>(a.phase), p->nx, p->ny, p->nz, kv);
    HIP_LAUNCHED();
  }
  hipLaunchKernelGGL(k_state_init, dim3(1), dim3(64), 0, p->stream, p->state, o->tol,
                     o->max_iter, (o->flags & CBS_RECORD_HISTORY) ? 1 : 0);
  HIP_LAUNCHED();
  if (a.src == SRC_POINT) {
    const long long idx = ((long long)src->r0[2] * p->ny + src->r0[1]) * p->nx + src->r0[0];
    hipLaunchKernelGGL(k_point_amp, dim3(1), dim3(64), 0, p->stream, p->state,
                       static_cast<const float2*>(E_fwd), idx, a.sE, E_fwd ? 1 : 0,
                       (float)(p->pitch * p->pitch),
                       make_float2((float)src->amp[0][0], (float)src->amp[0][1]),
                       make_float2((float)src->amp[1][0], (float)src->amp[1][1]),
                       make_float2((float)src->amp[2][0], (float)src->amp[2][1]));
    HIP_LAUNCHED();
  }
  a.warm = (o->flags & CBS_WARM_START) ? 1 : 0;
  if (a.warm && a.src == SRC_PLANE) {
    hipLaunchKernelGGL(k_incident, dim3(2048), dim3(256), 0, p->stream, a, -1.0f);
    HIP_LAUNCHED();
  }
  return CBS_OK;
}

int begin_solve(cbs_plan_s* p, CbsArgs& a, const cbs_opts* o, const cbs_source* src,
                const void* E_fwd, const Kvec& kv) {
  auto& A = p->act;
  if (A.on) return fail(CBS_E_STATE, "a solve is already in progress on this plan");
  if (int rc = enqueue_solve_start(p, a, o, src, E_fwd, kv)) return rc;
  const bool plane = a.src == SRC_PLANE;
  HIP_TRY(hipEventRecord(p->ev0, p->stream));
  if (!a.fused && (a.src == SRC_FIELD || a.src == SRC_FIELD_CONJ)) {
    a.rows = p->rows;   // 256-byte aligned and padded: cleared in words
    const int words = (3 * p->nz * p->ny + 3) / 4;
    hipLaunchKernelGGL(k_clear_words, dim3((words + 255) / 256), dim3(256), 0, p->stream,
                       reinterpret_cast<unsigned*>(a.rows), words);
    HIP_LAUNCHED();
  }
  enqueue_prologue(p, a);
  HIP_LAUNCHED();
  A.on = true;
  A.stopped = false;
  A.plane = plane;
  A.flags = o->flags;
  A.max_iter = o->max_iter;
  A.tol = o->tol;
  A.enqueued = 0;
  A.head = A.count = 0;
  A.ms = 0.f;
  A.args = a;
  std::memset(&p->last, 0, sizeof(DevState));
  return CBS_OK;
}

// Enqueue up to `iters` iterations and an asynchronous copy of the device
// state into the next pinned slot; never blocks.
int advance_solve(cbs_plan_s* p, int iters) {
  auto& A = p->act;
  if (!A.on) return fail(CBS_E_STATE, "no solve in progress (cbs_solve_begin first)");
  if (iters < 1) return fail(CBS_E_INVALID, "iters must be >= 1");
  if (A.stopped || A.enqueued >= A.max_iter) return CBS_OK;
  if (A.count == cbs_plan_s::kRing)
    return fail(CBS_E_STATE, "%d quanta already outstanding; poll before advancing", A.count);
  const int q = std::min(iters, A.max_iter - A.enqueued);
  for (int i = 0; i < q; ++i) {
    int rc = enqueue_iteration(p, A.args, A.enqueued + i + 1 >= A.max_iter);
    if (rc != CBS_OK) return rc;
  }
  A.enqueued += q;
  if (int rc = enqueue_residual(p, A.args)) return rc;
  const int slot = (A.head + A.count) % cbs_plan_s::kRing;
  HIP_TRY(hipMemcpyAsync(&p->mirror[slot], p->state, sizeof(DevState), hipMemcpyDeviceToHost,
                         p->stream));
  HIP_TRY(hipEventRecord(p->evq[slot], p->stream));
  A.count++;
  return CBS_OK;
}

// Retire completed quanta in order; never blocks.
int poll_solve(cbs_plan_s* p, int* done) {
  auto& A = p->act;
  if (!A.on) return fail(CBS_E_STATE, "no solve in progress");
  while (A.count > 0) {
    const hipError_t e = hipEventQuery(p->evq[A.head]);
    if (e == hipErrorNotReady) break;
    if (e != hipSuccess) return fail(CBS_E_HIP, "hipEventQuery: %s", hipGetErrorString(e));
    p->last = p->mirror[A.head];
    if (p->last.done && !A.stopped) {
      A.stopped = true;
      HIP_TRY(hipEventElapsedTime(&A.ms, p->ev0, p->evq[A.head]));
    }
    A.head = (A.head + 1) % cbs_plan_s::kRing;
    A.count--;
  }
  if (done) *done = A.stopped ? 1 : 0;
  return CBS_OK;
}

int wait_solve(cbs_plan_s* p) {
  auto& A = p->act;
  if (A.count > 0) {
    const int tail = (A.head + A.count - 1) % cbs_plan_s::kRing;
    HIP_TRY(hipEventSynchronize(p->evq[tail]));
  }
  return poll_solve(p, nullptr);
}

// Finish: add E_inc for plane-wave solves (enqueued), report stats and status.
int end_solve(cbs_plan_s* p, cbs_stats* stats) {
  auto& A = p->act;
  if (!A.on) return fail(CBS_E_STATE, "no solve in progress");
  int rc = wait_solve(p);
  if (rc) return rc;
  if (!A.stopped) return fail(CBS_E_STATE, "solve has not stopped yet (advance further)");
  A.on = false;
  if (A.plane && !(A.flags & CBS_RETURN_SCATTERED)) {
    hipLaunchKernelGGL(k_incident, dim3(2048), dim3(256), 0, p->stream, A.args, 1.0f);
    HIP_LAUNCHED();
  }
  const DevState& hs = p->last;
  p->hist_len = (A.flags & CBS_RECORD_HISTORY) ? std::min(hs.iter, kHistCap) : 0;
  if (stats) {
    stats->iterations = hs.iter;
    stats->converged = hs.status == 1;
    stats->residual = hs.eta;
    stats->eps_shift = p->eps;
    stats->ms = A.ms;
  }
  if (hs.status == 3) return fail(CBS_E_DIVERGED, "non-finite residual after %d iterations", hs.iter);
  if (hs.status == 1) return CBS_OK;
  g_err = "max_iter reached before the residual met tol";
  return CBS_NOT_CONVERGED;
}

// Blocking solve on top of the primitives: quanta of at most check_every iterations,
// two of them in flight, so the device has work while the host reads the state of
// the one before (a 64^3 iteration takes 20 us and a host round trip about as long:
// 100 iterations 2.13 -> 2.05 ms, 40 iterations of 32^3 0.54 -> 0.51), and sized by
// the residual so that a solve that meets tol leaves little behind (pace.hpp).
int run_blocking(cbs_plan_s* p, int check_every, cbs_stats* stats) {
  auto& A = p->act;
  Pace pace(A.tol, check_every, (A.flags & CBS_WARM_START) != 0, long_iteration(p));
  int done = 0, rc = CBS_OK;
  while (!done) {
    while (!rc && A.count < 2 && A.enqueued < A.max_iter) {
      const int q = pace.next(A.enqueued - p->last.iter);
      if (q == 0) break;
      rc = advance_solve(p, q);
    }
    if (!rc && A.count == 0) rc = fail(CBS_E_STATE, "the device did not stop at max_iter");
    if (rc) break;
    const hipError_t e = hipEventSynchronize(p->evq[A.head]);
    if (e != hipSuccess) rc = fail(CBS_E_HIP, "hipEventSynchronize: %s", hipGetErrorString(e));
    if (rc || (rc = poll_solve(p, &done))) break;
    pace.read(p->last.iter, p->last.eta);
  }
  if (rc) {
    A.on = false;
    (void)hipStreamSynchronize(p->stream);
    return rc;
  }
  rc = end_solve(p, stats);
  const hipError_t e = hipStreamSynchronize(p->stream);
  if (e != hipSuccess) return fail(CBS_E_HIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
  return rc;
}

// Argument checks and source set-up shared by the blocking and the
// asynchronous entry points.
int prepare(cbs_plan_s* p, int adjoint, const cbs_source* src, void* E, const cbs_opts* o,
            CbsArgs& a, Kvec& kv);

// Illumination b of a plane-wave source: polarisation (x if all zero) and the
// wave vector from the transverse direction cosines (normal incidence if zero).
int set_plane_wave(cbs_plan_s* p, CbsArgs& a, Kvec& kv, int b, const cbs_source* src) {
  for (int c = 0; c < 3; ++c) kv.pol[b][c][0] = kv.pol[b][c][1] = 0.0;
  kv.pol[b][0][0] = 1.0;
  double sx = 0.0, sy = 0.0;
  if (src) {
    bool any = false;
    for (int c = 0; c < 3; ++c) any |= (src->pol[c][0] != 0.0 || src->pol[c][1] != 0.0);
    if (any)
      for (int c = 0; c < 3; ++c) {
        kv.pol[b][c][0] = src->pol[c][0];
        kv.pol[b][c][1] = src->pol[c][1];
      }
    sx = src->dir[0];
    sy = src->dir[1];
  }
  if (!std::isfinite(sx) || !std::isfinite(sy) || !(sx * sx + sy * sy < 1.0))
    return fail(CBS_E_INVALID, "plane-wave direction (%g, %g): need sx^2 + sy^2 < 1", sx, sy);
  for (int c = 0; c < 3; ++c)
    if (kv.pol[b][c][0] != 0.0 || kv.pol[b][c][1] != 0.0) a.pol_mask |= 1u << (3 * b + c);
  const double kbd = p->kb * p->pitch;
  kv.kd[b][0] = kbd * sx;
  kv.kd[b][1] = kbd * sy;
  kv.kd[b][2] = kbd * std::sqrt(1.0 - sx * sx - sy * sy);
  if (sx != 0.0 || sy != 0.0) a.oblique = 1;
  return CBS_OK;
}

int set_source(cbs_plan_s* p, CbsArgs& a, const cbs_source* src, bool adjoint, Kvec& kv) {
  const int kind = src ? src->kind : CBS_SRC_PLANE_WAVE;
  kv.nb = 1;
  for (int c = 0; c < 3; ++c) kv.kd[0][c] = kv.pol[0][c][0] = kv.pol[0][c][1] = 0.0;
  kv.pol[0][0][0] = 1.0;
  switch (kind) {
    case CBS_SRC_NONE:
      a.src = SRC_NONE;
      break;
    case CBS_SRC_PLANE_WAVE: {
      if (adjoint) return fail(CBS_E_INVALID, "adjoint source cannot be a plane wave");
      a.src = SRC_PLANE;
      if (int rc = set_plane_wave(p, a, kv, 0, src)) return rc;
      break;
    }
    case CBS_SRC_FIELD:
    case CBS_SRC_FIELD_CONJ:
      if (!src->field) return fail(CBS_E_INVALID, "FIELD source without a field pointer");
      a.src = kind == CBS_SRC_FIELD ? SRC_FIELD : SRC_FIELD_CONJ;
      a.fin = static_cast<const float2*>(src->field);
      break;
    case CBS_SRC_POINT:
      for (int c = 0; c < 3; ++c) {
        const int n = c == 0 ? p->nx : (c == 1 ? p->ny : p->nz);
        if (src->r0[c] < 0 || src->r0[c] >= n)
          return fail(CBS_E_INVALID, "point source r0[%d]=%d outside [0,%d)", c, src->r0[c], n);
      }
      a.src = SRC_POINT;
      a.r0x = src->r0[0];
      a.r0y = src->r0[1];
      a.r0z = src->r0[2];
      break;
    default:
      return fail(CBS_E_INVALID, "unknown source kind %d", kind);
  }
  return CBS_OK;
}

int prepare(cbs_plan_s* p, int adjoint, const cbs_source* src, void* E, const cbs_opts* o,
            CbsArgs& a, Kvec& kv) {
  int rc = check_plan(p, true);
  if (rc) return rc;
  if ((rc = check_opts(o))) return rc;
  if (!E) return fail(CBS_E_INVALID, "output field is NULL");
  if (adjoint) {
    if (!src) return fail(CBS_E_INVALID, "adjoint source is NULL");
    if (src->kind != CBS_SRC_POINT && src->kind != CBS_SRC_FIELD &&
        src->kind != CBS_SRC_FIELD_CONJ)
      return fail(CBS_E_INVALID, "adjoint source must be POINT, FIELD or FIELD_CONJ");
  }
  a = base_args(p);
  if ((rc = set_source(p, a, src, adjoint != 0, kv))) return rc;
  a.E = static_cast<float2*>(E);
  return CBS_OK;
}

// ---------------------------------------------------------------------------
// allocation-free solve: the workspace of one plan in a static device array
// ---------------------------------------------------------------------------
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];   // device address of cbs_scratch, per device

int static_scratch(void** out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(CBS_E_HIP, "device index %d out of range", dev);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(cbs_scratch)));
    if (!ptr || reinterpret_cast<uintptr_t>(ptr) % 256 != 0)
      return fail(CBS_E_HIP, "static scratch of device %d has no usable address", dev);
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return CBS_OK;
}

// The blocking solve loop without events or a pinned ring: enqueue
// check_every iterations and the residual, read the device state back
// synchronously, repeat until the device has stopped.
int run_static(cbs_plan_s* p, CbsArgs& a, const cbs_opts* o, const cbs_source* src,
               const Kvec& kv, cbs_stats* stats) {
  const auto t0 = std::chrono::steady_clock::now();
  if (int rc = enqueue_solve_start(p, a, o, src, nullptr, kv)) return rc;
  enqueue_prologue(p, a);
  HIP_LAUNCHED();
  DevState hs;
  std::memset(&hs, 0, sizeof(hs));
  int enqueued = 0;
  Pace pace(o->tol, o->check_every, a.warm != 0, long_iteration(p));
  for (;;) {
    const int q = std::min(pace.next(0), o->max_iter - enqueued);
    for (int i = 0; i < q; ++i)
      if (int rc = enqueue_iteration(p, a, enqueued + i + 1 >= o->max_iter)) return rc;
    enqueued += q;
    if (int rc = enqueue_residual(p, a)) return rc;
    HIP_TRY(hipMemcpyAsync(&hs, p->state, sizeof(DevState), hipMemcpyDeviceToHost, p->stream));
    HIP_TRY(hipStreamSynchronize(p->stream));
    if (hs.done || enqueued >= o->max_iter) break;
    pace.read(hs.iter, hs.eta);
  }
  if (a.src == SRC_PLANE && !(o->flags & CBS_RETURN_SCATTERED)) {
    hipLaunchKernelGGL(k_incident, dim3(2048), dim3(256), 0, p->stream, a, 1.0f);
    HIP_LAUNCHED();
  }
  HIP_TRY(hipStreamSynchronize(p->stream));
  const double ms =
      std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  if (stats) {
    stats->iterations = hs.iter;
    stats->converged = hs.status == 1;
    stats->residual = hs.eta;
    stats->eps_shift = p->eps;
    stats->ms = (float)ms;
  }
  if (hs.status == 3) return fail(CBS_E_DIVERGED, "non-finite residual after %d iterations", hs.iter);
  if (hs.status == 1) return CBS_OK;
  g_err = "max_iter reached before the residual met tol";
  return CBS_NOT_CONVERGED;
}

}  // namespace

extern "C" {

int cbs_solve_static(int nx, int ny, int nz, double pitch_m, double lambda0_m, double n_bg,
                     const int pml[3], const void* eps_r_dev, int dtype, const cbs_source* src,
                     void* E_dev, const cbs_opts* opts, cbs_stats* stats, void* stream) {
  int pm[3];
  if (int rc = check_grid(nx, ny, nz, pitch_m, lambda0_m, n_bg, pml, pm)) return rc;
  Layout L;
  layout_of(nx, ny, nz, L);
  if (L.total > CBS_STATIC_SCRATCH_BYTES)
    return fail(CBS_E_WORKSPACE,
                "grid %dx%dx%d needs %zu bytes of scratch; the static scratch holds %zu "
                "(use cbs_plan_create with a workspace)",
                nx, ny, nz, L.total, (size_t)CBS_STATIC_SCRATCH_BYTES);
  if (int rc = check_opts(opts)) return rc;
  if (!eps_r_dev || !E_dev) return fail(CBS_E_INVALID, "eps_r or the output field is NULL");
  void* base = nullptr;
  if (int rc = static_scratch(&base)) return rc;
  cbs_plan_s p{};   // on the stack: no events, no pinned memory
  init_plan(&p, nx, ny, nz, pitch_m, lambda0_m, n_bg, pm, base, static_cast<hipStream_t>(stream));
  Tables t;         // host staging of the tables, consumed before set-up returns
  HIP_TRY(upload_tables(&p, t));
  hipLaunchKernelGGL(k_clear_words, dim3(1), dim3(64), 0, p.stream,
                     reinterpret_cast<unsigned*>(p.state), (int)(sizeof(DevState) / 4));
  HIP_LAUNCHED();
  if (int rc = set_permittivity_impl(&p, eps_r_dev, dtype)) return rc;   // synchronises
  CbsArgs a;
  Kvec kv;
  if (int rc = prepare(&p, 0, src, E_dev, opts, a, kv)) return rc;
  return run_static(&p, a, opts, src, kv, stats);
}


size_t cbs_plan_workspace_bytes(int nx, int ny, int nz) {
  if (nx < 2 || ny < 2 || nz < 2) return 0;
  if (!cbs_axis_supported(0, nx) || !cbs_axis_supported(1, ny) || !cbs_axis_supported(2, nz))
    return 0;
  Layout L;
  if (!layout_of(nx, ny, nz, L)) return 0;
  return L.total;
}

int cbs_axis_supported(int axis, int n) {
  const SizeOps* o = find_size(n);
  if (!o) return 0;
  if (axis == 2) return o->kz != nullptr;
  return (axis == 0 || axis == 1) ? 1 : 0;
}

int cbs_plan_create(cbs_plan_t* out, int nx, int ny, int nz, double pitch_m, double lambda0_m,
                    double n_bg, const int pml[3], void* workspace, size_t workspace_bytes,
                    void* stream) {
  if (!out) return fail(CBS_E_INVALID, "out is NULL");
  *out = nullptr;
  int pm[3];
  if (int rc = check_grid(nx, ny, nz, pitch_m, lambda0_m, n_bg, pml, pm)) return rc;
  Layout L;
  layout_of(nx, ny, nz, L);
  if (!workspace) return fail(CBS_E_WORKSPACE, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
    return fail(CBS_E_WORKSPACE, "workspace must be 256-byte aligned");
  if (workspace_bytes < L.total)
    return fail(CBS_E_WORKSPACE, "workspace %zu bytes < required %zu", workspace_bytes, L.total);

  cbs_plan_s* p = new (std::nothrow) cbs_plan_s();
  if (!p) return fail(CBS_E_INVALID, "out of host memory");
  init_plan(p, nx, ny, nz, pitch_m, lambda0_m, n_bg, pm, workspace,
            static_cast<hipStream_t>(stream));
  // events are created null and destroyed by cleanup whatever succeeded
  auto cleanup = [&](int rc) {
    if (p->ev0) (void)hipEventDestroy(p->ev0);
    if (p->ev1) (void)hipEventDestroy(p->ev1);
    for (int i = 0; i < 5; ++i)
      if (p->evp[i]) (void)hipEventDestroy(p->evp[i]);
    for (int i = 0; i < cbs_plan_s::kRing; ++i)
      if (p->evq[i]) (void)hipEventDestroy(p->evq[i]);
    if (p->mirror) (void)hipHostFree(p->mirror);
    delete p;
    return rc;
  };
  if (hipEventCreate(&p->ev0) != hipSuccess || hipEventCreate(&p->ev1) != hipSuccess)
    return cleanup(fail(CBS_E_HIP, "hipEventCreate failed"));
  for (int i = 0; i < 5; ++i)
    if (hipEventCreate(&p->evp[i]) != hipSuccess) return cleanup(fail(CBS_E_HIP, "hipEventCreate failed"));
  for (int i = 0; i < cbs_plan_s::kRing; ++i)
    if (hipEventCreate(&p->evq[i]) != hipSuccess) return cleanup(fail(CBS_E_HIP, "hipEventCreate failed"));
  if (hipHostMalloc((void**)&p->mirror, cbs_plan_s::kRing * sizeof(DevState), hipHostMallocDefault) != hipSuccess)
    return cleanup(fail(CBS_E_HIP, "hipHostMalloc of the state mirror failed"));
  Tables* t = new (std::nothrow) Tables;
  if (!t) return cleanup(fail(CBS_E_INVALID, "out of host memory"));
  hipError_t e = upload_tables(p, *t);
  e = e == hipSuccess ? hipMemsetAsync(p->W, 0, L.V0 - L.W, p->stream) : e;
  e = e == hipSuccess ? hipMemsetAsync(p->state, 0, sizeof(DevState), p->stream) : e;
  const hipError_t es = hipStreamSynchronize(p->stream);
  delete t;
  e = e == hipSuccess ? es : e;
  if (e != hipSuccess) return cleanup(fail(CBS_E_HIP, "plan upload: %s", hipGetErrorString(e)));
  *out = p;
  return CBS_OK;
}

int cbs_plan_set_pml_profile(cbs_plan_t p, int order, double sigma_max) {
  int rc = check_plan(p, false);
  if (rc) return rc;
  if (order < 1 || order > 8) return fail(CBS_E_INVALID, "order must be in [1, 8]");
  if (!(sigma_max >= 0) || !std::isfinite(sigma_max)) return fail(CBS_E_INVALID, "sigma_max must be >= 0");
  p->order = order;
  p->sigma_max = sigma_max;
  p->have_eps = false;
  p->eps = -1.0;
  return CBS_OK;
}

int cbs_plan_set_shift_factor(cbs_plan_t p, double kappa) {
  int rc = check_plan(p, false);
  if (rc) return rc;
  if (!(kappa >= 1.0) || !std::isfinite(kappa)) return fail(CBS_E_INVALID, "shift factor must be >= 1 (got %g)", kappa);
  p->shift_factor = kappa;
  p->have_eps = false;
  p->eps = -1.0;
  return CBS_OK;
}

int cbs_set_permittivity(cbs_plan_t p, const void* eps_r, int dtype) {
  int rc = check_plan(p, false);
  if (rc) return rc;
  return set_permittivity_impl(p, eps_r, dtype);
}

double cbs_eps_shift(cbs_plan_t p) { return (p && p->have_eps) ? p->eps : -1.0; }

int cbs_solve(cbs_plan_t p, const cbs_source* src, void* E_dev, const cbs_opts* o,
              cbs_stats* stats) {
  CbsArgs a;
  Kvec kv;
  int rc = prepare(p, 0, src, E_dev, o, a, kv);
  if (rc) return rc;
  if ((rc = begin_solve(p, a, o, src, nullptr, kv))) return rc;
  return run_blocking(p, o->check_every, stats);
}

int cbs_adjoint_solve(cbs_plan_t p, const void* E_fwd, const cbs_source* adj, void* E_adj,
                      const cbs_opts* o, cbs_stats* stats) {
  CbsArgs a;
  Kvec kv;
  int rc = prepare(p, 1, adj, E_adj, o, a, kv);
  if (rc) return rc;
  if ((rc = begin_solve(p, a, o, adj, E_fwd, kv))) return rc;
  return run_blocking(p, o->check_every, stats);
}

int cbs_solve_begin(cbs_plan_t p, int adjoint, const void* E_fwd, const cbs_source* src,
                    void* E_dev, const cbs_opts* o) {
  CbsArgs a;
  Kvec kv;
  int rc = prepare(p, adjoint, src, E_dev, o, a, kv);
  if (rc) return rc;
  // The caller's quanta, several of them in flight, may stay behind a solve that meets
  // tol: past the L2s' 32 MB a stopped pass looks before it reads.  Two quanta of 29
  // (17) behind one iteration: 121 x 189 x 100 2.48 -> 0.80 ms, 189 x 189 x 121 2.50 ->
  // 0.75, 128^3 (quanta of 31) 1.26 -> 0.89; their iterations 0 to 0.5% longer.
  if (24LL * p->nxp * p->ny * p->nz > 32LL << 20) a.flag_first = a.z_first = 1;
  return begin_solve(p, a, o, src, adjoint ? E_fwd : nullptr, kv);
}

int cbs_solve_advance(cbs_plan_t p, int iters) {
  int rc = check_plan(p, true);
  if (rc) return rc;
  return advance_solve(p, iters);
}

int cbs_solve_poll(cbs_plan_t p, int* done, int* outstanding) {
  int rc = check_plan(p, true);
  if (rc) return rc;
  rc = poll_solve(p, done);
  if (outstanding) *outstanding = p->act.count;
  return rc;
}

int cbs_solve_end(cbs_plan_t p, cbs_stats* stats) {
  int rc = check_plan(p, true);
  if (rc) return rc;
  return end_solve(p, stats);
}

namespace {
struct BatchLayout {
  size_t W, partials, phx, phy, phz, total;
};
bool batch_layout(int nx, int ny, int nz, int count, BatchLayout& B) {
  const SizeOps* ox = find_size(nx);
  if (!ox || count < 1 || count > kMaxIllum) return false;
  const long long k1b = 3LL * ((ny + ox->k1_rows - 1) / ox->k1_rows) * nz;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  // the fields follow each other with no padding: W_b = W_0 + 3 b sW
  B.W = take((size_t)count * 3 * nz * ny * padded_pitch(nx) * sizeof(float2));
  B.partials = take((size_t)count * 2 * k1b * sizeof(double));
  B.phx = take((size_t)count * nx * sizeof(float2));
  B.phy = take((size_t)count * ny * sizeof(float2));
  B.phz = take((size_t)count * 3 * nz * sizeof(float2));
  B.total = off;
  return true;
}
}  // namespace

size_t cbs_batch_workspace_bytes(int nx, int ny, int nz, int count) {
  if (!cbs_plan_workspace_bytes(nx, ny, nz)) return 0;
  BatchLayout B;
  return batch_layout(nx, ny, nz, count, B) ? B.total : 0;
}

int cbs_solve_batch(cbs_plan_t p, int count, const cbs_source* srcs, void* E_dev,
                    const cbs_opts* o, cbs_stats* stats, void* work, size_t work_bytes) {
  int rc = check_plan(p, true);
  if (rc) return rc;
  if ((rc = check_opts(o))) return rc;
  if (count < 1 || count > kMaxIllum)
    return fail(CBS_E_INVALID, "count %d outside [1, %d]", count, kMaxIllum);
  if (!srcs || !E_dev) return fail(CBS_E_INVALID, "sources or the output field is NULL");
  BatchLayout B;
  batch_layout(p->nx, p->ny, p->nz, count, B);
  if (!work) return fail(CBS_E_WORKSPACE, "batch workspace is NULL");
  if (reinterpret_cast<uintptr_t>(work) % 256 != 0)
    return fail(CBS_E_WORKSPACE, "batch workspace must be 256-byte aligned");
  if (work_bytes < B.total)
    return fail(CBS_E_WORKSPACE, "batch workspace %zu bytes < required %zu", work_bytes, B.total);
  CbsArgs a = base_args(p);
  Kvec kv;
  kv.nb = count;
  a.src = SRC_PLANE;
  for (int b = 0; b < count; ++b) {
    if (srcs[b].kind != CBS_SRC_PLANE_WAVE)
      return fail(CBS_E_INVALID, "batched source %d is not a plane wave", b);
    if ((rc = set_plane_wave(p, a, kv, b, &srcs[b]))) return rc;
  }
  char* base = static_cast<char*>(work);
  set_illuminations(p, a, count);
  a.W = reinterpret_cast<float2*>(base + B.W);
  a.partials = reinterpret_cast<double*>(base + B.partials);
  a.phx = reinterpret_cast<float2*>(base + B.phx);
  a.phy = reinterpret_cast<float2*>(base + B.phy);
  a.phase = reinterpret_cast<float2*>(base + B.phz);
  a.E = static_cast<float2*>(E_dev);
  if ((rc = begin_solve(p, a, o, nullptr, nullptr, kv))) return rc;
  cbs_stats st;
  rc = run_blocking(p, o->check_every, &st);
  if (rc < 0 && rc != CBS_E_DIVERGED) return rc;
  if (stats)
    for (int b = 0; b < count; ++b) {
      stats[b] = st;
      stats[b].residual = p->last.eta_b[b];
      stats[b].converged = p->last.eta_b[b] <= o->tol ? 1 : 0;
    }
  return rc;
}

int cbs_batch_step(cbs_plan_t* plans, int count, int iters, int* done_out) {
  if (count < 0 || (count > 0 && (!plans || !done_out)))
    return fail(CBS_E_INVALID, "bad plan array");
  for (int i = 0; i < count; ++i) {
    int rc = check_plan(plans[i], true);
    if (rc) return rc;
    if (!plans[i]->act.on) return fail(CBS_E_STATE, "plan %d has no solve in progress", i);
  }
  // enqueue every plan's quantum first (each on its own stream), then wait
  for (int i = 0; i < count; ++i) {
    int rc = advance_solve(plans[i], iters);
    if (rc) return rc;
  }
  for (int i = 0; i < count; ++i) {
    int rc = wait_solve(plans[i]);
    if (rc) return rc;
    done_out[i] = plans[i]->act.stopped ? 1 : 0;
  }
  return CBS_OK;
}

int cbs_gradient(cbs_plan_t p, const void* E, const void* Ea, const int lo[3], const int hi[3],
                 double scale, float* grad) {
  int rc = check_plan(p, false);
  if (rc) return rc;
  if (!E || !Ea || !grad || !lo || !hi) return fail(CBS_E_INVALID, "NULL argument");
  const int dims[3] = {p->nx, p->ny, p->nz};
  for (int a = 0; a < 3; ++a)
    if (lo[a] < 0 || hi[a] > dims[a] || lo[a] > hi[a])
      return fail(CBS_E_INVALID, "box axis %d [%d,%d) outside [0,%d)", a, lo[a], hi[a], dims[a]);
  const int bx = hi[0] - lo[0], by = hi[1] - lo[1], bz = hi[2] - lo[2];
  if ((long long)bx * by * bz == 0) return CBS_OK;
  hipLaunchKernelGGL(k_gradient, dim3(2048), dim3(256), 0, p->stream,
                     static_cast<const float2*>(E), static_cast<const float2*>(Ea),
                     (long long)p->nx * p->ny * p->nz, p->nx, p->ny, lo[0], lo[1], lo[2], bx, by,
                     bz, scale * p->k0 * p->k0, grad);
  HIP_LAUNCHED();
  return CBS_OK;
}

namespace {
// Full width at half maximum of the profile v[0, n) around its sample i0, with
// the half-maximum crossings interpolated linearly between samples; NaN when
// the profile does not fall below half on both sides inside [0, n).
double fwhm_of(const double* v, int n, int i0, double pitch) {
  const double half = 0.5 * v[i0];
  int l = i0;
  while (l > 0 && v[l - 1] >= half) --l;
  int r = i0;
  while (r < n - 1 && v[r + 1] >= half) ++r;
  if (l == 0 || r == n - 1) return std::nan("");
  const double xl = (l - 1) + (half - v[l - 1]) / (v[l] - v[l - 1]);
  const double xr = r + (v[r] - half) / (v[r] - v[r + 1]);
  return (xr - xl) * pitch;
}
}  // namespace

int cbs_lens_metrics(cbs_plan_t p, const void* E, const int lo[3], const int hi[3],
                     double disc_factor, double aperture_m, double e0, cbs_lens_figures* out) {
  int rc = check_plan(p, false);
  if (rc) return rc;
  if (!E || !lo || !hi || !out) return fail(CBS_E_INVALID, "NULL argument");
  if (!(disc_factor > 0) || !(aperture_m > 0) || !(e0 > 0))
    return fail(CBS_E_INVALID, "disc_factor, aperture and e0 must be > 0");
  const int dims[3] = {p->nx, p->ny, p->nz};
  for (int a = 0; a < 3; ++a)
    if (lo[a] < 0 || hi[a] > dims[a] || lo[a] >= hi[a])
      return fail(CBS_E_INVALID, "search box axis %d [%d,%d) empty or outside [0,%d)", a, lo[a],
                  hi[a], dims[a]);
  const float2* F = static_cast<const float2*>(E);
  const long long sE = (long long)p->nx * p->ny * p->nz;
  const int bx = hi[0] - lo[0], by = hi[1] - lo[1], bz = hi[2] - lo[2];
  const long long NB = (long long)bx * by * bz;
  const int nb = (int)std::min<long long>(kMetricBlocks, (NB + kMetricThreads - 1) / kMetricThreads);
  // 1. focus: the maximum of |E|^2 in the box, 2. the profiles through it, and
  // the spectral fields of its plane; the host waits once for focus and profiles
  const int nx = p->nx, ny = p->ny;
  const long long NP = (long long)nx * ny;
  const int nl = nx + ny + p->nz;
  double* focus = p->metrics + 2 * kMetricBlocks;   // 2 values, then the profiles
  double* lines = focus + 2;
  double2* twx = reinterpret_cast<double2*>(lines + ((nl + 1) & ~1));   // 16-byte aligned
  double2* twy = twx + nx;
  double2* pl = twy + ny;   // 4 planes
  hipLaunchKernelGGL(k_argmax_intensity, dim3(nb), dim3(kMetricThreads), 0, p->stream, F, sE, nx, ny,
                     lo[0], lo[1], lo[2], bx, by, bz, p->metrics);
  HIP_LAUNCHED();
  hipLaunchKernelGGL(k_argmax_finish, dim3(1), dim3(64), 0, p->stream, p->metrics, nb, focus);
  HIP_LAUNCHED();
  hipLaunchKernelGGL(k_line_intensity, dim3((nl + 255) / 256), dim3(256), 0, p->stream, F, sE, nx, ny,
                     p->nz, focus, lines);
  HIP_LAUNCHED();
  std::vector<double> prof(nl + 2);
  HIP_TRY(hipMemcpyAsync(prof.data(), focus, (nl + 2) * sizeof(double), hipMemcpyDeviceToHost,
                         p->stream));
  HIP_TRY(hipStreamSynchronize(p->stream));
  const double* lp = prof.data() + 2;
  const double best = prof[0];
  const long long bi = (long long)prof[1];
  const int fx = (int)(bi % nx), fy = (int)((bi / nx) % ny), fz = (int)(bi / NP);
  out->focus[0] = fx;
  out->focus[1] = fy;
  out->focus[2] = fz;
  out->peak = best;
  out->fwhm[0] = fwhm_of(lp, nx, fx, p->pitch);
  out->fwhm[1] = fwhm_of(lp + nx, ny, fy, p->pitch);
  out->fwhm[2] = fwhm_of(lp + nx + ny, p->nz, fz, p->pitch);
  // 3. power through the disc of diameter disc_factor x lateral FWHM: the
  // Poynting flux of the plane's propagating angular spectrum
  out->disc_flux = std::nan("");
  out->eta_f = std::nan("");
  if (std::isfinite(out->fwhm[0]) && std::isfinite(out->fwhm[1])) {
    std::vector<double2> t(nx + ny);
    for (int m = 0; m < nx; ++m) t[m] = make_double2(std::cos(2 * M_PI * m / nx), -std::sin(2 * M_PI * m / nx));
    for (int m = 0; m < ny; ++m) t[nx + m] = make_double2(std::cos(2 * M_PI * m / ny), -std::sin(2 * M_PI * m / ny));
    HIP_TRY(hipMemcpyAsync(twx, t.data(), (nx + ny) * sizeof(double2), hipMemcpyHostToDevice, p->stream));
    const dim3 g((unsigned)std::min<long long>(4096, (NP + 255) / 256)), b(256);
    hipLaunchKernelGGL(k_plane_extract, g, b, 0, p->stream, F, sE, nx, ny, focus, pl, pl + NP);
    HIP_LAUNCHED();
    // 2D DFTs of the first `fields` planes in place
    auto dft2 = [&](int fields, int sign) -> int {
      for (int axis = 0; axis < 2; ++axis) {
        const SizeOps* o = axis == 0 ? p->ox : p->oy;
        const int n = axis == 0 ? nx : ny, ln = axis == 0 ? ny : nx;
        hipLaunchKernelGGL(k_plane_dft, dim3((ln + kDftLines - 1) / kDftLines, fields),
                           dim3(kDftThreads), (size_t)(2 * kDftLines + 1) * n * sizeof(double2),
                           p->stream, pl, nx, ny, axis, sign, o->n1, o->n2, axis == 0 ? twx : twy);
        HIP_LAUNCHED();
      }
      return CBS_OK;
    };
    if ((rc = dft2(2, -1))) return rc;
    const double k = 2.0 * M_PI * p->n_bg / p->lambda0;
    hipLaunchKernelGGL(k_angular_h, g, b, 0, p->stream, pl, pl + NP, pl + 2 * NP, pl + 3 * NP, nx, ny,
                       2.0 * M_PI / (nx * p->pitch), 2.0 * M_PI / (ny * p->pitch), k);
    HIP_LAUNCHED();
    if ((rc = dft2(4, +1))) return rc;
    const double radius = 0.5 * disc_factor * 0.5 * (out->fwhm[0] + out->fwhm[1]) / p->pitch;
    const int nd = (int)std::min<long long>(256, (NP + kMetricThreads - 1) / kMetricThreads);
    const double scale = 1.0 / ((double)NP * (double)NP);   // two unscaled inverse transforms
    hipLaunchKernelGGL(k_disc_flux, dim3(nd), dim3(kMetricThreads), 0, p->stream, pl, pl + NP,
                       pl + 2 * NP, pl + 3 * NP, nx, ny, (double)fx, (double)fy, radius * radius, scale,
                       p->metrics);
    HIP_LAUNCHED();
    double part[256];
    HIP_TRY(hipMemcpyAsync(part, p->metrics, nd * sizeof(double), hipMemcpyDeviceToHost, p->stream));
    HIP_TRY(hipStreamSynchronize(p->stream));
    double sum = 0.0;
    for (int q = 0; q < nd; ++q) sum += part[q];
    out->disc_flux = sum * p->pitch * p->pitch;
    out->eta_f = out->disc_flux / (e0 * e0 * M_PI * 0.25 * aperture_m * aperture_m);
  }
  return CBS_OK;
}

int cbs_tfsf_source(cbs_plan_t p, const cbs_source* src, const int lo[3], const int hi[3],
                    void* S_dev) {
  int rc = check_plan(p, false);
  if (rc) return rc;
  if (!S_dev || !lo || !hi) return fail(CBS_E_INVALID, "NULL argument");
  if (src && src->kind != CBS_SRC_PLANE_WAVE)
    return fail(CBS_E_INVALID, "the TF/SF source injects a plane wave (kind PLANE_WAVE)");
  if (p->act.on) return fail(CBS_E_STATE, "a solve is in progress on this plan");
  const int dims[3] = {p->nx, p->ny, p->nz};
  for (int a = 0; a < 3; ++a)
    if (lo[a] < 0 || hi[a] > dims[a] || lo[a] >= hi[a])
      return fail(CBS_E_INVALID, "box axis %d [%d,%d) empty or outside [0,%d)", a, lo[a], hi[a],
                  dims[a]);
  CbsArgs a = base_args(p);
  Kvec kv;
  kv.nb = 1;
  if ((rc = set_plane_wave(p, a, kv, 0, src))) return rc;
  TfsfAssemble A;
  TfsfArgs& t = A.t;
  t.ntot = p->nx + p->ny + p->nz;
  for (int ax = 0; ax < 3; ++ax) {
    t.n[ax] = dims[ax];
    t.lo[ax] = lo[ax];
    t.hi[ax] = hi[ax];
    t.kd[ax] = kv.kd[0][ax];
  }
  t.off[0] = 0;
  t.off[1] = p->nx;
  t.off[2] = p->nx + p->ny;
  t.pitch = p->pitch;
  t.tab = reinterpret_cast<double2*>(p->W);   // the spectral work field is free between solves
  A.nx = p->nx;
  A.ny = p->ny;
  A.nz = p->nz;
  A.px = p->pml[0];
  A.py = p->pml[1];
  A.pz = p->pml[2];
  A.order = p->order;
  A.sigma_max = p->sigma_max;
  A.kb2 = p->kb * p->kb;
  for (int c = 0; c < 3; ++c) {
    double re = c == 0 ? 1.0 : 0.0, im = 0.0;
    if (src) {
      bool any = false;
      for (int k = 0; k < 3; ++k) any |= (src->pol[k][0] != 0.0 || src->pol[k][1] != 0.0);
      if (any) {
        re = src->pol[c][0];
        im = src->pol[c][1];
      }
    }
    A.q[c] = make_double2(re, im);
  }
  A.S = static_cast<float2*>(S_dev);
  const dim3 g1(t.ntot), b1(64);
  hipLaunchKernelGGL(k_tfsf_forward, g1, b1, 0, p->stream, t);
  HIP_LAUNCHED();
  hipLaunchKernelGGL(k_tfsf_inverse, g1, b1, 0, p->stream, t);
  HIP_LAUNCHED();
  hipLaunchKernelGGL(k_tfsf_assemble, dim3(2048), dim3(256), 0, p->stream, A);
  HIP_LAUNCHED();
  return CBS_OK;
}

int cbs_apply_green(cbs_plan_t p, const void* in, void* out) {
  int rc = check_plan(p, true);
  if (rc) return rc;
  if (!in || !out) return fail(CBS_E_INVALID, "NULL field");
  if (in == out) return fail(CBS_E_INVALID, "in and out must not alias");
  CbsArgs a = base_args(p);
  a.green_in = 1;
  a.fin = static_cast<const float2*>(in);
  a.fout = static_cast<float2*>(out);
  hipLaunchKernelGGL(k_state_init, dim3(1), dim3(64), 0, p->stream, p->state, 0.0, 1, 0);
  HIP_LAUNCHED();
  p->ox->k1(a, K1_FWD, p->stream);
  p->oy->ky(a, -1, p->stream);
  p->oz->kz(a, p->stream);
  p->oy->ky(a, +1, p->stream);
  p->ox->k1(a, K1_INV, p->stream);
  HIP_LAUNCHED();
  return CBS_OK;
}

int cbs_time_passes(cbs_plan_t p, void* E_dev, int iters, float* ms_out) {
  int rc = check_plan(p, true);
  if (rc) return rc;
  if (!E_dev || !ms_out || iters < 1) return fail(CBS_E_INVALID, "bad arguments");
  CbsArgs a = base_args(p);
  Kvec kv;
  if ((rc = set_source(p, a, nullptr, false, kv))) return rc;
  a.E = static_cast<float2*>(E_dev);
  hipLaunchKernelGGL(k_phase_tables, dim3(8), dim3(256), 0, p->stream, p->phx, p->phy, p->phase,
                     p->nx, p->ny, p->nz, kv);
  hipLaunchKernelGGL(k_state_init, dim3(1), dim3(64), 0, p->stream, p->state, 0.0, iters, 0);
  HIP_LAUNCHED();
  enqueue_prologue(p, a);
  constexpr int kSlot[4] = {1, 2, 3, 0};   // launch order -> place in ms_out
  double acc[5] = {0, 0, 0, 0, 0};         // what is not launched stays 0 (events alone: 4 us)
  for (int it = 0; it < iters; ++it) {
    HIP_TRY(hipEventRecord(p->evp[0], p->stream));
    p->oz->kz(a, p->stream);   // reduces the residual, as in a solve
    HIP_TRY(hipEventRecord(p->evp[1], p->stream));
    if (!a.fused) p->oy->ky(a, +1, p->stream);
    HIP_TRY(hipEventRecord(p->evp[2], p->stream));
    if (a.fused)
      p->ox->kxy(a, K1_ITER, p->stream);
    else
      p->ox->k1(a, K1_ITER, p->stream);
    HIP_TRY(hipEventRecord(p->evp[3], p->stream));
    if (!a.fused) p->oy->ky(a, -1, p->stream);
    HIP_TRY(hipEventRecord(p->evp[4], p->stream));
    HIP_LAUNCHED();
    HIP_TRY(hipEventSynchronize(p->evp[4]));
    for (int k = 0; k < 4; ++k) {
      if (a.fused && (k == 1 || k == 3)) continue;   // no y launch
      float ms = 0.f;
      HIP_TRY(hipEventElapsedTime(&ms, p->evp[k], p->evp[k + 1]));
      acc[kSlot[k]] += ms;
    }
  }
  for (int k = 0; k < 5; ++k) ms_out[k] = (float)(acc[k] / iters);
  return CBS_OK;
}

int cbs_bandwidth_probe(const void* src, void* dst, size_t bytes, int reps, void* stream,
                        float* ms_out) {
  if (!src || !dst || !ms_out || reps < 1 || bytes == 0 || bytes % 16 != 0)
    return fail(CBS_E_INVALID, "bandwidth probe: bad arguments");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const long long n4 = (long long)(bytes / 16);
  const long long nb = (n4 + kCopyThreads - 1) / kCopyThreads;
  if (nb > 0x7fffffffLL) return fail(CBS_E_INVALID, "bandwidth probe: buffer too large");
  hipEvent_t e0, e1;
  HIP_TRY(hipEventCreate(&e0));
  HIP_TRY(hipEventCreate(&e1));
  int rc = CBS_OK;
  hipLaunchKernelGGL(k_copy, dim3((unsigned)nb), dim3(kCopyThreads), 0, s,
                     static_cast<const float4*>(src), static_cast<float4*>(dst), n4);
  if (hipEventRecord(e0, s) != hipSuccess) rc = fail(CBS_E_HIP, "hipEventRecord failed");
  for (int r = 0; r < reps && rc == CBS_OK; ++r)
    hipLaunchKernelGGL(k_copy, dim3((unsigned)nb), dim3(kCopyThreads), 0, s,
                       static_cast<const float4*>(src), static_cast<float4*>(dst), n4);
  hipError_t e = hipGetLastError();
  if (rc == CBS_OK && e != hipSuccess) rc = fail(CBS_E_HIP, "kernel launch: %s", hipGetErrorString(e));
  if (rc == CBS_OK && hipEventRecord(e1, s) != hipSuccess) rc = fail(CBS_E_HIP, "hipEventRecord failed");
  if (rc == CBS_OK && hipEventSynchronize(e1) != hipSuccess) rc = fail(CBS_E_HIP, "hipEventSynchronize failed");
  float ms = 0.f;
  if (rc == CBS_OK && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) rc = fail(CBS_E_HIP, "hipEventElapsedTime failed");
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc == CBS_OK) *ms_out = ms / reps;
  return rc;
}

// ---------------------------------------------------------------------------
// stretched-coordinate layer (reference [31]): per-axis operators, the
// operator of the preconditioned system and its GMRES solve
// ---------------------------------------------------------------------------
namespace {

struct ScpmlLayout {
  size_t basis, b, F, u, lam[3], w64[3], part, h, y, total;
};

bool scpml_layout(int nx, int ny, int nz, int restart, ScpmlLayout& S) {
  if (restart < 1 || restart > kScpmlMaxRestart) return false;
  const int dims[3] = {nx, ny, nz};
  for (int a = 0; a < 3; ++a)
    if (dims[a] < 2 || dims[a] > kScpmlMaxAxis) return false;
  const size_t N = (size_t)nx * ny * nz;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  S.basis = take((size_t)(restart + 1) * 3 * N * sizeof(float2));
  S.b = take(3 * N * sizeof(float2));
  S.F = take(3 * N * sizeof(float2));
  S.u = take(3 * N * sizeof(float2));
  for (int a = 0; a < 3; ++a) S.lam[a] = take((size_t)dims[a] * sizeof(float2));
  for (int a = 0; a < 3; ++a) S.w64[a] = take((size_t)dims[a] * sizeof(double2));
  S.part = take((size_t)(kScpmlMaxRestart + 1) * kGmBlocks * sizeof(double2));
  S.h = take((size_t)3 * (kScpmlMaxRestart + 1) * sizeof(double2));
  S.y = take((size_t)(kScpmlMaxRestart + 1) * sizeof(double2));
  S.total = off;
  return true;
}

struct Scpml {
  cbs_plan_s* p;
  int dims[3];
  long long N, n3;            // voxels; complex values of a vector field
  float2 *basis, *b, *F, *u;
  const float2* lam[3];       // 1 - 1/s along each axis
  const double2* w64[3];      // exp(-2 pi i m / n) of each axis
  double2 *part, *h, *y;
  float2* vec(int i) const { return basis + (long long)i * n3; }
};

int scpml_setup(cbs_plan_s* p, const cbs_scpml* layer, int restart, void* work, size_t bytes,
                Scpml& s) {
  if (!layer) return fail(CBS_E_INVALID, "layer parameters are NULL");
  if (!(layer->alpha_max >= 0.0) || !std::isfinite(layer->alpha_max))
    return fail(CBS_E_INVALID, "alpha_max must be finite and >= 0");
  if (layer->order < 1 || layer->order > 8) return fail(CBS_E_INVALID, "order must be in [1, 8]");
  ScpmlLayout S;
  if (!scpml_layout(p->nx, p->ny, p->nz, restart, S))
    return fail(CBS_E_INVALID, "restart must be in [1, %d] and every axis <= %d", kScpmlMaxRestart,
                kScpmlMaxAxis);
  if (!work) return fail(CBS_E_WORKSPACE, "stretched-layer workspace is NULL");
  if (reinterpret_cast<uintptr_t>(work) % 256 != 0)
    return fail(CBS_E_WORKSPACE, "stretched-layer workspace must be 256-byte aligned");
  if (bytes < S.total)
    return fail(CBS_E_WORKSPACE, "stretched-layer workspace %zu bytes < required %zu", bytes, S.total);
  char* base = static_cast<char*>(work);
  s.p = p;
  s.dims[0] = p->nx;
  s.dims[1] = p->ny;
  s.dims[2] = p->nz;
  s.N = (long long)p->nx * p->ny * p->nz;
  s.n3 = 3 * s.N;
  s.basis = reinterpret_cast<float2*>(base + S.basis);
  s.b = reinterpret_cast<float2*>(base + S.b);
  s.F = reinterpret_cast<float2*>(base + S.F);
  s.u = reinterpret_cast<float2*>(base + S.u);
  s.part = reinterpret_cast<double2*>(base + S.part);
  s.h = reinterpret_cast<double2*>(base + S.h);
  s.y = reinterpret_cast<double2*>(base + S.y);
  for (int a = 0; a < 3; ++a) {
    const int n = s.dims[a];
    float2* lam = reinterpret_cast<float2*>(base + S.lam[a]);
    s.lam[a] = lam;
    double2* w64 = reinterpret_cast<double2*>(base + S.w64[a]);
    s.w64[a] = w64;
    hipLaunchKernelGGL(k_scpml_lambda, dim3((n + 127) / 128), dim3(128), 0, p->stream, n, p->pml[a],
                       layer->order, layer->alpha_max, lam, w64);
    HIP_LAUNCHED();
  }
  return CBS_OK;
}

void gm_grid(long long n, dim3& g) {
  g = dim3((unsigned)std::min<long long>((n + kGmThreads - 1) / kGmThreads, 8192));
}

// F = alpha (L_s - L) v:  per component c, sum_{b != c} A_b v_c + B_c v_c +
// T_c Z + (S_c^-1 - I) T_c X with X = sum_b S_b^-1 T_b v_b and Z = sum_b (S_b^-1 -
// I) T_b v_b.  The first launch of each axis b forms its A_b and B_b terms of
// every component and u_b = T_b v_b, the second the X and Z terms of component b
// (an axis without a layer has A = B = 0 and S^-1 = I exactly).
int enqueue_delta(const Scpml& s, const float2* v, float2* F, float alpha) {
  cbs_plan_s* p = s.p;
  ScAxis a;
  a.v = v;
  a.F = F;
  a.u = s.u;
  for (int b = 0; b < 3; ++b) a.lam[b] = s.lam[b];
  a.nx = p->nx;
  a.ny = p->ny;
  a.nz = p->nz;
  a.alpha = alpha;
  const LaunchSc launch[3] = {p->ox->scx, p->oy->scy, p->oz->scz};
  const float2* tw[3] = {p->twx, p->twy, p->twz};
  for (int grad = 0; grad < 2; ++grad) {
    if (grad) {
      dim3 g;
      gm_grid(s.N, g);
      hipLaunchKernelGGL(sc_combine, g, dim3(256), 0, p->stream, a);
      HIP_LAUNCHED();
    }
    for (int b = 0; b < 3; ++b) {
      a.axis = b;
      a.first = b == 0 ? 1 : 0;
      a.p = p->pml[b];
      a.tw = tw[b];
      a.w64 = s.w64[b];
      launch[b](a, grad != 0, p->stream);
      HIP_LAUNCHED();
    }
  }
  return CBS_OK;
}


// w = B v = v - (the CBS step from v with the field source -(L_s - L) v):
// B = gamma [I - G (V - (L_s - L))], the CBS-preconditioned stretched operator.
// v minus its step is the negative of the step's update, which the x pass writes
// to w itself (K1_RES): v is neither copied nor subtracted from.  w = scale B v.
int enqueue_operator(const Scpml& s, const float2* v, float2* w, double scale) {
  cbs_plan_s* p = s.p;
  int rc = enqueue_delta(s, v, s.F, -1.0f);
  if (rc) return rc;
  CbsArgs a = base_args(p);
  a.E = const_cast<float2*>(v);   // read only: warm prologue and K1_RES
  a.fout = w;
  a.res_scale = (float)scale;
  a.src = SRC_FIELD;
  a.fin = s.F;
  a.src_scale = 1.0f;   // F is already in units of the pitch
  a.warm = 1;
  enqueue_prologue(p, a);
  p->oz->kz(a, p->stream);
  if (a.fused) {
    p->ox->kxy(a, K1_RES, p->stream);
  } else {
    p->oy->ky(a, +1, p->stream);
    p->ox->k1(a, K1_RES, p->stream);
  }
  HIP_LAUNCHED();
  return CBS_OK;
}

// h[0..cnt) = V[0..cnt)^H w (vectors of n3 values, V_i = V + i n3); with self,
// h[cnt] = |w|^2 too
int enqueue_dots(const Scpml& s, const float2* V, int cnt, const float2* w, double2* h,
                 bool self = false) {
  const int all = cnt + (self ? 1 : 0);
  hipLaunchKernelGGL(k_gm_dots, dim3(kGmBlocks, (all + kGmGroup - 1) / kGmGroup), dim3(kGmThreads),
                     0, s.p->stream, V, s.n3, cnt, all, w, s.n3, s.part);
  HIP_LAUNCHED();
  hipLaunchKernelGGL(k_gm_dots_finish, dim3(all), dim3(kGmThreads), 0, s.p->stream, s.part,
                     kGmBlocks, h);
  HIP_LAUNCHED();
  return CBS_OK;
}

// w += sign sum_i c_i / nrm_i V_i (nrm null: 1); with norm, *norm = |w|^2 afterwards
int enqueue_update(const Scpml& s, int cnt, const double2* c, const double2* nrm, float sign,
                   float2* w, double2* norm = nullptr) {
  hipLaunchKernelGGL(k_gm_update, dim3(kGmUpdateBlocks), dim3(kGmThreads), 0, s.p->stream, s.basis,
                     s.n3, cnt, c, nrm, sign, w, s.n3, norm ? s.part : nullptr);
  HIP_LAUNCHED();
  if (norm) {
    hipLaunchKernelGGL(k_gm_dots_finish, dim3(1), dim3(kGmThreads), 0, s.p->stream, s.part,
                       kGmUpdateBlocks, norm);
    HIP_LAUNCHED();
  }
  return CBS_OK;
}

int enqueue_scale(const Scpml& s, float2* w, double f, double2* nrm) {
  dim3 g;
  gm_grid(s.n3, g);
  hipLaunchKernelGGL(k_gm_scale, g, dim3(kGmThreads), 0, s.p->stream, w, s.n3, (float)f, nrm);
  HIP_LAUNCHED();
  return CBS_OK;
}

// copy n device double2 to the host and wait for the stream
int read_back(cbs_plan_s* p, const double2* dev, std::complex<double>* host, int n) {
  HIP_TRY(hipMemcpyAsync(host, dev, n * sizeof(double2), hipMemcpyDeviceToHost, p->stream));
  HIP_TRY(hipStreamSynchronize(p->stream));
  return CBS_OK;
}

// |w| from the sum of its squares.  A NaN stays one and is refused by the caller's
// finiteness test (std::max(0.0, NaN) is 0: a vector that overflowed would read as
// a residual of zero).
double norm_of(double sq) { return sq < 0.0 ? 0.0 : std::sqrt(sq); }

// Restarted GMRES(m) on B x = b from x = 0 (x in E_dev).  Arnoldi with
// classical Gram-Schmidt (fused dot and update passes over the basis),
// repeated for a step whose projection shortened w more than tenfold;
// V_j of a step is kept as the update leaves it, with its length: 1 / |V_j| goes
// into the operator's output, the dots and the coefficients instead of a pass
// over the vector (0.2 of 9.8 ms a step at 275 x 275 x 315);
// Givens rotations on the host in FP64; at the end of each cycle the true
// residual b - B x gives the restart vector and the reported residual.
int scpml_gmres(const Scpml& s, float2* x, int m, const cbs_opts* o, double beta0, int* iters,
                double* rel_out, std::vector<double>& hist) {
  cbs_plan_s* p = s.p;
  using cd = std::complex<double>;
  std::vector<cd> H((size_t)(m + 1) * m), cs(m), sn(m), g(m + 1), hv(3 * (m + 1)), y(m + 1);
  std::vector<double> sig(m + 1, 1.0);   // 1 / |V_j|
  double2* h0 = s.h;                     // V^H w
  double2* h1 = s.h + (m + 1);           // the second projection's
  double2* nrm = s.h + 2 * (m + 1);      // |V_j|^2
  auto Hij = [&](int i, int j) -> cd& { return H[(size_t)j * (m + 1) + i]; };
  int total = 0, rc;
  double beta = beta0, rel = 1.0;
  // V_0 = b / beta0
  dim3 gg;
  gm_grid(s.n3, gg);
  hipLaunchKernelGGL(k_gm_copy, gg, dim3(kGmThreads), 0, p->stream, s.b, s.vec(0), s.n3);
  HIP_LAUNCHED();
  if ((rc = enqueue_scale(s, s.vec(0), 1.0 / beta0, nrm))) return rc;
  while (true) {
    std::fill(g.begin(), g.end(), cd(0));
    g[0] = beta;
    int k = 0;
    for (int j = 0; j < m && total < o->max_iter; ++j) {
      float2* w = s.vec(j + 1);
      if ((rc = enqueue_operator(s, s.vec(j), w, sig[j]))) return rc;
      // classical Gram-Schmidt; the sweep over V_0..V_j also gives |w|^2 before
      // the projection (h0[j+1]), the update |w|^2 after it
      if ((rc = enqueue_dots(s, s.basis, j + 1, w, h0, true))) return rc;
      if ((rc = enqueue_update(s, j + 1, h0, nrm, -1.0f, w, nrm + j + 1))) return rc;
      if ((rc = read_back(p, s.h, hv.data(), 3 * (m + 1)))) return rc;
      for (int i = 0; i <= j; ++i) Hij(i, j) = sig[i] * hv[i];
      double nn = hv[2 * (m + 1) + j + 1].real();
      // the projection shortened w more than tenfold: FP32 rounding of the
      // update may have left components along the basis of about 10 ulp of the
      // original length, so project once more (a DGKS-type test)
      if (nn < 1e-2 * hv[j + 1].real()) {
        if ((rc = enqueue_dots(s, s.basis, j + 1, w, h1))) return rc;
        if ((rc = enqueue_update(s, j + 1, h1, nrm, -1.0f, w, nrm + j + 1))) return rc;
        if ((rc = read_back(p, s.h, hv.data(), 3 * (m + 1)))) return rc;
        for (int i = 0; i <= j; ++i) Hij(i, j) += sig[i] * hv[(m + 1) + i];
        nn = hv[2 * (m + 1) + j + 1].real();
      }
      const double hn = norm_of(nn);
      Hij(j + 1, j) = hn;
      for (int i = 0; i <= j; ++i)
        if (!std::isfinite(Hij(i, j).real()) || !std::isfinite(Hij(i, j).imag()))
          return fail(CBS_E_DIVERGED, "non-finite Arnoldi coefficient after %d steps", total);
      if (!std::isfinite(hn)) return fail(CBS_E_DIVERGED, "non-finite norm after %d steps", total);
      sig[j + 1] = hn > 0.0 ? 1.0 / hn : 1.0;
      // previous rotations, then the one that zeroes H(j+1, j)
      for (int i = 0; i < j; ++i) {
        const cd t = cs[i] * Hij(i, j) + sn[i] * Hij(i + 1, j);
        Hij(i + 1, j) = -std::conj(sn[i]) * Hij(i, j) + cs[i] * Hij(i + 1, j);
        Hij(i, j) = t;
      }
      const cd a = Hij(j, j);
      const double r = std::hypot(std::abs(a), hn);
      cs[j] = r > 0 ? cd(std::abs(a) / r) : cd(1.0);
      sn[j] = r > 0 ? (std::abs(a) > 0 ? (a / std::abs(a)) * hn / r : cd(1.0)) : cd(0.0);
      Hij(j, j) = cs[j] * a + sn[j] * hn;
      Hij(j + 1, j) = 0.0;
      g[j + 1] = -std::conj(sn[j]) * g[j];
      g[j] = cs[j] * g[j];
      ++total;
      ++k;
      const double est = std::abs(g[j + 1]) / beta0;
      hist.push_back(est);
      if (est <= o->tol || hn <= 1e-300) break;
    }
    // x += V y, H(0..k, 0..k) y = g
    for (int i = k - 1; i >= 0; --i) {
      cd t = g[i];
      for (int l = i + 1; l < k; ++l) t -= Hij(i, l) * y[l];
      y[i] = t / Hij(i, i);
    }
    for (int i = 0; i < k; ++i) y[i] *= sig[i];
    if (k > 0) {
      HIP_TRY(hipMemcpyAsync(s.y, y.data(), k * sizeof(double2), hipMemcpyHostToDevice, p->stream));
      if ((rc = enqueue_update(s, k, s.y, nullptr, 1.0f, x))) return rc;
    }
    // true residual r = b - B x into V_0
    if ((rc = enqueue_operator(s, x, s.vec(0), 1.0))) return rc;
    hipLaunchKernelGGL(k_gm_rsub, gg, dim3(kGmThreads), 0, p->stream, s.b, s.vec(0), s.n3);
    HIP_LAUNCHED();
    if ((rc = enqueue_dots(s, nullptr, 0, s.vec(0), s.h, true))) return rc;
    if ((rc = read_back(p, s.h, hv.data(), 1))) return rc;   // also retires the y upload
    beta = norm_of(hv[0].real());
    if (!std::isfinite(beta)) return fail(CBS_E_DIVERGED, "non-finite residual after %d steps", total);
    rel = beta / beta0;
    if (rel <= o->tol || total >= o->max_iter || k == 0) break;
    if ((rc = enqueue_scale(s, s.vec(0), 1.0 / beta, nrm))) return rc;
  }
  *iters = total;
  *rel_out = rel;
  return CBS_OK;
}

}  // namespace

size_t cbs_scpml_workspace_bytes(int nx, int ny, int nz, int restart) {
  ScpmlLayout S;
  if (!find_size(nx) || !find_size(ny) || !find_size(nz)) return 0;
  return scpml_layout(nx, ny, nz, restart, S) ? S.total : 0;
}

int cbs_scpml_operator(cbs_plan_t p, const cbs_scpml* layer, const void* in, void* out,
                       void* work, size_t work_bytes) {
  int rc = check_plan(p, false);
  if (rc) return rc;
  if (!in || !out) return fail(CBS_E_INVALID, "NULL field");
  if (in == out) return fail(CBS_E_INVALID, "in and out must not alias");
  if (p->act.on) return fail(CBS_E_STATE, "a solve is in progress on this plan");
  Scpml s;
  if ((rc = scpml_setup(p, layer, 1, work, work_bytes, s))) return rc;
  // the operators are in units of the pitch: 1/d^2 gives 1/m^2
  return enqueue_delta(s, static_cast<const float2*>(in), static_cast<float2*>(out),
                       (float)(1.0 / (p->pitch * p->pitch)));
}

int cbs_solve_scpml(cbs_plan_t p, const cbs_source* src, void* E_dev, const cbs_opts* o,
                    const cbs_scpml* layer, cbs_stats* stats, void* work, size_t work_bytes) {
  int rc = check_plan(p, true);
  if (rc) return rc;
  if ((rc = check_opts(o))) return rc;
  if (!E_dev) return fail(CBS_E_INVALID, "output field is NULL");
  if (p->act.on) return fail(CBS_E_STATE, "a solve is in progress on this plan");
  if (p->sigma_max != 0.0)
    return fail(CBS_E_STATE, "the stretched layer replaces the graded potential: set the "
                             "plan's sigma_max to 0 (cbs_plan_set_pml_profile) first");
  if (o->flags & CBS_WARM_START)
    return fail(CBS_E_INVALID, "the stretched-layer solve starts from zero (no CBS_WARM_START)");
  if (!layer) return fail(CBS_E_INVALID, "layer parameters are NULL");
  Scpml s;
  if ((rc = scpml_setup(p, layer, layer->restart, work, work_bytes, s))) return rc;
  const auto t0 = std::chrono::steady_clock::now();
  // b = gamma G S: one CBS step from zero with the solve's source
  CbsArgs a = base_args(p);
  Kvec kv;
  if ((rc = set_source(p, a, src, false, kv))) return rc;
  cbs_opts so = *o;
  so.flags = 0;
  so.tol = -1.0;            // the step count never stops the passes
  so.max_iter = INT_MAX;
  if ((rc = enqueue_solve_start(p, a, &so, src, nullptr, kv))) return rc;
  a.E = s.b;
  a.warm = 0;
  enqueue_prologue(p, a);
  if ((rc = enqueue_iteration(p, a, true))) return rc;
  float2* x = static_cast<float2*>(E_dev);
  dim3 gg;
  gm_grid(s.n3, gg);
  hipLaunchKernelGGL(k_gm_copy, gg, dim3(kGmThreads), 0, p->stream, nullptr, x, s.n3);
  HIP_LAUNCHED();
  std::complex<double> bb;
  if ((rc = enqueue_dots(s, nullptr, 0, s.b, s.h, true))) return rc;
  if ((rc = read_back(p, s.h, &bb, 1))) return rc;
  const double beta0 = norm_of(bb.real());
  if (!std::isfinite(beta0)) return fail(CBS_E_DIVERGED, "non-finite source");
  std::vector<double> hist;
  int iters = 0;
  double rel = 0.0;
  if (beta0 > 0.0 && (rc = scpml_gmres(s, x, layer->restart, o, beta0, &iters, &rel, hist)))
    return rc;
  if (a.src == SRC_PLANE && !(o->flags & CBS_RETURN_SCATTERED)) {
    CbsArgs ai = a;
    ai.E = x;
    hipLaunchKernelGGL(k_incident, dim3(2048), dim3(256), 0, p->stream, ai, 1.0f);
    HIP_LAUNCHED();
  }
  DevState ds;
  HIP_TRY(hipMemcpyAsync(&ds, p->state, sizeof(DevState), hipMemcpyDeviceToHost, p->stream));
  HIP_TRY(hipStreamSynchronize(p->stream));
  if (ds.status == 3) return fail(CBS_E_DIVERGED, "non-finite field in a CBS step");
  p->hist_len = 0;
  if ((o->flags & CBS_RECORD_HISTORY) && !hist.empty()) {
    const int n = std::min<int>((int)hist.size(), kHistCap);
    HIP_TRY(hipMemcpy(p->hist, hist.data(), n * sizeof(double), hipMemcpyHostToDevice));
    p->hist_len = n;
  }
  const bool ok = rel <= o->tol;
  if (stats) {
    stats->iterations = iters;
    stats->converged = ok ? 1 : 0;
    stats->residual = rel;
    stats->eps_shift = p->eps;
    stats->ms = std::chrono::duration<float, std::milli>(std::chrono::steady_clock::now() - t0).count();
  }
  if (ok) return CBS_OK;
  g_err = "max_iter reached before the residual met tol";
  return CBS_NOT_CONVERGED;
}

int cbs_history(cbs_plan_t p, double* out, int max) {
  int rc = check_plan(p, false);
  if (rc) return rc;
  const int n = std::min(max, p->hist_len);
  if (n > 0 && out)
    HIP_TRY(hipMemcpy(out, p->hist, n * sizeof(double), hipMemcpyDeviceToHost));
  return p->hist_len;
}

int cbs_plan_destroy(cbs_plan_t p) {
  if (!p) return CBS_OK;
  // outstanding asynchronous copies target the pinned mirror: drain first
  if (p->act.on || p->act.count > 0) (void)hipStreamSynchronize(p->stream);
  (void)hipEventDestroy(p->ev0);
  (void)hipEventDestroy(p->ev1);
  for (int i = 0; i < 5; ++i) (void)hipEventDestroy(p->evp[i]);
  for (int i = 0; i < cbs_plan_s::kRing; ++i) (void)hipEventDestroy(p->evq[i]);
  (void)hipHostFree(p->mirror);
  delete p;
  return CBS_OK;
}

const char* cbs_last_error(void) { return g_err.c_str(); }

}  // extern "C"
