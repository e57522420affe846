// Stretched-coordinate absorbing layer (reference [31] of arXiv 2506.15411,
// named in its simulation-setup paragraph) for the spectral vector operator,
// and the vector kernels of the GMRES solve that uses it.
//
// In a stretched layer every derivative d/da becomes (1/s_a) d/da with
// s_a = 1 + i alpha_max u_a^m (u_a the depth into the layer of axis a, the
// graded potential's u).  With the solver's spectral derivatives D_a (symbol
// i p), T_a (symbol i pt, pt = p except 0 at the Nyquist bin of an even axis)
// and S_a = diag(s_a), the stretched operator differs from L = F^-1 (|p|^2 I -
// pt pt^T) F by
//
//   ((L_s - L) E)_c = sum_{b != c} A_b E_c + B_c E_c + C_c X - T_c Y,
//   X = sum_b C_b E_b,   Y = sum_b T_b E_b,
//   A_a = D_a^2 - S_a^-1 D_a S_a^-1 D_a,  B_a = T_a^2 - S_a^-1 T_a S_a^-1 T_a,
//   C_a = S_a^-1 T_a,
//
// every term a 1D operator along one axis, applied to all lines of a field by
// FFTs along the axis (scpml_axis.hpp).  Since S^-1 - I vanishes outside the
// layer, C_c X - T_c Y is evaluated as T_c Z + (S_c^-1 - I) T_c X with Z = X - Y =
// sum_b (S_b^-1 - I) T_b E_b: one product T_b E_b per axis gives both X and Z.
// One launch per axis forms its share of sum A E + B E, X and Z from the three
// components, a second one per axis adds the X and Z terms.  Work is in units of
// the pitch (p d in [-pi, pi]).
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace cbs {

constexpr int kScpmlMaxRestart = 64;   // GMRES basis <= 65 vectors
constexpr int kScpmlMaxAxis = 1024;
constexpr int kGmBlocks = 512;         // fixed grid of the FP64 dot products
constexpr int kGmThreads = 256;

__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 zadd(double2 a, double2 b) {
  return make_double2(a.x + b.x, a.y + b.y);
}

// depth u in (0, 1] into a layer of p voxels on each side of an axis of n
// voxels (outermost voxel 1, first layer voxel next to the interior 1/p), else 0
__device__ __forceinline__ double stretch_depth(int i, int n, int p) {
  if (p <= 0) return 0.0;
  if (i < p) return double(p - i) / double(p);
  if (i >= n - p) return double(i - (n - p - 1)) / double(p);
  return 0.0;
}

// lambda = 1 - 1/s over an axis, one thread per voxel, FP64 rounded to FP32 once (1
// minus a rounded 1/s loses what of lambda is below 6e-8: its whole real part where
// a^2 is less).  1/s is applied as 1 - lambda.  w64 = exp(-2 pi i m / n), the twiddles
// of the 64-bit transform.
__global__ void k_scpml_lambda(int n, int pml, int order, double alpha, float2* lam,
                               double2* w64) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n) return;
  const double u = stretch_depth(m, n, pml);
  double um = 1.0;
  for (int k = 0; k < order; ++k) um *= u;
  const double a = alpha * um;   // s = 1 + i a, lambda = (a^2 + i a) / (1 + a^2)
  const double r = a / (1.0 + a * a);
  lam[m] = make_float2((float)(a * r), (float)r);
  double sn, cs;
  sincospi(2.0 * m / n, &sn, &cs);
  w64[m] = make_double2(cs, -sn);
}

// ---------------------------------------------------------------------------
// GMRES vector kernels: fields of n complex FP32 values, reductions in FP64
// ---------------------------------------------------------------------------
__device__ __forceinline__ double2 block_sum_z(double sx, double sy, double2* red) {
  for (int o = 32; o > 0; o >>= 1) {
    sx += __shfl_down(sx, o);
    sy += __shfl_down(sy, o);
  }
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
  if (lane == 0) red[wv] = make_double2(sx, sy);
  __syncthreads();
  double2 r = make_double2(0, 0);
  if (threadIdx.x == 0)
    for (int k = 0; k < (int)blockDim.x / 64; ++k) r = zadd(r, red[k]);
  return r;   // valid in thread 0
}

// part[i][blk] = partial of sum_e conj(V_i[e]) w[e] for i < cnt, and of |w[e]|^2 for
// i = cnt when all = cnt + 1; fixed grid, fixed order, so the result does not
// depend on timing.  A work-group takes kGmGroup vectors, so w is read once for
// all of them, and the group's loads are in flight together: 2.24 ms a step on
// average over a GMRES(40) cycle of 275 x 275 x 315 (6.0 TB/s; one vector per
// work-group, reading w again for each, 3.1 ms).  Non-temporal loads: 2.27 ms.
constexpr int kGmGroup = 8;
__global__ void __launch_bounds__(kGmThreads)
k_gm_dots(const float2* V, long long vstride, int cnt, int all, const float2* w, long long n,
          double2* part) {
  __shared__ double2 red[kGmGroup][kGmThreads / 64];
  const int i0 = (int)blockIdx.y * kGmGroup;
  const float2* v[kGmGroup];
  // a slot past cnt reads w itself: the norm's slot, or one whose sum is not kept
#pragma unroll
  for (int q = 0; q < kGmGroup; ++q) v[q] = i0 + q < cnt ? V + (i0 + q) * vstride : w;
  double sx[kGmGroup], sy[kGmGroup];
#pragma unroll
  for (int q = 0; q < kGmGroup; ++q) sx[q] = sy[q] = 0.0;
  for (long long e = (long long)blockIdx.x * kGmThreads + threadIdx.x; e < n;
       e += (long long)gridDim.x * kGmThreads) {
    const float2 b = w[e];
    float2 a[kGmGroup];
#pragma unroll
    for (int q = 0; q < kGmGroup; ++q)
      if (i0 + q < all) a[q] = v[q][e];
#pragma unroll
    for (int q = 0; q < kGmGroup; ++q)
      if (i0 + q < all) {
        sx[q] += (double)a[q].x * b.x + (double)a[q].y * b.y;
        sy[q] += (double)a[q].x * b.y - (double)a[q].y * b.x;
      }
  }
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
#pragma unroll
  for (int q = 0; q < kGmGroup; ++q) {
    for (int o = 32; o > 0; o >>= 1) {
      sx[q] += __shfl_down(sx[q], o);
      sy[q] += __shfl_down(sy[q], o);
    }
    if (lane == 0) red[q][wv] = make_double2(sx[q], sy[q]);
  }
  __syncthreads();
  const int q = threadIdx.x;
  if (q < kGmGroup && i0 + q < all) {
    double2 r = red[q][0];
    for (int k = 1; k < kGmThreads / 64; ++k) r = zadd(r, red[q][k]);
    part[(i0 + q) * gridDim.x + blockIdx.x] = r;
  }
}

// h[i] = sum over blocks of part[i][.], one work-group per i
__global__ void __launch_bounds__(kGmThreads)
k_gm_dots_finish(const double2* part, int nblk, double2* h) {
  __shared__ double2 red[kGmThreads / 64];
  const double2* p = part + blockIdx.x * nblk;
  double sx = 0, sy = 0;
  for (int k = threadIdx.x; k < nblk; k += kGmThreads) {
    sx += p[k].x;
    sy += p[k].y;
  }
  const double2 r = block_sum_z(sx, sy, red);
  if (threadIdx.x == 0) h[blockIdx.x] = r;
}

// w += sign sum_{i < cnt} c_i / nrm_i V_i, coefficients c (FP64) and squared norms
// nrm (null: 1) in device memory; with part, part[blk] is a partial of |w|^2 after the update (a sweep over w of its
// own before).  Vectors are added in order; a work-group takes 16 KB pieces of
// each, two vectors' loads in flight together: 2.60 ms a step on average over a
// GMRES(40) cycle of 275 x 275 x 315 (4.9 TB/s), element by element 2.70 with
// eight vectors in flight; more work-groups, non-temporal loads: no faster.
constexpr int kGmUpdateBlocks = 2048;
static_assert(kGmUpdateBlocks <= (kScpmlMaxRestart + 1) * kGmBlocks, "partials fit");
__global__ void __launch_bounds__(kGmThreads)
k_gm_update(const float2* V, long long vstride, int cnt, const double2* c, const double2* nrm,
            float sign, float2* w, long long n, double2* part) {
  __shared__ float2 cf[kScpmlMaxRestart + 1];
  __shared__ double2 red[kGmThreads / 64];
  if (threadIdx.x < cnt) {
    const double f = nrm ? sign / nrm[threadIdx.x].x : sign;
    cf[threadIdx.x] = make_float2((float)(f * c[threadIdx.x].x), (float)(f * c[threadIdx.x].y));
  }
  __syncthreads();
  double s2 = 0.0;
  constexpr int E = 8, G = 2;   // elements of a thread, vectors in flight
  for (long long e0 = (long long)blockIdx.x * (E * kGmThreads) + threadIdx.x; e0 < n;
       e0 += (long long)gridDim.x * (E * kGmThreads)) {
    float2 acc[E];
    bool ok[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
      ok[k] = e0 + k * kGmThreads < n;
      acc[k] = ok[k] ? w[e0 + k * kGmThreads] : make_float2(0.f, 0.f);
    }
    auto add = [&](int i, float2 v, float2& r) {
      r.x = fmaf(cf[i].x, v.x, fmaf(-cf[i].y, v.y, r.x));
      r.y = fmaf(cf[i].x, v.y, fmaf(cf[i].y, v.x, r.y));
    };
    int i = 0;
    for (; i + G <= cnt; i += G) {
      float2 v[G][E];
#pragma unroll
      for (int q = 0; q < G; ++q)
#pragma unroll
        for (int k = 0; k < E; ++k)
          v[q][k] = ok[k] ? V[(i + q) * vstride + e0 + k * kGmThreads] : make_float2(0.f, 0.f);
#pragma unroll
      for (int q = 0; q < G; ++q)
#pragma unroll
        for (int k = 0; k < E; ++k) add(i + q, v[q][k], acc[k]);
    }
    for (; i < cnt; ++i)
#pragma unroll
      for (int k = 0; k < E; ++k)
        if (ok[k]) add(i, V[i * vstride + e0 + k * kGmThreads], acc[k]);
#pragma unroll
    for (int k = 0; k < E; ++k)
      if (ok[k]) {
        w[e0 + k * kGmThreads] = acc[k];
        s2 += (double)acc[k].x * acc[k].x + (double)acc[k].y * acc[k].y;
      }
  }
  if (part) {
    const double2 r = block_sum_z(s2, 0.0, red);
    if (threadIdx.x == 0) part[blockIdx.x] = r;
  }
}

// w = s w, a unit vector: *nrm = 1
__global__ void k_gm_scale(float2* w, long long n, float s, double2* nrm) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *nrm = make_double2(1.0, 0.0);
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x) {
    const float2 v = w[e];
    w[e] = make_float2(s * v.x, s * v.y);
  }
}

// w = a - w
__global__ void k_gm_rsub(const float2* a, float2* w, long long n) {
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x) {
    const float2 x = a[e], v = w[e];
    w[e] = make_float2(x.x - v.x, x.y - v.y);
  }
}

// dst = src (or 0 when src is null)
__global__ void k_gm_copy(const float2* src, float2* dst, long long n) {
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    dst[e] = src ? src[e] : make_float2(0.f, 0.f);
}

}  // namespace cbs
