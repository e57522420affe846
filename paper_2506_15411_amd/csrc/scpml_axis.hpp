// Stretched-derivative products of one axis, by FFTs along the axis's lines.
//
// With D = F^-1 (i p) F, T = F^-1 (i pt) F along an axis, s the layer's stretch
// and lambda = 1 - 1/s (zero outside the layer), the axis's operators of the
// stretched layer (scpml.hpp) are
//   A v = D^2 v - s^-1 D s^-1 D v = lambda (D^2 v) + s^-1 D (lambda (D v)),
//   B v = the same with T,
// the second form with no cancellation outside the layer.  A line takes five
// transforms: forward, the inverses of i p v^ and -p^2 v^, and forward and
// inverse again for D of lambda D v; T v, needed for X and Z, is the first
// inverse of B.  The transforms are the passes' two-level register form
// (kernels.hpp): a work-group holds a few lines in LDS, the spectrum stays in the
// registers of the level-B threads and every level writes where it read.
// Vector work bounds them (five transforms per 104 bytes moved); components are
// separate work-groups, since a loop over them keeps the tables of all three in
// registers.  The operator at 275 x 275 x 315 takes 2.60 ms, dense matrix products
// on the FP32 matrix cores 7.04 ms; at 64^3 89 us against 460; relative error
// against FP64 at 275 x 275 x 315 1.8e-7 (products 6.4e-7) on noise and 9.8e-7 (2.6e-6)
// on a spherical wave at lambda / 16.
#pragma once

namespace cbs {

struct ScAxis {
  const float2* v;      // phase 1: the field [3][nz][ny][nx]
  float2* F;            // result [3][nz][ny][nx]
  float2* u;            // T_b v_b of every axis b, [3][nz][ny][nx]
  const float2* lam[3]; // lambda = 1 - 1/s along x, y and z
  const float2* tw;     // the axis's twiddle table
  const double2* w64;   // exp(-2 pi i m / n) of the axis, m < n, in 64 bits
  int nx, ny, nz;
  int axis;             // 0 = x, 1 = y, 2 = z
  int p;                // layer voxels per side
  int first;            // F is written instead of added to
  float alpha;          // F += alpha ...
};

// Lines per work-group: eight, whose two exchange buffers leave room for four
// work-groups per CU at 275 points (16 columns, two work-groups: y axis of 275 x
// 275 x 315 885 us against 760 in the whole-transform form), four on axes above
// about 600.
template <int N1, int N2, bool ROW>
struct ScGeom {
  static constexpr int N = N1 * N2;
  static constexpr int TX = 2 * N * 8 * 8 <= 76 * 1024 ? 8 : 4;
  static constexpr int P = N % 2 ? N : N + 1;   // ROW: line pitch in LDS
  static constexpr int SIZE = ROW ? TX * P : TX * N;
  static constexpr int THREADS = round64(TX * cmax(N1, N2));
};

// Position of a work-group's lines: line l's element j sits at base + j stride
// (elements of one scalar field: below 2^29, so byte offsets fit 32 bits).
struct ScTile {
  unsigned base;
  unsigned stride;
  bool ok;
};
__device__ __forceinline__ float2& sc_at(float2* f, unsigned e) {
  return *reinterpret_cast<float2*>(reinterpret_cast<char*>(f) + e * 8u);
}
__device__ __forceinline__ float2 sc_at(const float2* f, unsigned e) {
  return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(f) + e * 8u);
}
template <bool ROW, int TX>
__device__ __forceinline__ ScTile sc_tile(const ScAxis& a, unsigned L, int line) {
  ScTile t;
  if constexpr (ROW) {
    const unsigned l = L * TX + line;
    t.ok = line < TX && l < (unsigned)(a.ny * a.nz);
    t.base = l * (unsigned)a.nx;
    t.stride = 1;
  } else {
    const unsigned gx = (unsigned)(a.nx + TX - 1) / TX;
    const int x = (int)(L % gx) * TX + line;
    const unsigned o = L / gx;    // z (y lines) or y (z lines)
    t.ok = line < TX && x < a.nx;
    t.base = o * (unsigned)(a.axis == 1 ? a.nx * a.ny : a.nx) + (unsigned)x;
    t.stride = (unsigned)(a.axis == 1 ? a.nx : a.nx * a.ny);
  }
  return t;
}

// the frequency p of index k (pt when t: 0 at the Nyquist index), and i q v
template <int N>
__device__ __forceinline__ float sc_freq(int k, bool t) {
  const int m = (k < (N + 1) / 2) ? k : k - N;
  if (t && 2 * k == N) return 0.f;
  return (float)((2.0 * 3.14159265358979323846 / N) * (double)m);
}
__device__ __forceinline__ float2 imul(float q, float2 v) { return make_float2(-q * v.y, q * v.x); }

// A layer of at most N2 voxels a side holds elements j2 + N2 q of a level-A task
// for q = 0 and q = N1 - 1 alone (THIN): what lambda multiplies is needed there
// only, and lambda D v is zero elsewhere.  The inverse DFT-N1 for those two
// outputs, and the forward one of those two inputs, are sums of N1 terms, a third
// of the work of a DFT-25 (275 x 275 x 315, layers of 8: x axis 630 -> 457 us, y
// axis 760 -> 573, before the first transform went to 64 bits: 510 and 612; four edge elements or more a side would cost what the full
// transform does, the 48-voxel z layer keeps it).
template <int N1>
__device__ __forceinline__ void edge_out(const float2* b, float2& o0, float2& o1) {
  o0 = o1 = b[0];
  sfor<1, N1>([&](auto K) {
    o0 = cadd(o0, b[CV(K)]);
    o1 = cadd(o1, rot<N1, -CV(K)>(b[CV(K)]));
  });
}
template <int N1>
__device__ __forceinline__ void edge_in(float2 i0, float2 i1, float2* b) {
  sfor<0, N1>([&](auto K) { b[CV(K)] = cadd(i0, rot<N1, CV(K)>(i1)); });
}
constexpr bool sc_thin(int n1, int n2, int p) { return n1 >= 5 && p <= n2; }

// The forward transform of v is taken in 64 bits and rounded once between its
// levels: the symbols p and p^2 multiply what is rounded there by up to 10, where a
// smooth field has p^2 = 0.15 (lambda / 16), so this transform's round-off is most of
// the operator's error on a wave.  Products of 64 bits issue at the rate of those of
// 32 here and need no more registers at once than the later levels do.  Error against
// FP64 on a spherical wave, 32 bits -> 64: 64^3 1.86e-6 -> 6.5e-7, 192 x 192 x 256
// 1.98e-6 -> 6.6e-7, 275 x 275 x 315 2.99e-6 -> 9.8e-7 (dense matrix products: 1.03e-6,
// 1.64e-6, 2.61e-6); operator at 275 x 275 x 315 2.57 -> 2.60 ms, a GMRES step 9.21 ->
// 9.28, 189 x 189 x 121 1.633 -> 1.657.  This is level A, level B is in sc_apply.
template <int N1>
__device__ __forceinline__ void dft_wide(float2 (&b)[N1]) {
  double2 d[N1];
  sfor<0, N1>([&](auto J) { d[CV(J)] = make_double2(b[CV(J)].x, b[CV(J)].y); });
  dft<N1, -1>(d);
  sfor<0, N1>([&](auto J) { b[CV(J)] = make_float2((float)d[CV(J)].x, (float)d[CV(J)].y); });
}

// F_c (+)= alpha [A v_c for c != axis, B v_c for c = axis], u_axis = T v_axis
template <int N1, int N2, bool ROW, bool THIN>
__global__ void __launch_bounds__((ScGeom<N1, N2, ROW>::THREADS)) sc_apply(ScAxis a) {
  using G = ScGeom<N1, N2, ROW>;
  constexpr int N = G::N, TX = G::TX, T = G::THREADS;
  __shared__ float2 l1[G::SIZE], l2[G::SIZE];
  __shared__ float2 tw[N], lam[N];
  const int tid = threadIdx.x;
  for (int i = tid; i < N; i += T) {
    tw[i] = a.tw[i];
    lam[i] = a.lam[a.axis][i];
  }
  const int la = ROW ? tid / N2 : tid % TX, j2 = ROW ? tid % N2 : tid / TX;
  const int lb = ROW ? tid / N1 : tid % TX, k1 = ROW ? tid % N1 : tid / TX;
  const unsigned tiles = gridDim.x / 3, L = xcd_remap(blockIdx.x, gridDim.x);
  const int c = (int)(L / tiles);   // this work-group's component
  const ScTile ta = sc_tile<ROW, TX>(a, L % tiles, la);
  const bool oka = ta.ok && j2 < N2, okb = lb < TX && k1 < N1;
  const long long nvox = (long long)a.nx * a.ny * a.nz;
  // LDS offsets: level-A task's positions j2 + N2 q, level-B task's N2 k1 + q
  constexpr int SP = ROW ? 1 : TX;
  const int pa = ROW ? la * G::P + j2 : j2 * TX + la;
  const int pb = ROW ? lb * G::P + N2 * k1 : N2 * k1 * TX + lb;
  const unsigned g0 = ta.base + j2 * ta.stride;    // global: element j2 + N2 q
  const unsigned gs = N2 * ta.stride;
  const float2* twt = tw + j2 * N1;
  const bool own = c == a.axis;
  const float2* v = a.v + c * nvox;
  float2* F = a.F + c * nvox;
  if (!own && a.p == 0) {   // no layer: A = 0
    if (a.first && oka) sfor<0, N1>([&](auto J) { sc_at(F, g0 + CV(J) * gs) = make_float2(0.f, 0.f); });
    return;
  }
  {
    float2 b[N1];
    if (oka) sfor<0, N1>([&](auto J) { b[CV(J)] = sc_at(v, g0 + CV(J) * gs); });
    __syncthreads();   // the tables are in LDS
    if (oka) {
      dft_wide<N1>(b);
      sfor<0, N1>([&](auto K) { l1[pa + N2 * SP * CV(K)] = b[CV(K)]; });   // twiddled in level B
    }
  }
  const double2 w1 = a.w64[k1 < N1 ? k1 : 0];
  __syncthreads();
  if (okb) {
    float2 w[N2], g[N2];
    double2 d[N2], r = w1;   // r = exp(-2 pi i J k1 / n)
    sfor<0, N2>([&](auto J) {
      const float2 f = l1[pb + SP * CV(J)];
      d[CV(J)] = make_double2(f.x, f.y);
      if constexpr (CV(J) > 0) d[CV(J)] = cmul(d[CV(J)], r);
      if constexpr (CV(J) > 0 && CV(J) + 1 < N2) r = cmul(r, w1);
    });
    dft<N2, -1>(d);
    sfor<0, N2>([&](auto K) {
      w[CV(K)] = make_float2((float)d[CV(K)].x, (float)d[CV(K)].y);
      const float q = sc_freq<N>(k1 + N1 * CV(K), own);
      g[CV(K)] = imul(q * (1.0f / N), w[CV(K)]);
      w[CV(K)] = cscale(w[CV(K)], -q * q * (1.0f / N));
    });
    dft<N2, +1>(g);
    sfor<0, N2>([&](auto J) { l1[pb + SP * CV(J)] = g[CV(J)]; });
    if (a.p > 0) {
      dft<N2, +1>(w);
      sfor<0, N2>([&](auto J) { l2[pb + SP * CV(J)] = w[CV(J)]; });
    }
  }
  __syncthreads();
  if (oka) {
    float2 b[N1];
    sfor<0, N1>([&](auto K) { b[CV(K)] = cmulc(l1[pa + N2 * SP * CV(K)], twt[CV(K)]); });
    float2 e0, e1;
    if (!THIN || own) {
      dft<N1, +1>(b);   // D v (T v) at j2 + N2 q
      e0 = b[0];
      e1 = b[N1 - 1];
    } else {
      edge_out<N1>(b, e0, e1);
    }
    if (own) {
      float2* u = a.u + c * nvox;
      sfor<0, N1>([&](auto J) { sc_at(u, g0 + CV(J) * gs) = b[CV(J)]; });
    }
    if (THIN && a.p > 0) {
      const float2 m0 = lam[j2], m1 = lam[j2 + N2 * (N1 - 1)];
      edge_in<N1>(cmul(m0, e0), cmul(m1, e1), b);
      sfor<0, N1>([&](auto K) { l1[pa + N2 * SP * CV(K)] = cmul(b[CV(K)], twt[CV(K)]); });
      sfor<0, N1>([&](auto K) { b[CV(K)] = cmulc(l2[pa + N2 * SP * CV(K)], twt[CV(K)]); });
      edge_out<N1>(b, e0, e1);
      l2[pa] = e0;
      l2[pa + N2 * SP * (N1 - 1)] = e1;
    } else if (a.p > 0) {
      sfor<0, N1>([&](auto J) { b[CV(J)] = cmul(lam[j2 + N2 * CV(J)], b[CV(J)]); });
      dft<N1, -1>(b);
      sfor<0, N1>([&](auto K) { l1[pa + N2 * SP * CV(K)] = cmul(b[CV(K)], twt[CV(K)]); });
      // D^2 v waits in l2, at this task's own positions
      sfor<0, N1>([&](auto K) { b[CV(K)] = cmulc(l2[pa + N2 * SP * CV(K)], twt[CV(K)]); });
      dft<N1, +1>(b);
      sfor<0, N1>([&](auto J) { l2[pa + N2 * SP * CV(J)] = b[CV(J)]; });
    } else if (a.first) {   // own component without a layer: B = 0
      sfor<0, N1>([&](auto J) { sc_at(F, g0 + CV(J) * gs) = make_float2(0.f, 0.f); });
    }
  }
  if (a.p == 0) return;
  __syncthreads();
  if (okb) {
    float2 w[N2];
    sfor<0, N2>([&](auto J) { w[CV(J)] = l1[pb + SP * CV(J)]; });
    dft<N2, -1>(w);
    sfor<0, N2>([&](auto K) {
      w[CV(K)] = imul(sc_freq<N>(k1 + N1 * CV(K), own) * (1.0f / N), w[CV(K)]);
    });
    dft<N2, +1>(w);
    sfor<0, N2>([&](auto J) { l1[pb + SP * CV(J)] = w[CV(J)]; });
  }
  __syncthreads();
  if (oka) {
    float2 b[N1], f[N1];
    sfor<0, N1>([&](auto J) {
      f[CV(J)] = a.first ? make_float2(0.f, 0.f) : sc_at(F, g0 + CV(J) * gs);
    });
    sfor<0, N1>([&](auto K) { b[CV(K)] = cmulc(l1[pa + N2 * SP * CV(K)], twt[CV(K)]); });
    dft<N1, +1>(b);
    sfor<0, N1>([&](auto J) {
      constexpr bool IN = !THIN || CV(J) == 0 || CV(J) == N1 - 1;   // in the layer
      float2 w = b[CV(J)];
      // lambda D^2 v + s^-1 w with s^-1 = 1 - lambda
      if constexpr (IN) w = cadd(w, cmul(lam[j2 + N2 * CV(J)], csub(l2[pa + N2 * SP * CV(J)], w)));
      sc_at(F, g0 + CV(J) * gs) = make_float2(f[CV(J)].x + a.alpha * w.x, f[CV(J)].y + a.alpha * w.y);
    });
  }
}

// Z = sum_b (s_b^-1 - 1) u_b = -sum_b lambda_b u_b and X = sum_b s_b^-1 u_b = Z +
// sum_b u_b, in place of u_y and u_x.  A launch of its own: accumulated in sc_apply
// X and Z would be read and written by every axis, and formed in sc_grad from three
// fields they cost it its occupancy (256 registers; 586 us against 246 for the x
// axis of 275 x 275 x 315).
static __global__ void __launch_bounds__(256) sc_combine(ScAxis a) {
  const unsigned nvox = (unsigned)a.nx * a.ny * a.nz;
  float2 *u0 = a.u, *u1 = a.u + nvox, *u2 = u1 + nvox;
  for (unsigned i = blockIdx.x * 256 + threadIdx.x; i < nvox; i += gridDim.x * 256) {
    const unsigned l = i / (unsigned)a.nx, x = i - l * a.nx, z = l / (unsigned)a.ny, y = l - z * a.ny;
    const float2 v0 = u0[i], v1 = u1[i], v2 = u2[i];
    const float2 m = cadd(cmul(a.lam[0][x], v0), cadd(cmul(a.lam[1][y], v1), cmul(a.lam[2][z], v2)));
    u0[i] = csub(cadd(v0, cadd(v1, v2)), m);
    u1[i] = make_float2(-m.x, -m.y);
  }
}

// F_axis += alpha [T Z + (s^-1 - 1) T X] with X and Z of sc_combine
template <int N1, int N2, bool ROW, bool THIN>
__global__ void __launch_bounds__((ScGeom<N1, N2, ROW>::THREADS)) sc_grad(ScAxis a) {
  using G = ScGeom<N1, N2, ROW>;
  constexpr int N = G::N, TX = G::TX, T = G::THREADS;
  __shared__ float2 l1[G::SIZE], l2[G::SIZE];
  __shared__ float2 tw[N], lam[N];
  const int tid = threadIdx.x;
  for (int i = tid; i < N; i += T) {
    tw[i] = a.tw[i];
    lam[i] = a.lam[a.axis][i];
  }
  const int la = ROW ? tid / N2 : tid % TX, j2 = ROW ? tid % N2 : tid / TX;
  const int lb = ROW ? tid / N1 : tid % TX, k1 = ROW ? tid % N1 : tid / TX;
  const ScTile ta = sc_tile<ROW, TX>(a, xcd_remap(blockIdx.x, gridDim.x), la);
  const bool oka = ta.ok && j2 < N2, okb = lb < TX && k1 < N1;
  constexpr int SP = ROW ? 1 : TX;
  const int pa = ROW ? la * G::P + j2 : j2 * TX + la;
  const int pb = ROW ? lb * G::P + N2 * k1 : N2 * k1 * TX + lb;
  const unsigned g0 = ta.base + j2 * ta.stride;
  const unsigned gs = N2 * ta.stride;
  const bool layer = a.p > 0;
  const long long nvox = (long long)a.nx * a.ny * a.nz;
  float2* F = a.F + a.axis * nvox;
  const float2 *X = a.u, *Z = a.u + nvox;
  const float2* twt = tw + j2 * N1;
  float2 z[N1], f[N1];
  if (oka) {
    sfor<0, N1>([&](auto J) { z[CV(J)] = sc_at(Z, g0 + CV(J) * gs); });
    if (layer) sfor<0, N1>([&](auto J) { f[CV(J)] = sc_at(X, g0 + CV(J) * gs); });
  }
  __syncthreads();   // the tables are in LDS
  if (oka) {
    dft<N1, -1>(z);
    sfor<0, N1>([&](auto K) { l1[pa + N2 * SP * CV(K)] = cmul(z[CV(K)], twt[CV(K)]); });
    if (layer) {
      dft<N1, -1>(f);
      sfor<0, N1>([&](auto K) { l2[pa + N2 * SP * CV(K)] = cmul(f[CV(K)], twt[CV(K)]); });
    }
    sfor<0, N1>([&](auto J) { f[CV(J)] = sc_at(F, g0 + CV(J) * gs); });
  }
  __syncthreads();
  auto level_b = [&](float2* l) {
    float2 w[N2];
    sfor<0, N2>([&](auto J) { w[CV(J)] = l[pb + SP * CV(J)]; });
    dft<N2, -1>(w);
    sfor<0, N2>([&](auto K) {
      w[CV(K)] = imul(sc_freq<N>(k1 + N1 * CV(K), true) * (1.0f / N), w[CV(K)]);
    });
    dft<N2, +1>(w);
    sfor<0, N2>([&](auto J) { l[pb + SP * CV(J)] = w[CV(J)]; });
  };
  if (okb) {
    level_b(l1);
    if (layer) level_b(l2);
  }
  __syncthreads();
  if (oka) {
    if (layer) {
      sfor<0, N1>([&](auto K) { z[CV(K)] = cmulc(l2[pa + N2 * SP * CV(K)], twt[CV(K)]); });
      if constexpr (THIN) {
        float2 e0, e1;
        edge_out<N1>(z, e0, e1);
        z[0] = e0;
        z[N1 - 1] = e1;
      } else {
        dft<N1, +1>(z);
      }
      sfor<0, N1>([&](auto J) {
        if constexpr (THIN && CV(J) != 0 && CV(J) != N1 - 1) return;
        const float2 w = cmul(lam[j2 + N2 * CV(J)], z[CV(J)]);   // s^-1 - 1 = -lambda
        f[CV(J)] = make_float2(f[CV(J)].x - a.alpha * w.x, f[CV(J)].y - a.alpha * w.y);
      });
    }
    sfor<0, N1>([&](auto K) { z[CV(K)] = cmulc(l1[pa + N2 * SP * CV(K)], twt[CV(K)]); });
    dft<N1, +1>(z);
    sfor<0, N1>([&](auto J) {
      sc_at(F, g0 + CV(J) * gs) =
          make_float2(f[CV(J)].x + a.alpha * z[CV(J)].x, f[CV(J)].y + a.alpha * z[CV(J)].y);
    });
  }
}

// grad: sc_grad instead of sc_apply
template <int N1, int N2, bool ROW>
void launch_sc(const ScAxis& a, bool grad, hipStream_t s) {
  using G = ScGeom<N1, N2, ROW>;
  const long long tiles = ROW ? ((long long)a.ny * a.nz + G::TX - 1) / G::TX
                              : (long long)((a.nx + G::TX - 1) / G::TX) * (a.axis == 1 ? a.nz : a.ny);
  auto go = [&](auto thin) {
    constexpr bool THIN = CV(thin);
    if (grad)
      hipLaunchKernelGGL((sc_grad<N1, N2, ROW, THIN>), dim3((unsigned)tiles), dim3(G::THREADS), 0, s, a);
    else
      hipLaunchKernelGGL((sc_apply<N1, N2, ROW, THIN>), dim3(3u * (unsigned)tiles),
                         dim3(G::THREADS), 0, s, a);
  };
  if constexpr (sc_thin(N1, N2, 0)) {
    if (sc_thin(N1, N2, a.p)) return go(std::true_type{});
  }
  go(std::false_type{});
}

}  // namespace cbs
