// CBS iteration kernels for gfx950.
//
// One CBS iteration (vector CBS of references [25]/[26] of arXiv 2506.15411)
//     W = V E_s + S;  GW = F^-1 G^ F W;  E_s += gamma (GW - E_s)
// runs as four passes over HBM, each a batch of 1D FFTs along one axis:
//
//   KZ     forward FFT along z, G^(p) 3x3 multiply (1/N folded in),
//          inverse FFT along z; all three components of a z-column
//          are in one workgroup; one more workgroup reduces the
//          residual partials of the iteration before        (W in place)
//   KY(+)  inverse FFT along y                               (W in place)
//   K1     inverse FFT along x -> GW, CBS update of E_s with FP64 residual
//          partials, W = V E_s + S for the next iteration, forward FFT
//          along x                                           (W, E_s)
//   KY(-)  forward FFT along y, for the next iteration      (W in place)
//
// so the three passes that work within one z plane follow each other.
//
// Every 1D transform of length n = N1 * N2 is two register levels joined by
// one exchange through LDS: level A does N2 DFT-N1 over stride-N2 subsets
// (one per thread) and multiplies by exp(-+2 pi i j2 k1 / n); level B does
// N1 DFT-N2 over the contiguous groups (one per thread).  Level A writes its
// results to the LDS slots its inputs came from, so each exchange needs one
// buffer and one barrier.  The inter-level twiddles come from an FP64-built
// table stored [j2][k1], so each thread's twiddles are contiguous.  In K1 the
// inverse transform ends with thread t holding GW[t + N1 m]; the forward
// transform of the next W is chosen with the transposed split (DFT-N2 over
// exactly those elements first), so the update and the start of the forward
// transform run in registers without an LDS round trip.  In KZ the forward
// level B leaves each thread with all z-frequencies k1 + N1 k2 of its group
// for the three components, the Green multiply and the inverse level B run on
// those registers, and the z spectrum is never reordered.
//
// Work is in units of the voxel pitch: lengths are scaled by 1/d, potentials
// by d^2 (p d in [-pi, pi], kb^2 d^2, eps d^2), which leaves E_s unchanged.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "codelets.hpp"

namespace cbs {

enum SrcKind : int { SRC_NONE = 0, SRC_PLANE = 1, SRC_FIELD = 2, SRC_POINT = 3, SRC_FIELD_CONJ = 4 };
// Source forms the x and plane passes are compiled for (the launchers choose):
// plane waves at normal incidence, points and none; an oblique illumination among
// the plane waves (a per-element x phase); a field, loaded with the other
// pointwise operands (in the update loop its loads waited one by one behind the
// stores of E_s: x pass of 192 x 192 x 256 239 us, now 228; prologue of 275 x 275
// x 315 470, now 386).
enum SrcForm : int { FORM_PLAIN = 0, FORM_OBLIQUE = 1, FORM_FIELD = 2 };
// K1_RES: fout = -res_scale gamma (GW - E), the step's negative, and no forward
// transform
enum K1Mode : int { K1_FWD = 0, K1_ITER = 1, K1_INV = 2, K1_RES = 3 };

constexpr int kHistCap = 1 << 16;
// Illuminations one batched solve advances together (same medium, own sources).
constexpr int kMaxIllum = 8;

// The spectral work field W is stored in bricks of 8 x-columns:
//   W[c][z][x / 8][y][x % 8]   (x padded to nxp = 8 * gx columns)
// so a y-pass tile (8 columns x ny rows) is one contiguous block, a z-pass
// column of one brick row is a 64-byte piece per plane (rows y and y+1 share a
// 128-byte line), and R consecutive rows of an x-line form 64 R-byte pieces.
constexpr int kBrick = 8;

// Wave priority a pass raises to while its work-groups issue their first
// loads, where few waves share a SIMD (x pass: at most two, y pass: at most
// three; the launchers decide from the occupancy API).
constexpr int kLoadPrio = 2;

// Device-resident solve state (lives in the workspace).
struct DevState {
  int done;        // 1: stop iterating (kernels return at entry)
  int iter;        // iterations applied
  int status;      // 0 running, 1 converged, 2 max_iter, 3 diverged
  int max_iter;
  double tol;
  double eta;      // last relative update norm
  float2 amp[3];   // point-source amplitude (already scaled by d^2)
  int record;      // keep eta history
  int pending;     // the x pass wrote residual partials that are not reduced yet
  double eta_b[kMaxIllum];   // last relative update norm of each illumination
};

// Fixed-order sum of the per-block partials, then the stopping rule.  The
// partials are summed in kResStreams interleaved streams (stream s takes
// partials s, s + kResStreams, ... in order), the stream sums are combined by
// one wave in a fixed order, so the result is the same double whichever kernel
// and block shape runs it (the lagged reduction in the z pass and the
// quantum-end k_residual must agree bit for bit: which of them reduces a given
// iteration depends on where the host's quanta end).  A single work-group does
// it, so its time is the latency of its loads: eight pairs of a thread are in
// flight together (one at a time it was 50 us for the 18432 partials of
// 192 x 192 x 256, longer than the y pass it then ran in; now under 10 us, in
// the shadow of the pass's other work-groups: iteration 469 -> 432 us).  A batched solve has nb
// illuminations with per_b partials each: each gets its own eta, and the solve
// stops when the largest meets tol.  red holds 2 kResStreams doubles of LDS;
// THREADS is any multiple of 64.
constexpr int kResStreams = 256;
template <int THREADS>
__device__ __forceinline__ void residual_finish(const double* part, int per_b, int nb,
                                                DevState* st, double* hist, double* red) {
  static_assert(THREADS % 64 == 0, "whole waves");
  typedef double pair_t __attribute__((ext_vector_type(2)));
  constexpr int NS = (kResStreams + THREADS - 1) / THREADS;   // streams of a thread
  constexpr int U = NS >= 4 ? 2 : 8 / NS;                     // partials of each in flight
  double eta = 0.0;      // the largest eta (meaningful in thread 0)
  bool bad = false;      // a non-finite eta
  for (int ib = 0; ib < nb; ++ib) {
    const pair_t* pb = reinterpret_cast<const pair_t*>(part) + (long long)ib * per_b;
    double a[NS], b[NS];
    sfor<0, NS>([&](auto Q) { a[CV(Q)] = b[CV(Q)] = 0.0; });
    for (int i0 = threadIdx.x; i0 < per_b; i0 += U * kResStreams) {
      pair_t v[U][NS];
      sfor<0, U>([&](auto J) {
        sfor<0, NS>([&](auto Q) {
          const int s = threadIdx.x + CV(Q) * THREADS;
          const int i = i0 + CV(Q) * THREADS + CV(J) * kResStreams;
          v[CV(J)][CV(Q)] = pair_t{0.0, 0.0};
          if (s < kResStreams && i < per_b) v[CV(J)][CV(Q)] = __builtin_nontemporal_load(pb + i);
        });
      });
      sfor<0, U>([&](auto J) {
        sfor<0, NS>([&](auto Q) {
          a[CV(Q)] += v[CV(J)][CV(Q)].x;
          b[CV(Q)] += v[CV(J)][CV(Q)].y;
        });
      });
    }
    sfor<0, NS>([&](auto Q) {
      const int s = threadIdx.x + CV(Q) * THREADS;
      if (s < kResStreams) {
        red[s] = a[CV(Q)];
        red[kResStreams + s] = b[CV(Q)];
      }
    });
    __syncthreads();
    if (threadIdx.x < 64) {
      const int l = threadIdx.x;
      double nd = red[l], ne = red[kResStreams + l];
      #pragma unroll
      for (int q = 64; q < kResStreams; q += 64) {
        nd += red[l + q];
        ne += red[kResStreams + l + q];
      }
      #pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        nd += __shfl_xor(nd, o, 64);
        ne += __shfl_xor(ne, o, 64);
      }
      if (l == 0) {
        double e;
        if (ne > 0.0)
          e = sqrt(nd / ne);
        else
          e = (nd == 0.0) ? 0.0 : INFINITY;
        st->eta_b[ib] = e;
        if (!isfinite(e)) bad = true;
        else if (e > eta) eta = e;
      }
    }
    __syncthreads();   // red is rewritten for the next illumination
  }
  if (threadIdx.x == 0) {
    auto set_done = [&] {   // read by other blocks of the z pass meanwhile
      __hip_atomic_store(&st->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (bad) eta = NAN;
    {
      const int it = st->iter + 1;
      st->iter = it;
      st->eta = eta;
      if (st->record && it <= kHistCap) hist[it - 1] = eta;
      if (!isfinite(eta)) {
        st->status = 3;
        set_done();
      } else if (eta <= st->tol) {
        st->status = 1;
        set_done();
      } else if (it >= st->max_iter) {
        st->status = 2;
        set_done();
      }
    }
  }
}

struct CbsArgs {
  int nx, ny, nz, nxp;          // grid, padded row length of W (kBrick * gx)
  int gx, gy;                   // x bricks (nxp / kBrick), x-pass row groups (ceil(ny / rows))
  int px, py, pz;               // absorbing layer per side
  long long sW;                 // component stride of W  (nz * ny * nxp)
  long long sE;                 // component stride of E  (nz * ny * nx)
  float2* W;                    // spectral work field, bricked (see kBrick)
  float2* E;                    // E_s, caller layout [3][nz][ny][nx]
  const float2* V0;             // unshifted potential * d^2, [nz][ny][nx]
  const float2* twx;            // x split n1 x n2: twx[j2 n1 + k1] = exp(-2 pi i j2 k1 / nx)
  const float2* twy;            // same layout for the y split
  const float2* twz;            // same layout for the z split
  const float2* phase;          // [nb][3][nz] pol_c exp(i kz d z) of each illumination's wave
  const float2* fin;            // FIELD source / Green input
  unsigned char* rows;          // FIELD source: [3][nz][ny], 0 for rows of the field that are
                                // all zero (written by the prologue); null: not kept
  float2* fout;                 // Green output, K1_RES output
  double* partials;             // 2 doubles per K1 block
  int k1_blocks;                // K1 or KXY blocks per illumination (partials to reduce)
  int nb;                       // illuminations advanced together (1: an ordinary solve)
  int fused;                    // host: the plane's passes run as one (kxy)
  long long sWb, sEb;           // stride between illuminations in W (3 sW) and E (3 sE)
  const float2* phx;            // [nb][nx] exp(i kx d x) of each illumination's plane wave
  const float2* phy;            // [nb][ny] exp(i ky d y)
  unsigned pol_mask;            // bit 3 b + c: illumination b's polarisation has a component c
  int oblique;                  // some illumination has kx or ky != 0 (phx, phy not all 1)
  int k1_prio;                  // x-pass: raise wave priority for the load phase (set by launch_k1)
  int ky_prio;                  // y pass: the same (set by launch_ky)
  int flag_first;               // x and y pass: the stop flag before the first loads (large_grid)
  int z_first;                  // host: z pass the same (cbs_solve_begin)
  double* hist;                 // residual history
  DevState* st;
  int src;                      // SrcKind
  int warm;                     // K1_FWD: W = V E + S from E (else E = 0)
  int green_in;                 // K1_FWD: W = fin
  int r0x, r0y, r0z;
  float src_scale;              // d^2: physical (1/m^2) sources and Green inputs
  float res_scale;              // K1_RES
  float eps, inv_eps, kb2;      // eps d^2, 1/(eps d^2), kb^2 d^2
  float pfx, pfy, pfz;          // 2 pi / n_a
  float invN;                   // 1 / (nx ny nz)
};

// ---------------------------------------------------------------------------
// per-size geometry of the passes
// ---------------------------------------------------------------------------
constexpr int cmax(int a, int b) { return a > b ? a : b; }
constexpr int round64(int t) { return (t + 63) / 64 * 64; }

// Rows per x-pass workgroup.  A row of n = N1 N2 is N2 tasks of level A
// (DFT-N1, inverse and forward) and N1 tasks of level B (DFT-N2 twice and the
// update); R rows pack their R N2 and R N1 tasks onto whole waves.  The rule
// takes the R <= 8 with the least vector work per row, the waves of each level
// weighed by its operation count (an n-point codelet about n times the sum of
// its prime factors, the update about 25 per element), the larger R (longer
// pieces of W) on ties.  Workgroups are at most four waves; two where the estimate of
// a thread's registers is above 160, since with two waves per SIMD a larger group
// leaves part of the CU empty (621 = 27 x 23, 193 registers; 261 = 29 x 9 is estimated
// at 170 and holds 132).  Measured on these splits, x pass of n x n x 64 (621: 100
// rows) in us, rows: time, the rule's choice first:
// 96 = 12 x 8: 5: 15.8, 8: 15.9, 4: 16.6; 100 = 10 x 10: 6: 16.8, 5: 17.2, 8: 18.6;
// 121 = 11 x 11: 5: 21.6, 4: 23.2, 6: 26.3; 128 = 16 x 8: 8: 20.6, 7: 21.3, 5: 23.4;
// 189 = 21 x 9: 6: 41.4, 7: 41.8, 8: 43.0; 192 = 16 x 12: 8: 40.6, 4: 40.8, 5: 42.3;
// 256 = 16 x 16: 8: 68.6, 4: 68.6, 5: 74.6; 261: 4: 93.2, 6: 90.2, 8: 93.7, 5: 103;
// 275 = 25 x 11: 5: 106.8, 7: 110.9, 6: 115; 315 = 21 x 15: 8: 131.7, 3: 129.4, 5: 139;
// 621: 4: 80.7, 8: 84.3, 7: 91.4, 5: 104.
constexpr int codelet_ops(int n) {
  int ops = 0, m = n;
  for (int p = 2; m > 1; ++p)
    for (; m % p == 0; m /= p) ops += p;
  return n * ops;
}
constexpr int k1_rows_for(int n1, int n2) {
  const int regs = 2 * n1 * (n1 >= 17 && ct_is_prime(n1) ? 2 : 1) + 6 * n2;
  const int most = regs > 160 ? 128 : 256;
  const int wa = 2 * codelet_ops(n1), wb = 2 * codelet_ops(n2) + 25 * n2;
  int best = 1, cost = wa * (round64(n2) / 64) + wb * (round64(n1) / 64);
  for (int r = 2; r <= 8 && r * cmax(n1, n2) <= most; ++r) {
    const int c = wa * (round64(r * n2) / 64) + wb * (round64(r * n1) / 64);
    if (c * best <= cost * r) {
      best = r;
      cost = c;
    }
  }
  return best;
}
// Columns per z-pass workgroup: a whole brick row (8) unless the exchange
// buffer of 3 components x 8 columns (160 KB of LDS per CU) leaves room for
// fewer than three workgroups and those hold fewer than 12 waves per CU; then
// half a brick row (measured at 315: split 35 x 9 0.39 ms with 4 columns against
// 0.46 ms with 8; split 15 x 21, 8 waves per workgroup, 0.27 ms with 8 columns
// against 0.34 ms with 4).
constexpr int kz_tx_for(int n1, int n2) {
  const int n = n1 * n2;
  const int lds8 = 3 * n * 8 * 8 + n * 8;
  if (lds8 <= 53 * 1024) return 8;
  const int waves8 = round64(8 * cmax(3 * n2, n1)) / 64;
  return waves8 * ((160 * 1024) / lds8) >= 12 ? 8 : 4;
}

template <int N1, int N2>
struct XGeom {
  static constexpr int N = N1 * N2;
  static constexpr int LINES = k1_rows_for(N1, N2);
  static constexpr int THREADS = round64(LINES * cmax(N1, N2));
};
template <int N1, int N2, int TX>
struct YGeom {
  static constexpr int N = N1 * N2;
  static constexpr int TM = cmax(N1, N2);
  static constexpr int THREADS = round64(TX * TM);
};
template <int N1, int N2, int TX>
struct ZGeom {
  static constexpr int N = N1 * N2;
  static constexpr int TM = cmax(3 * N2, N1);
  static constexpr int THREADS = round64(TX * TM);
};

// dimensionless frequency 2 pi m / n of FFT index k (m in FFT order) and the
// same with the Nyquist index of an even axis flagged
__device__ __forceinline__ float freq_of(int k, int n, float pf, bool& nyq) {
  const int m = (k < (n + 1) / 2) ? k : k - n;
  nyq = ((n & 1) == 0) && (2 * k == n);
  return pf * float(m);
}

// Workgroups are dispatched round-robin over the 8 XCDs (block b runs on XCD
// b mod 8), and each XCD has its own L2.  The y and z passes read 64-byte
// column tiles, half a 128-byte L2 line; remapping the linear block index so
// that each XCD walks a contiguous range of tiles puts both halves of a line
// in the same L2 at about the same time.  Bijective for any block count.
constexpr int kXcds = 8;
__device__ __forceinline__ unsigned xcd_remap(unsigned b, unsigned total) {
  const unsigned q = total / kXcds, r = total % kXcds;
  const unsigned k = b % kXcds, j = b / kXcds;
  return k * q + (k < r ? k : r) + j;
}

// The stop flag before the first loads, on large grids and in solves the caller
// advances: in the x and y passes here, in the z pass by a form of its own.  The plane
// pass looks late whatever the size (128^3 iteration 78.6 us, with the flag first
// 80.1; 100 x 100 x 64 30.8 and 31.7).  A load of its own: waiting for flag_first
// would wait for the flag too if that were already in flight.
__device__ __forceinline__ bool stop_first(const CbsArgs& a) {
  const bool stop = a.flag_first && a.st->done;
  asm volatile("" ::: "memory");
  return stop;
}

// A pass's inter-level twiddle table is copied to LDS by every workgroup.
// Staged: issue() starts all of this thread's table loads at once, the caller
// then issues its first data loads, and commit() writes the table to LDS
// before the barrier, so the table's latency overlaps the data loads instead
// of preceding them.
template <int N, int THREADS>
struct TwStage {
  static constexpr int K = (N + THREADS - 1) / THREADS;
  float2 v[K];
  // rounds that lie wholly inside the table need no bounds test
  template <int I>
  static constexpr bool kFull = (I + 1) * THREADS <= N;
  __device__ __forceinline__ void issue(const float2* g, int tid) {
    sfor<0, K>([&](auto I) {
      const int i = tid + CV(I) * THREADS;
      if (kFull<CV(I)> || i < N) v[CV(I)] = g[i];
    });
  }
  __device__ __forceinline__ void commit(float2* s, int tid) const {
    sfor<0, K>([&](auto I) {
      const int i = tid + CV(I) * THREADS;
      if (kFull<CV(I)> || i < N) s[i] = v[CV(I)];
    });
  }
};

// ---------------------------------------------------------------------------
// block reduction of two doubles (residual partials)
// ---------------------------------------------------------------------------
template <int THREADS>
__device__ __forceinline__ void block_sum2(double a, double b, double* red, double* out) {
  #pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) {
    red[2 * wv] = a;
    red[2 * wv + 1] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double sa = 0.0, sb = 0.0;
    for (int w = 0; w < THREADS / 64; ++w) {
      sa += red[2 * w];
      sb += red[2 * w + 1];
    }
    out[0] = sa;
    out[1] = sb;
  }
}

// ---------------------------------------------------------------------------
// K1: x-pass with the fused CBS update
// ---------------------------------------------------------------------------
// A workgroup transforms R consecutive rows (y0 .. y0+R-1) of one component
// at one z.  W is read and written in place in its bricks: element x of row y
// sits at brick x/8, offset 8 y + x%8, so the R rows of one brick form one
// contiguous 64 R-byte piece.  The inverse transform, the update and the
// forward transform share one LDS exchange buffer per row.
template <int N1, int N2, int MODE, int FORM>
__global__ void __launch_bounds__((XGeom<N1, N2>::THREADS))
k1_xpass(CbsArgs a) {
  using G = XGeom<N1, N2>;
  constexpr int N = G::N, R = G::LINES;
  __shared__ float2 lds[R * N];     // R rows of one component, natural x order
  __shared__ double red[2 * (G::THREADS / 64)];

  if (MODE == K1_ITER && stop_first(a)) return;
  const int done = MODE == K1_ITER ? a.st->done : 0;
  const int tid = threadIdx.x;
  // with few waves per SIMD, a work-group's load phase would otherwise wait
  // behind the other waves' vector work
  if (a.k1_prio) __builtin_amdgcn_s_setprio(kLoadPrio);
  __shared__ float2 tw[N];
  TwStage<N, G::THREADS> tws;
  tws.issue(a.twx, tid);

  // block -> (illumination, component, row group, z); the 3 nb components of
  // the same rows are adjacent in the remapped order so V0 is shared in one L2
  const unsigned per = 3u * (unsigned)a.nb;
  const unsigned L = xcd_remap(blockIdx.x, per * (unsigned)a.gy * (unsigned)a.nz);
  const int cc = (int)(L % per);
  const int ib = cc / 3, c = cc - 3 * ib;
  const unsigned rest = L / per;
  const int yg = (int)(rest % (unsigned)a.gy);
  const int z = (int)(rest / (unsigned)a.gy);
  const int y0 = yg * R;
  const int rv = (a.ny - y0) < R ? (a.ny - y0) : R;   // valid rows in this group

  // The two levels of a row are different tasks: R N2 level-A tasks (row, j2),
  // R N1 level-B tasks (row, k1), each packed onto the first lanes of the
  // work-group, so waves without a task skip the level.
  const int ta = tid % N2, la = tid / N2;   // level A: j2, row
  const int t = tid % N1, line = tid / N1;  // level B: k1, row
  const bool oka = la < rv;
  const bool ok = line < rv;
  const int y = y0 + (ok ? line : 0);
  float2* La = lds + (oka ? la : 0) * N;
  float2* Lr = lds + (ok ? line : 0) * N;
  // W bricks of this (component, z, row group): brick xt starts at wb + xt * ny * 8
  float2* wb = a.W + ib * a.sWb + c * a.sW + ((long long)z * a.gx * a.ny + y0) * kBrick;
  const long long bstride = (long long)a.ny * kBrick;
  const long long ebase = ib * a.sEb + c * a.sE + ((long long)z * a.ny + y) * a.nx;  // E / fin / fout row
  const long long vbase = ((long long)z * a.ny + y) * a.nx;             // V0 row

  float2 v[N2];  // thread t (< N1): element t + N1 m, m < N2
  // the pointwise operands V0 and E_s, loaded between the levels of the inverse
  // transform: their latency hides behind the second, and the first does not
  // hold their registers (before it: 261 points 177 registers and 208 us, now
  // 168 us; 256 158 -> 150, 189 78 -> 73, 315 223 -> 214, 275 and 621 unchanged)
  constexpr bool PF = MODE != K1_INV;
  constexpr bool FIELD = FORM == FORM_FIELD && (MODE == K1_ITER || MODE == K1_FWD);
  float2 pv[PF ? N2 : 1], pe[PF ? N2 : 1], pf[FIELD ? N2 : 1];
  const float2* v0t = a.V0 + vbase + t;   // this thread's elements are t + N1 m
  float2* et = a.E + ebase + t;

  // a field source that is zero along the row is not read again every iteration
  // (the source of an objective at a point or in a plane: x pass of 189 x 189 x 121
  // 102 us with the field read, 70 without)
  const long long frow = ((long long)c * a.nz + z) * a.ny + y;
  const bool live = !(FIELD && MODE == K1_ITER) || !a.rows || a.rows[frow];
  auto load_operands = [&]() {
    if constexpr (PF) {
      if (!ok) return;
      if constexpr (FIELD) {
        sfor<0, N2>([&](auto M) { pf[CV(M)] = make_float2(0.f, 0.f); });
        if (live) sfor<0, N2>([&](auto M) { pf[CV(M)] = a.fin[ebase + t + N1 * CV(M)]; });
      }
      if (MODE == K1_FWD && a.green_in) return;
      sfor<0, N2>([&](auto M) { pv[CV(M)] = v0t[N1 * CV(M)]; });
      if (MODE != K1_FWD || a.warm) sfor<0, N2>([&](auto M) { pe[CV(M)] = et[N1 * CV(M)]; });
    }
  };
  if constexpr (MODE == K1_FWD) load_operands();

  // element x of this thread's row in the bricks
  float2* wrow = wb + la * kBrick;
  auto wat = [&](int x) -> float2& { return wrow[(x / kBrick) * bstride + (x % kBrick)]; };
  // inverse level A input: thread j2 = t < N2 holds row[j2 + N2 j1]
  float2 b[N1];
  auto load_a = [&]() {
    if (oka) sfor<0, N1>([&](auto J1) { b[CV(J1)] = wat(ta + N2 * CV(J1)); });
  };
  if constexpr (MODE != K1_FWD) load_a();
  if constexpr (MODE == K1_ITER) {
    asm volatile("" ::: "memory");   // the loads are issued before the flag is waited for
    if (done) return;
  }
  tws.commit(tw, tid);
  __syncthreads();   // the twiddle table is in LDS
  if (a.k1_prio) __builtin_amdgcn_s_setprio(0);

  if constexpr (MODE != K1_FWD) {
    // inverse level A: DFT-N1 over row[j2 + N2 j1]
    if (oka) {
      dft<N1, +1>(b);
      const float2* twt = tw + ta * N1;   // exp(-2 pi i j2 k1 / N), conjugated below
      sfor<0, N1>([&](auto K1) { b[CV(K1)] = cmulc(b[CV(K1)], twt[CV(K1)]); });
      sfor<0, N1>([&](auto K1) { La[ta + N2 * CV(K1)] = b[CV(K1)]; });
    }
    load_operands();
    __syncthreads();
    // inverse level B: thread k1 = t < N1, DFT-N2 over Lr[N2 k1 + j2]
    if (ok) {
      sfor<0, N2>([&](auto J2) { v[CV(J2)] = Lr[N2 * t + CV(J2)]; });
      dft<N2, +1>(v);
    }
    __syncthreads();  // lds is rewritten below
  }

  if constexpr (MODE == K1_INV) {
    if (ok) {
      sfor<0, N2>([&](auto M) { a.fout[ebase + t + N1 * CV(M)] = v[CV(M)]; });
    }
    return;
  }

  if constexpr (MODE == K1_RES) {
    if (ok) {
      sfor<0, N2>([&](auto M) {
        const float2 d = cmul(make_float2(1.0f - pv[CV(M)].y * a.inv_eps, pv[CV(M)].x * a.inv_eps),
                              csub(v[CV(M)], pe[CV(M)]));
        a.fout[ebase + t + N1 * CV(M)] = make_float2(-a.res_scale * d.x, -a.res_scale * d.y);
      });
    }
    return;
  }

  double sd = 0.0, se = 0.0;
  if (ok) {
    const bool yin = (y >= a.py) && (y < a.ny - a.py);
    const bool zin = (z >= a.pz) && (z < a.nz - a.pz);
    // pol_c exp(i (ky y + kz z)); the x phase joins per element when oblique
    const float2 ph = a.phase[(ib * 3 + c) * a.nz + z];
    const float2 spl = FORM == FORM_OBLIQUE ? cmul(ph, a.phy[ib * a.ny + y]) : ph;
    const float2* phxb = a.phx + ib * a.nx;
    const float fs = a.src_scale, fsi = a.src == SRC_FIELD_CONJ ? -fs : fs;
    const bool green = MODE == K1_FWD && a.green_in;
    if constexpr (FIELD && MODE == K1_FWD) {
      bool any = false;
      sfor<0, N2>([&](auto M) { any |= pf[CV(M)].x != 0.f || pf[CV(M)].y != 0.f; });
      if (any && a.rows) a.rows[frow] = 1;   // every thread that writes writes 1
    }
    sfor<0, N2>([&](auto M) {
      const int x = t + N1 * CV(M);
      float2 e = make_float2(0.f, 0.f);   // a cold start, whatever the output buffer held
      float2 w;
      if (FIELD && green) {
        w = cscale(pf[FIELD ? CV(M) : 0], fs);
      } else {
        const float2 v0 = pv[CV(M)];
        if (MODE != K1_FWD || a.warm) e = pe[CV(M)];
        if constexpr (MODE == K1_ITER) {
          // gamma = 1 + i V0 / eps
          const float2 gm = make_float2(1.0f - v0.y * a.inv_eps, v0.x * a.inv_eps);
          const float2 d = cmul(gm, csub(v[CV(M)], e));
          e = cadd(e, d);
          sd += (double)(d.x * d.x + d.y * d.y);
          se += (double)(e.x * e.x + e.y * e.y);
        }
        if (MODE == K1_ITER || !a.warm) et[N1 * CV(M)] = e;
        // W = (V0 - i eps) e + S
        w = cmul(make_float2(v0.x, v0.y - a.eps), e);
        if constexpr (FIELD) {
          const float2 f = pf[CV(M)];
          w = cadd(w, make_float2(f.x * fs, f.y * fsi));
        } else if (a.src == SRC_PLANE) {
          const bool xin = (x >= a.px) && (x < a.nx - a.px);
          if (xin && yin && zin) {
            if constexpr (FORM == FORM_OBLIQUE)
              w = cadd(w, cmul(v0, cmul(spl, phxb[x])));
            else
              w = cadd(w, cmul(v0, spl));
          }
        } else if (a.src == SRC_POINT) {
          if (x == a.r0x && y == a.r0y && z == a.r0z) w = cadd(w, a.st->amp[c]);
        }
      }
      v[CV(M)] = w;
    });
    // forward level A' (split N2 x N1): DFT-N2 over v, twiddle, to Lr[t + N1 k1']
    dft<N2, -1>(v);
    const float2* twc = tw + t;   // exp(-2 pi i t k / N) sits at [k][t] of the table
    sfor<0, N2>([&](auto K) { Lr[t + N1 * CV(K)] = cmul(v[CV(K)], twc[N1 * CV(K)]); });
  }
  __syncthreads();
  // forward level B': thread k1' = t < N2, DFT-N1 over Lr[N1 k1' + j2']
  float2 bo[N1];
  if (oka) {
    sfor<0, N1>([&](auto J) { bo[CV(J)] = La[N1 * ta + CV(J)]; });
    dft<N1, -1>(bo);
    sfor<0, N1>([&](auto K) { wat(ta + N2 * CV(K)) = bo[CV(K)]; });
  }
  if constexpr (MODE == K1_ITER) {
    const long long slot = (long long)ib * a.k1_blocks + (long long)rest * 3 + c;
    block_sum2<G::THREADS>(sd, se, red, a.partials + 2 * slot);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.st->pending = 1;
  }
}

// ---------------------------------------------------------------------------
// KY: FFT along y of TX adjacent columns of one (component, z) plane
// ---------------------------------------------------------------------------
template <int N1, int N2, int TX, int S>
__global__ void __launch_bounds__((YGeom<N1, N2, TX>::THREADS))
ky_pass(CbsArgs a) {
  using G = YGeom<N1, N2, TX>;
  constexpr int N = G::N;
  __shared__ float2 lds[N * TX];
  __shared__ float2 tw[N];
  if (stop_first(a)) return;
  const int done = a.st->done;
  const int tid = threadIdx.x;
  if (a.ky_prio) __builtin_amdgcn_s_setprio(kLoadPrio);
  TwStage<N, G::THREADS> tws;
  tws.issue(a.twy, tid);
  const int xi = tid % TX;
  const int t = tid / TX;
  const unsigned gx = (unsigned)(a.nx + TX - 1) / TX;
  // component c < 3 nb: the W fields of a batch follow each other (sWb = 3 sW)
  const unsigned L = xcd_remap(blockIdx.x, gx * (unsigned)a.nz * 3u * (unsigned)a.nb);
  const int bx = (int)(L % gx);
  const unsigned rest = L / gx;
  const int z = (int)(rest % (unsigned)a.nz), c = (int)(rest / (unsigned)a.nz);
  static_assert(TX == kBrick, "y-pass tiles are one brick wide");
  const int x = bx * TX + xi;
  const bool xok = x < a.nx;
  // the tile is brick (c, z, bx): ny rows of 8 columns, contiguous
  float2* col = a.W + c * a.sW + ((long long)z * a.gx + bx) * a.ny * kBrick + xi;
  const long long ps = kBrick;
  float2 b[N1];
  auto load_a = [&]() {
    if (t < N2) {
      if (xok) {
        // per-thread base once; each load then adds a uniform stride
        const float2* ct = col + (long long)t * ps;
        const long long st = (long long)N2 * ps;
        sfor<0, N1>([&](auto J1) { b[CV(J1)] = ct[CV(J1) * st]; });
      } else {
        sfor<0, N1>([&](auto J1) { b[CV(J1)] = make_float2(0.f, 0.f); });
      }
    }
  };
  load_a();
  asm volatile("" ::: "memory");   // the loads are issued before the flag is waited for
  if (done) return;
  tws.commit(tw, tid);
  __syncthreads();
  if (a.ky_prio) __builtin_amdgcn_s_setprio(0);
  if (t < N2) {
    dft<N1, S>(b);
    const float2* twt = tw + t * N1;
    sfor<0, N1>([&](auto K1) {
      const float2 w = twt[CV(K1)];
      b[CV(K1)] = (S < 0) ? cmul(b[CV(K1)], w) : cmulc(b[CV(K1)], w);
    });
    sfor<0, N1>([&](auto K1) { lds[(t + N2 * CV(K1)) * TX + xi] = b[CV(K1)]; });
  }
  __syncthreads();
  if (t < N1 && xok) {
    float2 v[N2];
    sfor<0, N2>([&](auto J2) { v[CV(J2)] = lds[(N2 * t + CV(J2)) * TX + xi]; });
    dft<N2, S>(v);
    float2* ct = col + (long long)t * ps;
    const long long st = (long long)N1 * ps;
    sfor<0, N2>([&](auto K2) { ct[CV(K2) * st] = v[CV(K2)]; });
  }
}

// ---------------------------------------------------------------------------
// KXY: the three passes of one square plane in one
// ---------------------------------------------------------------------------
// A workgroup holds one (component, z) plane of N x N points in LDS and runs
// KY(+), K1 and KY(-) on it: W crosses HBM once each way instead of three times.
// Every level works in place, so a level needs one barrier and no second buffer:
//   inverse A   task j2: points j2 + N2 j1, DFT-N1, twiddle, back to j2 + N2 k1
//   inverse B   task k1: positions N2 k1 + j2, DFT-N2 -> points k1 + N1 m, left
//               at N2 k1 + m
//   forward A'  task k1: those positions (points k1 + N1 m), DFT-N2, twiddle
//   forward B'  task k': positions N2 k1 + k', DFT-N1 -> k' + N2 K, natural order
// along y (a column per task) and, between, along x (a row per task); the row at
// position q holds y = q / N2 + N1 (q % N2) while the x levels run.
//
// One plane is one CU's work, and its time is the latency of seven dependent
// levels (about 13 us at 64 x 64, 24 at 128 x 128), bounded by vector
// instructions there (16 us of issue at 128 x 128).  The operands of the update are
// loaded behind the first level and held through the next two: the iteration form
// spills 8 (12 oblique) bytes a lane at 64 x 64, 32, 40 and 112 with a field at 121 x
// 121, 20, 36 and 128 at 128 x 128, none at the other lengths.  Threads: as few as keep the
// rounds of 1024 threads over the N N2 and N N1 tasks of the two levels (96 =
// 12 x 8: 768 threads 34.5 us, 576 36.6; 121: 704 threads 61.5, 1024 79.5 with a
// mostly empty second round).  Row pitch N + 8: rows then start 64 bytes apart in
// the banks and stay 16-byte aligned (128: 56.2 us, N + 2 59.3, N + 1 65.3).
// Where the LDS holds two planes or more and a thread has one round of tasks, six
// waves per SIMD are asked for, 80 registers: the lengths up to 48 take that or less by
// themselves, 64 = 8 x 8 takes 84 and then holds two planes a CU instead of three
// (iteration of 64 x 64 x 256 42.2 -> 38.5 us, eight illuminations 273 -> 267, at 8
// bytes of scratch; 64^3 equal).  A field source's operands are 5 registers more and
// lose by it (64 x 64 x 32 16.05 -> 17.3 us, 64 x 64 x 256 43.2 -> 44.5), two rounds
// (96 = 12 x 8) spill 140 bytes, and eight waves cost every length (48 x 48 x 256 with a
// field 30.6 -> 36.3, 64 x 64 x 256 38.5 -> 45.9).  Iteration in us, three passes -> fused:
// 16^3 14.5 -> 8.6, 32^3 16.4 -> 10.8, 64^3 29.5 -> 19.5, 96^3 52.6 -> 46.3,
// 121^3 88.4 -> 82.3, 128^3 95.7 -> 77.7, 128 x 128 x 256 172.7 -> 133.
template <int N1, int N2>
struct XYGeom {
  static constexpr int N = N1 * N2;
  static constexpr int P = N % 2 ? N : N + 8;       // row pitch in LDS
  static constexpr int GX = (N + kBrick - 1) / kBrick;
  static constexpr int RA = (N * N2 + 1023) / 1024, RB = (N * N1 + 1023) / 1024;   // rounds
  static constexpr int THREADS = round64(cmax((N * N2 + RA - 1) / RA, (N * N1 + RB - 1) / RB));
  static constexpr int QG = (GX * kBrick * N2 + THREADS - 1) / THREADS;   // columns x N2 tasks
  static constexpr int QA = (N * N2 + THREADS - 1) / THREADS;
  static constexpr int QB = (N * N1 + THREADS - 1) / THREADS;
  static constexpr int FIT = 160 * 1024 / (8 * N * (P + 1));   // planes the LDS of a CU holds
  // waves per SIMD, at least
  static constexpr int waves(bool field) {
    const int all = (FIT * (THREADS / 64) + 3) / 4;   // with every plane that fits
    return FIT >= 2 && QB == 1 && !field ? (all < 6 ? all : 6) : 1;
  }
};
// MODE as in K1: K1_ITER the whole iteration, K1_FWD (W from E and the source, x
// and y forward) and K1_RES (y and x inverse, fout = -res_scale gamma (GW - E)) its halves.
template <int N1, int N2, int MODE, int FORM>
__global__ void __launch_bounds__((XYGeom<N1, N2>::THREADS), (XYGeom<N1, N2>::waves(FORM == FORM_FIELD)))
kxy_pass(CbsArgs a) {
  using G = XYGeom<N1, N2>;
  constexpr int N = G::N, P = G::P, T = G::THREADS;
  __shared__ float2 lds[N * P];
  __shared__ float2 tw[N];
  __shared__ double red[2 * (T / 64)];
  const int done = MODE == K1_ITER ? a.st->done : 0;
  const int tid = threadIdx.x;
  TwStage<N, T> tws;
  tws.issue(a.twx, tid);
  // block -> (z, illumination, component), a z plane's components adjacent so
  // they share V0 in one L2
  const unsigned per = 3u * (unsigned)a.nb;
  const unsigned L = xcd_remap(blockIdx.x, per * (unsigned)a.nz);
  const int z = (int)(L / per);
  const int cc = (int)(L % per);
  const int ib = cc / 3, c = cc - 3 * ib;
  float2* wp = a.W + ib * a.sWb + c * a.sW + (long long)z * G::GX * N * kBrick;
  const float2* v0p = a.V0 + (long long)z * N * N;
  const long long ebase = ib * a.sEb + c * a.sE + (long long)z * N * N;
  float2* ep = a.E + ebase;

  // inverse y, level A: task (xi, j2, brick), a wave reads whole brick rows
  if constexpr (MODE == K1_FWD) {
    tws.commit(tw, tid);
  } else {
    float2 b[G::QG][N1];
    sfor<0, G::QG>([&](auto QQ) {
      const int i = tid + CV(QQ) * T;
      const int xi = i % kBrick, j2 = (i / kBrick) % N2, br = i / (kBrick * N2);
      if (br * kBrick + xi < N) {
        const float2* w = wp + ((long long)br * N + j2) * kBrick + xi;
        sfor<0, N1>([&](auto J) { b[CV(QQ)][CV(J)] = w[N2 * kBrick * CV(J)]; });
      }
    });
    // The stop flag, read first, is waited for behind the issued loads, here and, where
    // it does not come first, in the other passes: one round trip less per launch
    // (16^3 iteration 8.5 -> 7.9 us, 32^3 10.9 -> 10.1, 64^3 19.5 -> 19.1).
    asm volatile("" ::: "memory");
    if (done) return;
    tws.commit(tw, tid);
    __syncthreads();
    sfor<0, G::QG>([&](auto QQ) {
      const int i = tid + CV(QQ) * T;
      const int xi = i % kBrick, j2 = (i / kBrick) % N2, br = i / (kBrick * N2);
      const int x = br * kBrick + xi;
      if (x < N) {
        dft<N1, +1>(b[CV(QQ)]);
        const float2* t = tw + j2 * N1;
        sfor<0, N1>([&](auto K) { lds[(j2 + N2 * CV(K)) * P + x] = cmulc(b[CV(QQ)][CV(K)], t[CV(K)]); });
      }
    });
  }
  // the pointwise operands of this thread's x-level-B tasks (y, k1): elements
  // x = k1 + N1 m of row y, in flight during the levels before them
  constexpr bool FIELD = FORM == FORM_FIELD && MODE != K1_RES;
  float2 pv[G::QB][N2], pe[G::QB][N2], pf[FIELD ? G::QB : 1][FIELD ? N2 : 1];
  sfor<0, G::QB>([&](auto QQ) {
    const int i = tid + CV(QQ) * T;
    if (i < N * N1) {
      const int o = (i / N1) * N + i % N1;
      sfor<0, N2>([&](auto M) { pv[CV(QQ)][CV(M)] = v0p[o + N1 * CV(M)]; });
      if constexpr (FIELD)
        sfor<0, N2>([&](auto M) { pf[CV(QQ)][CV(M)] = a.fin[ebase + o + N1 * CV(M)]; });
      if (MODE != K1_FWD || a.warm)
        sfor<0, N2>([&](auto M) { pe[CV(QQ)][CV(M)] = ep[o + N1 * CV(M)]; });
    }
  });
  __syncthreads();
  if constexpr (MODE != K1_FWD) {
  // inverse y, level B: task (x, k1)
  sfor<0, G::QB>([&](auto QQ) {
    const int i = tid + CV(QQ) * T;
    if (i < N * N1) {
      float2* l = lds + N2 * (i / N) * P + i % N;
      float2 v[N2];
      sfor<0, N2>([&](auto J) { v[CV(J)] = l[CV(J) * P]; });
      dft<N2, +1>(v);
      sfor<0, N2>([&](auto J) { l[CV(J) * P] = v[CV(J)]; });
    }
  });
  __syncthreads();
  // inverse x, level A: task (row, j2)
  sfor<0, G::QA>([&](auto QQ) {
    const int i = tid + CV(QQ) * T;
    if (i < N * N2) {
      const int j2 = i % N2;
      float2* l = lds + (i / N2) * P + j2;
      float2 b[N1];
      sfor<0, N1>([&](auto J) { b[CV(J)] = l[N2 * CV(J)]; });
      dft<N1, +1>(b);
      const float2* t = tw + j2 * N1;
      sfor<0, N1>([&](auto K) { l[N2 * CV(K)] = cmulc(b[CV(K)], t[CV(K)]); });
    }
  });
  __syncthreads();
  }
  // inverse x, level B; update; W = V E_s + S; forward x, level A'
  const bool zin = (z >= a.pz) && (z < a.nz - a.pz);
  const float2 ph = a.phase[(ib * 3 + c) * a.nz + z];   // pol_c exp(i kz z)
  const float fs = a.src_scale, fsi = a.src == SRC_FIELD_CONJ ? -fs : fs;
  double sd = 0.0, se = 0.0;
  sfor<0, G::QB>([&](auto QQ) {
    const int i = tid + CV(QQ) * T;
    if (i < N * N1) {
      const int t = i % N1, y = i / N1;
      const int o = y * N + t;
      float2* l = lds + (N2 * (y % N1) + y / N1) * P + N2 * t;
      float2 v[N2];
      if constexpr (MODE != K1_FWD) {
        sfor<0, N2>([&](auto J) { v[CV(J)] = l[CV(J)]; });
        dft<N2, +1>(v);
      }
      if constexpr (MODE == K1_RES) {
        sfor<0, N2>([&](auto M) {
          const float2 v0 = pv[CV(QQ)][CV(M)];
          const float2 d = cmul(make_float2(1.0f - v0.y * a.inv_eps, v0.x * a.inv_eps),
                                csub(v[CV(M)], pe[CV(QQ)][CV(M)]));
          a.fout[ebase + o + N1 * CV(M)] = make_float2(-a.res_scale * d.x, -a.res_scale * d.y);
        });
        return;
      }
      const bool yzin = zin && (y >= a.py) && (y < a.ny - a.py);
      const float2 spl = FORM == FORM_OBLIQUE ? cmul(ph, a.phy[ib * a.ny + y]) : ph;
      const float2* phxb = a.phx + ib * a.nx;
      sfor<0, N2>([&](auto M) {
        const int x = t + N1 * CV(M);
        const float2 v0 = pv[CV(QQ)][CV(M)];
        float2 e = make_float2(0.f, 0.f);   // a cold start, whatever E held
        if (MODE != K1_FWD || a.warm) e = pe[CV(QQ)][CV(M)];
        if constexpr (MODE == K1_ITER) {
          const float2 gm = make_float2(1.0f - v0.y * a.inv_eps, v0.x * a.inv_eps);
          const float2 d = cmul(gm, csub(v[CV(M)], e));
          e = cadd(e, d);
          sd += (double)(d.x * d.x + d.y * d.y);
          se += (double)(e.x * e.x + e.y * e.y);
        }
        if (MODE == K1_ITER || !a.warm) ep[o + N1 * CV(M)] = e;
        float2 w = cmul(make_float2(v0.x, v0.y - a.eps), e);
        if constexpr (FIELD) {
          const float2 f = pf[CV(QQ)][CV(M)];
          w = cadd(w, make_float2(f.x * fs, f.y * fsi));
        } else if (a.src == SRC_PLANE) {
          if (yzin && (x >= a.px) && (x < a.nx - a.px)) {
            if constexpr (FORM == FORM_OBLIQUE)
              w = cadd(w, cmul(v0, cmul(spl, phxb[x])));
            else
              w = cadd(w, cmul(v0, spl));
          }
        } else if (a.src == SRC_POINT) {
          if (x == a.r0x && y == a.r0y && z == a.r0z) w = cadd(w, a.st->amp[c]);
        }
        v[CV(M)] = w;
      });
      dft<N2, -1>(v);
      const float2* tc = tw + t;
      sfor<0, N2>([&](auto K) { l[CV(K)] = cmul(v[CV(K)], tc[N1 * CV(K)]); });
    }
  });
  if constexpr (MODE == K1_RES) return;
  __syncthreads();
  // forward x, level B': task (row, k')
  sfor<0, G::QA>([&](auto QQ) {
    const int i = tid + CV(QQ) * T;
    if (i < N * N2) {
      float2* l = lds + (i / N2) * P + i % N2;
      float2 b[N1];
      sfor<0, N1>([&](auto J) { b[CV(J)] = l[N2 * CV(J)]; });
      dft<N1, -1>(b);
      sfor<0, N1>([&](auto K) { l[N2 * CV(K)] = b[CV(K)]; });
    }
  });
  __syncthreads();
  // forward y, level A': task (x, k1)
  sfor<0, G::QB>([&](auto QQ) {
    const int i = tid + CV(QQ) * T;
    if (i < N * N1) {
      const int t = i / N;
      float2* l = lds + N2 * t * P + i % N;
      float2 v[N2];
      sfor<0, N2>([&](auto J) { v[CV(J)] = l[CV(J) * P]; });
      dft<N2, -1>(v);
      const float2* tc = tw + t;
      sfor<0, N2>([&](auto K) { l[CV(K) * P] = cmul(v[CV(K)], tc[N1 * CV(K)]); });
    }
  });
  __syncthreads();
  // forward y, level B': task (xi, k', brick), written straight to the bricks
  sfor<0, G::QG>([&](auto QQ) {
    const int i = tid + CV(QQ) * T;
    const int xi = i % kBrick, k = (i / kBrick) % N2, br = i / (kBrick * N2);
    const int x = br * kBrick + xi;
    if (x < N) {
      float2 b[N1];
      sfor<0, N1>([&](auto J) { b[CV(J)] = lds[(N2 * CV(J) + k) * P + x]; });
      dft<N1, -1>(b);
      float2* w = wp + ((long long)br * N + k) * kBrick + xi;
      sfor<0, N1>([&](auto K) { w[N2 * kBrick * CV(K)] = b[CV(K)]; });
    }
  });
  if constexpr (MODE == K1_ITER) {
    block_sum2<T>(sd, se, red, a.partials + 2 * ((long long)ib * a.k1_blocks + (long long)z * 3 + c));
    if (blockIdx.x == 0 && tid == 0) a.st->pending = 1;
  }
}

// ---------------------------------------------------------------------------
// KZ: FFT along z, Green's tensor, inverse FFT along z (3 components)
// ---------------------------------------------------------------------------
// FIRST: the stop flag before the loads (z_first), a form of its own: a solve that
// leaves few launches behind does better without the wait (64^3 iteration 19.7 us,
// without 19.1; z pass of 275 x 275 x 315 261 us, without 255).
template <int N1, int N2, int TX, bool FIRST>
__global__ void __launch_bounds__((ZGeom<N1, N2, TX>::THREADS))
kz_pass(CbsArgs a) {
  using G = ZGeom<N1, N2, TX>;
  constexpr int N = G::N;
  __shared__ float2 lds[3 * N * TX];
  __shared__ float2 tw[N];
  __shared__ int stop;
  // block 0 transforms nothing: it finishes the previous iteration's residual
  // (stream order: the x pass that wrote the partials has completed) beside the
  // columns of the others
  if (blockIdx.x == 0) {
    if (a.st->done || !a.st->pending) return;
    constexpr bool kFits = sizeof(lds) >= 2 * kResStreams * sizeof(double);
    if constexpr (kFits) {
      residual_finish<G::THREADS>(a.partials, a.k1_blocks, a.nb, a.st, a.hist,
                                  reinterpret_cast<double*>(lds));
    } else {
      __shared__ double red[2 * kResStreams];
      residual_finish<G::THREADS>(a.partials, a.k1_blocks, a.nb, a.st, a.hist, red);
    }
    if (threadIdx.x == 0) a.st->pending = 0;
    return;
  }
  // Block 0 may raise the stop flag while the others look at it, so a work-group
  // takes one thread's reading of it: whole groups go on or leave.  Some columns of
  // W are then transformed and some are not, and W is dead: the passes behind this
  // one see the flag, E is whole, and a solve's prologue forms W anew.
  const int tid = threadIdx.x;
  int flag = 0;
  if (tid == 0) flag = __hip_atomic_load(&a.st->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if constexpr (FIRST) {
    if (tid == 0) stop = flag;
    __syncthreads();
    if (stop) return;
  }
  TwStage<N, G::THREADS> tws;
  tws.issue(a.twz, tid);
  const int xi = tid % TX;
  const int t = tid / TX;
  // remapped order: the kBrick / TX parts of one brick row, then y, then the
  // brick; rows y, y+1 of a brick share a 128-byte line
  static_assert(kBrick % TX == 0, "z-pass tiles split a brick row evenly");
  constexpr int PARTS = kBrick / TX;
  const unsigned per_b = (unsigned)(a.nxp / TX) * (unsigned)a.ny;
  const unsigned Lb = xcd_remap(blockIdx.x - 1, per_b * (unsigned)a.nb);
  const int ib = (int)(Lb / per_b);
  const unsigned L = Lb - (unsigned)ib * per_b;
  const int part = (int)(L % PARTS);
  const int y = (int)((L / PARTS) % (unsigned)a.ny);
  const int brick = (int)(L / (PARTS * (unsigned)a.ny));
  const int bx = brick * PARTS + part;      // tile index along x
  const int x = bx * TX + xi;
  const bool xok = x < a.nx;
  const long long plane = (long long)a.ny * a.nxp;   // z stride (gx bricks of ny x 8)
  float2* colbase = a.W + ib * a.sWb + ((long long)brick * a.ny + y) * kBrick + part * TX + xi;

  const long long zst = (long long)N2 * plane;  // z stride between the samples of one DFT-N1
  // forward level A: thread (c, j2), DFT-N1 over z = j2 + N2 j1
  const int ca = t / N2;
  const int j2 = t - ca * N2;
  float2 b[N1];
  auto load_a = [&]() {
    if (t < 3 * N2) {
      const float2* col = colbase + ca * a.sW + (long long)j2 * plane;
      if (xok) {
        sfor<0, N1>([&](auto J1) { b[CV(J1)] = col[CV(J1) * zst]; });
      } else {
        sfor<0, N1>([&](auto J1) { b[CV(J1)] = make_float2(0.f, 0.f); });
      }
    }
  };
  load_a();
  asm volatile("" ::: "memory");   // the loads are issued before the flag is waited for
  if (!FIRST && tid == 0) stop = flag;
  tws.commit(tw, tid);
  __syncthreads();
  if (!FIRST && stop) return;
  if (t < 3 * N2) {
    dft<N1, -1>(b);
    const float2* twt = tw + j2 * N1;
    sfor<0, N1>([&](auto K1) { b[CV(K1)] = cmul(b[CV(K1)], twt[CV(K1)]); });
    float2* Lc = lds + ca * N * TX;
    sfor<0, N1>([&](auto K1) { Lc[(j2 + N2 * CV(K1)) * TX + xi] = b[CV(K1)]; });
  }
  __syncthreads();

  // Green's tensor of the column's modes: the x/y parts are fixed per thread
  float2* L0 = lds;
  float2* L1 = lds + N * TX;
  float2* L2 = lds + 2 * N * TX;
  bool nyx, nyy;
  const float px = freq_of(x, a.nx, a.pfx, nyx);
  const float py = freq_of(y, a.ny, a.pfy, nyy);
  const float ptx = nyx ? 0.f : px, pty = nyy ? 0.f : py;
  const float pxy2 = px * px + py * py;
  const float nq_xy = (nyx ? px * px : 0.f) + (nyy ? py * py : 0.f);
  const float eps = a.eps, e2 = eps * eps;
  const bool nq_any = nyx || nyy;
  const float sb = __builtin_amdgcn_rcpf(a.kb2 * a.kb2 + e2);
  const float2 gb0 = make_float2(-a.kb2 * sb, eps * sb);
  // v <- G^(p) v / N at z-frequency index kz
  auto green = [&](float2& u0, float2& u1, float2& u2, int kz) {
    bool nyz;
    const float pz = freq_of(kz, a.nz, a.pfz, nyz);
    const float ptz = nyz ? 0.f : pz;
    const float p2 = pxy2 + pz * pz;
    // a = invN / (p2 - kb2 - i eps), b = 1 / (p2 - |pt|^2 - kb2 - i eps)
    const float r1 = p2 - a.kb2;
    const float s1 = a.invN * __builtin_amdgcn_rcpf(r1 * r1 + e2);
    const float2 ga = make_float2(r1 * s1, eps * s1);
    float2 gb = gb0;   // 1 / (-kb2 - i eps): every mode without a Nyquist component
    if (nq_any || nyz) {
      const float r2 = (nq_xy + (nyz ? pz * pz : 0.f)) - a.kb2;
      const float s2 = __builtin_amdgcn_rcpf(r2 * r2 + e2);
      gb = make_float2(r2 * s2, eps * s2);
    }
    const float2 sp = make_float2(ptx * u0.x + pty * u1.x + ptz * u2.x,
                                  ptx * u0.y + pty * u1.y + ptz * u2.y);
    const float2 bs = cmul(gb, sp);
    u0 = cmul(ga, make_float2(u0.x + ptx * bs.x, u0.y + ptx * bs.y));
    u1 = cmul(ga, make_float2(u1.x + pty * bs.x, u1.y + pty * bs.y));
    u2 = cmul(ga, make_float2(u2.x + ptz * bs.x, u2.y + ptz * bs.y));
  };

  if constexpr (N1 > N2) {
    // level B: thread k1 = t, all three components, Green multiply, inverse B
    if (t < N1) {
      float2 v0[N2], v1[N2], v2[N2];
      sfor<0, N2>([&](auto J) {
        const int o = (N2 * t + CV(J)) * TX + xi;
        v0[CV(J)] = L0[o];
        v1[CV(J)] = L1[o];
        v2[CV(J)] = L2[o];
      });
      dft<N2, -1>(v0);
      dft<N2, -1>(v1);
      dft<N2, -1>(v2);
      sfor<0, N2>([&](auto K2) {
        constexpr int k2 = CV(K2);
        green(v0[k2], v1[k2], v2[k2], t + N1 * k2);
      });
      dft<N2, +1>(v0);
      dft<N2, +1>(v1);
      dft<N2, +1>(v2);
      sfor<0, N2>([&](auto J) {
        const int o = (N2 * t + CV(J)) * TX + xi;
        L0[o] = v0[CV(J)];
        L1[o] = v1[CV(J)];
        L2[o] = v2[CV(J)];
      });
    }
  } else {
    // N1 <= N2: one thread per k1 would leave most lanes idle and hold 3 N2
    // values.  Split level B over the 3 N1 threads (component, k1): forward
    // DFT-N2 per component, the Green multiply spread over the same threads by
    // frequency, inverse DFT-N2 per component, with the spectra in LDS between.
    const int cb = t / N1, kb = t - cb * N1;
    float2* Lb = lds + (cb < 3 ? cb : 0) * N * TX;
    auto level_b = [&](auto sign) {
      if (t < 3 * N1) {
        float2 v[N2];
        sfor<0, N2>([&](auto J) { v[CV(J)] = Lb[(N2 * kb + CV(J)) * TX + xi]; });
        dft<N2, decltype(sign)::value>(v);
        sfor<0, N2>([&](auto J) { Lb[(N2 * kb + CV(J)) * TX + xi] = v[CV(J)]; });
      }
    };
    level_b(std::integral_constant<int, -1>{});
    __syncthreads();
    if (t < 3 * N1) {
      // thread (part, k1) handles k2 = part, part + 3, ...
      for (int k2 = cb; k2 < N2; k2 += 3) {
        const int o = (N2 * kb + k2) * TX + xi;
        float2 u0 = L0[o], u1 = L1[o], u2 = L2[o];
        green(u0, u1, u2, kb + N1 * k2);
        L0[o] = u0;
        L1[o] = u1;
        L2[o] = u2;
      }
    }
    __syncthreads();
    level_b(std::integral_constant<int, +1>{});
  }
  __syncthreads();

  // inverse level A: conj twiddle, inverse DFT-N1, store z = j2 + N2 j1
  if (t < 3 * N2 && xok) {
    float2* Lc = lds + ca * N * TX;
    float2 b[N1];
    sfor<0, N1>([&](auto K1) { b[CV(K1)] = Lc[(j2 + N2 * CV(K1)) * TX + xi]; });
    const float2* twt = tw + j2 * N1;
    sfor<0, N1>([&](auto K1) { b[CV(K1)] = cmulc(b[CV(K1)], twt[CV(K1)]); });
    dft<N1, +1>(b);
    float2* col = colbase + ca * a.sW + (long long)j2 * plane;
    sfor<0, N1>([&](auto J1) { col[CV(J1) * zst] = b[CV(J1)]; });
  }
}

}  // namespace cbs
#include "scpml_axis.hpp"
namespace cbs {

// ---------------------------------------------------------------------------
// launchers and the per-size registry
// ---------------------------------------------------------------------------
using LaunchK1 = void (*)(const CbsArgs&, int mode, hipStream_t);
using LaunchKY = void (*)(const CbsArgs&, int sign, hipStream_t);
using LaunchKZ = void (*)(const CbsArgs&, hipStream_t);
using LaunchSc = void (*)(const ScAxis&, bool grad, hipStream_t);

struct SizeOps {
  int n;
  LaunchK1 kxy;       // the fused plane pass of an n x n plane (nullptr: none)
  LaunchK1 k1;        // x axis
  LaunchKY ky;        // y axis
  LaunchKZ kz;        // z axis (nullptr: unsupported on z)
  LaunchSc scx, scy, scz;   // stretched-layer products along x, y and z (z: nullptr as kz)
  int n1, n2;         // split of the x/y passes (twiddle table layout)
  int z1, z2;         // split of the z pass
  int k1_rows;         // rows per x-pass workgroup when this length is the x axis
};

constexpr int kTY = kBrick;   // columns per y-pass block

// Whether the iteration kernel holds at most two waves per SIMD (occupancy
// API, once per size): then its work-groups raise their priority for the load
// phase (measured at 621 = 27 x 23, two waves: x-pass 2.36 -> 2.30 ms; at
// 275 = 25 x 11, three waves: 0.58 -> 0.60 ms, so not there).
template <int N1, int N2>
int k1_low_occupancy() {
  static int v = -1;
  if (v < 0) {
    using G = XGeom<N1, N2>;
    int b = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k1_xpass<N1, N2, K1_ITER, FORM_PLAIN>, G::THREADS,
                                                     0) != hipSuccess || b <= 0)
      v = 0;
    else
      v = b * (G::THREADS / 64) <= 2 * 4 ? 1 : 0;   // 4 SIMDs per CU
  }
  return v;
}

// the instantiation of a mode and source: go(mode, form)
template <class F>
void with_form(const CbsArgs& a, int mode, F&& go) {
  using std::integral_constant;
  auto forms = [&](auto MD) {
    if (a.src == SRC_FIELD || a.src == SRC_FIELD_CONJ || a.green_in)
      go(MD, integral_constant<int, FORM_FIELD>{});
    else if (a.oblique && a.src == SRC_PLANE)
      go(MD, integral_constant<int, FORM_OBLIQUE>{});
    else
      go(MD, integral_constant<int, FORM_PLAIN>{});
  };
  if (mode == K1_FWD)
    forms(integral_constant<int, K1_FWD>{});
  else if (mode == K1_ITER)
    forms(integral_constant<int, K1_ITER>{});
  else if (mode == K1_RES)
    go(integral_constant<int, K1_RES>{}, integral_constant<int, FORM_PLAIN>{});
  else
    go(integral_constant<int, K1_INV>{}, integral_constant<int, FORM_PLAIN>{});
}

template <int N1, int N2>
void launch_k1(const CbsArgs& a_in, int mode, hipStream_t s) {
  using G = XGeom<N1, N2>;
  CbsArgs a = a_in;
  a.k1_prio = k1_low_occupancy<N1, N2>();
  const unsigned nb = 3u * (unsigned)a.nb * (unsigned)a.gy * (unsigned)a.nz;
  auto go = [&](auto MD, auto FM) {
    hipLaunchKernelGGL((k1_xpass<N1, N2, CV(MD), CV(FM)>), dim3(nb), dim3(G::THREADS), 0, s, a);
  };
  with_form(a, mode, go);
}

template <int N1, int N2>
int ky_low_occupancy() {
  static int v = -1;
  if (v < 0) {
    using G = YGeom<N1, N2, kTY>;
    int b = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, ky_pass<N1, N2, kTY, -1>, G::THREADS,
                                                     0) != hipSuccess || b <= 0)
      v = 0;
    else
      v = b * (G::THREADS / 64) <= 3 * 4 ? 1 : 0;
  }
  return v;
}

template <int N1, int N2>
void launch_ky(const CbsArgs& a_in, int sign, hipStream_t s) {
  using G = YGeom<N1, N2, kTY>;
  CbsArgs a = a_in;
  a.ky_prio = ky_low_occupancy<N1, N2>();
  dim3 grid((unsigned)((long long)((a.nx + kTY - 1) / kTY) * a.nz * 3 * a.nb));
  if (sign < 0)
    hipLaunchKernelGGL((ky_pass<N1, N2, kTY, -1>), grid, dim3(G::THREADS), 0, s, a);
  else
    hipLaunchKernelGGL((ky_pass<N1, N2, kTY, +1>), grid, dim3(G::THREADS), 0, s, a);
}

template <int N1, int N2>
void launch_kz(const CbsArgs& a, hipStream_t s) {
  constexpr int TX = kz_tx_for(N1, N2);
  using G = ZGeom<N1, N2, TX>;
  dim3 grid((unsigned)((long long)(a.nxp / TX) * a.ny * a.nb) + 1);   // + the residual's block
  if (a.z_first)
    hipLaunchKernelGGL((kz_pass<N1, N2, TX, true>), grid, dim3(G::THREADS), 0, s, a);
  else
    hipLaunchKernelGGL((kz_pass<N1, N2, TX, false>), grid, dim3(G::THREADS), 0, s, a);
}

template <int N1, int N2>
void launch_kxy(const CbsArgs& a, int mode, hipStream_t s) {
  using G = XYGeom<N1, N2>;
  const dim3 grid(3u * (unsigned)a.nb * (unsigned)a.nz), block(G::THREADS);
  with_form(a, mode, [&](auto MD, auto FM) {
    if constexpr (CV(MD) != K1_INV)   // cbs_apply_green's x pass has no plane form
      hipLaunchKernelGGL((kxy_pass<N1, N2, CV(MD), CV(FM)>), grid, block, 0, s, a);
  });
}
// the fused plane pass needs a plane of N x N complex values in 160 KB of LDS
template <int N1, int N2>
constexpr LaunchK1 kxy_for() {
  if constexpr (N2 > 1 && N1 * N2 <= 128)
    return &launch_kxy<N1, N2>;
  else
    return nullptr;
}

#define CBS_SIZE_XYZ(n, a1, a2, z1, z2)                                                         \
  SizeOps {                                                                                     \
    n, kxy_for<a1, a2>(), &launch_k1<a1, a2>, &launch_ky<a1, a2>, &launch_kz<z1, z2>,           \
        &launch_sc<a1, a2, true>, &launch_sc<a1, a2, false>, &launch_sc<z1, z2, false>, a1, a2, \
        z1, z2, XGeom<a1, a2>::LINES                                                            \
  }
#define CBS_SIZE_XY(n, a1, a2)                                                           \
  SizeOps {                                                                              \
    n, nullptr, &launch_k1<a1, a2>, &launch_ky<a1, a2>, nullptr, &launch_sc<a1, a2, true>, \
        &launch_sc<a1, a2, false>, nullptr, a1, a2, 0, 0, XGeom<a1, a2>::LINES           \
  }

// registry, defined in the size translation units
const SizeOps* find_size(int n);

}  // namespace cbs
