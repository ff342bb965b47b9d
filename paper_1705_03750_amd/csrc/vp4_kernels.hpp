// vp4_kernels.hpp -- HIP kernels (gfx950) of the metric semi-Lagrangian
// method in 4D phase space: 2D periodic space (x, y) x 2D velocity (u, w)
// (Colombi & Alard, arXiv:1705.03750: 60 numbers per element, section 2.1;
// 15-point interpolation, section 2.2.1; Fourier solution of Poisson's
// equation for periodic systems, section 2.5).
//
// Arithmetic is written operation by operation (-ffp-contract=off).
//
// Device data (inside the caller's workspace):
//   F, C, f  [nv][nv][ns][ns] (x fastest): F_ini, spline coefficients and a
//            scratch f; no padding -- the interpolations wrap x and y and
//            treat u and w as zero (F) or mirrored (C) outside the grid.
//   state    SoA [60][E]; rec AoS [E][64]: X (4), A = T^-1 (16), the
//            element's cull constants (R_K, R_DELTA; two words unused), and
//            -H/2 with the off-diagonal terms doubled (40).
//   lists    per query block of 4^4 sites: a count and cap element ids;
//            every element whose validity window can reach a site of the
//            block is listed.  Block boundaries sit half an element spacing
//            (mod 4) off the grid origin, on the element lattice, so that an
//            undeformed lattice puts 2 elements per axis in each list; the
//            first and last block of an axis may be partial, and on x and y
//            they are the two halves of the seam block, which share a list.
//   part     density partials [velocity blocks][ns^2] (one row of partial
//            sums per velocity block); rho [ns^2]; transforms and the 12 force
//            fields (a_x, a_y, grad a, Hessian of a) [12][ns^2].
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vp4k {

constexpr int NST = 60;
constexpr int S_P = 0, S_T = 4, S_H = 20;  // state rows
constexpr int RS = 64;                     // record doubles (512 bytes)
constexpr int R_A = 4, R_K = 20, R_DELTA = 21, R_G = 24;  // record offsets
constexpr int BLK = 4;                     // sites per axis of a block
constexpr int SPAN = 4096;                 // max blocks of one element
// Grids without lists: at most DIRECT_FEW elements, or DIRECT_MAX where a ring
// holds at most two (a window of the undeformed lattice then covers it already,
// and lists hold every element, most of them more than once).  us for f with
// lists / without: 8^4, stride 4, 16 elements 44 / 28; 16^4, stride 8 43 / 29;
// 32^4, stride 16 106 / 88; 16^2 x 8^2, strides 4 and 8, sheared 39 / 28; 8^2 x
// 16^2, stride 4, 64 elements, sheared 67 / 54.  Above: 36 elements, three per
// ring (24^2 x 8^2) 32 / 41; 144 elements (8^2 x 24^2) 77 / 109.
constexpr int DIRECT_FEW = 16;
constexpr int DIRECT_MAX = 64;
enum { FL_NUMERIC = 1, FL_WIDE = 2 };
enum { M_DENSITY = 0, M_F = 1, M_ASSIGN = 2 };

// symmetric pair (b, c), b <= c: 00 01 02 03 11 12 13 22 23 33
__device__ __constant__ const int PB[10] = {0, 0, 0, 0, 1, 1, 1, 2, 2, 3};
__device__ __constant__ const int PC[10] = {0, 1, 2, 3, 1, 2, 3, 2, 3, 3};

struct KP {
  int ns, nv, ss, sv, ms, mv, E;
  int o[4];      // block origin offset per axis, (spacing / 2) mod 4
  int ob[4];     // 1 when o > 0 (a partial first block)
  int nb[4];     // blocks per axis
  int nls;       // list columns per space axis (ns / 4)
  int cap;       // list slots per block
  int direct;    // no lists, queries scan the elements (DIRECT_MAX)
  double L, hL, vmax, dx, du, inv_dx, inv_du, G, dt, h, beta;
  double inv_ms, inv_mv;  // 1 / ms, 1 / mv (lat_index)
  double Dm[4], rD[4];  // element spacings and their inverses; the two space
                        // axes' are equal, and the two velocity axes'
};

__device__ __forceinline__ double coord(const KP &p, int a, int i) {
  return a < 2 ? ((double)i + 0.5) * p.dx : -p.vmax + ((double)i + 0.5) * p.du;
}
__device__ __forceinline__ double lat_q(const KP &p, int a, int k) {
  const int s = a < 2 ? p.ss : p.sv;
  return coord(p, a, s * k + s / 2);
}
// Lattice indices of element e < 2^24: the quotients by ms and mv (at most
// 2^9) from a multiplication, (e + 1/2) / m being at least 2^-10 away from
// an integer.
__device__ __forceinline__ void lat_index(const KP &p, int e, int k[4]) {
  int q = (int)(((double)e + 0.5) * p.inv_ms);
  k[0] = e - q * p.ms;
  e = q;
  q = (int)(((double)e + 0.5) * p.inv_ms);
  k[1] = e - q * p.ms;
  e = q;
  q = (int)(((double)e + 0.5) * p.inv_mv);
  k[2] = e - q * p.mv;
  k[3] = q;
}
__device__ __forceinline__ double wrapL(const KP &p, double x) {
  if (x < 0.0) {
    x = x + p.L;
    if (x >= p.L) x = 0.0;
  } else if (x >= p.L) {
    x = x - p.L;
    if (x < 0.0) x = 0.0;
  }
  return x;
}
__device__ __forceinline__ double image(const KP &p, double d) {
  if (d > p.hL) return d - p.L;
  if (d < -p.hL) return d + p.L;
  return d;
}

// Query-block geometry: block b of axis a starts at site o_a + 4 (b - ob_a),
// o_a = (element spacing / 2) mod 4, the element lattice's offset.
__device__ __forceinline__ int floordiv4(int i) {
  return (i >= 0) ? i / BLK : -((-i + BLK - 1) / BLK);
}
__device__ __forceinline__ int blk_of(const KP &p, int a, int i) {
  return floordiv4(i - p.o[a]) + p.ob[a];
}
__device__ __forceinline__ int blk_first(const KP &p, int a, int b) {
  return p.o[a] + BLK * (b - p.ob[a]);
}
// List of block (bx, by, bu, bw): x and y wrap onto ns / 4 list columns.
__device__ __forceinline__ long long list_of(const KP &p, int bx, int by, int bu,
                                             int bw) {
  const int lx = ((bx % p.nls) + p.nls) % p.nls;
  const int ly = ((by % p.nls) + p.nls) % p.nls;
  return (((long long)bw * p.nb[2] + bu) * p.nls + ly) * p.nls + lx;
}

// LDS written by a lane of the wavefront, read by another.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------- elements

__global__ __launch_bounds__(256) void k4_reset(KP p, double *__restrict__ st) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= p.E) return;
  const size_t E = (size_t)p.E;
  int k[4];
  lat_index(p, e, k);
  for (int s = 0; s < NST; ++s) st[s * E + e] = 0.0;
  for (int a = 0; a < 4; ++a) {
    st[(S_P + a) * E + e] = lat_q(p, a, k[a]);
    st[(S_T + 5 * a) * E + e] = 1.0;
  }
}

__global__ __launch_bounds__(256) void k4_zero(int *__restrict__ a, long long n) {
  const long long gsz = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += gsz)
    a[i] = 0;
}

// A = T^-1 by the adjugate (2 x 2 minors of rows 0-1 and rows 2-3); false
// when det T is not positive and finite.
__device__ __forceinline__ bool inv4(const double *m, double *r, double &det) {
  const double a0 = m[0] * m[5] - m[4] * m[1];
  const double a1 = m[0] * m[6] - m[4] * m[2];
  const double a2 = m[0] * m[7] - m[4] * m[3];
  const double a3 = m[1] * m[6] - m[5] * m[2];
  const double a4 = m[1] * m[7] - m[5] * m[3];
  const double a5 = m[2] * m[7] - m[6] * m[3];
  const double b5 = m[10] * m[15] - m[14] * m[11];
  const double b4 = m[9] * m[15] - m[13] * m[11];
  const double b3 = m[9] * m[14] - m[13] * m[10];
  const double b2 = m[8] * m[15] - m[12] * m[11];
  const double b1 = m[8] * m[14] - m[12] * m[10];
  const double b0 = m[8] * m[13] - m[12] * m[9];
  det = ((((a0 * b5 - a1 * b4) + a2 * b3) + a3 * b2) - a4 * b1) + a5 * b0;
  if (!(det > 0.0) || !isfinite(det)) return false;
  const double q = 1.0 / det;
  r[0] = ((m[5] * b5 - m[6] * b4) + m[7] * b3) * q;
  r[1] = ((-m[1] * b5 + m[2] * b4) - m[3] * b3) * q;
  r[2] = ((m[13] * a5 - m[14] * a4) + m[15] * a3) * q;
  r[3] = ((-m[9] * a5 + m[10] * a4) - m[11] * a3) * q;
  r[4] = ((-m[4] * b5 + m[6] * b2) - m[7] * b1) * q;
  r[5] = ((m[0] * b5 - m[2] * b2) + m[3] * b1) * q;
  r[6] = ((-m[12] * a5 + m[14] * a2) - m[15] * a1) * q;
  r[7] = ((m[8] * a5 - m[10] * a2) + m[11] * a1) * q;
  r[8] = ((m[4] * b4 - m[5] * b2) + m[7] * b0) * q;
  r[9] = ((-m[0] * b4 + m[1] * b2) - m[3] * b0) * q;
  r[10] = ((m[12] * a4 - m[13] * a2) + m[15] * a0) * q;
  r[11] = ((-m[8] * a4 + m[9] * a2) - m[11] * a0) * q;
  r[12] = ((-m[4] * b3 + m[5] * b1) - m[6] * b0) * q;
  r[13] = ((m[0] * b3 - m[1] * b1) + m[2] * b0) * q;
  r[14] = ((-m[12] * a3 + m[13] * a1) - m[14] * a0) * q;
  r[15] = ((m[8] * a3 - m[9] * a1) + m[10] * a0) * q;
  return true;
}

// One field of the force at (x, y): 3 x 3 dual TSC.
__device__ __forceinline__ double tsc_field(const KP &p,
                                            const double *__restrict__ A,
                                            double x, double y) {
  const int n = p.ns;
  double u[2] = {x * p.inv_dx - 0.5, y * p.inv_dx - 0.5};
  double w[2][3];
  int at[2][3];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    if (!(u[a] >= -3.0)) u[a] = -3.0;
    if (u[a] > (double)n + 2.0) u[a] = (double)n + 2.0;
    const double fi = floor(u[a] + 0.5), d = u[a] - fi;
    const double tm = 0.5 - d, tp = 0.5 + d;
    w[a][0] = 0.5 * (tm * tm);
    w[a][1] = 0.75 - d * d;
    w[a][2] = 0.5 * (tp * tp);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      // sites in [-4, n + 3] and n >= 8: at most one period off
      const int i = (int)fi - 1 + q;
      at[a][q] = i < 0 ? i + n : (i >= n ? i - n : i);
    }
  }
  double row[3];
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const double *R = A + (size_t)at[1][b] * n;
    row[b] = fma(w[0][2], R[at[0][2]],
                 fma(w[0][1], R[at[0][1]], w[0][0] * R[at[0][0]]));
  }
  return fma(w[1][2], row[2], fma(w[1][1], row[1], w[1][0] * row[0]));
}

// The element pass (section 2.4): kick over dt and corrector drift (when
// `kick`), predictor drift (when `drift`), then (when `predict`) the inverse,
// the query record and the registration in every block the validity window
// can reach, counted in cnt_reg; cnt_zero (nzero counts) is cleared.
//
// A workgroup takes EPW consecutive elements with their states in LDS, and
// its threads the entries of the states (the kick and the drifts act entry by
// entry), then the (element, block) pairs of the registration.  One thread
// per element kept 60 entries in registers and walked its 81 or more blocks
// one after another, each with an atomic to wait for: 159 us at 64^4 (65536
// elements) and 126 us at 16^4 (256), against 97 and 11 us on average for this
// pass, the kick (18 and 9 us as its own launch) included.  It waits on the
// slot claims' device atomics.
//
// EPW from the number of elements (elem_epw): 16 share the lines of the state
// rows, but a workgroup's claims are a chain of rounds, up to 16 x 4096 pairs of
// sheared elements on a narrow ring, so that a pass of few elements is spread
// over more workgroups.  us per step with 16 / 4 / 1 (stride 4, sheared): 256
// elements 24 / 13 / 11, 1024 25 / 16 / 15, 2304 29 / 20 / 27, 4096 30 / 23 / 34,
// 6400 33 / 32 / 47, 9216 36 / 37 / 61, 65536 149 / 167 / 394; stride 8 on 32 and
// 64 sites, 256 elements 93 / 34 / 15, 4096 133 / 75 / 70.
constexpr int REG_AHEAD = 4;  // pairs in flight per thread
inline int elem_epw(int E) { return E <= 1024 ? 1 : E <= 8192 ? 4 : 16; }
template <int EPW>
struct ElemLds {
  static constexpr int EP1 = EPW + 1;  // pitch
  double s[NST][EP1], A[16][EP1], f[12][EP1], u[4][EP1];
  double k[EPW], delta[EPW];
  int blo[4][EP1], ext[4][EP1], at[EP1];
};

// Entry r of the 30 that a drift (or a kick) changes: its state row and the
// row of its rate (a drift adds h times the velocity row).
__device__ __forceinline__ void moving_row(int r, int &space, int &vel) {
  if (r < 2) {
    space = S_P + r;
    vel = space + 2;
  } else if (r < 10) {
    space = S_T + r - 2;
    vel = space + 8;
  } else {
    space = S_H + r - 10;
    vel = space + 20;
  }
}

// Can the validity window of element e of the workgroup hold a site of the
// block whose sites span [g0, g1] per axis (space columns unwrapped)?  l = A dP is
// linear, so over the block's box each l_a ranges over its centre value +-
// sum_b |A_ab| half-width_b; rounding margins as in the 2D engine.
template <int EPW>
__device__ __forceinline__ bool block_meets(const KP &p, const ElemLds<EPW> &S,
                                            int e, const int g0[4],
                                            const int g1[4]) {
  double m[4], h[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const double lo = coord(p, a, g0[a]), hi = coord(p, a, g1[a]);
    m[a] = 0.5 * (lo + hi) - S.s[S_P + a][e];
    h[a] = 0.5 * (hi - lo);
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    double c = 0.0, rad = 0.0, mag = 0.0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const double A = S.A[4 * a + b][e];
      c = fma(A, m[b], c);
      rad = fma(fabs(A), h[b], rad);
      mag = fma(fabs(A), fabs(m[b]) + h[b] + 1.0, mag);
    }
    const double tol = 0x1p-36 * (mag + p.Dm[a]);
    if (!(fabs(c) - rad < p.Dm[a] + tol)) return false;
  }
  return true;
}

template <int EPW>
__global__ __launch_bounds__(256) void k4_elem(
    KP p, double *__restrict__ st, const double *__restrict__ fld,
    double *__restrict__ rec, int *__restrict__ cnt_zero, long long nzero,
    int *__restrict__ cnt_reg, int *__restrict__ lst, int *__restrict__ flags,
    int kick, int drift, int predict) {
  __shared__ ElemLds<EPW> S;
  const int tid = threadIdx.x;
  const long long gsz = (long long)gridDim.x * 256;
  for (long long i = (long long)blockIdx.x * 256 + tid; i < nzero; i += gsz)
    cnt_zero[i] = 0;
  const int e0 = blockIdx.x * EPW, ne = min(EPW, p.E - e0);
  if (ne <= 0) return;
  const size_t E = (size_t)p.E;
  for (int q = tid; q < NST * EPW; q += 256) {
    const int r = q / EPW, e = q % EPW;
    if (e < ne) S.s[r][e] = st[r * E + e0 + e];
  }
  __syncthreads();
  if (kick) {
    const int k = tid / EPW, e = tid % EPW;
    if (k < 12 && e < ne)
      S.f[k][e] = tsc_field(p, fld + (size_t)k * p.ns * p.ns, S.s[S_P][e],
                            S.s[S_P + 1][e]);
    __syncthreads();
    // v, T_v. and H_v.. (reading R5: the right-hand sides use the half-step
    // T and H of the space rows, which the kick leaves alone)
    const double dt = p.dt;
    for (int q = tid; q < 30 * EPW; q += 256) {
      const int r = q / EPW, e = q % EPW;
      if (e >= ne) continue;
      int space, vel;
      moving_row(r, space, vel);
      double v;
      int i;
      if (r < 2) {
        v = S.f[r][e];
      } else if (r < 10) {
        i = (r - 2) >> 2;
        const int j = (r - 2) & 3;
        v = fma(S.f[3 + 2 * i][e], S.s[S_T + 4 + j][e],
                S.f[2 + 2 * i][e] * S.s[S_T + j][e]);
      } else {
        i = (r - 10) / 10;
        const int h = (r - 10) % 10, jb = PB[h], kc = PC[h];
        const double t0j = S.s[S_T + jb][e], t1j = S.s[S_T + 4 + jb][e];
        const double t0k = S.s[S_T + kc][e], t1k = S.s[S_T + 4 + kc][e];
        v = S.f[2 + 2 * i][e] * S.s[S_H + h][e];
        v = fma(S.f[3 + 2 * i][e], S.s[S_H + 10 + h][e], v);
        v = fma(S.f[6 + 3 * i][e], t0j * t0k, v);
        v = fma(S.f[7 + 3 * i][e], fma(t0j, t1k, t1j * t0k), v);
        v = fma(S.f[8 + 3 * i][e], t1j * t1k, v);
      }
      const double x = fma(dt, v, S.s[vel][e]);
      S.s[vel][e] = x;
      st[vel * E + e0 + e] = x;
    }
    __syncthreads();
  }
  if (kick || drift) {
    // the corrector and the next predictor as two roundings, as two passes
    for (int q = tid; q < 30 * EPW; q += 256) {
      const int r = q / EPW, e = q % EPW;
      if (e >= ne) continue;
      int space, vel;
      moving_row(r, space, vel);
      const double v = S.s[vel][e];
      double x = S.s[space][e];
      for (int t = 0; t < kick + drift; ++t) {
        x = fma(p.h, v, x);
        if (r < 2) x = wrapL(p, x);
      }
      S.s[space][e] = x;
      st[space * E + e0 + e] = x;
    }
    __syncthreads();
  }
  if (!predict) return;
  int bad = 0;
  double det = 1.0;
  if (tid < EPW) {
    // A = T^-1, one thread per element
    double T[16], A[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) T[q] = tid < ne ? S.s[S_T + q][tid] : 0.0;
    bad = !inv4(T, A, det);
#pragma unroll
    for (int q = 0; q < 16; ++q) S.A[q][tid] = bad ? 0.0 : A[q];
#pragma unroll
    for (int a = 0; a < 4; ++a) bad = bad || !isfinite(S.s[S_P + a][tid]);
    if (tid < ne && bad) atomicOr(flags, FL_NUMERIC);
  }
  if (tid < 4 * EPW) {
    // four threads per element, one per axis (wavefront 0)
    const int e = tid >> 2, a = tid & 3;
    bad = __shfl(bad, e);
    det = __shfl(det, e);
    wave_sync();
    double x = 0.0;
#pragma unroll
    for (int q = 0; q < 10; ++q)
      x += (PB[q] == PC[q] ? 0.5 : 1.0) * fabs(S.s[S_H + 10 * a + q][e]) *
           (p.Dm[PB[q]] * p.Dm[PC[q]]);
    S.u[a][e] = x;
    wave_sync();
    // Bound of the map's quadratic part, for the query's cull.  On the
    // validity window |l_a| < Dm_a, |u_c| <= sum_bd |H_cbd| Dm_b Dm_d, and
    // the Lagrangian distance between dQ = l - A u / 2 and l (element
    // spacings) is at most delta = |rD_a sum_c |A_ac| |u_c| / 2|, so |z(dQ)|
    // >= |z(l)| - delta.  A site whose best squared distance is bd cannot
    // take the element when |z(l)|^2 > (sqrt(bd) + delta)^2; with 2 delta
    // sqrt(bd) <= delta (1 + bd) it is enough that |z(l)|^2 k - delta > bd,
    // k = 1 / (1 + delta).  The margins (2^-20 relative and 2^-36 absolute
    // on delta, 2^-30 on k) exceed the rounding of dQ and of the test by
    // far, so a culled element loses strictly.
    double t = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) t += fabs(S.A[4 * a + c][e]) * S.u[c][e];
    t *= p.rD[a];
    t *= t;
    t += __shfl_xor(t, 1);
    t += __shfl_xor(t, 2);
    const double delta = sqrt(t) * (1.0 + 0x1p-20) + 0x1p-36;
    if (a == 0) {
      S.delta[e] = delta;
      S.k[e] = (1.0 - 0x1p-30) / (1.0 + delta);
    }
    // Eulerian reach along the axis: |dP_a| <= sum_b |T_ab| Dm_b, in sites,
    // with a relative margin for the rounding of l = A dP
    double reach = 0.0, tsum = 0.0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const double v = fabs(S.s[S_T + 4 * a + b][e]);
      reach = fma(v, p.Dm[b], reach);
      tsum += v;
    }
    const double rel = 0x1p-20 + 0x1p-40 * (tsum * tsum) * fabs(1.0 / det);
    const double inv_d = a < 2 ? p.inv_dx : p.inv_du;
    const double rs = reach * inv_d * (1.0 + rel) + 0x1p-20;
    const double X = S.s[S_P + a][e];
    const double c = (a < 2 ? X : X + p.vmax) * inv_d - 0.5;
    int lo = (int)ceil(c - rs), hi = (int)floor(c + rs);
    bool far = false;
    if (a >= 2) {
      lo = max(lo, 0);
      hi = min(hi, p.nv - 1);
    } else {
      // images lie within half a period of an element at most half a period
      // off the square; a window reaching further enters every list column
      // (the seam's twice: a harmless repetition).  Of an element further off
      // a site sees an image beyond half a period (one period is taken off),
      // which such a window may reach: not listed
      const int reach_lo = (int)floor(c) - p.ns / 2;
      const int reach_hi = (int)ceil(c) + p.ns / 2;
      far = (lo < reach_lo || hi > reach_hi) && !(fabs(X - p.hL) <= p.L);
      lo = max(lo, reach_lo);
      hi = min(hi, reach_hi);
    }
    const int b0 = blk_of(p, a, lo);
    const int n = far || p.direct ? SPAN + 1 : blk_of(p, a, hi) - b0 + 1;
    S.blo[a][e] = b0;  // unwrapped on x and y
    S.ext[a][e] = n;
    // the blocks of the element's box: none for a bad element or a window
    // off the grid; too many of them: the queries scan every element
    int box = (e >= ne || bad || lo > hi) ? 0 : min(n, SPAN + 1);
    int m = __shfl_xor(box, 1);
    box = min(box * m, SPAN + 1);
    m = __shfl_xor(box, 2);
    box = min(box * m, SPAN + 1);
    if (a == 0) {
      if (box > SPAN) {
        atomicOr(flags, FL_WIDE);
        box = 0;
      }
      S.at[e] = box;
    }
    wave_sync();
    // first pair of every element
    if (tid == 0) {
      int sum = 0;
      for (int q = 0; q < EPW; ++q) {
        const int b = S.at[q];
        S.at[q] = sum;
        sum += b;
      }
      S.at[EPW] = sum;
    }
  }
  __syncthreads();
  for (int q = tid; q < RS * ne; q += 256) {
    const int e = q / RS, o = q % RS;
    double v = 0.0;
    if (o < R_A)
      v = S.s[S_P + o][e];
    else if (o < R_K)
      v = S.A[o - R_A][e];
    else if (o == R_K)
      v = S.k[e];
    else if (o == R_DELTA)
      v = S.delta[e];
    else if (o >= R_G)
      v = (PB[(o - R_G) % 10] == PC[(o - R_G) % 10] ? -0.5 : -1.0) *
          S.s[S_H + o - R_G][e];
    rec[(size_t)(e0 + e) * RS + o] = v;
  }
  const int total = S.at[EPW];
  for (int q0 = tid; q0 < total; q0 += 256 * REG_AHEAD) {
    long long blk[REG_AHEAD];
    int id[REG_AHEAD], slot[REG_AHEAD];
#pragma unroll
    for (int k = 0; k < REG_AHEAD; ++k) {
      const int q = q0 + 256 * k;
      blk[k] = -1;
      if (q < total) {
        int e = 0;  // last element whose first pair is <= q
#pragma unroll
        for (int h = EPW / 2; h > 0; h /= 2)
          if (S.at[e + h] <= q) e += h;
        // pair -> block, x fastest (quotients of numbers below 2^12: a float
        // product is exact enough)
        int r = q - S.at[e], b[4], g0[4], g1[4];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const int n = S.ext[a][e];
          const int d = (int)(((float)r + 0.5f) * (1.0f / (float)n));
          b[a] = S.blo[a][e] + (r - d * n);
          r = d;
        }
        b[3] = S.blo[3][e] + r;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          g0[a] = blk_first(p, a, b[a]);
          g1[a] = g0[a] + BLK - 1;
          if (a >= 2) {  // the live sites of a partial velocity block
            g0[a] = max(g0[a], 0);
            g1[a] = min(g1[a], p.nv - 1);
          }
        }
        if (block_meets(p, S, e, g0, g1)) {
          blk[k] = list_of(p, b[0], b[1], b[2], b[3]);
          id[k] = e0 + e;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < REG_AHEAD; ++k)
      slot[k] = blk[k] >= 0 ? atomicAdd(&cnt_reg[blk[k]], 1) : p.cap;
#pragma unroll
    for (int k = 0; k < REG_AHEAD; ++k)
      if (slot[k] < p.cap) lst[blk[k] * p.cap + slot[k]] = id[k];
  }
}

// Second-order inverse map of one element (record r) at offset d = P - X: l
// = A d, then u'_c = l^T (-H_c / 2) l over the symmetric pairs and dQ = l +
// A u' (equal bit for bit to l - A u / 2: scaling by a power of two commutes
// with every rounding).  R is a pointer to the record in any address space.
template <typename R>
__device__ __forceinline__ void map4_l(R r, const double d[4], double l[4]) {
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    R A = r + R_A + 4 * a;
    l[a] = fma(A[3], d[3], fma(A[2], d[2], fma(A[1], d[1], A[0] * d[0])));
  }
}

template <typename R>
__device__ __forceinline__ void map4_q(R r, const double l[4], double dq[4]) {
  double pr[10], u[4];
#pragma unroll
  for (int q = 0; q < 10; ++q) pr[q] = l[PB[q]] * l[PC[q]];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    R G = r + R_G + 10 * a;
    double s = G[0] * pr[0];
#pragma unroll
    for (int q = 1; q < 10; ++q) s = fma(G[q], pr[q], s);
    u[a] = s;
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    R A = r + R_A + 4 * a;
    double s = l[a];
#pragma unroll
    for (int b = 0; b < 4; ++b) s = fma(A[b], u[b], s);
    dq[a] = s;
  }
}

// Offset of site P from an element at the nearest image in x and y.
template <typename R>
__device__ __forceinline__ void offset4(const KP &p, R r, const double P[4],
                                        double d[4]) {
  d[0] = image(p, P[0] - r[0]);
  d[1] = image(p, P[1] - r[1]);
  d[2] = P[2] - r[2];
  d[3] = P[3] - r[3];
}

__device__ __forceinline__ void map4(const KP &p, const double *r,
                                     const double P[4], double dq[4]) {
  double d[4], l[4];
  offset4(p, r, P, d);
  map4_l(r, d, l);
  map4_q(r, l, dq);
}

__device__ __forceinline__ double dist2(const KP &p, const double dq[4]) {
  const double z0 = dq[0] * p.rD[0], z1 = dq[1] * p.rD[0];
  const double z2 = dq[2] * p.rD[2], z3 = dq[3] * p.rD[2];
  return fma(z3, z3, fma(z2, z2, fma(z1, z1, z0 * z0)));
}

// Site of thread t of block blk (blocks numbered x fastest): (i, j, k, l),
// its coordinates, whether it lies on the grid, and the block's list.  A
// wavefront takes 4 x 4 x 2 x 2 sites (sub-block u1 + 2 w1 = t >> 6 of the
// block's four): the more cubic the sub-block, the fewer windows it meets.
// loc is the site's index in the block, x fastest.
__device__ __forceinline__ bool block_site(const KP &p, int blk, int t,
                                           int g[4], double P[4], int bb[4],
                                           int &loc, long long &list) {
  unsigned b = (unsigned)blk;
  bb[0] = (int)(b % (unsigned)p.nb[0]);
  b /= (unsigned)p.nb[0];
  bb[1] = (int)(b % (unsigned)p.nb[1]);
  b /= (unsigned)p.nb[1];
  bb[2] = (int)(b % (unsigned)p.nb[2]);
  bb[3] = (int)(b / (unsigned)p.nb[2]);
  const int lc[4] = {t & 3, (t >> 2) & 3, ((t >> 4) & 1) | ((t >> 5) & 2),
                     ((t >> 5) & 1) | ((t >> 6) & 2)};
  bool live = true;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    g[a] = blk_first(p, a, bb[a]) + lc[a];
    P[a] = coord(p, a, g[a]);
    live = live && g[a] >= 0 && g[a] < (a < 2 ? p.ns : p.nv);
  }
  loc = ((lc[3] * 4 + lc[2]) * 4 + lc[1]) * 4 + lc[0];
  list = list_of(p, bb[0], bb[1], bb[2], bb[3]);
  return live;
}

// LDS of the query, per list slot: the entry (element id, the image shift of
// x and y, 0 none, 1 -L, 2 +L, 3 per site), the sub-blocks its window can
// reach (bits 0-3) and those whose centre it is near (bits 4-7), and per
// sub-block a lower bound of its Lagrangian distance.
struct QueryLds {
  int *ent, *sub;
  float *low;  // [slot][4]
  __device__ __forceinline__ QueryLds(const KP &p, char *lds)
      : ent(reinterpret_cast<int *>(lds)), sub(ent + p.cap),
        low(reinterpret_cast<float *>(sub + p.cap)) {}
};
constexpr int QUERY_SLOT_BYTES = 24;

// Entries k = tid, tid + 256, .. of the block's list, one per thread: from l
// at the block's centre, l is linear in P, so over a sub-block's box it
// ranges over its centre value +- sum_b |A_ab| half-width_b (rounding margins
// as in block_meets).  The distance bound leaves out the rounding of the
// square roots, which the float's own margin covers.
__device__ __forceinline__ void query_filter(const KP &p,
                                             const double *__restrict__ rec,
                                             const int *__restrict__ L, int n,
                                             const int bb[4], QueryLds Q) {
  const double hw[4] = {1.5 * p.dx, 1.5 * p.dx, 0.5 * p.du, 0.5 * p.du};
  for (int k = threadIdx.x; k < n; k += 256) {
    const int e = L[k];
    const double *r = rec + (size_t)e * RS;
    int code = 0;
    double m[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int g0 = blk_first(p, a, bb[a]);
      m[a] = 0.5 * (coord(p, a, g0) + coord(p, a, g0 + BLK - 1)) - r[a];
      if (a < 2) {
        int s = 0;
        if (m[a] > p.hL) {
          m[a] = m[a] - p.L;
          s = 1;
        } else if (m[a] < -p.hL) {
          m[a] = m[a] + p.L;
          s = 2;
        }
        // the block's sites on both sides of the half period
        if (fabs(m[a]) + 2.0 * p.dx > p.hL) s = 3;
        code |= s << (24 + 2 * a);
      }
    }
    const bool split = ((code >> 24) & 3) == 3 || ((code >> 26) & 3) == 3;
    int bits = 0;
    double zc2[4] = {0.0, 0.0, 0.0, 0.0}, zr2 = 0.0;
    bool ok[4] = {true, true, true, true};
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const double *A = r + R_A + 4 * a;
      double c = 0.0, rad = 0.0, mag = 0.0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        c = fma(A[b], m[b], c);
        rad = fma(fabs(A[b]), hw[b], rad);
        mag = fma(fabs(A[b]), fabs(m[b]) + 2.0 * (hw[b] + p.du) + 1.0, mag);
      }
      const double lim = p.Dm[a] + 0x1p-36 * (mag + p.Dm[a]) + rad;
      const double z = rad * p.rD[a];
      zr2 = fma(z, z, zr2);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const double ls = c + (((s & 1) ? A[2] : -A[2]) +
                               ((s & 2) ? A[3] : -A[3])) * p.du;
        ok[s] = ok[s] && fabs(ls) < lim;
        const double zs = ls * p.rD[a];
        zc2[s] = fma(zs, zs, zc2[s]);
      }
    }
    const double out = sqrt(zr2) + r[R_DELTA];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (ok[s] || split) bits |= 1 << s;
      if (zc2[s] < 1.0) bits |= 16 << s;
      Q.low[4 * k + s] =
          split ? -1.0f : (float)(sqrt(zc2[s]) - out) * 0.9999f - 1e-4f;
    }
    Q.ent[k] = e | code;
    Q.sub[k] = bits;
  }
}

// One candidate at this lane's site: l, validity, the cull against the best
// distance so far (whole wavefronts skip the quadratic part), and the
// (d^2, id) update.
template <typename R>
__device__ __forceinline__ void query_candidate(const KP &p, R r, int e,
                                                bool live, const double d[4],
                                                double &bd, int &best,
                                                double bdq[4]) {
  double l[4], zl[4];
  map4_l(r, d, l);
  // every lane, no short cuts: the tests combine as lane masks
  bool valid = live;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    valid = valid & (fabs(l[a]) < p.Dm[a & 2]);
    zl[a] = l[a] * p.rD[a & 2];
  }
  const double z2 = fma(zl[3], zl[3], fma(zl[2], zl[2], fma(zl[1], zl[1],
                                                            zl[0] * zl[0])));
  if (__ballot(valid & !(z2 * r[R_K] - r[R_DELTA] > bd)) == 0ull) return;
  double dq[4];
  map4_q(r, l, dq);
  const double d2 = dist2(p, dq);
  if (valid & ((d2 < bd) | ((d2 == bd) & (e < best)))) {
    bd = d2;
    best = e;
#pragma unroll
    for (int a = 0; a < 4; ++a) bdq[a] = dq[a];
  }
}

// Can the validity window of an element (record r) reach the sub-block of
// centre ctr?  The bound of query_filter; a sub-block with sites on both sides
// of the half period is taken as reached.
__device__ __forceinline__ bool reaches(const KP &p, const double *r,
                                        const double ctr[4]) {
  const double hw[4] = {1.5 * p.dx, 1.5 * p.dx, 0.5 * p.du, 0.5 * p.du};
  double m[4];
  bool split = false, ok = true;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    m[a] = ctr[a] - r[a];
    if (a < 2) {
      m[a] = image(p, m[a]);
      split = split || fabs(m[a]) + 2.0 * p.dx > p.hL;
    }
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const double *A = r + R_A + 4 * a;
    double c = 0.0, rad = 0.0, mag = 0.0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      c = fma(A[b], m[b], c);
      rad = fma(fabs(A[b]), hw[b], rad);
      mag = fma(fabs(A[b]), fabs(m[b]) + 2.0 * hw[b] + 1.0, mag);
    }
    ok = ok && fabs(c) < p.Dm[a] + 0x1p-36 * (mag + p.Dm[a]) + rad;
  }
  return ok || split;
}

// Nearest valid element (smallest (d^2, id)) of every site of the workgroup's
// block.  The workgroup first sorts the list's entries by sub-block, one per
// thread (query_filter); each wavefront then walks its own sub-block's
// candidates, the near ones (centre closer than one spacing, about the
// undeformed lattice's nearest few) first, so that the far ones can be
// dropped by their distance bound (a lane per candidate) and by the cull.
// Records are read through the scalar cache: they are uniform over the
// wavefront, and the operands come straight from scalar registers.
//
// With an overflowed list, a too-wide element or no lists every element is
// scanned.  SORTED: a wavefront first tests 64 of them at a time against its
// sub-block (reaches) and walks those that pass; else it walks them all, each
// record waited for.  4096 elements at 256^2 x 4^2 (stride 4), walked: 29.0 ms
// in the reconstruction, 39.7 in the resampling, which has three wavefronts per
// SIMD to hide the waits; sorted: 3.0 and 4.1, but the test's registers cost
// the reconstruction's lists 0.4 (64^4) to 1.5 % (16^4), so that it walks.
typedef const __attribute__((address_space(4))) double cdouble;
template <bool SORTED>
__device__ __forceinline__ int query4(const KP &p, const double *__restrict__ rec,
                                      const int *__restrict__ L, int n,
                                      bool scan_all, bool live, const int bb[4],
                                      const double P[4], double bdq[4],
                                      char *lds) {
  double bd = __builtin_inf();
  int best = -1;
  for (int a = 0; a < 4; ++a) bdq[a] = 0.0;
  auto record = [&](int e) {
    return (cdouble *)(unsigned long long)(rec + (size_t)e * RS);
  };
  if (!SORTED && scan_all) {
    for (int e = 0; e < p.E; ++e) {
      cdouble *r = record(e);
      double d[4];
      offset4(p, r, P, d);
      query_candidate(p, r, e, live, d, bd, best, bdq);
    }
    return best;
  }
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (SORTED && scan_all) {
    double ctr[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int g0 = blk_first(p, a, bb[a]);
      ctr[a] = 0.5 * (coord(p, a, g0) + coord(p, a, g0 + BLK - 1));
    }
    ctr[2] += (w & 1) ? p.du : -p.du;
    ctr[3] += (w & 2) ? p.du : -p.du;
    for (int e0 = 0; e0 < p.E; e0 += 64) {
      const int el = min(e0 + lane, p.E - 1);
      unsigned long long todo = __ballot(
          e0 + lane < p.E && reaches(p, rec + (size_t)el * RS, ctr));
      while (todo) {
        const int e = e0 + __builtin_ctzll(todo);
        todo &= todo - 1;
        cdouble *r = record(e);
        double d[4];
        offset4(p, r, P, d);
        query_candidate(p, r, e, live, d, bd, best, bdq);
      }
    }
    return best;
  }
  const QueryLds Q(p, lds);
  query_filter(p, rec, L, n, bb, Q);
  __syncthreads();
  float top = __builtin_inff();
  for (int far = 0; far < 2; ++far) {
    if (far) {
      // no site of the sub-block takes an element beyond its worst distance
      top = live ? (float)sqrt(bd) * 1.0001f : 0.0f;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1)
        top = fmaxf(top, __shfl_xor(top, off));
    }
    for (int c0 = 0; c0 < n; c0 += 64) {
      const int k = c0 + lane;
      int ent = 0, sub = 0;
      float low = 0.0f;
      if (k < n) {
        ent = Q.ent[k];
        sub = Q.sub[k] >> w;
        low = Q.low[4 * k + w];
      }
      unsigned long long todo =
          __ballot((sub & 1) && ((sub >> 4) & 1) == (far ? 0 : 1) && !(low > top));
      while (todo) {
        const int j = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int en = __builtin_amdgcn_readlane(ent, j);
        const int e = en & 0xffffff, sx = (en >> 24) & 3, sy = (en >> 26) & 3;
        cdouble *r = record(e);
        double d[4];
        if (sx == 3 || sy == 3) {
          offset4(p, r, P, d);
        } else {
          const double hx = sx == 1 ? -p.L : (sx == 2 ? p.L : 0.0);
          const double hy = sy == 1 ? -p.L : (sy == 2 ? p.L : 0.0);
          d[0] = (P[0] - r[0]) + hx;
          d[1] = (P[1] - r[1]) + hy;
          d[2] = P[2] - r[2];
          d[3] = P[3] - r[3];
        }
        query_candidate(p, r, e, live, d, bd, best, bdq);
      }
    }
  }
  return best;
}

// ------------------------------------------------------- interpolations

// 15-point second-order interpolation (section 2.2.1 in four dimensions):
// nearest node, its 8 axis neighbours (Lagrange signs), and one cross term
// per axis pair at the floor corner of that plane.  x, y positions clamped
// to [-12, ns + 11] and wrapped; zero outside the u, w grid.  Every stencil
// index along an axis is the nearest node's -1, 0 or +1 (the floor corner
// is the nearest node or the one below), so 15 values serve the 33 terms.
// (Grids hold at most 2^31 values: 32-bit indices.)
template <typename FT>
__device__ __forceinline__ FT int15(const KP &p, const FT *__restrict__ F,
                                    const double sin_[4]) {
  double s[4];
  for (int a = 0; a < 4; ++a) s[a] = sin_[a];
  for (int a = 0; a < 2; ++a) {
    if (s[a] < -12.0) s[a] = -12.0;
    if (s[a] > (double)p.ns + 11.0) s[a] = (double)p.ns + 11.0;
  }
  for (int a = 2; a < 4; ++a)
    if (!(s[a] > -4.0 && s[a] < p.nv + 3.0)) return (FT)0;
  // nearest node, whether the floor node is the nearest one (else the one
  // below), the offset from it; index steps to the nodes below and above
  const int str[4] = {1, p.ns, p.ns * p.ns, p.ns * p.ns * p.nv};
  bool fl[4], in[4][3];
  FT dq[4];
  int at0 = 0, step[4][3];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const double fn = floor(s[a] + 0.5);
    int n = (int)fn;
    fl[a] = (int)floor(s[a]) == n;
    dq[a] = (FT)(s[a] - fn);
    int lo = n - 1, hi = n + 1;
    if (a < 2) {
      // positions in [-14, ns + 13] and ns >= 8: at most two periods off
      auto wrap = [&](int i) {
        i += i < 0 ? p.ns : 0;
        i += i < 0 ? p.ns : 0;
        i -= i >= p.ns ? p.ns : 0;
        i -= i >= p.ns ? p.ns : 0;
        return i;
      };
      lo = wrap(lo);
      n = wrap(n);
      hi = wrap(hi);
    } else {
      // off the u, w grid: zero (read from a node that exists)
      in[a][0] = lo >= 0 && lo < p.nv;
      in[a][1] = n >= 0 && n < p.nv;
      in[a][2] = hi >= 0 && hi < p.nv;
      lo = min(max(lo, 0), p.nv - 1);
      n = min(max(n, 0), p.nv - 1);
      hi = min(max(hi, 0), p.nv - 1);
    }
    at0 += n * str[a];
    step[a][0] = (lo - n) * str[a];
    step[a][1] = 0;
    step[a][2] = (hi - n) * str[a];
  }
  auto at = [&](int i, bool ok) -> FT {
    const FT v = F[(unsigned)i];
    return ok ? v : (FT)0;
  };
  // the nearest node, its axis neighbours, and per axis the neighbour on the
  // other side of the cell (index o): 2 where the floor node is the nearest
  const FT c = at(at0, in[2][1] & in[3][1]);
  FT w0 = (FT)1 - dq[0] * dq[0];
#pragma unroll
  for (int a = 1; a < 4; ++a) w0 = w0 - dq[a] * dq[a];
  FT f = c * w0, nb[4];
  int so[4];
  bool ino[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const bool other = (a == 2 ? in[3][1] : a == 3 ? in[2][1] : in[2][1] & in[3][1]);
    const FT up = at(at0 + step[a][2], a < 2 ? other : other & in[a][2]);
    const FT dn = at(at0 + step[a][0], a < 2 ? other : other & in[a][0]);
    const FT h = (FT)0.5 * dq[a];
    const FT wp = h * ((FT)1 + dq[a]), wm = h * ((FT)1 - dq[a]);
    f = fma(up, wp, f);
    f = fma(-dn, wm, f);
    nb[a] = fl[a] ? up : dn;
    so[a] = fl[a] ? step[a][2] : step[a][0];
    ino[a] = a < 2 ? true : (fl[a] ? in[a][2] : in[a][0]);
  }
  // cross terms f11 + f00 - f10 - f01 at the cell's low corner: of the four
  // corners one is the nearest node, two are axis neighbours, one is a
  // diagonal; which is which follows from the floor flags
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = a + 1; b < 4; ++b) {
      bool ok = true;
      if (a >= 2) ok = ok & ino[a];
      if (b >= 2) ok = ok & ino[b];
      if (a != 2 && b != 2) ok = ok & in[2][1];
      if (a != 3 && b != 3) ok = ok & in[3][1];
      const FT dg = at(at0 + so[a] + so[b], ok);
      const bool same = fl[a] == fl[b];
      const FT pl = same ? c + dg : nb[a] + nb[b];
      const FT m1 = same ? (fl[a] ? nb[a] : nb[b]) : (fl[a] ? dg : c);
      const FT m2 = same ? (fl[a] ? nb[b] : nb[a]) : (fl[a] ? c : dg);
      f = fma((pl - m1) - m2, dq[a] * dq[b], f);
    }
  return f;
}

// Cubic B-spline weights.  Double precision: each times the rounded 1/6.
// Single precision: six times the weights, the 1/6^4 of the four axes
// applied once to the sum (two-float constant), because float(1/6) is 3e-8
// too large and that shared rounding would scale every resampled value by
// 1 + 1.2e-7 at each resampling.
template <typename FT>
__device__ __forceinline__ void bspw(double ud, FT b[4]) {
  const FT u = (FT)ud;
  const FT t = (FT)1 - u;
  const FT u2 = u * u, u3 = u2 * u;
  if constexpr (sizeof(FT) == 8) {
    const FT sixth = (FT)(1.0 / 6.0);
    b[0] = ((t * t) * t) * sixth;
    b[1] = (((FT)3 * u3 - (FT)6 * u2) + (FT)4) * sixth;
    b[2] = ((((FT)-3 * u3 + (FT)3 * u2) + (FT)3 * u) + (FT)1) * sixth;
    b[3] = u3 * sixth;
  } else {
    b[0] = (t * t) * t;
    b[1] = ((FT)3 * u3 - (FT)6 * u2) + (FT)4;
    b[2] = (((FT)-3 * u3 + (FT)3 * u2) + (FT)3 * u) + (FT)1;
    b[3] = u3;
  }
}

constexpr float INV1296_HI = (float)(1.0 / 1296.0);
constexpr float INV1296_LO =
    (float)(1.0 / 1296.0 - (double)(float)(1.0 / 1296.0));

// Tensor cubic B-spline (x, y periodic, clamped to [-12, ns + 11]; u, w on
// [0, nv - 1] with mirror ghosts c(-1) = c(1), c(n) = c(n - 2); 0 outside).
template <typename FT>
__device__ __forceinline__ FT spline4(const KP &p, const FT *__restrict__ C,
                                      const double sin_[4]) {
  double s[4];
  for (int a = 0; a < 4; ++a) s[a] = sin_[a];
  for (int a = 0; a < 2; ++a) {
    if (s[a] < -12.0) s[a] = -12.0;
    if (s[a] > (double)p.ns + 11.0) s[a] = (double)p.ns + 11.0;
  }
  for (int a = 2; a < 4; ++a)
    if (!(s[a] >= 0.0 && s[a] <= (double)(p.nv - 1))) return (FT)0;
  int i0[4];
  FT w[4][4];
  for (int a = 0; a < 4; ++a) {
    int i = (int)floor(s[a]);
    if (a >= 2 && i > p.nv - 2) i = p.nv - 2;
    i0[a] = i;
    bspw<FT>(s[a] - (double)i, w[a]);
  }
  // row offsets along y, u, w (grids hold at most 2^31 values); the first
  // column of the four along x, and the step to each from it
  auto wrap = [&](int i) {  // positions in [-14, ns + 13], ns >= 8
    i += i < 0 ? p.ns : 0;
    i += i < 0 ? p.ns : 0;
    i -= i >= p.ns ? p.ns : 0;
    i -= i >= p.ns ? p.ns : 0;
    return i;
  };
  const int x0 = wrap(i0[0] - 1);
  unsigned yj[4], uk[4], wl[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    int k = i0[2] - 1 + q, l = i0[3] - 1 + q;
    if (k < 0) k = -k;
    if (k > p.nv - 1) k = 2 * (p.nv - 1) - k;
    if (l < 0) l = -l;
    if (l > p.nv - 1) l = 2 * (p.nv - 1) - l;
    yj[q] = (unsigned)(wrap(i0[1] - 1 + q) * p.ns);
    uk[q] = (unsigned)(k * p.ns * p.ns);
    wl[q] = (unsigned)(l * p.ns * p.ns) * (unsigned)p.nv;
  }
  FT f = (FT)0;
  constexpr int AHEAD = 8;
  // the sum of a row's four terms given its values
  auto row4 = [&](const FT *c) {
    FT r = w[0][0] * c[0];
    r = fma(w[0][1], c[1], r);
    r = fma(w[0][2], c[2], r);
    return fma(w[0][3], c[3], r);
  };
  auto tensor = [&](auto row) {
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      FT fu = (FT)0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        FT fy = (FT)0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const FT r = row(wl[l] + uk[k] + yj[j]);
          fy = (j == 0) ? w[1][0] * r : fma(w[1][j], r, fy);
        }
        fu = (k == 0) ? w[2][0] * fy : fma(w[2][k], fy, fu);
        // at most AHEAD rows in flight: more of them spill
        if (k % (AHEAD / 4) == AHEAD / 4 - 1) __builtin_amdgcn_sched_barrier(0);
      }
      f = (l == 0) ? w[3][0] * fu : fma(w[3][l], fu, f);
    }
  };
  // four neighbouring columns are one load (aligned to a value only) unless a
  // lane's cell lies across the seam
  if (__ballot(x0 + 3 >= p.ns) == 0ull) {
    tensor([&](unsigned at) {
      FT c[4];
      __builtin_memcpy(c, C + (size_t)(at + (unsigned)x0), sizeof(c));
      return row4(c);
    });
  } else {
    const int x1 = x0 + 1 < p.ns ? x0 + 1 : x0 + 1 - p.ns;
    const int x2 = x0 + 2 < p.ns ? x0 + 2 : x0 + 2 - p.ns;
    const int x3 = x0 + 3 < p.ns ? x0 + 3 : x0 + 3 - p.ns;
    tensor([&](unsigned at) {
      const FT *r = C + (size_t)at;
      const FT c[4] = {r[x0], r[x1], r[x2], r[x3]};
      return row4(c);
    });
  }
  if constexpr (sizeof(FT) == 4) f = fmaf(f, INV1296_HI, f * INV1296_LO);
  return f;
}

__device__ __forceinline__ double Wk(double x) {
  if (x <= 1.0) {
    const double x2 = x * x;
    return fma(0.75 * x, x2, fma(-1.5, x2, 1.0));
  }
  if (x <= 2.0) {
    const double t = 2.0 - x;
    return ((0.25 * t) * t) * t;
  }
  return 0.0;
}

__device__ __forceinline__ void index_pos(const KP &p, const double Q[4],
                                          double s[4]) {
  s[0] = Q[0] * p.inv_dx - 0.5;
  s[1] = Q[1] * p.inv_dx - 0.5;
  s[2] = (Q[2] + p.vmax) * p.inv_du - 0.5;
  s[3] = (Q[3] + p.vmax) * p.inv_du - 0.5;
}

// ------------------------------------------------------- reconstruction

// One workgroup of 256 threads per 4^4-site block, one thread per site.
// M_DENSITY: the block's 16 velocity sites per (x, y) column are summed (w
// outer, u inner) into part[velocity block][y][x]; M_F: f; M_ASSIGN: ids.
//
// Bound by FP64 vector instructions.  A block's list holds 69 to 81 elements
// of which a site needs one; sorting the list per sub-block, culling, reading
// records as scalar operands and the 15-value interpolation took a wavefront
// from 8500 vector instructions to 2200 and a launch at 64^4 (mixed,
// stride 4) from 5650 to 1720 us; at 16^4, where every element used to be
// scanned, from 156 to 31 us.  Six wavefronts per SIMD (80 VGPRs, the spills
// outside the candidate loop) against the 4 the compiler takes by itself and
// 7 or 8: 1720, 2100, 1820 and 1920 us.
template <typename FT, int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k4_recon(
    KP p, const double *__restrict__ rec, const int *__restrict__ cnt,
    const int *__restrict__ lst, const int *__restrict__ flags,
    const FT *__restrict__ F, double *__restrict__ part, FT *__restrict__ fout,
    int *__restrict__ aout) {
  extern __shared__ char lds[];  // QUERY_SLOT_BYTES per list slot
  __shared__ double sf[256];
  const int t = threadIdx.x;
  int g[4], bb[4], loc;
  double P[4];
  long long list;
  const bool live = block_site(p, blockIdx.x, t, g, P, bb, loc, list);
  const int n = cnt[list];
  const bool scan_all = (n > p.cap) || (flags[0] & FL_WIDE);
  double dq[4];
  const int best = query4<false>(p, rec, lst + list * p.cap, n, scan_all, live,
                                 bb, P, dq, lds);
  const size_t site =
      (((size_t)g[3] * p.nv + g[2]) * p.ns + g[1]) * p.ns + g[0];
  FT fv = (FT)0;
  if (MODE != M_ASSIGN && live && best >= 0) {
    int k[4];
    lat_index(p, best, k);
    double Q[4], s[4];
    for (int a = 0; a < 4; ++a) Q[a] = lat_q(p, a, k[a]) + dq[a];
    index_pos(p, Q, s);
    fv = int15<FT>(p, F, s);
  }
  if (MODE == M_F && live) fout[site] = fv;
  if (MODE == M_ASSIGN && live) aout[site] = best;
  if (MODE == M_DENSITY) {
    sf[loc] = (double)fv;  // 0 off the grid
    __syncthreads();
    const int i = blk_first(p, 0, bb[0]) + (t & 3);
    const int j = blk_first(p, 1, bb[1]) + ((t >> 2) & 3);
    if (t < 16 && i >= 0 && i < p.ns && j >= 0 && j < p.ns) {
      double s = 0.0;
      for (int l = 0; l < 4; ++l)
        for (int k = 0; k < 4; ++k) s += sf[l * 64 + k * 16 + t];
      const long long vb = (long long)bb[3] * p.nb[2] + bb[2];
      part[(size_t)vb * p.ns * p.ns + (size_t)j * p.ns + i] = s;
    }
  }
}

// Resampling value of every site (section 2.3.2 axis by axis): nearest
// element, beta-restricted lattice neighbours (no offsets in more than one
// axis when an axis needs three; x, y wrap with a one-period shift), W(2d)
// blend of their Q, tensor spline of F_ini at Q_r; u, w edge rows zero.
// Writes into out (F_ini when resampling).
//
// Bound by the per-lane gathers: the neighbours' records (480 bytes a slot)
// and the spline's 256 coefficients.  The four columns of a row as one load
// and wraps without remainders: 9.30 -> 7.40 ms per launch at 64^4 (mixed,
// 10 steps), 362 -> 343 us at 32^2 x 24^2 (FP64).  Three wavefronts per SIMD
// (at most 168 VGPRs): with four (128) the double form spills 100 registers
// (374 us) and the float form is 1 % slower.
//
// The slot offsets and the lattice wrap are selects, not branches that store
// into small arrays: the branch form, once the register budget made the
// compiler keep the offsets as one 4-lane vector, was miscompiled (the
// control-flow structurizer rebuilt that vector's phi with an undefined
// incoming value on the path q > 7 of the third axis, so slot 8 re-used slot
// 7's offsets, the diagonal (0, 0, +1, +1) with zero weight, and the +1
// neighbour along the fourth axis dropped out of the blend).
template <typename FT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k4_remap(
    KP p, const double *__restrict__ rec, const int *__restrict__ cnt,
    const int *__restrict__ lst, const int *__restrict__ flags,
    const FT *__restrict__ C, FT *__restrict__ out) {
  extern __shared__ char lds[];  // QUERY_SLOT_BYTES per list slot
  int g[4], bb[4], loc;
  double P[4];
  long long list;
  const bool live = block_site(p, blockIdx.x, threadIdx.x, g, P, bb, loc, list);
  const int n = cnt[list];
  const bool scan_all = (n > p.cap) || (flags[0] & FL_WIDE);
  double dq[4];
  const int best = query4<true>(p, rec, lst + list * p.cap, n, scan_all, live,
                                bb, P, dq, lds);
  if (!live) return;
  const size_t site =
      (((size_t)g[3] * p.nv + g[2]) * p.ns + g[1]) * p.ns + g[0];
  const bool edge = g[2] == 0 || g[2] == p.nv - 1 || g[3] == 0 || g[3] == p.nv - 1;
  if (edge || best < 0) {
    out[site] = (FT)0;
    return;
  }
  int k0[4], lo[4], hi[4];
  bool three = false;
  lat_index(p, best, k0);
  for (int a = 0; a < 4; ++a) {
    const double z = dq[a] * p.rD[a];
    lo[a] = (z < p.beta) ? -1 : 0;
    hi[a] = (z < -p.beta) ? 0 : 1;
    three = three || (hi[a] - lo[a] == 2);
  }
  // The beta-set in the order of the nested loops over the offsets (axis 3
  // slowest, axis 0 fastest), one slot per trip so that a wavefront runs at
  // most 16 neighbour maps whatever its lanes' sets: without a three-valued
  // axis the 16 corners d_a = lo_a + bit a of q; with one, the 9 slots
  // -1 on axes 3, 2, 1, 0, the centre, +1 on axes 0, 1, 2, 3, those outside
  // [lo, hi] skipped.
  double sw = 0.0, sq[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int q = 0; q < 16; ++q) {
    int d[4];
    bool use = !three || q == 4;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      if (!three) {
        d[a] = lo[a] + ((q >> a) & 1);
      } else if (q == 3 - a) {
        d[a] = -1;
        use = lo[a] == -1;
      } else if (q == 5 + a) {
        d[a] = 1;
        use = hi[a] == 1;
      } else {
        d[a] = 0;
      }
    }
    int kk[4];
    double shift[2];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int k = k0[a] + d[a];
      if (a < 2) {  // x, y wrap with a one-period shift
        shift[a] = k < 0 ? -p.L : (k >= p.ms ? p.L : 0.0);
        kk[a] = k < 0 ? k + p.ms : (k >= p.ms ? k - p.ms : k);
      } else {      // u, w: no neighbour beyond the lattice
        use = use && k >= 0 && k < p.mv;
        kk[a] = k;
      }
    }
    if (!use) continue;
    const int m = ((kk[3] * p.mv + kk[2]) * p.ms + kk[1]) * p.ms + kk[0];
    double ex[4];
    map4(p, rec + (size_t)m * RS, P, ex);
    const double wgt = Wk(2.0 * sqrt(dist2(p, ex)));
    sw += wgt;
    for (int a = 0; a < 4; ++a) {
      const double Qa = (lat_q(p, a, kk[a]) + (a < 2 ? shift[a] : 0.0)) + ex[a];
      sq[a] = fma(wgt, Qa, sq[a]);
    }
  }
  double Q[4], s[4];
  for (int a = 0; a < 4; ++a)
    Q[a] = (sw > 0.0) ? sq[a] / sw : lat_q(p, a, k0[a]) + dq[a];
  index_pos(p, Q, s);
  out[site] = spline4<FT>(p, C, s);
}

// ------------------------------------------------------------- the field

// The discrete Fourier solution of Poisson's equation on the periodic square
// in three launches of one workgroup per row or column, each holding what its
// transforms read in LDS (the sums in index order; tw = cos, sin of 2 pi m /
// ns, the index p i mod ns formed by steps of p).  As six launches of one
// thread per output, the transforms reading global memory with a 64-bit
// remainder per term and k4_rho walking its 289 partials on 16 workgroups,
// the field took 164 us per step at 64^2 (rho 79, x 13, y 26, inverse 26 +
// 14, differences 5); as three, 32 us (16 + 8 + 8).  Bound by launches and the serial sums.
constexpr int FT_WG = 256;

// cos, sin of 2 pi m / n into LDS.
__device__ __forceinline__ void load_tw(const double *__restrict__ tw, int n,
                                        double *cs) {
  for (int i = threadIdx.x; i < 2 * n; i += FT_WG) cs[i] = tw[i];
}

// Row j = blockIdx.x: rho(i, j) = du dw sum over velocity blocks (in order)
// of the partials (part != null, rho written) or rho as given, then R1[j][p]
// = sum_i rho[j][i] e^{-2 pi i p i / ns}.  The partials are requested 32
// ahead of their additions.
__global__ __launch_bounds__(FT_WG) void k4_rho_dft_x(
    KP p, const double *__restrict__ part, double *__restrict__ rho,
    const double *__restrict__ tw, double *__restrict__ re,
    double *__restrict__ im) {
  extern __shared__ double ft[];  // 3 ns doubles
  const int n = p.ns, j = blockIdx.x;
  double *row = ft, *cs = ft + n, *sn = cs + n;
  load_tw(tw, n, cs);
  const size_t n2 = (size_t)n * n;
  for (int i = threadIdx.x; i < n; i += FT_WG) {
    const size_t q = (size_t)j * n + i;
    if (part) {
      const int nvb = p.nb[2] * p.nb[3];
      double s = 0.0;
      for (int v0 = 0; v0 < nvb; v0 += 32) {
        double x[32];
#pragma unroll
        for (int u = 0; u < 32; ++u)
          x[u] = v0 + u < nvb ? part[(size_t)(v0 + u) * n2 + q] : 0.0;
#pragma unroll
        for (int u = 0; u < 32; ++u)
          if (v0 + u < nvb) s += x[u];
      }
      row[i] = (p.du * p.du) * s;
      rho[q] = row[i];
    } else {
      row[i] = rho[q];
    }
  }
  __syncthreads();
  for (int pf = threadIdx.x; pf < n; pf += FT_WG) {
    double sr = 0.0, si = 0.0;
    int m = 0;
    for (int i = 0; i < n; ++i) {
      const double v = row[i];
      sr = fma(v, cs[m], sr);
      si = fma(-v, sn[m], si);
      m += pf;
      m -= m >= n ? n : 0;
    }
    re[(size_t)j * n + pf] = sr;
    im[(size_t)j * n + pf] = si;
  }
}

// Spectra of a_x and a_y from rho^ = (sr, si) at wave numbers (pf, qy): phi^ =
// -2 G rho^ / |k|^2, a^ = -i k phi^ (k = 0 and the Nyquist derivative zero).
__device__ __forceinline__ void force_spectrum(const KP &p, int pf, int qy,
                                               double sr, double si,
                                               double r[2], double i[2]) {
  const int n = p.ns;
  const double twopi = 6.283185307179586476925286766559;
  const int half = (n % 2 == 0) ? n / 2 - 1 : n / 2;
  const int pp = (pf <= half) ? pf : pf - n, qq = (qy <= half) ? qy : qy - n;
  const double kx = twopi * (double)pp / p.L, ky = twopi * (double)qq / p.L;
  const double k2 = kx * kx + ky * ky;
  const double gk = (-2.0 * p.G) / k2;
  const double pr = gk * sr, pi = gk * si;
#pragma unroll
  for (int comp = 0; comp < 2; ++comp) {
    double kd = comp == 0 ? kx : ky;
    if ((comp == 0 ? pf : qy) * 2 == n) kd = 0.0;
    const bool mean = pf == 0 && qy == 0;
    r[comp] = mean ? 0.0 : kd * pi;
    i[comp] = mean ? 0.0 : -(kd * pr);
  }
}

// Fields of component c at site q = (i, j) of n2: 0 and 1 = a_x and a_y, 2-5 =
// d a_x/dx, d a_x/dy, d a_y/dx, d a_y/dy, 6-8 = a_x,xx a_x,xy a_x,yy, 9-11 the
// same of a_y, by centred differences of the rows j - 1, j and j + 1.
__device__ __forceinline__ void force_fields(const KP &p, int c, int i,
                                             size_t q, size_t n2,
                                             const double *lo,
                                             const double *mid,
                                             const double *hi,
                                             double *__restrict__ fld) {
  const int ip = i + 1 < p.ns ? i + 1 : 0, im = i > 0 ? i - 1 : p.ns - 1;
  const double dx = p.dx;
  fld[c * n2 + q] = mid[i];
  fld[(2 + 2 * c) * n2 + q] = (mid[ip] - mid[im]) / (2.0 * dx);
  fld[(3 + 2 * c) * n2 + q] = (hi[i] - lo[i]) / (2.0 * dx);
  fld[(6 + 3 * c) * n2 + q] = ((mid[ip] + mid[im]) - 2.0 * mid[i]) / (dx * dx);
  fld[(7 + 3 * c) * n2 + q] =
      (((hi[ip] - lo[ip]) - hi[im]) + lo[im]) / (4.0 * (dx * dx));
  fld[(8 + 3 * c) * n2 + q] = ((hi[i] + lo[i]) - 2.0 * mid[i]) / (dx * dx);
}

// Column pf = blockIdx.x: R2[q][pf] = sum_j R1[j][pf] e^{-2 pi i q j / ns};
// the spectra of a_x and a_y, phi^ = -2 G rho^ / |k|^2, a^ = -i k phi^ (k = 0
// and the Nyquist derivative zero); back along y, T[c][j][pf] = sum_q
// a^[c][q][pf] e^{+2 pi i q j / ns}.  tr/ti hold [2][ns^2].
__global__ __launch_bounds__(FT_WG) void k4_spectrum_y(
    KP p, const double *__restrict__ re, const double *__restrict__ im,
    const double *__restrict__ tw, double *__restrict__ tr,
    double *__restrict__ ti) {
  extern __shared__ double ft[];  // 8 ns doubles
  const int n = p.ns, pf = blockIdx.x;
  double *cs = ft, *sn = cs + n, *rr = sn + n, *ri = rr + n, *ar = ri + n,
         *ai = ar + 2 * n;
  load_tw(tw, n, cs);
  for (int j = threadIdx.x; j < n; j += FT_WG) {
    rr[j] = re[(size_t)j * n + pf];
    ri[j] = im[(size_t)j * n + pf];
  }
  __syncthreads();
  for (int qy = threadIdx.x; qy < n; qy += FT_WG) {
    double sr = 0.0, si = 0.0;
    int m = 0;
    for (int j = 0; j < n; ++j) {
      const double a = rr[j], b = ri[j];
      sr = fma(a, cs[m], fma(b, sn[m], sr));
      si = fma(b, cs[m], fma(-a, sn[m], si));
      m += qy;
      m -= m >= n ? n : 0;
    }
    double r[2], i[2];
    force_spectrum(p, pf, qy, sr, si, r, i);
#pragma unroll
    for (int comp = 0; comp < 2; ++comp) {
      ar[comp * n + qy] = r[comp];
      ai[comp * n + qy] = i[comp];
    }
  }
  __syncthreads();
  const size_t n2 = (size_t)n * n;
  for (int o = threadIdx.x; o < 2 * n; o += FT_WG) {
    const int comp = o / n, j = o - comp * n;
    double sr = 0.0, si = 0.0;
    int m = 0;
    for (int qy = 0; qy < n; ++qy) {
      const double a = ar[comp * n + qy], b = ai[comp * n + qy];
      sr = fma(a, cs[m], fma(-b, sn[m], sr));
      si = fma(b, cs[m], fma(a, sn[m], si));
      m += j;
      m -= m >= n ? n : 0;
    }
    tr[comp * n2 + (size_t)j * n + pf] = sr;
    ti[comp * n2 + (size_t)j * n + pf] = si;
  }
}

// Row j = blockIdx.x: the inverse along x, real part / ns^2, of rows j - 1, j
// and j + 1, then the fields of row j.
__global__ __launch_bounds__(FT_WG) void k4_force_x(KP p,
                                                    const double *__restrict__ tr,
                                                    const double *__restrict__ ti,
                                                    const double *__restrict__ tw,
                                                    double *__restrict__ fld) {
  extern __shared__ double ft[];  // 8 ns doubles
  const int n = p.ns, j = blockIdx.x;
  const size_t n2 = (size_t)n * n;
  double *cs = ft, *sn = cs + n, *a6 = sn + n;  // a6[comp][row j-1, j, j+1][i]
  load_tw(tw, n, cs);
  __syncthreads();
  for (int o = threadIdx.x; o < 6 * n; o += FT_WG) {
    const int g = o / n, i = o - g * n, comp = g / 3;
    const int jj = j + g % 3 - 1, jr = jj < 0 ? n - 1 : (jj >= n ? 0 : jj);
    const double *re = tr + comp * n2 + (size_t)jr * n;
    const double *im = ti + comp * n2 + (size_t)jr * n;
    double sr = 0.0;
    int m = 0;
#pragma unroll 8
    for (int pf = 0; pf < n; ++pf) {
      sr = fma(re[pf], cs[m], fma(-im[pf], sn[m], sr));
      m += i;
      m -= m >= n ? n : 0;
    }
    a6[o] = sr * (1.0 / ((double)n * (double)n));
  }
  __syncthreads();
  for (int o = threadIdx.x; o < 2 * n; o += FT_WG) {
    const int c = o / n, i = o - c * n;
    const double *A = a6 + c * 3 * n;  // row r of the three at A + r n
    force_fields(p, c, i, (size_t)j * n + i, n2, A, A + n, A + 2 * n, fld);
  }
}

// The whole field in one workgroup, every transform in LDS, for grids of at
// most FS_MAX sites per axis, by the operations of the three launches in their
// order.  Bound by the round trip of the partials and the chains of the sums;
// the work grows as ns^3 on one compute unit while the three launches cost
// about 14 us whatever the size.  us per step, three launches / one: 8 sites
// (12 per velocity axis) 12.4 / 8.3, 12 13.8 / 10.5, 16 (16) 14.1 / 11.4, 16
// (40) 17.0 / 15.9, 20 (12) 14.8 / 16.9, 24 15.1 / 20.8.
constexpr int FS_MAX = 16;
constexpr int FS_WG = 512;

__global__ __launch_bounds__(FS_WG) void k4_field_small(
    KP p, const double *__restrict__ part, double *__restrict__ rho,
    const double *__restrict__ tw, double *__restrict__ fld) {
  extern __shared__ double ft[];  // 2 ns + 8 ns^2 doubles
  const int n = p.ns, n2 = n * n, tid = threadIdx.x;
  double *cs = ft, *sn = cs + n, *X = sn + n, *Y = X + 4 * n2;
  for (int i = tid; i < 2 * n; i += FS_WG) cs[i] = tw[i];
  for (int q = tid; q < n2; q += FS_WG) {
    if (part) {
      const int nvb = p.nb[2] * p.nb[3];
      double s = 0.0;
      for (int v0 = 0; v0 < nvb; v0 += 32) {
        double x[32];
#pragma unroll
        for (int u = 0; u < 32; ++u)
          x[u] = v0 + u < nvb ? part[(size_t)(v0 + u) * n2 + q] : 0.0;
#pragma unroll
        for (int u = 0; u < 32; ++u)
          if (v0 + u < nvb) s += x[u];
      }
      Y[q] = (p.du * p.du) * s;
      rho[q] = Y[q];
    } else {
      Y[q] = rho[q];
    }
  }
  __syncthreads();
  // along x: X = R1[j][pf], real and imaginary
  for (int o = tid; o < n2; o += FS_WG) {
    const int j = o / n, pf = o - j * n;
    double sr = 0.0, si = 0.0;
    int m = 0;
#pragma unroll 8
    for (int i = 0; i < n; ++i) {
      const double v = Y[j * n + i];
      sr = fma(v, cs[m], sr);
      si = fma(-v, sn[m], si);
      m += pf;
      m -= m >= n ? n : 0;
    }
    X[o] = sr;
    X[n2 + o] = si;
  }
  __syncthreads();
  // along y and the spectra: Y = a^[comp][real, imaginary][qy][pf]
  for (int o = tid; o < n2; o += FS_WG) {
    const int qy = o / n, pf = o - qy * n;
    double sr = 0.0, si = 0.0;
    int m = 0;
#pragma unroll 8
    for (int j = 0; j < n; ++j) {
      const double a = X[j * n + pf], b = X[n2 + j * n + pf];
      sr = fma(a, cs[m], fma(b, sn[m], sr));
      si = fma(b, cs[m], fma(-a, sn[m], si));
      m += qy;
      m -= m >= n ? n : 0;
    }
    double r[2], i[2];
    force_spectrum(p, pf, qy, sr, si, r, i);
#pragma unroll
    for (int comp = 0; comp < 2; ++comp) {
      Y[2 * comp * n2 + o] = r[comp];
      Y[(2 * comp + 1) * n2 + o] = i[comp];
    }
  }
  __syncthreads();
  // back along y: X = T[comp][real, imaginary][j][pf]
  for (int o = tid; o < 2 * n2; o += FS_WG) {
    const int comp = o / n2, g = o - comp * n2, j = g / n, pf = g - j * n;
    const double *A = Y + 2 * comp * n2 + pf;
    double sr = 0.0, si = 0.0;
    int m = 0;
#pragma unroll 8
    for (int qy = 0; qy < n; ++qy) {
      const double a = A[qy * n], b = A[n2 + qy * n];
      sr = fma(a, cs[m], fma(-b, sn[m], sr));
      si = fma(b, cs[m], fma(a, sn[m], si));
      m += j;
      m -= m >= n ? n : 0;
    }
    X[2 * comp * n2 + g] = sr;
    X[(2 * comp + 1) * n2 + g] = si;
  }
  __syncthreads();
  // back along x: Y = a[comp][j][i]
  for (int o = tid; o < 2 * n2; o += FS_WG) {
    const int comp = o / n2, g = o - comp * n2, j = g / n, i = g - j * n;
    const double *T = X + 2 * comp * n2 + j * n;
    double sr = 0.0;
    int m = 0;
#pragma unroll 8
    for (int pf = 0; pf < n; ++pf) {
      sr = fma(T[pf], cs[m], fma(-T[n2 + pf], sn[m], sr));
      m += i;
      m -= m >= n ? n : 0;
    }
    Y[o] = sr * (1.0 / ((double)n * (double)n));
  }
  __syncthreads();
  for (int o = tid; o < 2 * n2; o += FS_WG) {
    const int c = o / n2, g = o - c * n2, j = g / n, i = g - j * n;
    const double *A = Y + c * n2;
    const int jm = j > 0 ? j - 1 : n - 1, jp = j + 1 < n ? j + 1 : 0;
    force_fields(p, c, i, (size_t)g, (size_t)n2, A + jm * n, A + j * n,
                 A + jp * n, fld);
  }
}

// ------------------------------------------------------------- the spline

// The tridiagonal (1, 4, 1) solves with precomputed pivots, axis by axis (0
// x, 1 y, 2 u, 3 w): mirror end rows (4, 2) / (2, 4) on u and w, the cyclic
// system's tridiagonal part plus the Sherman-Morrison correction y - [(y_0 -
// y_{n-1}/4) / den] z on x and y.  tab: cp[n], ri[n] (and z[n], den on the
// periodic axes).  fit_line solves one line of n values, `stride` apart, of
// `in` into x (in place when equal).
template <typename FT>
__device__ __forceinline__ void fit_line(const FT *in, FT *x, int n,
                                         long long stride, bool per,
                                         const FT *__restrict__ tab) {
  const FT *cp = tab, *ri = tab + n;
  FT acc = (FT)0;
#pragma unroll 4
  for (int i = 0; i < n; ++i) {
    const FT sub = (!per && i == n - 1) ? (FT)2 : (FT)1;
    acc = ((FT)6 * in[i * stride] - sub * acc) * ri[i];
    x[i * stride] = acc;
  }
#pragma unroll 4
  for (int i = n - 2; i >= 0; --i) {
    acc = x[i * stride] - cp[i] * acc;
    x[i * stride] = acc;
  }
  if (per) {
    const FT *z = tab + 2 * n, den = tab[3 * n];
    const FT fact = (x[0] - (FT)0.25 * x[(long long)(n - 1) * stride]) / den;
    for (int i = 0; i < n; ++i) x[i * stride] = x[i * stride] - fact * z[i];
  }
}

// Axis 0, F -> C: a workgroup brings its lines (contiguous in memory) into
// LDS with coalesced accesses, a thread solves each there.  With a thread
// per line on global memory every access touched its own cache line: 1017 us
// at 64^4 (mixed) after a copy of F; 37 us this way.
constexpr int FITX_BYTES = 49152;
template <typename FT>
__host__ __device__ __forceinline__ int fitx_lines(int n) {
  const int l = FITX_BYTES / ((n + 1) * (int)sizeof(FT));
  return l < 64 ? l : 64;
}
template <typename FT>
__global__ __launch_bounds__(256) void k4_fit_x(KP p, const FT *__restrict__ F,
                                                FT *__restrict__ C,
                                                const FT *__restrict__ tab) {
  extern __shared__ char fitx[];  // fitx_lines rows of n + 1 values
  FT *buf = reinterpret_cast<FT *>(fitx);
  const int n = p.ns, nl = fitx_lines<FT>(n);
  const long long lines = (long long)p.ns * p.nv * p.nv;
  const long long l0 = (long long)blockIdx.x * nl;
  const int m = (int)min((long long)nl, lines - l0);
  for (int q = threadIdx.x; q < m * n; q += 256) {
    const int l = q / n;
    buf[q + l] = F[l0 * n + q];
  }
  __syncthreads();
  if ((int)threadIdx.x < m) {
    FT *x = buf + threadIdx.x * (n + 1);
    fit_line<FT>(x, x, n, 1, true, tab);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < m * n; q += 256) {
    const int l = q / n;
    C[l0 * n + q] = buf[q + l];
  }
}

// Axes 1 to 3, in place: one thread per line, neighbouring threads on
// neighbouring x.
template <typename FT>
__global__ __launch_bounds__(256) void k4_fit(KP p, FT *__restrict__ C, int ax,
                                              const FT *__restrict__ tab) {
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long ns = p.ns, nv = p.nv;
  const long long N4 = ns * ns * nv * nv;
  const int n = ax < 2 ? p.ns : p.nv;
  const long long stride = ax == 1 ? ns : ax == 2 ? ns * ns : ns * ns * nv;
  if (q >= N4 / n) return;
  const long long low = q % stride, high = q / stride;
  FT *x = C + high * stride * n + low;
  fit_line<FT>(x, x, n, stride, ax < 2, tab);
}

// f0 (device doubles) -> F, u and w edge rows zero.
template <typename FT>
__global__ __launch_bounds__(256) void k4_load(KP p, const double *__restrict__ src,
                                               FT *__restrict__ F) {
  const long long N4 = (long long)p.ns * p.ns * p.nv * p.nv;
  const long long gsz = (long long)gridDim.x * blockDim.x;
  for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < N4;
       q += gsz) {
    const long long r = q / ((long long)p.ns * p.ns);
    const int k = (int)(r % p.nv), l = (int)(r / p.nv);
    const bool edge = k == 0 || k == p.nv - 1 || l == 0 || l == p.nv - 1;
    F[q] = edge ? (FT)0 : (FT)src[q];
  }
}

// ------------------------------------------------------------ diagnostics

// Per-workgroup partial sums of f, (u^2 + w^2) f and f ln|f| over a range
// of sites (tree order within the workgroup).
template <typename FT>
__global__ __launch_bounds__(256) void k4_diag_part(KP p, const FT *__restrict__ f,
                                                    double *__restrict__ part) {
  __shared__ double s0[256], s1[256], s2[256];
  const long long N4 = (long long)p.ns * p.ns * p.nv * p.nv;
  const long long gsz = (long long)gridDim.x * blockDim.x;
  double m = 0.0, k = 0.0, en = 0.0;
  for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < N4;
       q += gsz) {
    const long long r = q / ((long long)p.ns * p.ns);
    const double u = coord(p, 2, (int)(r % p.nv)), w = coord(p, 3, (int)(r / p.nv));
    const double v = (double)f[q];
    m += v;
    k += (u * u + w * w) * v;
    if (v != 0.0) en += v * log(fabs(v));
  }
  const int t = threadIdx.x;
  s0[t] = m;
  s1[t] = k;
  s2[t] = en;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s) {
      s0[t] += s0[t + s];
      s1[t] += s1[t + s];
      s2[t] += s2[t + s];
    }
    __syncthreads();
  }
  if (t == 0) {
    part[3 * blockIdx.x] = s0[0];
    part[3 * blockIdx.x + 1] = s1[0];
    part[3 * blockIdx.x + 2] = s2[0];
  }
}

__global__ __launch_bounds__(256) void k4_diag_final(KP p,
                                                     const double *__restrict__ part,
                                                     int nparts,
                                                     const double *__restrict__ fld,
                                                     double *__restrict__ out) {
  __shared__ double s3[256];
  const int t = threadIdx.x;
  const int n2 = p.ns * p.ns;
  double pot = 0.0;
  for (int q = t; q < n2; q += 256) pot += fld[q] * fld[q] + fld[n2 + q] * fld[n2 + q];
  s3[t] = pot;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s) s3[t] += s3[t + s];
    __syncthreads();
  }
  if (t == 0) {
    double m = 0.0, k = 0.0, en = 0.0;
    for (int q = 0; q < nparts; ++q) {
      m += part[3 * q];
      k += part[3 * q + 1];
      en += part[3 * q + 2];
    }
    const double dV = (p.dx * p.dx) * (p.du * p.du);
    out[0] = m * dV;
    out[1] = 0.5 * k * dV;
    out[2] = (p.G != 0.0) ? -s3[0] * (p.dx * p.dx) / (4.0 * p.G) : 0.0;
    out[3] = out[1] + out[2];
    out[4] = -en * dV;
  }
}

}  // namespace vp4k
