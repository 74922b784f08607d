// particles.hip -- per-macroparticle kernels of the cylindrical envelope PIC
// step (arXiv:1912.04674): the momentum pass (gather of E, Bbar, Phi and
// grad Phi, ponderomotive Boris push, chi deposit, scatter into the tile
// order of the next pass), the position pass (gather of Phi^{n+1/2}, push,
// current deposit, tile histogram), loading and injection.
//
// Work decomposition: particles are counting-sorted by 16 x 16-cell tiles
// every SORT_EVERY steps (SORT_EVERY - 1 for quadratic shapes); a work item
// is (tile, contiguous range of at most g.chunk particles).  A work group
// stages the fields of its tile plus a
// HALO-cell margin in LDS, accumulates the deposits of its particles in LDS
// and flushes them to HBM once (atomic adds, since halos overlap).
// Particles drift at most one cell per step (dt < dx, dt < dr), so between
// two sorts they stay inside the margin.
//
// Positions: lab cell (column, row) in one word plus offsets in the cell
// along x and r and the azimuth; the push is Cartesian (Sec. 3), and the
// new radius is obtained from the radial and azimuthal components of the
// displacement without cancellation, so the offsets keep their resolution at
// any radius.
#include <algorithm>
#include <limits>

#include "common.hpp"
#include "cplx.hpp"
#include "elem.hpp"
#include "launch.hpp"
#include "scan.hpp"

namespace envpic {

// ------------------------------------------------------------ shapes --
template <class R> struct Lin {
  int i;   // first node (local LDS index)
  R a, b;  // weights of nodes i and i+1
};

template <class R> __device__ inline Lin<R> primal_w(int c, R f) { return Lin<R>{c, (R)1 - f, f}; }
// floor as an integer and fractional part (in [0, 1): the hardware's result
// for a tiny negative number is the largest value below 1)
__device__ inline int floor_int(float x) {
  int i;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(x));
  return i;
}
__device__ inline int floor_int(double x) { return (int)floor(x); }
__device__ inline float fract_r(float x) { return __builtin_amdgcn_fractf(x); }
__device__ inline double fract_r(double x) { return __builtin_amdgcn_fract(x); }
// a constant in the type of the path (the FP32 copy comes in as a kernel
// argument, which stays in a scalar register; one converted on the device
// would take a vector register)
template <class R> __device__ inline R pick(double x, float xf) {
  if constexpr (sizeof(R) == 4) return xf;
  else return x;
}
// x clamped to [lo, hi]; a NaN gives lo
__device__ inline float clamp_r(float x, float lo, float hi) { return __builtin_amdgcn_fmed3f(x, lo, hi); }
__device__ inline double clamp_r(double x, double lo, double hi) { return fmin(fmax(x, lo), hi); }
template <class R> __device__ inline Lin<R> dual_w(int c, R f) {
  const R v = f - (R)0.5, w = fract_r(v);
  return Lin<R>{v < (R)0 ? c - 1 : c, (R)1 - w, w};
}

// (RL: the row length of the LDS region the values are staged in)
template <class R, int RL = LR> __device__ inline R interp2(const R* a, Lin<R> sx, Lin<R> sr) {
  return sx.a * (sr.a * a[sx.i * RL + sr.i] + sr.b * a[sx.i * RL + sr.i + 1]) +
         sx.b * (sr.a * a[(sx.i + 1) * RL + sr.i] + sr.b * a[(sx.i + 1) * RL + sr.i + 1]);
}
// the same from the four weight products
template <class R, int RL = LR> __device__ inline R interp2w(const R* a, Lin<R> sx, Lin<R> sr) {
  const R* n = &a[sx.i * RL + sr.i];
  return sx.a * sr.a * n[0] + sx.a * sr.b * n[1] + sx.b * sr.a * n[RL] + sx.b * sr.b * n[RL + 1];
}
template <class C, class R, int RL = LR> __device__ inline C interp2c(const C* a, Lin<R> sx, Lin<R> sr) {
  C v00 = a[sx.i * RL + sr.i], v01 = a[sx.i * RL + sr.i + 1];
  C v10 = a[(sx.i + 1) * RL + sr.i], v11 = a[(sx.i + 1) * RL + sr.i + 1];
  R w00 = sx.a * sr.a, w01 = sx.a * sr.b, w10 = sx.b * sr.a, w11 = sx.b * sr.b;
  return mk<C>(w00 * v00.x + w01 * v01.x + w10 * v10.x + w11 * v11.x,
               w00 * v00.y + w01 * v01.y + w10 * v10.y + w11 * v11.y);
}

// Quadratic B-spline (order 2) on three nodes i, i+1, i+2 around the nearest
// node m = i + 1, d = u - m in [-1/2, 1/2): (1/2 - d)^2/2, 3/4 - d^2,
// (1/2 + d)^2/2.  Primal nodes sit at the cell corners (nearest node a or
// a + 1), dual nodes at the cell centres (nearest node always a).
// The outer weights differ by d, so the last is formed as the first plus d
// (four operations per stencil instead of seven; the absolute error stays
// within an ulp of 1/2).
template <class R> struct Quad {
  int i;
  R w[3];
};
template <class R> __device__ inline Quad<R> quad_of(int i, R d) {
  const R w0 = fma(d, fma(d, (R)0.5, (R)-0.5), (R)0.125);  // (1/2 - d)^2 / 2
  return Quad<R>{i, {w0, fma(-d, d, (R)0.75), w0 + d}};
}
template <class R> __device__ inline Quad<R> quad_primal(int c, R f) {
  return f < (R)0.5 ? quad_of<R>(c - 1, f) : quad_of<R>(c, f - (R)1);
}
template <class R> __device__ inline Quad<R> quad_dual(int c, R f) { return quad_of<R>(c - 1, f - (R)0.5); }

template <class R, int RL = LR> __device__ inline R interp3(const R* a, const Quad<R>& sx, const Quad<R>& sr) {
  R acc = 0;
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const R* col = a + (sx.i + u) * RL + sr.i;
    acc += sx.w[u] * (sr.w[0] * col[0] + sr.w[1] * col[1] + sr.w[2] * col[2]);
  }
  return acc;
}
template <class C, class R, int RL = LR>
__device__ inline C interp3c(const C* a, const Quad<R>& sx, const Quad<R>& sr) {
  R re = 0, im = 0;
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const C* col = a + (sx.i + u) * RL + sr.i;
    re += sx.w[u] * (sr.w[0] * col[0].x + sr.w[1] * col[1].x + sr.w[2] * col[2].x);
    im += sx.w[u] * (sr.w[0] * col[0].y + sr.w[1] * col[1].y + sr.w[2] * col[2].y);
  }
  return mk<C>(re, im);
}

// Phi and its centred differences (times 1/(2 dx), 1/(2 dr)) interpolated
// with one quadratic stencil, from Phi on the 5 x 5 nodes around the 3 x 3 of
// the stencil (corners unused).  j0 is the grid row of the stencil's first
// node (at least -1): the radial difference is zero on the axis row and, on
// the ghost row below it, minus its value on row 1.
template <class R, int RL>
__device__ inline void phi_grad3(const R* phi, const Quad<R>& sx, const Quad<R>& sr, int j0, R i2dx, R i2dr,
                                 R& ph, R& gx, R& gr) {
  // the differences taken through the weights: a node's Phi enters the x
  // difference with the weight of the node behind it minus that of the node
  // ahead; the radial weights of the axis row and the ghost row are moved
  // (zero on the axis, the ghost row folded onto row 1 with a sign)
  const R k0 = j0 >= 1 ? sr.w[0] : (R)0, k1 = j0 >= 0 ? sr.w[1] : (R)0;
  const R k2 = j0 == -1 ? sr.w[2] - sr.w[0] : sr.w[2];
  const R dx[5] = {-sx.w[0], -sx.w[1], sx.w[0] - sx.w[2], sx.w[1], sx.w[2]};
  const R dr[5] = {-k0, -k1, k0 - k2, k1, k2};
  const R* p = phi + sx.i * RL + sr.i;
  R a = 0, b = 0, d = 0;
#pragma unroll
  for (int u = -1; u < 4; ++u) {
    const R* c = p + u * RL;
    if (u >= 0 && u <= 2) {
      const R c0 = c[0], c1 = c[1], c2 = c[2];
      a += sx.w[u] * (sr.w[0] * c0 + sr.w[1] * c1 + sr.w[2] * c2);
      d += sx.w[u] * (dr[0] * c[-1] + dr[1] * c0 + dr[2] * c1 + dr[3] * c2 + dr[4] * c[3]);
      b += dx[u + 1] * (sr.w[0] * c0 + sr.w[1] * c1 + sr.w[2] * c2);
    } else {
      b += dx[u + 1] * (sr.w[0] * c[0] + sr.w[1] * c[1] + sr.w[2] * c[2]);
    }
  }
  ph = a;
  gx = b * i2dx;
  gr = d * i2dr;
}

// v clamped to [lo, hi]; bad is set when it was outside (one min/max and one
// compare)
__device__ inline int clampi(int v, int lo, int hi, bool& bad) {
  const int c = min(max(v, lo), hi);
  bad |= c != v;
  return c;
}

__device__ inline void lds_add(float* a, float v) { atomicAdd(a, v); }
__device__ inline void lds_add(double* a, double v) { atomicAdd(a, v); }

// Mode-1 current accumulators.  The FP64 path sums in FP64 LDS words.  The
// FP32 path sums fixed-point integers in 64-bit LDS words: on gfx950 integer
// LDS atomics issue faster than FP64 ones (and FP32 LDS atomics are far
// slower than either, measured), and an integer sum is exact and independent
// of the order in which the lanes land.  Each contribution is scaled by
// g.fix = 2^32 / (2 w_max / V_0), the bound of any |2 q w v S / V| (|v| < 1,
// S <= 1, V_0 the smallest node volume), so one contribution is at most 2^32
// in magnitude.  The particles of a work item and its riders add at most two
// each to one node, below 2^45.4, and a fold of two such nodes stays below
// 2^46.4.
//
// The float -> fixed conversion is one FP64 FMA: u x + 1.5 2^52 rounds u x
// to the nearest integer v and its bit pattern is 0x4338 2^48 + v (exact for
// |v| < 2^51).  The words add those patterns as they are; the constant parts
// only reach bits 48..63, so the low 48 bits of a word hold the sum of the v
// modulo 2^48, which is the sum itself, as |sum| < 2^47 (fixed_sum reads it).
// On the hot path this saves the subtraction of the constant per atomic.
// add_prod(a, u, x, y) adds u x and u y, formed in FP64.
template <class R> struct Acc1;
template <> struct Acc1<double> {
  using T = double2;
  using S = double;  // one word (real or imaginary part)
  __device__ static T zero() { return make_double2(0.0, 0.0); }
  __device__ static double scale(const Geo&) { return 1.0; }
  template <class A> __device__ static void add_prod(A& a, int k, double u, double x, double y) {
    atomicAdd(&a.re[k], u * x);
    atomicAdd(&a.im[k], u * y);
  }
  __device__ static bool nonzero(const T& v) { return v.x != 0.0 || v.y != 0.0; }
  __device__ static double re(const T& v, const Geo&) { return v.x; }
  __device__ static double im(const T& v, const Geo&) { return v.y; }
};
// bit pattern of u x + 1.5 2^52: 0x4338 2^48 + the nearest integer to u x
// (|u x| < 2^51)
__device__ inline unsigned long long fixed_bits(double u, double x) {
  return (unsigned long long)__double_as_longlong(fma(u, x, 6755399441055744.0));  // 1.5 * 2^52
}
// The sum held by a word of fixed_bits patterns: its low 48 bits, signed.
// Offset by 2^47 they become the low mantissa bits of a double in
// [2^52, 2^53), from which the offset is subtracted (exact: two integer
// operations on the high word and one FP64 addition).
__device__ inline double fixed_sum(long long w) {
  const int hi = (int)((((unsigned long long)w >> 32) & 0xFFFFu) ^ 0x8000u) | 0x43300000;
  return __hiloint2double(hi, (int)w) - 4644337115725824.0;  // 2^52 + 2^47
}
static_assert(4LL * (CHUNK + MAX_RIDERS) << 32 < 1LL << 47 && TR * 256 <= CHUNK + MAX_RIDERS,
              "two contributions of 2^32 a particle, two nodes folded (an injected item: TR cells of at most 256)");
__device__ inline bool fixed_nonzero(long long w) { return ((unsigned long long)w << 16) != 0; }
template <> struct Acc1<float> {
  using T = longlong2;
  using S = long long;  // one word (real or imaginary part)
  __device__ static T zero() { return make_longlong2(0, 0); }
  __device__ static float scale(const Geo& g) { return g.fix; }
  template <class A> __device__ static void add_prod(A& a, int k, double u, double x, double y) {  // already scaled
    atomicAdd((unsigned long long*)&a.re[k], fixed_bits(u, x));
    atomicAdd((unsigned long long*)&a.im[k], fixed_bits(u, y));
  }
  __device__ static bool nonzero(const T& v) { return fixed_nonzero(v.x | v.y); }
  __device__ static float re(const T& v, const Geo& g) { return (float)(fixed_sum(v.x) * g.unfix); }
  __device__ static float im(const T& v, const Geo& g) { return (float)(fixed_sum(v.y) * g.unfix); }
};

// Mode-0 deposit accumulators (chi, and J_x, J_r of the Esirkepov scheme).
// A contribution is w S: the weight times shape factors (or, for the
// currents, a partial sum of shape differences in [-1, 1]) without the
// inverse node volume or face area, which depend on the row only and are
// applied once per node at the flush.  The FP64 path sums FP64 words; the
// FP32 path sums fixed point as the mode-1 accumulators do, scaled by g.fix0
// = 2^32 / w_max, so a contribution is at most 2^32 and the sums have the same
// bound (exact, order-independent).
template <class R> struct Acc0;
template <> struct Acc0<double> {
  using T = double;
  __device__ static double scale(const Geo&) { return 1.0; }
  __device__ static void add_prod(T* a, double u, double x) { atomicAdd(a, u * x); }
  __device__ static bool nonzero(T v) { return v != 0.0; }
  __device__ static double val(T v, const Geo&) { return v; }
};
template <> struct Acc0<float> {
  using T = long long;
  __device__ static double scale(const Geo& g) { return g.fix0; }
  __device__ static void add_prod(T* a, double u, double x) { atomicAdd((unsigned long long*)a, fixed_bits(u, x)); }
  __device__ static bool nonzero(T v) { return fixed_nonzero(v); }
  __device__ static double val(T v, const Geo& g) { return fixed_sum(v) * g.unfix0; }
};

// Elementary functions.  The FP32 path uses the hardware reciprocal, square
// root, reciprocal square root and sine/cosine (about 1 ulp, or ~1e-6 for
// the direction cosines of the azimuth, far inside the FP32 path's
// tolerance).  The FP64 path refines the hardware's approximations to FP64
// and sums its own series, for the ranges met here: no scaling of extreme
// arguments and no reduction of large angles, whose code took the position
// pass to 169 registers (one work group per CU): 279 us at 8.4 M particles, 167
// with these.
__device__ inline float rsqrt_r(float x) { return __builtin_amdgcn_rsqf(x); }  // x >= 1 here
__device__ inline float sqrt_r(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ inline float rcp_r(float x) { return __builtin_amdgcn_rcpf(x); }
// 1 / sqrt(x), x >= 1 and finite: with e = 1 - x y^2, y (1 - e)^(-1/2) to
// third order
__device__ inline double rsqrt_r(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}
// For the arguments that the state alone bounds (1 + p^2 + Phi, 1 + t^2): the
// same, with 0 for an infinite argument, where the refinement would make a
// NaN.  The high word of the correction (of the result) is cleared there, a
// compare and one select each: 24 steps of 8.4 M particles take 10.41 ms, 10.38
// without (10.41 against 10.36 when the whole result of every root was
// selected, 10.61 against 10.40 with a minimum that avoids the NaN, which
// spilled).
__device__ inline float rsqrt1_r(float x) { return rsqrt_r(x); }
__device__ inline float rcp1_r(float x) { return rcp_r(x); }
__device__ inline double rsqrt1_r(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double e = fma(-(x * y), y, 1.0);
  e = __hiloint2double(y == 0.0 ? 0 : __double2hiint(e), __double2loint(e));
  return fma(y * e, fma(e, 0.375, 0.5), y);
}
// Newton's steps for 1 / x (x not denormal; 0 and infinities give a NaN)
__device__ inline double rcp_r(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}
__device__ inline double rcp1_r(double x) {
  const double y = rcp_r(x);
  return __hiloint2double(x == INFINITY ? 0 : __double2hiint(y), __double2loint(y));
}
__device__ inline double sqrt_r(double x) {  // x >= 0
  const double s = x * rsqrt_r(x);
  return x > 0.0 ? fma(fma(-s, s, x), 0.5 * rcp_r(s), s) : 0.0;
}
__device__ inline void sincos_r(float t, float* s, float* c) {
  *s = __sinf(t);
  *c = __cosf(t);
}
// Series in b2 = beta^2 for |beta| < SMALL_BETA, the displacement of a step
// against its radius: (sqrt(1 + b2) - 1) / b2, 1 / sqrt(1 + b2) and
// atan(beta) / beta, to the rounding of the type (binomial and arctangent
// series; the first omitted terms are at most 1.3e-9, 4.9e-9 and 2.2e-9 of the
// sum in FP32 and 8e-18, 5.5e-17 and 1e-19 in FP64).
// They replace a square root, a reciprocal square root and two reciprocals
// per particle; only waves with a lane closer to the axis take the general
// forms.
constexpr double SMALL_BETA = 0.05;
__device__ inline float sqrt1_series(float b2) { return fmaf(b2, fmaf(b2, 0.0625f, -0.125f), 0.5f); }
__device__ inline double sqrt1_series(double b2) {
  double s = -21.0 / 1024;
  s = fma(b2, s, 7.0 / 256);
  s = fma(b2, s, -5.0 / 128);
  s = fma(b2, s, 1.0 / 16);
  s = fma(b2, s, -1.0 / 8);
  return fma(b2, s, 0.5);
}
__device__ inline float rhyp_series(float b2) { return fmaf(b2, fmaf(b2, 0.375f, -0.5f), 1.0f); }
__device__ inline double rhyp_series(double b2) {
  double s = -63.0 / 256;
  s = fma(b2, s, 35.0 / 128);
  s = fma(b2, s, -5.0 / 16);
  s = fma(b2, s, 3.0 / 8);
  s = fma(b2, s, -0.5);
  return fma(b2, s, 1.0);
}
__device__ inline float atan_series(float b2) { return fmaf(-b2, fmaf(-b2, 0.2f, 1.0f / 3.0f), 1.0f); }
__device__ inline double atan_series(double b2) {
  double s = 1.0 / 13;
  s = fma(-b2, s, 1.0 / 11);
  s = fma(-b2, s, 1.0 / 9);
  s = fma(-b2, s, 1.0 / 7);
  s = fma(-b2, s, 1.0 / 5);
  s = fma(-b2, s, 1.0 / 3);
  return fma(-b2, s, 1.0);
}
__device__ inline float dtheta(float b, float ra) { return atan2f(b, ra); }
// atan2(b, ra) by halving the angle (tan(x/2) = sin x / (1 + cos x)) four
// times, to at most pi/32, and the series
__device__ inline double dtheta(double b, double ra) {
  const double h = sqrt_r(ra * ra + b * b);
  if (!(h > 0.0)) return 0.0;
  double t = fabs(b) * rcp_r(h + fabs(ra));  // tan of half the angle to the nearer end of the axis
#pragma unroll 1
  for (int k = 0; k < 3; ++k) t *= rcp_r(1.0 + sqrt_r(fma(t, t, 1.0)));
  const double t2 = t * t;
  double s = -1.0 / 15;
  s = fma(t2, s, 1.0 / 13);
  s = fma(t2, s, -1.0 / 11);
  s = fma(t2, s, 1.0 / 9);
  s = fma(t2, s, -1.0 / 7);
  s = fma(t2, s, 1.0 / 5);
  s = fma(t2, s, -1.0 / 3);
  double x = 16.0 * fma(t2 * s, t, t);
  x = ra < 0.0 ? 3.14159265358979323846 - x : x;
  return copysign(x, b);
}

// New radius and azimuth after a Cartesian transverse displacement with
// radial component a and azimuthal component b (lengths) from radius r:
// r' = |(r + a, b)|, written r' - r = a + (r + a)(sqrt(1 + beta^2) - 1) with
// beta = b/(r + a) so that small displacements keep full relative precision.
// Returns whether |beta| < SMALL_BETA with r + a > 0: the displacement's
// mid-point has then an even smaller beta, (b/2)/(r + a/2).
template <class R> __device__ inline bool radial_step(R r, R a, R b, R& dr_out, R& dth) {
  const R ra = r + a;
  const R beta = b * rcp_r(ra);
  if (ra > (R)0 && fabs(beta) < (R)SMALL_BETA) {
    const R b2 = beta * beta;
    dr_out = fma(b * beta, sqrt1_series(b2), a);
    dth = beta * atan_series(b2);
    return true;
  }
  if (ra > (R)0) {
    const R q = sqrt_r((R)1 + beta * beta);
    dr_out = a + ra * beta * beta * rcp_r((R)1 + q);
  } else {
    dr_out = sqrt_r(ra * ra + b * b) - r;
  }
  dth = dtheta(b, ra);
  return false;
}

// t (less than a turn beyond the range) brought back into [-pi, pi]
template <class R> __device__ inline R wrap_angle(R t) {
  const R two_pi = (R)6.28318530717958647692, inv = (R)0.15915494309189533577;
  return fma(-rint(t * inv), two_pi, t);
}

// Access to the particle records.  Each pass reads and writes a record once;
// when a simulation's particle buffers are larger than the last-level cache
// (NT), the records are read and written with non-temporal hints so that
// streaming them does not evict the grids, which the tiles' regions re-read
// and the field stage reads next (measured: the field stage of the
// 2048 x 256 LWFA workload 37 -> 28 us, its step 5.6 % shorter).  Runs whose
// buffers fit in that cache keep ordinary accesses, which let the next pass
// find the records there.
template <bool NT, class T> __device__ inline T pld(const T* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, class T> __device__ inline void pst(T* p, T v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}
// Element i of a record array: for 4-byte elements the byte offset is formed
// in 32 bits (slots < 2^30), so the access takes the array's address from
// scalar registers and the 32-bit offset from a vector register, with no
// 64-bit address arithmetic per lane.
template <class T> __device__ inline T* elem(T* a, int i) {
  if constexpr (sizeof(T) == 4) return (T*)((char*)a + (unsigned)i * 4u);
  else return a + i;
}
template <class T> __device__ inline const T* elem(const T* a, int i) {
  if constexpr (sizeof(T) == 4) return (const T*)((const char*)a + (unsigned)i * 4u);
  else return a + i;
}

// Loading order inside a tile: the R particles of a tile, enumerated cell
// by cell, fill a K-column matrix row by row (K = ceil(R/64)) and are stored
// column by column.  The 64 lanes of a wavefront then hold particles K apart
// in the enumeration, i.e. from cells at least four rows apart, so their
// deposit stencils do not share LDS addresses.  The per-step scatter keeps
// the relative order of the particles it moves, so the interleaving made at
// loading persists while every pass reads and writes contiguously.
__device__ inline int transpose_rank(int r, int R) {
  const int K = (R + 63) / 64;
  const int rows = (R + K - 1) / K;
  const int L = R - (rows - 1) * K;  // columns holding `rows` entries
  const int m = r % K, q = r / K;
  return m * rows - max(0, m - L) + q;
}

// slot of the r-th particle (in cell order) of a tile of v particles: the
// tile splits into nm = ceil(v / chunk) work items of item_share particles
// (as the scan makes them), and inside an item the particles are placed as at loading.  With
// linear shapes (O = 1) an item takes a contiguous range of ranks.  With
// quadratic shapes the ranks are dealt to the items in turn (listed by
// r mod nm, then r / nm, and cut at the items' sizes), so that every item
// spans all cells of the tile and a wavefront's lanes stay four cells apart
// in cell order with the smaller items of that order (measured: the
// position pass 5 % faster on the LWFA workload; with linear shapes the
// 8192 x 768 workload, six particles per cell more than an item holds,
// became 5 % slower, so they keep contiguous ranges)
template <int O> __device__ inline int placed_rank(int r, int v, int chunk) {
  const int nm = (v + chunk - 1) / chunk;
  int t = r;
  if constexpr (O == 2) {
    if (nm == 1) return transpose_rank(r, v);
    const int a = v / nm, b = v - a * nm, m = r % nm;
    t = m * a + min(m, b) + r / nm;  // (the first b residues hold a + 1 ranks)
  }
  const int sh = item_share(v, chunk), lo = t / sh * sh, hi = min(lo + sh, v);
  return lo + transpose_rank(t - lo, hi - lo);
}

// the tile region of a work item with a margin of h cells: lab column
// X0 = T TX - h, row R0 = tcr TR - h
struct Region {
  int T, tcx, tcr;
  int X0;  // lab column (lab columns fit 20 bits)
  int relX0, R0;
};
__device__ inline Region region_of(const Geo& g, int key, int h = HALO) {
  Region q;
  q.tcx = key / g.ntr;
  q.tcr = key - q.tcx * g.ntr;
  q.T = lab_tile(g, q.tcx);
  q.X0 = q.T * TX - h;
  q.relX0 = (int)((long long)q.X0 - g.shift);
  q.R0 = q.tcr * TR - h;
  return q;
}

// ================================================== momentum pass ==
// The chi deposit accumulates in 64-bit LDS words (Acc0): 64-bit atomics
// run at a much higher rate than ds_add_f32 on gfx950 (measured), and the
// accumulated sums are rounded once, at the flush.
// A region with a margin of H cells: (TX + 2H + 1) x (TR + 2H + 1) nodes.
template <int H> struct Halo {
  static constexpr int X = TX + 2 * H + 1, R = TR + 2 * H + 1, N = X * R;
};
// The gradient of Phi is staged only by the scattering passes with quadratic
// shapes (their registers are the tighter limit); the others difference the
// staged Phi where they read it.  The sort counters exist only in the
// scattering variants.
template <class R, bool M1, int H, int O, bool SC, bool CS> struct SmemMom {
  using C = typename cplx_of<R>::type;
  static constexpr int N = Halo<H>::N;
  static constexpr int NG = (O == 2 && SC) ? N : 1;
  R ex[N], er[N], bt[N], phi[N], gx[NG], gr[NG];
  typename Acc0<R>::T chi[N];
  C ex1[M1 ? N : 1], er1[M1 ? N : 1], et1[M1 ? N : 1];
  C bx1[M1 ? N : 1], br1[M1 ? N : 1], bt1[M1 ? N : 1];
  R ivol[Halo<H>::R];
  int ccell[CS ? CRN : 1];  // cell sort: particles per destination cell, then their next rank
};

// Work item of work group b (of n groups).  Work groups are dealt to the 8
// XCDs in turn; runs of XG consecutive items (radially adjacent tiles, whose
// LDS regions overlap) are given to one XCD so that the halo lines they
// share are fetched into that XCD's L2 once, and the runs rotate over the
// XCDs, which keeps their loads even.  A bijection of [0, n).
constexpr int XCDS = 8, XG = 4;
__device__ inline int item_of(int b, int n) {
  constexpr int sg = XCDS * XG;
  if (b >= (n / sg) * sg) return b;
  const int q = b / XCDS, x = b - q * XCDS;
  return ((q / XG) * XCDS + x) * XG + (q - (q / XG) * XG);
}

// Work item `item` of a layout, and whether there is one: its entry is read
// along with the number of items (every work group's index lies in the
// list's memory), one memory latency instead of two before a group can start.
// The groups of a launch start together, so what they wait for before the
// first particle is time in which nothing streams: with this, the first
// records fetched while the region is staged and all staging loads issued
// before the first is used, the position pass takes 93.3 us instead of 96.9 at
// 8.4 M particles, 14.9 instead of 16.4 at 0.8 M, and the in-place momentum
// pass 12.6 instead of 13.6 there (163 instead of 175 in FP64 at 8.4 M).
__device__ inline bool take_item(const Layout& L, int item, int4& it) {
  it = L.items[item];
  const int n = *L.n_items;
  asm volatile("" ::"s"(it.x), "s"(it.y), "s"(it.z), "s"(it.w));  // (keeps the load before the branch)
  return item < n;
}

// A ticket per lane from the global counter of its key (key < 0: none), with
// one atomic per distinct key in the wavefront; tickets follow lane order
// within a key.  Call from wavefront-uniform control flow.  (Only particles that
// change tile take one: ranking every particle in LDS first, a pass of its
// own, cost the 4096 x 512 workload, which sorts every step, 8 % of a step.)
__device__ inline int wave_ticket(int key, int* counters) {
  const int lane = (int)__lane_id();
  const unsigned long long below = (1ull << lane) - 1ull;
  unsigned long long pending = __ballot(key >= 0);
  int ticket = 0;
  while (pending) {
    const int leader = __ffsll((unsigned long long)pending) - 1;
    const int k = __shfl(key, leader);
    const unsigned long long m = __ballot(key == k);
    int base = 0;
    if (lane == leader) base = atomicAdd(&counters[k], (int)__popcll(m));
    base = __shfl(base, leader);
    if (key == k) ticket = base + (int)__popcll(m & below);
    pending &= ~m;
  }
  return ticket;
}
// counter of a particle's cell in a group's SCAT_CELL counters (the tile and
// SORT_EVERY cells around it)
__device__ inline int sort_cell(const Region& q, unsigned cw, bool& bad) {
  const int sx = clampi(cell_ix(cw) - (q.T * TX - SORT_EVERY), 0, CR - 1, bad);
  const int sr = clampi(cell_jr(cw) - (q.tcr * TR - SORT_EVERY), 0, CR - 1, bad);
  return sx * CR + sr;
}

// SCAT: SCAT_NONE updates p in place and keeps the layout.  SCAT_TILE
// re-sorts by tile into the next layout (the tiles of x^n), as its scan
// made it: incrementally (LAYOUT_MOVE: a particle that stays in its tile
// keeps its slot and has p updated in place; one that changed tile is
// written, whole, to a free slot of its new tile's segment or to that
// tile's overflow range, and its old slot is marked removed), or, when the
// scan found no room (LAYOUT_FULL), every particle is written into the other
// buffer keeping the particles' relative order (coalesced writes), from where
// settle_copy copies them back (in the envelope stage's launch).  SCAT_CELL
// orders each tile by cell and places every work item as at loading, so that
// the lanes of a wavefront hold particles of distinct cells again (the
// deposits' LDS atomics do not collide), at the price of strided writes.
// O: particle shape order (1 linear, 2 quadratic; order 2 re-sorts every
// second step, so its wider stencil stays inside the same halo).
// Waves per SIMD the compiler must allow.  FP32: the in-place pass fits four
// work groups per CU in LDS (its smaller region, no staged gradient) and is
// held to 64 registers per lane (eight waves per SIMD); a tile sort fits three
// (80 registers), or eight waves with mode 0 alone.  FP64: two work groups in
// place (128 registers), one in a sort.
// The in-place pass moves 44 B a particle at 4.3 TB/s (86.6 us) at 8.4 M
// particles and at 5.2 TB/s (1286 us) at 151 M, where a large copy reaches 5.9:
// the rest is the region's staging and the vector instructions.  A tile sort
// takes 102 us there, a scattering cell sort 190 to 310 as the order is lost, a
// gathered one 135 and its copy 105 to 160.
template <class R, bool M1, bool DEFER, int SCAT, int O> constexpr int mom_waves_per_simd() {
  if (DEFER || SCAT == SCAT_CELL) return 1;
  if (sizeof(R) == 8) return SCAT == SCAT_NONE ? 4 : 1;
  return SCAT == SCAT_NONE || !M1 ? 8 : 6;
}

// Margin: a scattering pass gathers at most SORT_EVERY cells of drift from
// the tile (SORT_EVERY - 1 with quadratic shapes) and needs the full HALO;
// the passes in between have drifted one cell less and stage a region with
// one cell less of margin (fewer bytes staged, less LDS per work group).
template <class R, bool M1, bool DEFER, int SCAT, int O, bool NT>
__global__ __launch_bounds__(WG, (mom_waves_per_simd<R, M1, DEFER, SCAT, O>())) void k_momentum(
    Geo g, Grids<R> f, R* __restrict__ chi_out,
                                                 Parts<R> src, Parts<R> dst, Layout Ls, Layout Ld,
                                                 int* __restrict__ ccur, R* __restrict__ gscr,
                                                 unsigned* __restrict__ inv, int* err) {
  using C = typename cplx_of<R>::type;
  constexpr int H = (SCAT == SCAT_NONE && !DEFER) ? HALO - 1 : HALO;
  constexpr int RX = Halo<H>::X, RL = Halo<H>::R, RN = Halo<H>::N;
  __shared__ SmemMom<R, M1, H, O, SCAT != SCAT_NONE, SCAT == SCAT_CELL> sm;
  int4 it;
  if (!take_item(Ls, item_of(blockIdx.x, gridDim.x), it)) return;
  const Region q = region_of(g, it.x, H);
  const R hdt = pick<R>(0.5 * g.dt, g.hdt_f);
  // the particles of the item: its range and, for the last item of a tile,
  // the tile's overflow range riding with it
  const int total = it.z + it.w, ov_base = (it.w > 0 ? Ls.ovb[it.x] : 0) - it.z;
  auto slot_of = [&](int k) { return k + (k < it.z ? it.y : ov_base); };
  // The cell word of the next particle is loaded one turn ahead: the rest of
  // the record follows it at once (the compiler places those loads behind
  // the test for a removed particle).  In the FP32 in-place pass of large
  // runs the rest is loaded at the end of the turn before (the first one while
  // the region is staged): 86.4 us instead of 90.8 at 8.4 M particles, 1279
  // instead of 1314 at 151 M.  Where the records are still in the last-level
  // cache it gives nothing (29.8 and 30.1 at 2.2 M), and the others lose by it,
  // to registers (FP64 in place 161 -> 174) or to what a sort does between the
  // loads and their use (102.5 -> 109).
  constexpr bool AHEAD = SCAT == SCAT_NONE && sizeof(R) == 4 && NT;
  struct Rec {
    R fx, fr, th, w, p[3];
  };
  auto fetch = [&](int p) {
    Rec v;
    v.fx = pld<NT>(elem(src.fx, p));
    v.fr = pld<NT>(elem(src.fr, p));
    v.th = pld<NT>(elem(src.th, p));
    v.w = pld<NT>(elem(src.w, p));
    v.p[0] = pld<NT>(elem(src.px, p));
    v.p[1] = pld<NT>(elem(src.py, p));
    v.p[2] = pld<NT>(elem(src.pz, p));
    return v;
  };
  unsigned cw_next = kDead;
  if (threadIdx.x < total) cw_next = pld<NT>(elem(src.cell, slot_of(threadIdx.x)));
  Rec rec{};
  if (AHEAD && threadIdx.x < total) rec = fetch(slot_of(threadIdx.x));

  // ---- stage E, Bbar, Phi (and mode 1) of the region in LDS.  Every load
  // reads a valid address (the index falls back to the column start) and the
  // value is selected afterwards; outside the grid the value is zero, and on
  // the ghost row j = -1 the radial-staggered values mirror row 1/2 with the
  // parity of the component (odd for mode-0 E_r and Bbar_t and mode-1 B_x).
  // The quadratic stencil also reaches the primal ghost row j = -1, which
  // mirrors row 1 (odd: mode-1 E_x; even: the others).  The loads of a
  // thread's nodes are all issued before the first is stored.
  constexpr int NS = (RN + WG - 1) / WG;
  struct Node {
    R ex, er, bt;
    C env, e1, r1, t1, bx, br, b1;
  } nd[NS];
  struct At {
    bool px, dxok, pv, pg;
    R hs, hp;
    size_t in, ih;
  };
  auto locate = [&](int k) {
    At t;
    const int a = k / RL, b = k - (k / RL) * RL;
    const int rel = q.relX0 + a, j = q.R0 + b;
    t.px = rel >= 0 && rel <= g.nx;
    t.dxok = rel >= 0 && rel <= g.nx - 1;
    const size_t o = (t.px || t.dxok) ? (size_t)phys_col(g, rel) * g.pitch : 0;
    const bool pr = j >= 0 && j <= g.nr, drok = j >= 0 && j <= g.nr - 1, ghost = j == -1;
    t.pg = O == 2 && ghost && g.nr >= 1;        // primal ghost row (order 2)
    t.pv = pr || t.pg;
    t.in = pr ? o + j : (t.pg ? o + 1 : o);     // primal row (clamped), ghost -> row 1
    t.ih = drok ? o + j : o;                    // half row, ghost -> row 1/2
    t.hs = drok ? (R)1 : (ghost ? (R)-1 : (R)0);  // odd parity on the ghost row
    t.hp = drok ? (R)1 : (ghost ? (R)1 : (R)0);   // even parity on the ghost row
    return t;
  };
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    const int k = threadIdx.x + u * WG;
    if (k >= RN) continue;
    const At t = locate(k);
    nd[u].ex = f.ex[t.in];
    nd[u].er = f.er[t.ih];
    nd[u].bt = f.btb[t.ih];
    nd[u].env = f.env[t.in];
    if (M1) {
      nd[u].e1 = f.ex1[t.in];
      nd[u].r1 = f.er1[t.ih];
      nd[u].t1 = f.et1[t.in];
      nd[u].bx = f.bxb1[t.ih];
      nd[u].br = f.brb1[t.in];
      nd[u].b1 = f.btb1[t.ih];
    }
  }
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    const int k = threadIdx.x + u * WG;
    if (k >= RN) continue;
    const At t = locate(k);
    sm.ex[k] = (t.dxok && t.pv) ? nd[u].ex : (R)0;
    sm.er[k] = t.px ? t.hs * nd[u].er : (R)0;
    sm.bt[k] = t.dxok ? t.hs * nd[u].bt : (R)0;
    sm.phi[k] = (t.px && t.pv) ? (R)0.5 * cnorm(nd[u].env) : (R)0;
    sm.chi[k] = 0;
    if (M1) {
      // (selected by component: a select of whole pairs goes through scratch
      // memory on the FP64 path)
      auto scaled = [](bool ok, C v, R by) { return mk<C>(ok ? v.x * by : (R)0, ok ? v.y * by : (R)0); };
      sm.ex1[k] = scaled(t.dxok && t.pv, nd[u].e1, t.pg ? (R)-1 : (R)1);
      sm.er1[k] = scaled(t.px, nd[u].r1, t.hp);
      sm.et1[k] = scaled(t.px && t.pv, nd[u].t1, (R)1);
      sm.bx1[k] = scaled(t.px, nd[u].bx, t.hs);
      sm.br1[k] = scaled(t.dxok && t.pv, nd[u].br, (R)1);
      sm.bt1[k] = scaled(t.dxok, nd[u].b1, t.hp);
    }
  }
  // (the last threads: the first ones hold the regions' second nodes)
  for (int k = WG - 1 - (int)threadIdx.x; k < RL; k += WG) {
    const int j = q.R0 + k;
    sm.ivol[k] = (j >= 0 && j <= g.nr) ? inv_vol_node<R>(g, j) : (R)0;
  }
  if (SCAT == SCAT_CELL)
    for (int k = threadIdx.x; k < CRN; k += WG) sm.ccell[k] = 0;
  __syncthreads();
  // grad Phi by centred differences on the primal nodes (zero radial
  // derivative on the axis, odd below it).  A scattering pass with quadratic
  // shapes stages it (the outermost ring of the region is unused); the
  // other gathers form it from the staged Phi (below).
  const R i2dx = pick<R>(0.5 * g.rdx, g.hrdx_f), i2dr = pick<R>(0.5 * g.rdr, g.hrdr_f);
  if constexpr (O == 2 && SCAT != SCAT_NONE) {
    for (int k = threadIdx.x; k < RN; k += WG) {
      const int a = k / RL, b = k - (k / RL) * RL;
      R vx = 0, vr = 0;
      if (a >= 1 && a <= RX - 2 && b >= 1 && b <= RL - 2) {
        vx = (sm.phi[k + RL] - sm.phi[k - RL]) * i2dx;
        if (q.R0 + b == -1)  // odd below the axis: minus the value on row 1
          vr = -((sm.phi[k + 3] - sm.phi[k + 1]) * i2dr);
        else if (q.R0 + b != 0)
          vr = (sm.phi[k + 1] - sm.phi[k - 1]) * i2dr;
      }
      sm.gx[k] = vx;
      sm.gr[k] = vr;
    }
  }

  bool bad = false, lost = false;
  // gather, push and chi deposit of one particle (p updated); d: the slot of
  // a deferred deposit
  auto push = [&](unsigned cw, R fx, R fr, R th, R w, R(&pv)[3], int d) {
    // the cell relative to the region: [1, RX - 3] for the linear stencils
    // (and the differences of Phi one node further out); order 2 keeps
    // [2, RX - 4], the range its position pass needs for the current
    // stencil of the old and new cells
    const int a = O == 2 ? clampi(cell_ix(cw) - q.X0, 2, RX - 4, bad) : clampi(cell_ix(cw) - q.X0, 1, RX - 3, bad);
    const int b = O == 2 ? clampi(cell_jr(cw) - q.R0, 2, RL - 4, bad) : clampi(cell_jr(cw) - q.R0, 1, RL - 3, bad);
    R s, c;
    sincos_r(th, &s, &c);
    R ex, er, bt, et = 0, bx = 0, br = 0, ph, gx, gr;
    Lin<R> Px, Pr;
    Quad<R> Qx, Qr;
    if constexpr (O == 2) {
      Qx = quad_primal<R>(a, fx);
      Qr = quad_primal<R>(b, fr);
      const Quad<R> Ux = quad_dual<R>(a, fx), Ur = quad_dual<R>(b, fr);
      ex = interp3<R, RL>(sm.ex, Ux, Qr);
      er = interp3<R, RL>(sm.er, Qx, Ur);
      bt = interp3<R, RL>(sm.bt, Ux, Ur);
      if constexpr (SCAT != SCAT_NONE) {
        ph = interp3<R, RL>(sm.phi, Qx, Qr);
        gx = interp3<R, RL>(sm.gx, Qx, Qr);
        gr = interp3<R, RL>(sm.gr, Qx, Qr);
      } else {
        phi_grad3<R, RL>(sm.phi, Qx, Qr, q.R0 + Qr.i, i2dx, i2dr, ph, gx, gr);
      }
      if (M1) {
        ex += mode1_at<C, R>(interp3c<C, R, RL>(sm.ex1, Ux, Qr), c, s);
        er += mode1_at<C, R>(interp3c<C, R, RL>(sm.er1, Qx, Ur), c, s);
        et = mode1_at<C, R>(interp3c<C, R, RL>(sm.et1, Qx, Qr), c, s);
        bx = mode1_at<C, R>(interp3c<C, R, RL>(sm.bx1, Qx, Ur), c, s);
        br = mode1_at<C, R>(interp3c<C, R, RL>(sm.br1, Ux, Qr), c, s);
        bt += mode1_at<C, R>(interp3c<C, R, RL>(sm.bt1, Ux, Ur), c, s);
      }
    } else {
      Px = primal_w<R>(a, fx);
      Pr = primal_w<R>(b, fr);
      // Phi on the 4 x 4 nodes around the cell (corners unused): interpolated
      // along r on the four columns, whose differences interpolated along x
      // give the x derivative, and along x on the four rows (the radial
      // difference at the axis row is zero)
      const R* pc = &sm.phi[a * RL + b];
      const R p00 = pc[0], p01 = pc[1], p10 = pc[RL], p11 = pc[RL + 1];
      const R um = Pr.a * pc[-RL] + Pr.b * pc[1 - RL], u0 = Pr.a * p00 + Pr.b * p01;
      const R u1 = Pr.a * p10 + Pr.b * p11, u2 = Pr.a * pc[2 * RL] + Pr.b * pc[2 * RL + 1];
      ph = Px.a * u0 + Px.b * u1;
      gx = (Px.a * (u1 - um) + Px.b * (u2 - u0)) * i2dx;
      const R vm = Px.a * pc[-1] + Px.b * pc[RL - 1], v0 = Px.a * p00 + Px.b * p10;
      const R v1 = Px.a * p01 + Px.b * p11, v2 = Px.a * pc[2] + Px.b * pc[RL + 2];
      const R d0 = q.R0 + b == 0 ? (R)0 : v1 - vm;
      gr = (Pr.a * d0 + Pr.b * (v2 - v0)) * i2dr;
      const Lin<R> Dx = dual_w<R>(a, fx), Dr = dual_w<R>(b, fr);
      if (M1) {
        // (the weight products are those of the mode-1 gathers below)
        ex = interp2w<R, RL>(sm.ex, Dx, Pr);
        er = interp2w<R, RL>(sm.er, Px, Dr);
        bt = interp2w<R, RL>(sm.bt, Dx, Dr);
      } else {
        ex = interp2<R, RL>(sm.ex, Dx, Pr);
        er = interp2<R, RL>(sm.er, Px, Dr);
        bt = interp2<R, RL>(sm.bt, Dx, Dr);
      }
      if (M1) {
        ex += mode1_at<C, R>(interp2c<C, R, RL>(sm.ex1, Dx, Pr), c, s);
        er += mode1_at<C, R>(interp2c<C, R, RL>(sm.er1, Px, Dr), c, s);
        et = mode1_at<C, R>(interp2c<C, R, RL>(sm.et1, Px, Pr), c, s);
        bx = mode1_at<C, R>(interp2c<C, R, RL>(sm.bx1, Px, Dr), c, s);
        br = mode1_at<C, R>(interp2c<C, R, RL>(sm.br1, Dx, Pr), c, s);
        bt += mode1_at<C, R>(interp2c<C, R, RL>(sm.bt1, Dx, Dr), c, s);
      }
    }
    // (x, r, theta) -> Cartesian, r-hat = (0, c, s), theta-hat = (0, -s, c)
    const R E[3] = {ex, er * c - et * s, er * s + et * c};
    const R B[3] = {bx, br * c - bt * s, br * s + bt * c};
    const R G[3] = {gx, gr * c, gr * s};
    // ponderomotive Boris: half kick with gbar(p^{n-1/2}), rotation and chi
    // with gbar of the half-kicked momentum, second half kick
    const R ig0 = (R)0.5 * rsqrt1_r((R)1 + pv[0] * pv[0] + pv[1] * pv[1] + pv[2] * pv[2] + ph);
    R F[3], pm[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      F[e] = -E[e] - G[e] * ig0;
      pm[e] = pv[e] + hdt * F[e];
    }
    const R igb = rsqrt1_r((R)1 + pm[0] * pm[0] + pm[1] * pm[1] + pm[2] * pm[2] + ph);
    const R tf = -hdt * igb;
    const R t[3] = {tf * B[0], tf * B[1], tf * B[2]};
    const R sf = (R)2 * rcp1_r((R)1 + t[0] * t[0] + t[1] * t[1] + t[2] * t[2]);
    const R sv[3] = {sf * t[0], sf * t[1], sf * t[2]};
    const R pp[3] = {pm[0] + pm[1] * t[2] - pm[2] * t[1], pm[1] + pm[2] * t[0] - pm[0] * t[2],
                     pm[2] + pm[0] * t[1] - pm[1] * t[0]};
    pv[0] = pm[0] + pp[1] * sv[2] - pp[2] * sv[1] + hdt * F[0];
    pv[1] = pm[1] + pp[2] * sv[0] - pp[0] * sv[2] + hdt * F[1];
    pv[2] = pm[2] + pp[0] * sv[1] - pp[1] * sv[0] + hdt * F[2];
    if (DEFER) {
      gscr[d] = (R)1 / igb;
    } else if constexpr (O == 2) {
      // rows below the axis are folded onto their mirrors at the flush
      const R wg = w * igb * (R)Acc0<R>::scale(g);
#pragma unroll
      for (int aa = 0; aa < 3; ++aa) {
        const double wa = (double)(wg * Qx.w[aa]);
#pragma unroll
        for (int bb = 0; bb < 3; ++bb)
          Acc0<R>::add_prod(&sm.chi[(Qx.i + aa) * RL + Qr.i + bb], wa, (double)Qr.w[bb]);
      }
    } else {
      const R wg = w * igb * (R)Acc0<R>::scale(g);
#pragma unroll
      for (int aa = 0; aa < 2; ++aa) {
        const double wa = (double)(wg * (aa ? Px.b : Px.a));
#pragma unroll
        for (int bb = 0; bb < 2; ++bb)
          Acc0<R>::add_prod(&sm.chi[(Px.i + aa) * RL + Pr.i + bb], wa, (double)(bb ? Pr.b : Pr.a));
      }
    }
  };

  // a tile sort that moves only the particles that change tile
  const bool move = SCAT == SCAT_TILE && *Ld.mode == LAYOUT_MOVE;
  // a cell sort whose copy is gathered afterwards (k_permute)
  const bool gather = SCAT == SCAT_CELL && !DEFER && (*Ld.mode & LAYOUT_GATHER) != 0;
  if constexpr (SCAT == SCAT_CELL) {
    // particles per destination cell, then one reservation per cell: each
    // counter becomes the first rank of the group's particles in its cell
    // (the loop below hands the ranks out)
    for (int k = threadIdx.x; k < total; k += WG) {
      const unsigned cw = *elem(src.cell, slot_of(k));
      if (cw != kDead) atomicAdd(&sm.ccell[sort_cell(q, cw, bad)], 1);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < CRN; k += WG) {
      const int c = sm.ccell[k];
      if (c > 0) {
        const int rel = (int)((long long)q.T * TX - SORT_EVERY + k / CR - g.shift);
        const int j = q.tcr * TR - SORT_EVERY + k % CR;
        sm.ccell[k] = atomicAdd(&ccur[(size_t)phys_col(g, rel) * g.pitch + j], c);
      }
    }
  }
  if (SCAT == SCAT_CELL || (O == 2 && SCAT != SCAT_NONE)) __syncthreads();
  const int seg_end = SCAT == SCAT_TILE ? Ls.offsets[g.ntiles] : 0;

  // ---- gather, push, deposit, scatter
  if constexpr (AHEAD) {
    for (int k = threadIdx.x; k < total; k += WG) {
      const unsigned cw = cw_next;
      const int p = slot_of(k), pn = slot_of(k + WG);
      const bool more = k + WG < total;
      if (more) cw_next = pld<NT>(elem(src.cell, pn));
      if (cw != kDead) {
        push(cw, rec.fx, rec.fr, rec.th, rec.w, rec.p, p);
        pst<NT>(elem(src.px, p), rec.p[0]);
        pst<NT>(elem(src.py, p), rec.p[1]);
        pst<NT>(elem(src.pz, p), rec.p[2]);
      }
      if (more) rec = fetch(pn);
    }
  } else {
    // (SCAT_TILE ranks over whole wavefronts: uniform trip count)
    const int trips = SCAT == SCAT_TILE ? (total + 63) & ~63 : total;
    for (int k = threadIdx.x; k < trips; k += WG) {
      const bool valid = SCAT != SCAT_TILE || k < total;
      const int p = slot_of(valid ? k : 0);
      const unsigned cw = cw_next;
      if (k + WG < total) cw_next = pld<NT>(elem(src.cell, slot_of(k + WG)));
      const R fx = pld<NT>(elem(src.fx, p)), fr = pld<NT>(elem(src.fr, p)), th = pld<NT>(elem(src.th, p)), w = pld<NT>(elem(src.w, p));
      R pv[3] = {pld<NT>(elem(src.px, p)), pld<NT>(elem(src.py, p)), pld<NT>(elem(src.pz, p))};
      bool live = valid && cw != kDead;
      int d = p;
      bool stay = true;
      if constexpr (SCAT == SCAT_TILE) {
        // The particle's slot in the new layout, unless it keeps its own: it
        // does when an incremental sort finds it in its tile's segment and
        // still in that tile (nearly all).  The others take tickets, one
        // global atomic per destination tile in a wavefront.
        int key = -1;
        if (live) {
          const int tx = cell_ix(cw) - q.T * TX, tr = cell_jr(cw) - q.tcr * TR;
          const bool same = (unsigned)tx < (unsigned)TX && (unsigned)tr < (unsigned)TR;
          if (!same || !move || p >= seg_end) {
            int tx2 = q.tcx + clampi((tx + TX) / TX - 1, -1, 1, bad);
            if (tx2 < 0) tx2 += g.ntxa;
            if (tx2 >= g.ntxa) tx2 -= g.ntxa;
            const int tr2 = q.tcr + clampi((tr + TR) / TR - 1, -1, 1, bad);
            stay = false;
            if (tr2 < 0 || tr2 >= g.ntr) {
              bad = true;  // no cell lies there: flagged, not written
              live = false;
            } else {
              key = tx2 * g.ntr + tr2;
            }
          }
        }
        if (__ballot(key >= 0)) {
          const int tk = wave_ticket(key, Ld.cursor);
          if (key >= 0) {
            d = tk;
            if (move) {
              // ticket tk of the destination: its free slots, then its overflow
              const int e = Ls.ext[key], room = Ld.ext[key] - e;
              d = tk < room ? Ls.offsets[key] + e + tk : (tk - room < Ld.ovn[key] ? Ld.ovb[key] + tk - room : -1);
            }
            if (d < 0) {  // more arrivals than the scan counted: never written
              lost = true;
              live = false;
            } else if ((long long)d >= g.cap) {  // the scan has flagged the overflow
              bad = true;
              live = false;
            }
          }
        }
      }
      if (!live) continue;
      if constexpr (SCAT == SCAT_CELL) {
        // rank in the destination tile's cell order, then the transposed
        // placement inside its work item (as at loading)
        const int r = atomicAdd(&sm.ccell[sort_cell(q, cw, bad)], 1);
        const int key = tile_key(g, cell_ix(cw), cell_jr(cw));
        const int off = Ld.offsets[key], v = Ld.ext[key];
        if (r >= v) {  // counts and particles disagree: flagged, never written
          bad = true;
          continue;
        }
        d = off + placed_rank<O>(r, v, g.chunk);
        if ((long long)d >= g.cap) {  // the scan has flagged the overflow
          bad = true;
          continue;
        }
        stay = gather;
      }
      push(cw, fx, fr, th, w, pv, d);
      if (SCAT == SCAT_NONE || stay) {
        pst<NT>(elem(src.px, p), pv[0]);
        pst<NT>(elem(src.py, p), pv[1]);
        pst<NT>(elem(src.pz, p), pv[2]);
        // the cell-ordered copy is gathered afterwards (k_permute): the
        // destination slot records where it comes from
        if (SCAT == SCAT_CELL) *elem(inv, d) = (unsigned)p;
      } else {
        // an incremental sort writes within the same buffer, into slots no
        // work item of this pass reads (free or overflow slots)
        const Parts<R>& out = move ? src : dst;
        pst<NT>(elem(out.cell, d), cw);
        pst<NT>(elem(out.fx, d), fx);
        pst<NT>(elem(out.fr, d), fr);
        pst<NT>(elem(out.th, d), th);
        pst<NT>(elem(out.px, d), pv[0]);
        pst<NT>(elem(out.py, d), pv[1]);
        pst<NT>(elem(out.pz, d), pv[2]);
        pst<NT>(elem(out.w, d), w);
        pst<NT>(elem(out.id, d), pld<NT>(elem(src.id, p)));
        if (move && p < seg_end) *elem(src.cell, p) = kDead;  // its old slot
      }
    }
  }
  if (bad) atomicOr(err, ERR_HALO);
  if (lost) atomicOr(err, ERR_LAYOUT);
  if (DEFER) return;
  __syncthreads();
  for (int k = threadIdx.x; k < RN; k += WG) {
    const int a = k / RL, b = k - (k / RL) * RL;
    const int rel = q.relX0 + a, j = q.R0 + b;
    typename Acc0<R>::T v = sm.chi[k];
    // order 2: the row below the axis (two LDS rows down) belongs to row 1
    if (O == 2 && j == 1 && b >= 2) v += sm.chi[k - 2];
    if (!Acc0<R>::nonzero(v)) continue;
    if (rel < 0 || rel > g.nx || j < 0 || j > g.nr) continue;
    atomicAdd(&chi_out[(size_t)phys_col(g, rel) * g.pitch + j], (R)(Acc0<R>::val(v, g) * sm.ivol[b]));
  }
}

// ================================================== position pass ==
// A mode-1 accumulator grid of N nodes, real and imaginary words in
// separate arrays: one atomic instruction then touches words 8 bytes apart
// across the lanes' nodes, not 16 as with interleaved pairs, which halves the
// LDS bank conflicts of the deposit (measured: they took 40 % of the
// position pass's LDS cycles with pairs).
template <class R, int N> struct Acc1Grid {
  using T = typename Acc1<R>::T;
  typename Acc1<R>::S re[N], im[N];
  __device__ T operator[](int k) const {
    T v;
    v.x = re[k];
    v.y = im[k];
    return v;
  }
  __device__ void clear(int k) {
    re[k] = 0;
    im[k] = 0;
  }
};

template <class R, bool M1> struct SmemPos {
  using C = typename cplx_of<R>::type;
  R phh[LN];
  typename Acc0<R>::T jx[LN], jr[LN];
  Acc1Grid<R, M1 ? LN : 1> jx1, jr1, jt1;
  R iax[LR], iar[LR], ivn[LR], ivh[LR];
  int ccell[CRN];  // before a cell sort: particles per cell of x^{n+1}
  int tcnt[11];    // per-tile counts of the work item (flush_tiles)
};

// The largest value of the type below 2: an offset in [0, 1) after a step of
// less than a cell (dt < dr; the stability limit accepts up to 0.97 dr)
template <class R> constexpr R BELOW_TWO = (R)2 - std::numeric_limits<R>::epsilon();

// one particle's move: old and new cells/offsets, transverse displacement
// (radial a, azimuthal b, lengths) at the old azimuth, new azimuth, velocity
template <class R> struct Move {
  int ix0, jr0, ix1, jr1;
  int dix, djr;  // steps in cells, -1, 0 or 1 (less than a cell: dt < dx, dt < dr)
  R fx0, fr0, fx1, fr1;
  R th0, th1, a, b;
  R c0, s0;  // cos, sin of the old azimuth
  bool refl;
  bool small;  // not reflected, and the step is short against its radius (radial_step)
  R vx, vy, vz;
};

// The push x^{n+1} = x^n + dt v in Cartesian space, expressed on the cell
// representation; specular reflection at r_max (p updated).
template <class R>
__device__ inline void push_position(const Geo& g, unsigned cw, R fx, R fr, R th, R& py, R& pz, R vx, R vy, R vz,
                                     Move<R>& mv) {
  const R dt = pick<R>(g.dt, g.dt_f), dr = pick<R>(g.dr, g.dr_f);
  mv.ix0 = cell_ix(cw);
  mv.jr0 = cell_jr(cw);
  mv.fx0 = fx;
  mv.fr0 = fr;
  mv.th0 = th;
  mv.vx = vx;
  mv.vy = vy;
  mv.vz = vz;
  // (|v| <= 1, so the floors below are -1, 0 or 1, whatever the state)
  const R x1 = fma(vx, pick<R>(g.dtdx, g.dtdx_f), fx);
  mv.dix = floor_int(x1);
  mv.ix1 = mv.ix0 + mv.dix;
  mv.fx1 = fract_r(x1);
  R s, c;
  sincos_r(th, &s, &c);
  mv.c0 = c;
  mv.s0 = s;
  const R dy = dt * vy, dz = dt * vz;
  mv.a = c * dy + s * dz;
  mv.b = -s * dy + c * dz;
  const R r = ((R)mv.jr0 + fr) * dr;
  R drad, dth;
  mv.small = radial_step(r, mv.a, mv.b, drad, dth);
  // (the radius stays >= 0 and the step below two cells whatever the rounding)
  const R r1 = clamp_r(fma(drad, pick<R>(g.rdr, g.rdr_f), fr), max((R)-1, -(R)mv.jr0), BELOW_TWO<R>);
  mv.djr = floor_int(r1);
  mv.jr1 = mv.jr0 + mv.djr;
  mv.fr1 = fract_r(r1);
  mv.th1 = wrap_angle(th + dth);
  mv.refl = false;
  if (mv.jr1 >= g.nr) {
    // r' = r_max + e with 0 <= e < dr  ->  r_max - e; reverse p_r
    const R e = (R)(mv.jr1 - g.nr) + mv.fr1;
    mv.jr1 = g.nr - 1;
    mv.djr = min(max(mv.jr1 - mv.jr0, -1), 1);
    mv.fr1 = (R)1 - e;
    if (mv.fr1 < (R)0) mv.fr1 = 0;
    R s1, c1;
    sincos_r(mv.th1, &s1, &c1);
    const R prad = py * c1 + pz * s1;
    py -= (R)2 * prad * c1;
    pz -= (R)2 * prad * s1;
    mv.refl = true;
    mv.small = false;
  }
}

// The Cartesian mid-point of a move, where mode 1 deposits, in the frame of
// the old azimuth at (r0 + a/2, b/2) (from both end points when the particle
// was reflected): its row as a step from the old one (at most one, as the
// move is shorter than a cell), its offset in that row, the cosine and sine
// of its azimuth.
template <class R>
__device__ inline void mid_point(const Geo& g, const Move<R>& mv, int& djm, R& frm, R& c, R& s) {
  const R dr = pick<R>(g.dr, g.dr_f), rdr = pick<R>(g.rdr, g.rdr_f);
  const R r0 = ((R)mv.jr0 + mv.fr0) * dr;
  const R u = r0 + (R)0.5 * mv.a, v = (R)0.5 * mv.b;
  R f;
  if (mv.small) {
    const R beta = v * rcp_r(u), b2 = beta * beta;
    const R cd = rhyp_series(b2), sd = beta * cd;
    f = fma(fma(v * beta, sqrt1_series(b2), (R)0.5 * mv.a), rdr, mv.fr0);
    c = mv.c0 * cd - mv.s0 * sd;
    s = mv.s0 * cd + mv.c0 * sd;
  } else if (!mv.refl) {
    const R rm = sqrt_r(u * u + v * v);
    const R cd = rm > (R)0 ? u / rm : (R)1, sd = rm > (R)0 ? v / rm : (R)0;
    // (for u > 0 the radius by its small difference from u)
    f = u > (R)0 ? mv.fr0 + ((R)0.5 * mv.a + v * v / (u + rm)) * rdr : mv.fr0 + (rm - r0) * rdr;
    c = mv.c0 * cd - mv.s0 * sd;
    s = mv.s0 * cd + mv.c0 * sd;
  } else {
    R s1, c1;
    sincos_r(mv.th1, &s1, &c1);
    const R r1 = ((R)mv.jr1 + mv.fr1) * dr;
    const R ym = (R)0.5 * (r0 * mv.c0 + r1 * c1), zm = (R)0.5 * (r0 * mv.s0 + r1 * s1);
    const R rm = sqrt_r(ym * ym + zm * zm);
    f = mv.fr0 + (rm - r0) * rdr;
    c = rm > (R)0 ? ym / rm : (R)1;
    s = rm > (R)0 ? zm / rm : (R)0;
  }
  f = clamp_r(f, max((R)-1, -(R)mv.jr0), BELOW_TWO<R>);
  djm = floor_int(f);
  frm = fract_r(f);
}

// Esirkepov current of one particle between two positions (mode 0) and the
// direct mid-point current of mode 1, into the LDS accumulators.
template <class R, bool M1>
__device__ inline void deposit_current(SmemPos<R, M1>& sm, const Region& q, const Geo& g, const Move<R>& mv, R w,
                                       bool& bad) {
  // the stencil spans min(a0, a1) .. min(a0, a1) + 2: the push moves a
  // particle less than a cell, so the new cell is the old one's neighbour or
  // itself, and every index is inside the region once the old cell is
  const int a0 = clampi(mv.ix0 - q.X0, 2, LX - 4, bad);
  const int b0 = clampi(mv.jr0 - q.R0, 2, LR - 4, bad);
  const int dxs = mv.dix, drs = mv.djr;
  // On the 3-node union of the old and new supports (first node amin), with
  // F0 and F1 the weights that the old and new position put beyond the first
  // node, the first partial sum of the flux along an axis is F0 - F1 and the
  // node sums S0 + S1 are 2 - (F0 + F1), (F0 + F1) - T2, T2.  The second
  // partial sum and the third node exist only when the particle changed
  // column (row).
  const int amin = a0 + min(dxs, 0), bmin = b0 + min(drs, 0);
  const R F0x = dxs < 0 ? (R)1 : mv.fx0, F1x = dxs > 0 ? (R)1 : mv.fx1;
  const R F0r = drs < 0 ? (R)1 : mv.fr0, F1r = drs > 0 ? (R)1 : mv.fr1;
  const R sx = F0x + F1x, sr = F0r + F1r;
  const R T2x = dxs > 0 ? mv.fx1 : (dxs < 0 ? mv.fx0 : (R)0), T2r = drs > 0 ? mv.fr1 : (drs < 0 ? mv.fr0 : (R)0);
  // J_x (i+1/2, j): flux accumulated along x; J_r (i, j+1/2): along r
  // (the face areas are applied at the flush)
  using A0 = Acc0<R>;
  typename A0::T* jx = &sm.jx[amin * LR + bmin];
  typename A0::T* jr = &sm.jr[amin * LR + bmin];
  const double hw = (double)w * (0.5 * A0::scale(g));
  const double cx0 = F0x - F1x, cr0 = F0r - F1r;
  const double wr0 = (double)((R)2 - sr) * hw, wr1 = (double)(sr - T2r) * hw;
  const double wx0 = (double)((R)2 - sx) * hw, wx1 = (double)(sx - T2x) * hw;
  A0::add_prod(&jx[0], cx0, wr0);
  A0::add_prod(&jx[1], cx0, wr1);
  A0::add_prod(&jr[0], cr0, wx0);
  A0::add_prod(&jr[LR], cr0, wx1);
  if (dxs != 0) {
    const double cx1 = dxs > 0 ? -mv.fx1 : mv.fx0;
    A0::add_prod(&jx[LR], cx1, wr0);
    A0::add_prod(&jx[LR + 1], cx1, wr1);
    A0::add_prod(&jr[2 * LR], cr0, (double)T2x * hw);
  }
  if (drs != 0) {
    const double cr1 = drs > 0 ? -mv.fr1 : mv.fr0;
    const double wr2 = (double)T2r * hw;
    A0::add_prod(&jr[1], cr1, wx0);
    A0::add_prod(&jr[LR + 1], cr1, wx1);
    A0::add_prod(&jx[2], cx0, wr2);
    if (dxs != 0) {
      A0::add_prod(&jx[LR + 2], (double)(dxs > 0 ? -mv.fx1 : mv.fx0), wr2);
      A0::add_prod(&jr[2 * LR + 1], cr1, (double)T2x * hw);
    }
  }
  if (M1) {
    int djm;
    R frm, c, s;
    mid_point<R>(g, mv, djm, frm, c, s);
    // the old cell's indices plus a step of at most one: inside the region
    const R um = fma(pick<R>(0.5 * g.dtdx, g.hdtdx_f), mv.vx, mv.fx0);
    const int am = a0 + floor_int(um), bm = b0 + djm;
    const R fm = fract_r(um);
    const Lin<R> Px = primal_w<R>(am, fm), Dx = dual_w<R>(am, fm);
    const Lin<R> Pr = primal_w<R>(bm, frm), Dr = dual_w<R>(bm, frm);
    // 2 q w v e^{i theta} per component (electrons, q = -1), with the
    // accumulator scale folded in; radial weights times inverse volumes
    const R q2 = w * ((R)-2 * Acc1<R>::scale(g));
    const R vx = q2 * mv.vx, vr = q2 * (mv.vy * c + mv.vz * s), vt = q2 * (mv.vz * c - mv.vy * s);
    const double xc = vx * c, xs = vx * s, rc = vr * c, rs = vr * s, tc = vt * c, ts = vt * s;
    const R pv[2] = {Pr.a * sm.ivn[Pr.i], Pr.b * sm.ivn[Pr.i + 1]};
    // (J_r1 of the half row -1/2 is folded onto +1/2 at the flush)
    const R dv[2] = {Dr.a * sm.ivh[Dr.i], Dr.b * sm.ivh[Dr.i + 1]};
#pragma unroll
    for (int aa = 0; aa < 2; ++aa) {
      const R wdx = aa ? Dx.b : Dx.a, wpx = aa ? Px.b : Px.a;
#pragma unroll
      for (int bb = 0; bb < 2; ++bb) {
        const double ux = wdx * pv[bb], ur = wpx * dv[bb], ut = wpx * pv[bb];
        Acc1<R>::add_prod(sm.jx1, (Dx.i + aa) * LR + Pr.i + bb, ux, xc, xs);  // (i+1/2, j)
        Acc1<R>::add_prod(sm.jr1, (Px.i + aa) * LR + Dr.i + bb, ur, rc, rs);  // (i, j+1/2)
        Acc1<R>::add_prod(sm.jt1, (Px.i + aa) * LR + Pr.i + bb, ut, tc, ts);  // (i, j)
      }
    }
  }
}

// Order-2 currents: the Esirkepov decomposition of the change between the
// old and new quadratic stencils on their 4-node union (mode 0), and the
// quadratic mid-point deposit of mode 1.  Contributions to the rows below
// the axis stay in the LDS ghost rows and are folded at the flush.
template <class R, bool M1>
__device__ inline void deposit_current2(SmemPos<R, M1>& sm, const Region& q, const Geo& g, const Move<R>& mv, R w,
                                        bool& bad) {
  const int a0 = clampi(mv.ix0 - q.X0, 2, LX - 4, bad);
  const int a1 = a0 + mv.dix;  // (a step of at most one cell)
  const int b0 = clampi(mv.jr0 - q.R0, 2, LR - 4, bad);
  const int b1 = b0 + mv.djr;
  const Quad<R> X0 = quad_primal<R>(a0, mv.fx0), X1 = quad_primal<R>(a1, mv.fx1);
  const Quad<R> Y0 = quad_primal<R>(b0, mv.fr0), Y1 = quad_primal<R>(b1, mv.fr1);
  // nearest nodes move by at most one (less than a cell per step)
  const int ax = min(X0.i, X1.i), by = min(Y0.i, Y1.i);
  const int ox0 = clampi(X0.i - ax, 0, 1, bad), ox1 = clampi(X1.i - ax, 0, 1, bad);
  const int or0 = clampi(Y0.i - by, 0, 1, bad), or1 = clampi(Y1.i - by, 0, 1, bad);
  // the stencils on the union (placed without indexing register arrays)
  auto place = [](const Quad<R>& Q, int o, R* S) {
    S[0] = o ? (R)0 : Q.w[0];
    S[1] = o ? Q.w[0] : Q.w[1];
    S[2] = o ? Q.w[1] : Q.w[2];
    S[3] = o ? Q.w[2] : (R)0;
  };
  R S0x[4], S1x[4], S0r[4], S1r[4];
  place(X0, ox0, S0x);
  place(X1, ox1, S1x);
  place(Y0, or0, S0r);
  place(Y1, or1, S1r);
  // partial sums of the change from the low side (the fourth is zero)
  R cx[3], cr[3];
  cx[0] = S1x[0] - S0x[0];
  cr[0] = S1r[0] - S0r[0];
#pragma unroll
  for (int k = 1; k < 3; ++k) {
    cx[k] = cx[k - 1] + (S1x[k] - S0x[k]);
    cr[k] = cr[k - 1] + (S1r[k] - S0r[k]);
  }
  using A0 = Acc0<R>;
  typename A0::T* jx = &sm.jx[ax * LR + by];
  typename A0::T* jr = &sm.jr[ax * LR + by];
  const double hw = (double)w * (0.5 * A0::scale(g));
#pragma unroll
  for (int bb = 0; bb < 4; ++bb) {
    const double sr = (double)(S0r[bb] + S1r[bb]) * hw;
#pragma unroll
    for (int aa = 0; aa < 3; ++aa)
      if (cx[aa] != (R)0) A0::add_prod(&jx[aa * LR + bb], (double)cx[aa], sr);
  }
#pragma unroll
  for (int aa = 0; aa < 4; ++aa) {
    const double sx = (double)(S0x[aa] + S1x[aa]) * hw;
#pragma unroll
    for (int bb = 0; bb < 3; ++bb)
      if (cr[bb] != (R)0) A0::add_prod(&jr[aa * LR + bb], (double)cr[bb], sx);
  }
  if (M1) {
    int djm;
    R frm, c, s;
    mid_point<R>(g, mv, djm, frm, c, s);
    const R um = fma(pick<R>(0.5 * g.dtdx, g.hdtdx_f), mv.vx, mv.fx0);
    const int am = a0 + floor_int(um), bm = b0 + djm;
    const R fm = fract_r(um);
    const Quad<R> Qx = quad_primal<R>(am, fm), Ux = quad_dual<R>(am, fm);
    const Quad<R> Qr = quad_primal<R>(bm, frm), Ur = quad_dual<R>(bm, frm);
    const R q2 = w * ((R)-2 * Acc1<R>::scale(g));
    const R vx = q2 * mv.vx, vr = q2 * (mv.vy * c + mv.vz * s), vt = q2 * (mv.vz * c - mv.vy * s);
    const double xc = vx * c, xs = vx * s, rc = vr * c, rs = vr * s, tc = vt * c, ts = vt * s;
    // radial weights times the inverse volume of the row they land on (the
    // ghost rows carry their mirrors'; their deposits are folded onto those
    // at the flush)
    R pv[3], dv[3];
#pragma unroll
    for (int bb = 0; bb < 3; ++bb) {
      pv[bb] = Qr.w[bb] * sm.ivn[Qr.i + bb];
      dv[bb] = Ur.w[bb] * sm.ivh[Ur.i + bb];
    }
    // each radial factor times the velocity's cosine and sine parts in FP64,
    // then one FMA per word with the axial weight (converted once per node)
#pragma unroll
    for (int bb = 0; bb < 3; ++bb) {
      const double p = pv[bb], d = dv[bb];
      const double pxc = p * xc, pxs = p * xs, drc = d * rc, drs = d * rs, ptc = p * tc, pts = p * ts;
#pragma unroll
      for (int aa = 0; aa < 3; ++aa) {
        const double ux = Ux.w[aa], qx = Qx.w[aa];
        Acc1<R>::add_prod(sm.jx1, (Ux.i + aa) * LR + Qr.i + bb, ux, pxc, pxs);  // (i+1/2, j)
        Acc1<R>::add_prod(sm.jr1, (Qx.i + aa) * LR + Ur.i + bb, qx, drc, drs);  // (i, j+1/2)
        Acc1<R>::add_prod(sm.jt1, (Qx.i + aa) * LR + Qr.i + bb, qx, ptc, pts);  // (i, j)
      }
    }
  }
}

template <class R, bool M1>
__device__ inline void stage_pos_constants(SmemPos<R, M1>& sm, const Region& q, const Geo& g) {
  // one constant per wavefront (of the first four), so that no wavefront
  // computes more than one FP64 division
  const double pi = 3.14159265358979323846;
  const int what = threadIdx.x >> 6, k = threadIdx.x & 63;
  static_assert(LR <= 64 && WG >= 256, "one wavefront per constant");
  if (k >= LR || what > 3) return;
  const int j = q.R0 + k;
  const bool node = j >= 0 && j <= g.nr, half = j >= 0 && j <= g.nr - 1;
  if (what == 0) {
    // 1 / (face area * dt): axial face of row j (V_j / dx), radial face at r_{j+1/2}
    const double ax = (j == 0 ? pi * g.dr * g.dr * 0.25 : 2.0 * pi * j * g.dr * g.dr);
    sm.iax[k] = node ? (R)(1.0 / (ax * g.dt)) : (R)0;
  } else if (what == 1) {
    const double ar = 2.0 * pi * (j + 0.5) * g.dr * g.dx;
    sm.iar[k] = half ? (R)(1.0 / (ar * g.dt)) : (R)0;
  } else if (what == 2) {
    // the primal ghost row j = -1 carries the volume of row 1, onto which
    // its (order-2) deposits are folded
    sm.ivn[k] = node ? inv_vol_node<R>(g, j) : (j == -1 ? inv_vol_node<R>(g, 1) : (R)0);
  } else {
    // (the ghost half row -1/2 that of +1/2)
    sm.ivh[k] = half ? inv_vol_half<R>(g, j) : (j == -1 ? inv_vol_half<R>(g, 0) : (R)0);
  }
}

template <class R, bool M1>
__device__ inline void zero_pos_acc(SmemPos<R, M1>& sm) {
  for (int k = threadIdx.x; k < LN; k += WG) {
    sm.jx[k] = 0;
    sm.jr[k] = 0;
    if (M1) {
      sm.jx1.clear(k);
      sm.jr1.clear(k);
      sm.jt1.clear(k);
    }
  }
  for (int k = threadIdx.x; k < CRN; k += WG) sm.ccell[k] = 0;
  if (threadIdx.x < 11) sm.tcnt[threadIdx.x] = 0;
}

// a + sg b of two mode-1 accumulator words (exact for the fixed point, whose
// words add modulo 2^64)
template <class T> __device__ inline T acc_axpy(T a, const T& b, int sg) {
  a.x += sg * b.x;
  a.y += sg * b.y;
  return a;
}

// O = 2: the deposits on the rows below the axis are folded onto their
// mirrors with the component's parity (R23): J_x row -1 onto row 1 (even for
// mode 0, odd for mode 1), J_r face -1/2 onto +1/2 (odd for mode 0), mode-1
// J_theta row -1 onto row 1 (even), and, for both orders, mode-1 J_r face
// -1/2 onto +1/2 (even).
template <class R, bool M1, int O>
__device__ inline void flush_current(SmemPos<R, M1>& sm, const Region& q, const Geo& g, R* jx_out,
                                     R* jr_out, typename cplx_of<R>::type* jx1_out,
                                     typename cplx_of<R>::type* jr1_out,
                                     typename cplx_of<R>::type* jt1_out) {
  for (int k = threadIdx.x; k < LN; k += WG) {
    const int a = k / LR, b = k - (k / LR) * LR;
    const int rel = q.relX0 + a, j = q.R0 + b;
    if (rel < 0 || rel > g.nx || j < 0 || j > g.nr) continue;
    const size_t o = (size_t)phys_col(g, rel) * g.pitch + j;
    const bool dxok = rel <= g.nx - 1, drok = j <= g.nr - 1;
    if constexpr (O == 2) {
      const bool fold_row = j == 1 && b >= 2, fold_face = j == 0 && b >= 1;
      typename Acc0<R>::T vjx = sm.jx[k], vjr = sm.jr[k];
      if (fold_row) vjx += sm.jx[k - 2];
      if (fold_face) vjr -= sm.jr[k - 1];
      if (dxok && Acc0<R>::nonzero(vjx)) atomicAdd(&jx_out[o], (R)(Acc0<R>::val(vjx, g) * sm.iax[b]));
      if (drok && Acc0<R>::nonzero(vjr)) atomicAdd(&jr_out[o], (R)(Acc0<R>::val(vjr, g) * sm.iar[b]));
      if (M1) {
        using A = Acc1<R>;
        typename A::T v1x = sm.jx1[k], v1t = sm.jt1[k];
        if (fold_row) {
          v1x = acc_axpy(v1x, sm.jx1[k - 2], -1);
          v1t = acc_axpy(v1t, sm.jt1[k - 2], 1);
        }
        if (dxok && A::nonzero(v1x)) {
          atomicAdd(&jx1_out[o].x, (R)A::re(v1x, g));
          atomicAdd(&jx1_out[o].y, (R)A::im(v1x, g));
        }
        typename A::T v1r = sm.jr1[k];
        if (j == 0 && b >= 1) v1r = acc_axpy(v1r, sm.jr1[k - 1], 1);
        if (drok && A::nonzero(v1r)) {
          atomicAdd(&jr1_out[o].x, (R)A::re(v1r, g));
          atomicAdd(&jr1_out[o].y, (R)A::im(v1r, g));
        }
        if (A::nonzero(v1t)) {
          atomicAdd(&jt1_out[o].x, (R)A::re(v1t, g));
          atomicAdd(&jt1_out[o].y, (R)A::im(v1t, g));
        }
      }
    } else {
      if (dxok && Acc0<R>::nonzero(sm.jx[k])) atomicAdd(&jx_out[o], (R)(Acc0<R>::val(sm.jx[k], g) * sm.iax[b]));
      if (drok && Acc0<R>::nonzero(sm.jr[k])) atomicAdd(&jr_out[o], (R)(Acc0<R>::val(sm.jr[k], g) * sm.iar[b]));
      if (M1) {
        using A = Acc1<R>;
        if (dxok && A::nonzero(sm.jx1[k])) {
          atomicAdd(&jx1_out[o].x, (R)A::re(sm.jx1[k], g));
          atomicAdd(&jx1_out[o].y, (R)A::im(sm.jx1[k], g));
        }
        typename A::T v1r = sm.jr1[k];
        if (j == 0 && b >= 1) v1r = acc_axpy(v1r, sm.jr1[k - 1], 1);
        if (drok && A::nonzero(v1r)) {
          atomicAdd(&jr1_out[o].x, (R)A::re(v1r, g));
          atomicAdd(&jr1_out[o].y, (R)A::im(v1r, g));
        }
        if (A::nonzero(sm.jt1[k])) {
          atomicAdd(&jt1_out[o].x, (R)A::re(sm.jt1[k], g));
          atomicAdd(&jt1_out[o].y, (R)A::im(sm.jt1[k], g));
        }
      }
    }
  }
}

// the per-cell counts of a work item into the global per-cell counts
__device__ inline void flush_cells(const int* cc, const Region& q, const Geo& g, int* ccount) {
  for (int k = threadIdx.x; k < CRN; k += WG) {
    const int c = cc[k];
    if (c > 0) {
      const int rel = (int)((long long)q.T * TX - SORT_EVERY + k / CR - g.shift);
      const int j = q.tcr * TR - SORT_EVERY + k % CR;
      atomicAdd(&ccount[(size_t)phys_col(g, rel) * g.pitch + j], c);
    }
  }
}

// The per-tile counts of a work item, t[d] for d = 3 (dx + 1) + (dr + 1)
// the particles that moved to the neighbouring tile (dx, dr) (counted
// before a tile sort), t[9] the particles removed, t[10] those of a range
// past the segments that stay in the tile (before a tile sort).  hist
// (particles per tile, kept current from step to step) loses the removed and
// moved ones and gains the moved ones at their new tiles; before a tile sort,
// arr gains the moved ones, and those that stay past the segments.
__device__ inline void flush_tiles(const int* t, const Region& q, const Geo& g, const SortCounts& sc) {
  if (threadIdx.x >= 9) return;
  const int d = threadIdx.x;
  int v = t[d];
  if (d == 4) {
    int moved = 0;
    for (int e = 0; e < 9; ++e) moved += e == 4 ? 0 : t[e];
    const int key = q.tcx * g.ntr + q.tcr;
    if (t[9] + moved != 0) atomicAdd(&sc.hist[key], -(t[9] + moved));
    if (t[10] != 0) atomicAdd(&sc.arr[key], t[10]);
    return;
  }
  if (v == 0) return;
  int tx = q.tcx + d / 3 - 1;
  if (tx < 0) tx += g.ntxa;
  if (tx >= g.ntxa) tx -= g.ntxa;
  const int tr = q.tcr + d % 3 - 1;
  if (tr < 0 || tr >= g.ntr) return;  // (no cell lies there)
  atomicAdd(&sc.hist[tx * g.ntr + tr], v);
  atomicAdd(&sc.arr[tx * g.ntr + tr], v);
}

// ============================================== loading / injection ==
// Plasma of lab cell column `col`, radial cell j: regular in x and r, one
// SplitMix64 angle per cell with equally spaced angles inside the cell,
// weights n 2 pi r (dr/N_r)(dx/N_x)/N_theta.  Particle k of the cell is
// stored at base + transpose_rank(r0 + k, n_range).  Returns 1 if live.
template <class R>
__device__ inline int load_particle(const Geo& g, const Plasma& pl, Parts<R> P, int base, int r0, int n_range,
                                    long long col, int j, int k) {
  const double pi = 3.14159265358979323846;
  const int ppc = g.ppc_x * g.ppc_r * g.ppc_t;
  const int t = k % g.ppc_t, b = (k / g.ppc_t) % g.ppc_r, a = k / (g.ppc_t * g.ppc_r);
  const double fx = (a + 0.5) / g.ppc_x, fr = (b + 0.5) / g.ppc_r;
  const double xl = ((double)col + fx) * g.dx;
  const double r = (j + fr) * g.dr;
  const double n = plasma_density(pl, xl, col, j);
  const int s = base + transpose_rank(r0 + k, n_range);
  P.px[s] = 0;
  P.py[s] = 0;
  P.pz[s] = 0;
  P.id[s] = (uint32_t)(col * (long long)g.nr * ppc + (long long)j * ppc + k);
  if (!(n > 0.0)) {
    P.cell[s] = kDead;
    P.fx[s] = 0;
    P.fr[s] = 0;
    P.th[s] = 0;
    P.w[s] = 0;
    return 0;
  }
  const double th0 = 2.0 * pi * counter_uniform(pl.seed, STREAM_ANGLE, col, j);
  double th = th0 + 2.0 * pi * t / g.ppc_t;  // in [0, 4 pi): fold into (-pi, pi]
  if (th > pi) th -= 2.0 * pi;
  if (th > pi) th -= 2.0 * pi;
  P.cell[s] = pack_cell((int)col, j);
  P.fx[s] = (R)fx;
  P.fr[s] = (R)fr;
  P.th[s] = (R)th;
  P.w[s] = (R)(n * 2.0 * pi * r * (g.dr / g.ppc_r) * (g.dx / g.ppc_x) / g.ppc_t);
  return 1;
}

// One work group (WG threads, group index blk) of the injection: the
// plasma of lab column gn.shift + nx - 1, tile by tile, with one work item
// per tile.  A row tile goes to the end of its tile's segment when the free
// slots hold it, else past the used slots (after the row tiles before it
// that went there); every group of the injection finds the same placement
// (the layout does not change during the pass).  s_cnt holds WG + 1 ints,
// s_base ntr + 1.  The field stage adds the items to the layout (and their
// slots to the segments or the fill pointer).
template <class R>
__device__ void inject_block(const InjectArgs& ia, Parts<R> P, const Layout& L, const SortCounts& sc, int* err,
                             int blk, int* s_cnt, int* s_base) {
  const Geo& g = ia.gn;
  const long long col = g.shift + g.nx - 1;
  const int ppc = g.ppc_x * g.ppc_r * g.ppc_t;
  const int total = *L.fill;  // end of the used slots
  const int base_items = *L.n_items;
  const int seg_end = L.offsets[g.ntiles];
  if ((long long)total + (long long)g.nr * ppc > ia.capacity || base_items + g.ntr > ia.max_items || col > COL_MAX) {
    if (blk == 0 && threadIdx.x == 0) atomicOr(err, ERR_CAPACITY);
    return;
  }
  // first slot of each row tile: its segment's end (>= 0) or, for now, the
  // negated slot count of a row tile that goes past the used slots
  for (int t = threadIdx.x; t < g.ntr; t += WG) {
    const int key = tile_key(g, col, t * TR), n = min(TR, g.nr - t * TR) * ppc;
    const int off = L.offsets[key], e = L.ext[key];
    s_base[t] = e + n <= L.offsets[key + 1] - off ? off + e : -n;
  }
  for (int k = threadIdx.x; k < WG + 1; k += WG) s_cnt[k] = 0;
  __syncthreads();
  if (threadIdx.x == 0) {
    int fill = total;
    for (int t = 0; t < g.ntr; ++t)
      if (s_base[t] < 0) {
        const int n = -s_base[t];
        s_base[t] = fill;
        fill += n;
      }
    s_base[g.ntr] = fill - total;  // slots past the used ones
  }
  __syncthreads();
  // live particles per cell (one cell = ppc consecutive threads), counted in
  // LDS first: a group spans WG / ppc + 1 rows at most
  const int idx = blk * WG + threadIdx.x;
  const int j_first = (blk * WG) / ppc;
  if (idx < g.nr * ppc) {
    const int j = idx / ppc, k = idx - (idx / ppc) * ppc;
    const int t = j / TR, trt = min(TR, g.nr - t * TR);
    if (load_particle<R>(g, ia.pl, P, s_base[t], (j - t * TR) * ppc, trt * ppc, col, j, k))
      atomicAdd(&s_cnt[j - j_first], 1);
  }
  __syncthreads();
  if (sc.mode == SCAT_CELL) {
    const int pc = phys_col(g, g.nx - 1);
    for (int k = threadIdx.x; k < WG + 1; k += WG)
      if (s_cnt[k] > 0 && j_first + k < g.nr) atomicAdd(&sc.ccount[(size_t)pc * g.pitch + j_first + k], s_cnt[k]);
  }
  // the particles per tile, kept current; before a tile sort the particles
  // of a row tile placed past the segments also arrive in their tile's
  // segment
  for (int k = threadIdx.x; k < WG + 1; k += WG)
    if (s_cnt[k] > 0 && j_first + k < g.nr) {
      const int j = j_first + k;
      const int key = tile_key(g, col, j);
      atomicAdd(&sc.hist[key], s_cnt[k]);
      if (sc.mode == SCAT_TILE && s_base[j / TR] >= seg_end) atomicAdd(&sc.arr[key], s_cnt[k]);
    }
  if (idx < g.ntr) {
    const int trt = min(TR, g.nr - idx * TR);
    L.items[base_items + idx] = make_int4(tile_key(g, col, idx * TR), s_base[idx], trt * ppc, 0);
  }
  if (idx == 0) {
    ia.pending[0] = g.ntr;           // items appended
    ia.pending[1] = s_base[g.ntr];   // slots appended past the used ones
  }
}

// vacate: 1 when the window moves after this step (particles whose new
// column is the window's first one are dropped after depositing); sc: what
// to count for a sort at the next step (SortCounts)
// Registers are held to what the LDS allows in flight: three work groups per
// CU with mode 1 (80 registers per lane, with some bytes of spills for the
// quadratic shapes), more with mode 0 alone; FP64: two groups (128).
// The pass moves 48 B a particle and issues 288 vector instructions per 64
// particles (367 before the steps' weights were shared and its constants came
// as arguments: 112 us at 8.4 M particles late in a run against 96): 93 us, 4.3
// TB/s there, 1345 us, 5.4 TB/s at 151 M, where a large copy reaches 5.9.  What
// the smaller run loses is the staging and flush that its three rounds of
// groups go through in step.
template <class R, bool M1, int O> constexpr int pos_waves_per_simd() {
  return sizeof(R) == 8 ? 4 : (M1 || O == 2) ? 6 : 8;
}

template <class R, bool M1, bool DEFER, int O, bool NT>
__global__ __launch_bounds__(WG, (pos_waves_per_simd<R, M1, O>())) void k_position(Geo g, Grids<R> f, R* __restrict__ jx_out,
                                                 R* __restrict__ jr_out,
                                                 typename cplx_of<R>::type* __restrict__ jx1_out,
                                                 typename cplx_of<R>::type* __restrict__ jr1_out,
                                                 typename cplx_of<R>::type* __restrict__ jt1_out,
                                                 Parts<R> P, Layout L, SortCounts sc, int vacate,
                                                 Parts<R> scr, int* err, int item_blocks,
                                                 InjectArgs inj) {
  __shared__ SmemPos<R, M1> sm;
  if ((int)blockIdx.x >= item_blocks) {
    // the phi staging area and the J_x accumulators are free in these
    // groups: they hold the row counts and the row tiles' first slots
    static_assert(sizeof(sm.phh) >= (WG + 1) * sizeof(int), "row counts do not fit");
    static_assert(sizeof(sm.jx) >= (NR_MAX / TR + 2) * sizeof(int), "row tile slots do not fit");
    inject_block<R>(inj, P, L, sc, err, blockIdx.x - item_blocks, reinterpret_cast<int*>(sm.phh),
                    reinterpret_cast<int*>(sm.jx));
    return;
  }
  int4 it;
  if (!take_item(L, item_of(blockIdx.x, item_blocks), it)) return;
  const Region q = region_of(g, it.x);
  // the next particle's record is loaded before this one is processed
  // (the stores below would otherwise keep the loads from moving up), the
  // first one while the region is staged
  struct Rec {
    unsigned cw;
    R fx, fr, th, w, px, py, pz;
  };
  auto fetch = [&](int p) {
    Rec r;
    r.cw = pld<NT>(elem(P.cell, p));
    r.fx = pld<NT>(elem(P.fx, p));
    r.fr = pld<NT>(elem(P.fr, p));
    r.th = pld<NT>(elem(P.th, p));
    r.w = pld<NT>(elem(P.w, p));
    r.px = pld<NT>(elem(P.px, p));
    r.py = pld<NT>(elem(P.py, p));
    r.pz = pld<NT>(elem(P.pz, p));
    return r;
  };
  // the item's range, then the overflow range riding with it
  const int total = it.z + it.w, ov_base = (it.w > 0 ? L.ovb[it.x] : 0) - it.z;
  auto slot_of = [&](int k) { return k + (k < it.z ? it.y : ov_base); };
  Rec nxt;
  if (threadIdx.x < total) nxt = fetch(slot_of(threadIdx.x));

  // Phi^{n+1/2} = (|A^{n+1}|^2 + |A^n|^2)/4 on the primal nodes (order 2:
  // the ghost row j = -1 mirrors row 1, even)
  constexpr int NS = (LN + WG - 1) / WG;  // (every load is issued before the first is used)
  R phi[NS];
  {
    typename cplx_of<R>::type e[NS], ep[NS];
    bool ok[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int k = min((int)threadIdx.x + u * WG, LN - 1);
      const int a = k / LR, b = k - (k / LR) * LR;
      const int rel = q.relX0 + a, j0 = q.R0 + b;
      const int j = (O == 2 && j0 == -1) ? 1 : j0;
      ok[u] = rel >= 0 && rel <= g.nx && j >= 0 && j <= g.nr;
      const size_t o = ok[u] ? (size_t)phys_col(g, rel) * g.pitch + j : 0;
      e[u] = f.env[o];
      ep[u] = f.envp[o];
    }
#pragma unroll
    for (int u = 0; u < NS; ++u) phi[u] = ok[u] ? (R)0.25 * (cnorm(e[u]) + cnorm(ep[u])) : (R)0;
  }
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    const int k = (int)threadIdx.x + u * WG;
    if (k < LN) sm.phh[k] = phi[u];
  }
  stage_pos_constants(sm, q, g);
  zero_pos_acc(sm);
  __syncthreads();
  const int seg_end = L.offsets[g.ntiles];
  bool bad = false;
  for (int k = threadIdx.x; k < total; k += WG) {
    const Rec cur = nxt;
    const int p = slot_of(k);
    if (k + WG < total) nxt = fetch(slot_of(k + WG));
    const unsigned cw = cur.cw;
    if (cw == kDead) continue;
    const R fx = cur.fx, fr = cur.fr, th = cur.th, w = cur.w;
    const R px = cur.px;
    R py = cur.py, pz = cur.pz;
    R ph;
    if constexpr (O == 2) {
      const int a = clampi(cell_ix(cw) - q.X0, 2, LX - 4, bad);
      const int b = clampi(cell_jr(cw) - q.R0, 2, LR - 4, bad);
      ph = interp3<R>(sm.phh, quad_primal<R>(a, fx), quad_primal<R>(b, fr));
    } else {
      // the old cell is at most two cells out of the tile: the range of the
      // current stencil's old cell, the same clamp as the deposit's (shared)
      const int a = clampi(cell_ix(cw) - q.X0, 2, LX - 4, bad);
      const int b = clampi(cell_jr(cw) - q.R0, 2, LR - 4, bad);
      ph = interp2<R>(sm.phh, primal_w<R>(a, fx), primal_w<R>(b, fr));
    }
    const R ig = rsqrt1_r((R)1 + px * px + py * py + pz * pz + ph);
    Move<R> mv;
    push_position<R>(g, cw, fx, fr, th, py, pz, px * ig, py * ig, pz * ig, mv);
    if (mv.refl) {
      *elem(P.py, p) = py;
      *elem(P.pz, p) = pz;
    }
    const int reln = mv.ix1 - (int)g.shift;  // (lab columns stay below COL_MAX)
    if ((unsigned)reln >= (unsigned)g.nx) {
      *elem(P.cell, p) = kDead;  // left the window: removed without deposit
      atomicAdd(&sm.tcnt[9], 1);
      continue;
    }
    if (DEFER) {
      scr.cell[p] = cw;
      scr.fx[p] = fx;
      scr.fr[p] = fr;
      scr.th[p] = th;
      scr.w[p] = mv.refl ? -ig : ig;
    } else if constexpr (O == 2) {
      deposit_current2<R, M1>(sm, q, g, mv, w, bad);
    } else {
      deposit_current<R, M1>(sm, q, g, mv, w, bad);
    }
    pst<NT>(elem(P.cell, p), pack_cell(mv.ix1, mv.jr1));
    pst<NT>(elem(P.fx, p), mv.fx1);
    pst<NT>(elem(P.fr, p), mv.fr1);
    pst<NT>(elem(P.th, p), mv.th1);
    if (vacate && reln < 1) {
      if (!DEFER) *elem(P.cell, p) = kDead;  // vacated column: dropped after depositing
      atomicAdd(&sm.tcnt[9], 1);
      continue;
    }
    if (sc.mode == SCAT_CELL) {
      const int sx = clampi(mv.ix1 - (q.T * TX - SORT_EVERY), 0, CR - 1, bad);
      const int sr = clampi(mv.jr1 - (q.tcr * TR - SORT_EVERY), 0, CR - 1, bad);
      atomicAdd(&sm.ccell[sx * CR + sr], 1);
    } else if (sc.mode == SCAT_TILE) {
      // a particle that changes tile (rare) counts for its new tile
      const int tx = mv.ix1 - q.T * TX, tr = mv.jr1 - q.tcr * TR;
      if ((unsigned)tx >= (unsigned)TX || (unsigned)tr >= (unsigned)TR) {
        const int dtx = clampi((tx + TX) / TX - 1, -1, 1, bad);
        const int dtr = clampi((tr + TR) / TR - 1, -1, 1, bad);
        atomicAdd(&sm.tcnt[(dtx + 1) * 3 + dtr + 1], 1);
      } else if (p >= seg_end) {
        // past the segments (an injected column, an overflow range): it joins
        // its tile's segment
        atomicAdd(&sm.tcnt[10], 1);
      }
    }
  }
  if (bad) atomicOr(err, ERR_HALO);
  __syncthreads();
  if (!DEFER) flush_current<R, M1, O>(sm, q, g, jx_out, jr_out, jx1_out, jr1_out, jt1_out);
  if (sc.mode == SCAT_CELL) flush_cells(sm.ccell, q, g, sc.ccount);
  flush_tiles(sm.tcnt, q, g, sc);
}

// ============================= deferred deposits (stage-by-stage API) ==
// chi^n from x^n and the gbar^n kept by a deferred momentum pass
template <class R>
__global__ __launch_bounds__(WG) void k_deposit_chi(Geo g, R* __restrict__ chi_out, Parts<R> P,
                                                    Layout L, const R* __restrict__ gscr, int* err) {
  __shared__ double acc[LN];
  __shared__ R ivol[LR];
  const int item = item_of(blockIdx.x, gridDim.x);
  if (item >= *L.n_items) return;
  const int4 it = L.items[item];
  const Region q = region_of(g, it.x);
  for (int k = threadIdx.x; k < LN; k += WG) acc[k] = 0;
  for (int k = threadIdx.x; k < LR; k += WG) {
    const int j = q.R0 + k;
    ivol[k] = (j >= 0 && j <= g.nr) ? inv_vol_node<R>(g, j) : (R)0;
  }
  __syncthreads();
  bool bad = false;
  for (int k = threadIdx.x; k < it.z + it.w; k += WG) {
    const int p = item_slot(L, it, k);
    const unsigned cw = P.cell[p];
    if (cw == kDead) continue;
    const int a = clampi(cell_ix(cw) - q.X0, 0, LX - 2, bad);
    const int b = clampi(cell_jr(cw) - q.R0, 0, LR - 2, bad);
    const Lin<R> Px = primal_w<R>(a, P.fx[p]), Pr = primal_w<R>(b, P.fr[p]);
    const R wg = P.w[p] / gscr[p];
#pragma unroll
    for (int aa = 0; aa < 2; ++aa)
#pragma unroll
      for (int bb = 0; bb < 2; ++bb)
        lds_add(&acc[(Px.i + aa) * LR + Pr.i + bb], (double)(wg * (aa ? Px.b : Px.a) * (bb ? Pr.b : Pr.a) * ivol[Pr.i + bb]));
  }
  if (bad) atomicOr(err, ERR_HALO);
  __syncthreads();
  for (int k = threadIdx.x; k < LN; k += WG) {
    const R v = (R)acc[k];
    if (v == (R)0) continue;
    const int a = k / LR, b = k - (k / LR) * LR;
    const int rel = q.relX0 + a, j = q.R0 + b;
    if (rel < 0 || rel > g.nx || j < 0 || j > g.nr) continue;
    atomicAdd(&chi_out[(size_t)phys_col(g, rel) * g.pitch + j], v);
  }
}

// J^{n+1/2} from the old positions and gbar kept by a deferred position pass
template <class R, bool M1>
__global__ __launch_bounds__(WG) void k_deposit_J(Geo g, R* __restrict__ jx_out, R* __restrict__ jr_out,
                                                  typename cplx_of<R>::type* __restrict__ jx1_out,
                                                  typename cplx_of<R>::type* __restrict__ jr1_out,
                                                  typename cplx_of<R>::type* __restrict__ jt1_out,
                                                  Parts<R> P, Layout L, int vacate, Parts<R> scr, int* err) {
  __shared__ SmemPos<R, M1> sm;
  const int item = item_of(blockIdx.x, gridDim.x);
  if (item >= *L.n_items) return;
  const int4 it = L.items[item];
  const Region q = region_of(g, it.x);
  stage_pos_constants(sm, q, g);
  zero_pos_acc(sm);
  __syncthreads();
  bool bad = false;
  for (int k = threadIdx.x; k < it.z + it.w; k += WG) {
    const int p = item_slot(L, it, k);
    const unsigned cw = P.cell[p];
    if (cw == kDead) continue;
    const R gm = scr.w[p];
    R py = P.py[p], pz = P.pz[p];
    if (gm < (R)0) {
      // undo the specular reflection of p (an involution about r-hat)
      R s1, c1;
      sincos_r(P.th[p], &s1, &c1);
      const R prad = py * c1 + pz * s1;
      py -= (R)2 * prad * c1;
      pz -= (R)2 * prad * s1;
    }
    const R ig = fabs(gm);
    // replay the push from the kept old position: the same arithmetic as the
    // fused position pass, hence the same move
    Move<R> mv;
    R py2 = py, pz2 = pz;
    push_position<R>(g, scr.cell[p], scr.fx[p], scr.fr[p], scr.th[p], py2, pz2, P.px[p] * ig, py * ig, pz * ig, mv);
    deposit_current<R, M1>(sm, q, g, mv, P.w[p], bad);
    if (vacate && (long long)cell_ix(cw) - g.shift < 1) P.cell[p] = kDead;
  }
  if (bad) atomicOr(err, ERR_HALO);
  __syncthreads();
  flush_current<R, M1, 1>(sm, q, g, jx_out, jr_out, jx1_out, jr1_out, jt1_out);
}

// The copy back of a tile sort whose scan rebuilt the layout, as a launch of
// its own (the deferred-deposit stages, which read the particles before the
// envelope stage that otherwise carries it).
template <class R>
__global__ __launch_bounds__(256) void k_settle(SettleArgs<R> sa) {
  settle_copy(sa, blockIdx.x, gridDim.x);
}

// initial loading of window cells in tile-major order (offsets per tile
// from the host, cells of a tile column-major inside the tile)
template <class R>
__global__ void k_init_particles(Geo g, Plasma pl, Parts<R> P, const int* __restrict__ offsets) {
  const long long cell = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= (long long)g.nx * g.nr) return;
  const int col = (int)(cell / g.nr), j = (int)(cell - (long long)col * g.nr);
  const int T = col / TX, tcr = j / TR;
  const int trt = min(TR, g.nr - tcr * TR);
  const int tct = min(TX, g.nx - T * TX);
  const int key = tile_key(g, col, j);
  const int local = (col - T * TX) * trt + (j - tcr * TR);
  const int ppc = g.ppc_x * g.ppc_r * g.ppc_t;
  for (int k = 0; k < ppc; ++k) load_particle<R>(g, pl, P, offsets[key], local * ppc, tct * trt * ppc, col, j, k);
}

// ====================================================== cell-sort copy ==
// The cell-ordered copy of a cell sort whose layout carries LAYOUT_GATHER:
// slot s of the new layout's work items takes the record of slot inv[s] of
// the buffer in use (the momentum pass wrote inv and updated p there).  One group per item moves one record
// array after the other, so the reads of a group stay within its tile's few
// tens of kilobytes of that array (cached in the L2) and every store is
// contiguous.  A direct scatter of whole records from the momentum pass
// wrote partial cache lines across every array of a tile at once once the
// particles had moved (measured: 2.5x its bytes written, 650 us for the
// cell sort late in the LWFA run).  A slot whose source index is not valid
// (possible only after a count mismatch, which the pass flags) gets a
// removed particle.
template <bool NT, int PPT, class T>
__device__ inline void gather_array(T* __restrict__ to, const T* __restrict__ from, const unsigned* sp, int start,
                                    int count, T none) {
  T v[PPT];
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    const int k = threadIdx.x + u * WG;
    v[u] = (k < count && sp[u] != ~0u) ? *elem(from, (int)sp[u]) : none;
  }
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    const int k = threadIdx.x + u * WG;
    if (k < count) pst<NT>(elem(to, start + k), v[u]);
  }
}
template <class R, bool NT>
__global__ __launch_bounds__(WG) void k_permute(Parts<R> src, Parts<R> dst, Layout L, const unsigned* __restrict__ inv,
                                                long long cap) {
  constexpr int PPT = CHUNK / WG;
  if ((*L.mode & LAYOUT_GATHER) == 0) return;  // the momentum pass scattered the records
  const int item = item_of(blockIdx.x, gridDim.x);
  if (item >= *L.n_items) return;
  const int4 it = L.items[item];
  const int start = it.y, count = it.z;  // count <= chunk <= CHUNK
  unsigned sp[PPT];
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    const int k = threadIdx.x + u * WG;
    const unsigned v = k < count ? *elem(inv, start + k) : ~0u;
    sp[u] = (long long)v < cap ? v : ~0u;
  }
  gather_array<NT, PPT>(dst.cell, src.cell, sp, start, count, kDead);
  gather_array<NT, PPT>(dst.fx, src.fx, sp, start, count, (R)0);
  gather_array<NT, PPT>(dst.fr, src.fr, sp, start, count, (R)0);
  gather_array<NT, PPT>(dst.th, src.th, sp, start, count, (R)0);
  gather_array<NT, PPT>(dst.px, src.px, sp, start, count, (R)0);
  gather_array<NT, PPT>(dst.py, src.py, sp, start, count, (R)0);
  gather_array<NT, PPT>(dst.pz, src.pz, sp, start, count, (R)0);
  gather_array<NT, PPT>(dst.w, src.w, sp, start, count, (R)0);
  gather_array<NT, PPT>(dst.id, src.id, sp, start, count, 0u);
}

// ============================================================ launchers ==
template <class R, bool M1, bool DEFER, int SCAT, int O, bool NT>
static void launch_momentum_k(const Geo& g, const Grids<R>& f, R* chi, const Parts<R>& src, const Parts<R>& dst,
                              const Layout& Ls, const Layout& Ld, int* ccur, R* gscr, unsigned* inv, int* err,
                              int max_items, hipStream_t st, const KEvents& ev) {
  launch_k(k_momentum<R, M1, DEFER, SCAT, O, NT>, dim3(max_items), dim3(WG), st, ev, g, f, chi, src, dst, Ls, Ld,
           ccur, gscr, inv, err);
}
template <class R, bool M1, bool DEFER, int O, bool NT>
static void launch_momentum_nt(const Geo& g, const Grids<R>& f, R* chi, const Parts<R>& src, const Parts<R>& dst,
                               const Layout& Ls, const Layout& Ld, int* ccur, R* gscr, unsigned* inv, int* err,
                               int grid, int scatter, hipStream_t st, const KEvents& ev) {
  if (scatter == SCAT_TILE && DEFER) {
    // the deferred chi deposit reads the particles before the envelope stage
    launch_momentum_k<R, M1, DEFER, SCAT_TILE, O, NT>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, st,
                                                      KEvents{ev.start, nullptr});
    launch_k(k_settle<R>, dim3(SETTLE_BLOCKS), dim3(256), st, KEvents{nullptr, ev.stop},
             SettleArgs<R>{src, dst, Ld, g.cap, SETTLE_BLOCKS});
  } else if (scatter == SCAT_TILE) {
    // (the envelope stage carries the copy back)
    launch_momentum_k<R, M1, DEFER, SCAT_TILE, O, NT>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, st, ev);
  } else if (scatter == SCAT_CELL && !DEFER) {
    // the pass scatters the records, or records their destinations for the
    // gather that follows (the layout scan chose)
    launch_momentum_k<R, M1, DEFER, SCAT_CELL, O, NT>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, st,
                                                      KEvents{ev.start, nullptr});
    launch_k(k_permute<R, NT>, dim3(grid), dim3(WG), st, KEvents{nullptr, ev.stop}, src, dst, Ld,
             (const unsigned*)inv, g.cap);
  } else if (scatter == SCAT_CELL) {
    launch_momentum_k<R, M1, DEFER, SCAT_CELL, O, NT>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, st, ev);
  } else {
    launch_momentum_k<R, M1, DEFER, SCAT_NONE, O, NT>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, st, ev);
  }
}
// non-temporal record access for the fused passes of large runs only
template <class R, bool M1, bool DEFER, int O>
static void launch_momentum_sc(const Geo& g, const Grids<R>& f, R* chi, const Parts<R>& src, const Parts<R>& dst,
                               const Layout& Ls, const Layout& Ld, int* ccur, R* gscr, unsigned* inv, int* err,
                               int grid, int scatter, hipStream_t st, const KEvents& ev) {
  if (!DEFER && g.stream_parts)
    launch_momentum_nt<R, M1, DEFER, O, true>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, scatter, st, ev);
  else
    launch_momentum_nt<R, M1, DEFER, O, false>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, scatter, st, ev);
}

// order 2 has no deferred-deposit variant (the library rejects the request)
template <class R>
void launch_momentum(const Geo& g, const Grids<R>& f, R* chi, const Parts<R>& src, const Parts<R>& dst,
                     const Layout& Ls, const Layout& Ld, int* ccur, R* gscr, unsigned* inv, int* err, int grid,
                     bool defer, int scatter, hipStream_t st, const KEvents& ev) {
  if (grid <= 0) return;
  if (g.order == 2) {
    if (g.modes >= 2)
      launch_momentum_sc<R, true, false, 2>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, scatter, st, ev);
    else
      launch_momentum_sc<R, false, false, 2>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, scatter, st, ev);
  } else if (g.modes >= 2) {
    if (defer)
      launch_momentum_sc<R, true, true, 1>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, scatter, st, ev);
    else
      launch_momentum_sc<R, true, false, 1>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, scatter, st, ev);
  } else {
    if (defer)
      launch_momentum_sc<R, false, true, 1>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, scatter, st, ev);
    else
      launch_momentum_sc<R, false, false, 1>(g, f, chi, src, dst, Ls, Ld, ccur, gscr, inv, err, grid, scatter, st, ev);
  }
}

template <class R> int inject_blocks(const Geo& g) {
  const int n = std::max(g.nr * g.ppc_x * g.ppc_r * g.ppc_t, g.ntr);
  return (n + WG - 1) / WG;
}

template <class R, bool M1, bool DEFER, int O, bool NT>
static void launch_position_nt(const Geo& g, const Grids<R>& f, const DepositBufs<R>& d, const Parts<R>& P,
                               const Layout& L, const SortCounts& sc, int vacate, const Parts<R>& scr, int* err,
                               int max_items, const InjectArgs& inj, hipStream_t st, const KEvents& ev) {
  launch_k(k_position<R, M1, DEFER, O, NT>, dim3(max_items + inj.blocks), dim3(WG), st, ev, g, f, d.jx, d.jr, d.jx1,
           d.jr1, d.jt1, P, L, sc, vacate, scr, err, max_items, inj);
}
template <class R, bool M1, bool DEFER, int O>
static void launch_position_k(const Geo& g, const Grids<R>& f, const DepositBufs<R>& d, const Parts<R>& P,
                              const Layout& L, const SortCounts& sc, int vacate, const Parts<R>& scr, int* err,
                              int grid, const InjectArgs& inj, hipStream_t st, const KEvents& ev) {
  if (!DEFER && g.stream_parts)
    launch_position_nt<R, M1, DEFER, O, true>(g, f, d, P, L, sc, vacate, scr, err, grid, inj, st, ev);
  else
    launch_position_nt<R, M1, DEFER, O, false>(g, f, d, P, L, sc, vacate, scr, err, grid, inj, st, ev);
}

template <class R>
void launch_position(const Geo& g, const Grids<R>& f, const DepositBufs<R>& d, const Parts<R>& P, const Layout& L,
                     const SortCounts& sc, int vacate, const Parts<R>& scr, int* err, int grid, bool defer,
                     const InjectArgs& inj, hipStream_t st, const KEvents& ev) {
  if (grid <= 0) return;
  if (g.order == 2) {
    if (g.modes >= 2)
      launch_position_k<R, true, false, 2>(g, f, d, P, L, sc, vacate, scr, err, grid, inj, st, ev);
    else
      launch_position_k<R, false, false, 2>(g, f, d, P, L, sc, vacate, scr, err, grid, inj, st, ev);
  } else if (g.modes >= 2) {
    if (defer)
      launch_position_k<R, true, true, 1>(g, f, d, P, L, sc, vacate, scr, err, grid, inj, st, ev);
    else
      launch_position_k<R, true, false, 1>(g, f, d, P, L, sc, vacate, scr, err, grid, inj, st, ev);
  } else {
    if (defer)
      launch_position_k<R, false, true, 1>(g, f, d, P, L, sc, vacate, scr, err, grid, inj, st, ev);
    else
      launch_position_k<R, false, false, 1>(g, f, d, P, L, sc, vacate, scr, err, grid, inj, st, ev);
  }
}

template <class R>
void launch_deposit_chi(const Geo& g, R* chi, const Parts<R>& P, const Layout& L, const R* gscr, int* err, int grid,
                        hipStream_t st) {
  if (grid <= 0) return;
  hipLaunchKernelGGL((k_deposit_chi<R>), dim3(grid), dim3(WG), 0, st, g, chi, P, L, gscr, err);
}

template <class R>
void launch_deposit_J(const Geo& g, const DepositBufs<R>& d, const Parts<R>& P, const Layout& L, int vacate,
                      const Parts<R>& scr, int* err, int grid, hipStream_t st) {
  if (grid <= 0) return;
  if (g.modes >= 2)
    hipLaunchKernelGGL((k_deposit_J<R, true>), dim3(grid), dim3(WG), 0, st, g, d.jx, d.jr, d.jx1, d.jr1, d.jt1, P, L, vacate, scr, err);
  else
    hipLaunchKernelGGL((k_deposit_J<R, false>), dim3(grid), dim3(WG), 0, st, g, d.jx, d.jr, d.jx1, d.jr1, d.jt1, P, L, vacate, scr, err);
}

template <class R>
void launch_init_particles(const Geo& g, const Plasma& pl, const Parts<R>& P, const int* offsets, hipStream_t st) {
  const long long cells = (long long)g.nx * g.nr;
  const int grid = (int)((cells + 255) / 256);
  hipLaunchKernelGGL((k_init_particles<R>), dim3(grid), dim3(256), 0, st, g, pl, P, offsets);
}



#define ENVPIC_INST(R)                                                                                          \
  template void launch_momentum<R>(const Geo&, const Grids<R>&, R*, const Parts<R>&, const Parts<R>&,           \
                                   const Layout&, const Layout&, int*, R*, unsigned*, int*, int, bool, int,     \
                                   hipStream_t, const KEvents&);                                                \
  template void launch_position<R>(const Geo&, const Grids<R>&, const DepositBufs<R>&, const Parts<R>&,         \
                                   const Layout&, const SortCounts&, int, const Parts<R>&, int*, int, bool,     \
                                   const InjectArgs&, hipStream_t, const KEvents&);                             \
  template int inject_blocks<R>(const Geo&);                                                                    \
  template void launch_deposit_chi<R>(const Geo&, R*, const Parts<R>&, const Layout&, const R*, int*, int,      \
                                      hipStream_t);                                                             \
  template void launch_deposit_J<R>(const Geo&, const DepositBufs<R>&, const Parts<R>&, const Layout&, int,     \
                                    const Parts<R>&, int*, int, hipStream_t);                                   \
  template void launch_init_particles<R>(const Geo&, const Plasma&, const Parts<R>&, const int*, hipStream_t);
ENVPIC_INST(float)
ENVPIC_INST(double)
#undef ENVPIC_INST

}  // namespace envpic
