// bunch.hip -- self-consistent initial fields of an externally injected
// relativistic electron bunch (arXiv:1912.04674, Sec. 3: the field
// initialisation of external injection carries over to cylindrical
// symmetry).  The bunch moves along x with velocity beta; its potential
// solves the relativistic Poisson equation
//     (1/gamma^2) d2phi/dx2 + (1/r) d/dr (r dphi/dr) = -rho
// on the primal nodes, discretised so that the Gauss law of the field update
// holds exactly:
//     E_x(i+1/2, j) = -(phi_{i+1,j} - phi_{i,j}) / (gamma^2 dx),
//     E_r(i, j+1/2) = -(phi_{i,j+1} - phi_{i,j}) / dr,
//     B_theta(i+1/2, j+1/2) = beta (E_r(i, j+1/2) + E_r(i+1, j+1/2)) / 2,
// with phi = 0 on the x ends and at r_max.  Multiplied by the node volume
// V_j the system K phi = q sum w S is symmetric positive definite:
//     (K phi)_{ij} = V_j/(gamma^2 dx^2) (2 phi_ij - phi_{i-1,j} - phi_{i+1,j})
//                  + A_{j+1/2}/dr (phi_ij - phi_{i,j+1})
//                  + A_{j-1/2}/dr (phi_ij - phi_{i,j-1}),
// A_{j+1/2} = 2 pi (j + 1/2) dr dx, A_{-1/2} = 0, V_0 = pi dr^2 dx / 4.
//
// Solved by conjugate gradients in FP64.  K has constant coefficients along
// x, so sine modes in x turn it into one tridiagonal system in r per mode;
// that exact inverse, carried out in FP32 (FP64 eliminations), is the
// preconditioner: each iteration shrinks the residual by three or more orders
// of magnitude, and FP64 residuals and directions decide the result.  Per
// iteration: z = S T^-1 S r, two products with the (nx - 1)^2 sine matrix
// S on the FP32 matrix cores (its entries looked up in a sine table in LDS,
// never stored) around a cyclic reduction per mode; the new direction
// p = z + beta p; q = K p; x and r.  Partial sums are added in a fixed order,
// so a solve is reproducible up to the order of the charge deposit's atomics.
// The scalars stay on the device; the host reads the residual every iteration.
//   A product costs (nx - 1)^2 nr multiply-adds, 37 to 40 us at 2048 x 256; the
// whole call with 200 000 bunch particles there takes 0.53 ms (3 iterations
// to 1e-12), against 82 ms for 3200 iterations with the diagonal as
// preconditioner (26 us each, launch and reduction latency).  Grids whose
// sine table exceeds the LDS (nx > PRE_NX_MAX) keep the diagonal: there the
// stencil kernel forms the direction p = r/diag + beta p_old on the fly for
// its node and the four neighbours (two direction buffers, swapped by the
// host), and the host reads the residual every CG_CHECK iterations.
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"

namespace envpic {

constexpr int SB = 256;  // threads of the grid kernels

struct CgOp {
  int ni, nj;       // unknowns: interior columns i = 1 .. nx-1, rows j = 0 .. nr-1
  double g2;        // 1 / gamma^2
  double dx, dr;
};

__device__ inline double vol_j(const CgOp& o, int j) {
  const double pi = 3.14159265358979323846;
  return j == 0 ? pi * o.dr * o.dr * o.dx * 0.25 : 2.0 * pi * j * o.dr * o.dr * o.dx;
}
__device__ inline double face_j(const CgOp& o, int j) {  // A_{j+1/2} / dr
  const double pi = 3.14159265358979323846;
  return 2.0 * pi * (j + 0.5) * o.dx;
}
__device__ inline double diag_j(const CgOp& o, int j) {
  const double cx = vol_j(o, j) * o.g2 / (o.dx * o.dx);
  return 2.0 * cx + face_j(o, j) + (j >= 1 ? face_j(o, j - 1) : 0.0);
}

// q sum w S of the particles with id in [id_lo, id_hi) onto the unknowns
// (boundary nodes hold none), with the loop's shape and the axis fold.  A
// bunch is dense (200 000 particles on some 500 cells at 2048 x 256), so
// atomics on its few nodes bound the pass: a work group adds its particles up
// in LDS, on the nodes of its tile and QH around it, and adds the sums to
// memory once (18 us; every term to memory: 209 us).  Q_SPLIT groups share a
// work item, as the bunch has few of them.
constexpr int QH = HALO + 1, QX = TX + 2 * QH + 1, QR = TR + 2 * QH + 1;
constexpr int Q_SPLIT = 4;
template <class R>
__global__ __launch_bounds__(SB) void k_bunch_charge(Geo g, Parts<R> P, Layout L, unsigned id_lo, unsigned id_hi,
                                                     CgOp o, double* __restrict__ rhs) {
  __shared__ double s_q[QX * QR];
  const int item = blockIdx.x;
  if (item >= *L.n_items) return;
  const int4 it = L.items[item];
  const int count = it.z + it.w;
  const int tcx = it.x / g.ntr;
  const int iq = (int)((long long)lab_tile(g, tcx) * TX - g.shift) - QH, jq = (it.x - tcx * g.ntr) * TR - QH;
  for (int q = threadIdx.x; q < QX * QR; q += SB) s_q[q] = 0.0;
  __syncthreads();
  for (int k = blockIdx.y * SB + threadIdx.x; k < count; k += Q_SPLIT * SB) {
    const int p = item_slot(L, it, k);
    const unsigned cw = P.cell[p];
    const unsigned id = P.id[p];
    if (cw == kDead || id < id_lo || id >= id_hi) continue;
    const double ux = (double)((long long)cell_ix(cw) - g.shift) + (double)P.fx[p];
    const double ur = (double)cell_jr(cw) + (double)P.fr[p];
    const double w = -(double)P.w[p];  // q = -1
    int i0, j0;
    double wx[3], wr[3];
    const int n = g.order == 2 ? 3 : 2;
    if (g.order == 2) {
      const double mx = floor(ux + 0.5), dxo = ux - mx, mr = floor(ur + 0.5), dro = ur - mr;
      i0 = (int)mx - 1;
      j0 = (int)mr - 1;
      wx[0] = 0.5 * (0.5 - dxo) * (0.5 - dxo);
      wx[1] = 0.75 - dxo * dxo;
      wx[2] = 0.5 * (0.5 + dxo) * (0.5 + dxo);
      wr[0] = 0.5 * (0.5 - dro) * (0.5 - dro);
      wr[1] = 0.75 - dro * dro;
      wr[2] = 0.5 * (0.5 + dro) * (0.5 + dro);
    } else {
      const double fx0 = floor(ux), fr0 = floor(ur);
      i0 = (int)fx0;
      j0 = (int)fr0;
      wx[0] = 1.0 - (ux - fx0);
      wx[1] = ux - fx0;
      wr[0] = 1.0 - (ur - fr0);
      wr[1] = ur - fr0;
      wx[2] = wr[2] = 0.0;
    }
    const bool near = i0 >= iq && i0 + n <= iq + QX && j0 >= jq && j0 + n <= jq + QR;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        if (a >= n || b >= n) continue;
        const double q = w * wx[a] * wr[b];
        const int i = i0 + a, j = abs(j0 + b);  // below the axis: the mirror row (charge is even)
        if (near)
          atomicAdd(&s_q[(i - iq) * QR + j0 + b - jq], q);
        else if (i >= 1 && i <= o.ni && j < o.nj)
          atomicAdd(&rhs[(size_t)(i - 1) * o.nj + j], q);
      }
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < QX * QR; k += SB) {
    const double q = s_q[k];
    const int i = iq + k / QR, j = abs(jq + k % QR);
    if (q != 0.0 && i >= 1 && i <= o.ni && j < o.nj) atomicAdd(&rhs[(size_t)(i - 1) * o.nj + j], q);
  }
}

template <int N>
__device__ inline void cg_block_sum(double (&v)[N], double* red /* [N][SB] */, double* out) {
  for (int k = 0; k < N; ++k) red[k * SB + threadIdx.x] = v[k];
  __syncthreads();
  for (int s = SB / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s)
      for (int k = 0; k < N; ++k) red[k * SB + threadIdx.x] += red[k * SB + threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x < N) out[(size_t)blockIdx.x * N + threadIdx.x] = red[threadIdx.x * SB];
}

// scalars on the device: [0] r.z, [1] alpha, [2] beta, [3] r.r, [4] b.b
enum { CG_RZ = 0, CG_ALPHA, CG_BETA, CG_RR, CG_BB, CG_RZ2, CG_ZERO };

__global__ __launch_bounds__(SB) void k_cg_zero(double* __restrict__ a, long long n) {
  const long long k = (long long)blockIdx.x * SB + threadIdx.x;
  if (k < n) a[k] = 0.0;
}

// the preconditioner: 1 / diag of each row (the diagonal depends on j only)
__global__ __launch_bounds__(SB) void k_cg_idiag(CgOp o, CgVecs v) {
  const int j = blockIdx.x * SB + threadIdx.x;
  if (j < o.nj) v.idiag[j] = 1.0 / diag_j(o, j);
}

// x = 0, p_old = 0 (so the first direction is z); partial sums of r.z, r.r
__global__ __launch_bounds__(SB) void k_cg_start(CgOp o, CgVecs v) {
  __shared__ double red[2 * SB];
  double s[2] = {0.0, 0.0};
  const long long k = (long long)blockIdx.x * SB + threadIdx.x;
  const long long n = (long long)o.ni * o.nj;
  if (k < n) {
    const int j = (int)(k % o.nj);
    const double r = v.r[k], z = r * v.idiag[j];
    v.x[k] = 0.0;
    v.p[k] = 0.0;
    s[0] = r * z;
    s[1] = r * r;
  }
  cg_block_sum<2>(s, red, v.part);
}

// p_new = r / diag + beta p_old (at the node and its neighbours), q = K p_new;
// partial sums of p_new.q
__global__ __launch_bounds__(SB) void k_cg_apply(CgOp o, CgVecs v, const double* __restrict__ p_old,
                                                 double* __restrict__ p_new) {
  __shared__ double red[SB];
  double s[1] = {0.0};
  const long long k = (long long)blockIdx.x * SB + threadIdx.x;
  const long long n = (long long)o.ni * o.nj;
  const double beta = v.s[CG_BETA];
  if (k < n) {
    const int i = (int)(k / o.nj), j = (int)(k - (long long)i * o.nj);
    auto dir = [&](long long m, int jj) { return v.r[m] * v.idiag[jj] + beta * p_old[m]; };
    const double pc = dir(k, j);
    const double cx = vol_j(o, j) * o.g2 / (o.dx * o.dx);
    const double pl = i > 0 ? dir(k - o.nj, j) : 0.0, pr = i < o.ni - 1 ? dir(k + o.nj, j) : 0.0;
    const double pu = j < o.nj - 1 ? dir(k + 1, j + 1) : 0.0, pd = j > 0 ? dir(k - 1, j - 1) : 0.0;
    double q = cx * (2.0 * pc - pl - pr) + face_j(o, j) * (pc - pu);
    if (j > 0) q += face_j(o, j - 1) * (pc - pd);
    p_new[k] = pc;
    v.q[k] = q;
    s[0] = pc * q;
  }
  cg_block_sum<1>(s, red, v.part);
}

// fixed-order sum of NQ partial sums per block into sums[0 .. NQ)
template <int NQ>
__device__ inline void cg_sum_parts(const double* part, int nb, double* sums) {
  __shared__ double lanes[NQ][256];
  const int l = threadIdx.x;
  for (int q = 0; q < NQ; ++q) {
    double s = 0.0;
    for (int b = l; b < nb; b += 256) s += part[(size_t)b * NQ + q];
    lanes[q][l] = s;
  }
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (l < h)
      for (int q = 0; q < NQ; ++q) lanes[q][l] += lanes[q][l + h];
    __syncthreads();
  }
  if (l == 0)
    for (int q = 0; q < NQ; ++q) sums[q] = lanes[q][0];
}

// after k_cg_start: r.z, r.r and b.b (= r.r at the start)
__global__ __launch_bounds__(256) void k_cg_init_scalars(int nb, CgVecs v) {
  __shared__ double t[2];
  cg_sum_parts<2>(v.part, nb, t);
  if (threadIdx.x == 0) {
    v.s[CG_RZ] = t[0];
    v.s[CG_RR] = t[1];
    v.s[CG_BB] = t[1];
    v.s[CG_BETA] = 0.0;
    v.s[CG_ZERO] = 0.0;
  }
}

// alpha = r.z / p.Kp
__global__ __launch_bounds__(256) void k_cg_alpha(int nb, CgVecs v) {
  __shared__ double t[1];
  cg_sum_parts<1>(v.part, nb, t);
  if (threadIdx.x == 0) v.s[CG_ALPHA] = t[0] != 0.0 ? v.s[CG_RZ] / t[0] : 0.0;
}

// x += alpha p, r -= alpha q; partial sums of r.z (z = r / diag) and r.r
__global__ __launch_bounds__(SB) void k_cg_update(CgOp o, CgVecs v, const double* __restrict__ p) {
  __shared__ double red[2 * SB];
  double s[2] = {0.0, 0.0};
  const long long k = (long long)blockIdx.x * SB + threadIdx.x;
  const long long n = (long long)o.ni * o.nj;
  const double alpha = v.s[CG_ALPHA];
  if (k < n) {
    const int j = (int)(k % o.nj);
    v.x[k] += alpha * p[k];
    const double r = v.r[k] - alpha * v.q[k];
    v.r[k] = r;
    s[0] = r * (r * v.idiag[j]);
    s[1] = r * r;
  }
  cg_block_sum<2>(s, red, v.part);
}

// beta = r.z(new) / r.z(old)
__global__ __launch_bounds__(256) void k_cg_beta(int nb, CgVecs v) {
  __shared__ double t[2];
  cg_sum_parts<2>(v.part, nb, t);
  if (threadIdx.x == 0) {
    v.s[CG_BETA] = v.s[CG_RZ] != 0.0 ? t[0] / v.s[CG_RZ] : 0.0;
    v.s[CG_RZ] = t[0];
    v.s[CG_RR] = t[1];
  }
}

// ------------------------------------------- sine-mode preconditioner --
// sin(pi t / nx), t = 0 .. 2 nx - 1
__global__ __launch_bounds__(SB) void k_sine_table(int nx, float* __restrict__ table) {
  const int t = blockIdx.x * SB + threadIdx.x;
  if (t < 2 * nx) table[t] = (float)sinpi((double)t / nx);
}

using f32x16 = __attribute__((__vector_size__(16 * sizeof(float)))) float;
constexpr int DT_M = 64, DT_N = 32;  // modes (or columns) and rows of a work group's tile
constexpr int DT_K = 16;             // columns per trip of a wavefront's loop
constexpr int DT_P = 8;              // wavefronts that share a 32 x 32 half, each with its stretches of columns
constexpr int DT_T = 2 * DT_P * 64;  // threads
// LDS of a work group: the sine table, then the wavefronts' sums in its place
inline size_t dst_lds(int nx) {
  return std::max(2 * (size_t)nx * sizeof(float), (size_t)2 * (DT_P - 1) * 16 * 64 * sizeof(float));
}

// out[m][j] = scale * sum_k sin(pi (m+1)(k+1) / nx) in[k][j] over the n = nx - 1
// columns k: a matrix product on the FP32 matrix cores.  A work group owns a
// 64 x 32 tile (one group per CU at 2048 x 256) and its two 32 x 32 halves are
// shared by eight wavefronts each, which take alternate stretches of 16
// columns (their sums are added through LDS in a fixed order): the loads of
// `in` come out of the L2 and a single wavefront per SIMD would wait for each
// stretch (168 us so at 2048 x 256, the matrix cores' time is 14; 37 us with
// four and the next stretch's loads issued a trip ahead; pad words against
// bank conflicts of the table reads gave nothing).  A lane's operands:
// row m = lane % 32 and k = lane / 32 of S, column j = lane % 32 and the same
// k of `in`; the table index (m+1)(k+1) mod 2 nx advances by 2 (m+1) per
// product.  The FP64 input is the residual, divided by its norm so that it
// stays in FP32's range whatever the charge's size (rr: its square).  DOT:
// also the partial sums of r . out, out taken times that norm, one per work
// group, in part[2 b].
template <class T, bool DOT>
__global__ __launch_bounds__(DT_T) void k_dst(int nx, int nj, const float* __restrict__ table,
                                              const T* __restrict__ in, float* __restrict__ out, float scale,
                                              const double* __restrict__ rr, const double* __restrict__ r,
                                              double* __restrict__ part) {
  extern __shared__ float s_tab[];  // [2 nx], then the sums of the wavefronts but the first of each half
  __shared__ double s_dot[2];
  const int n = nx - 1, two = 2 * nx;
  for (int t = threadIdx.x; t < two; t += DT_T) s_tab[t] = table[t];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = wave & 1, part_k = wave >> 1;
  const int l32 = lane & 31, lk = lane >> 5;
  const int m = blockIdx.x * DT_M + half * 32 + l32;  // (rows past the end are computed and not stored)
  const int j = blockIdx.y * DT_N + l32;
  const unsigned jc = min(j, nj - 1), off = lk * nj + jc;
  const int m1 = min(m, n - 1) + 1;
  const unsigned step = 2 * m1;                                             // < 2 nx
  const unsigned skip = ((long long)(DT_P - 1) * DT_K * m1) % two;          // over the other wavefronts' stretches
  unsigned idx = (unsigned)(((long long)m1 * (part_k * DT_K + lk + 1)) % two);
  const double norm = sqrt(*rr);
  const T unit = sizeof(T) == 8 ? (T)(1.0 / norm) : (T)1;
  const auto load = [&](int k0, T(&b)[DT_K / 2]) {
    if (k0 + DT_K <= n) {
      const T* at = in + (size_t)k0 * nj;
#pragma unroll
      for (int u = 0; u < DT_K / 2; ++u) b[u] = (at + (size_t)2 * u * nj)[off];
    } else {
#pragma unroll
      for (int u = 0; u < DT_K / 2; ++u) {
        const int k = k0 + 2 * u + lk;
        const T v = in[(size_t)min(k, n - 1) * nj + jc];
        b[u] = k < n ? v : (T)0;
      }
    }
  };
  T b[DT_K / 2];
  load(part_k * DT_K, b);
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
  __syncthreads();
  for (int k0 = part_k * DT_K; k0 < n; k0 += DT_P * DT_K) {
    float a[DT_K / 2], bv[DT_K / 2];
#pragma unroll
    for (int u = 0; u < DT_K / 2; ++u) {
      bv[u] = (float)(b[u] * unit);
      a[u] = s_tab[idx];
      idx += step;
      idx = min(idx, idx - two);  // (unsigned: the smaller is the one in range)
    }
    idx += skip;
    idx = min(idx, idx - two);
    if (k0 + DT_P * DT_K < n) load(k0 + DT_P * DT_K, b);
#pragma unroll
    for (int u = 0; u < DT_K / 2; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u], bv[u], acc, 0, 0, 0);
  }
  __syncthreads();
  float* s_sum = s_tab + (size_t)half * (DT_P - 1) * 16 * 64 + lane;
  if (part_k > 0)
#pragma unroll
    for (int e = 0; e < 16; ++e) s_sum[((part_k - 1) * 16 + e) * 64] = acc[e];
  __syncthreads();
  double dot = 0.0;
  if (part_k == 0) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      // element e of a lane: row 8 (e / 4) + 4 (lane / 32) + e % 4, column lane % 32
      const int row = blockIdx.x * DT_M + half * 32 + 8 * (e >> 2) + 4 * lk + (e & 3);
      float v = acc[e];
      for (int q = 0; q < DT_P - 1; ++q) v += s_sum[(q * 16 + e) * 64];
      if (row < n && j < nj) {
        v *= scale;
        const size_t o = (size_t)row * nj + j;
        out[o] = v;
        if (DOT) dot += r[o] * (double)v;
      }
    }
  }
  if constexpr (DOT) {
    for (int o = 32; o >= 1; o >>= 1) dot += __shfl_xor(dot, o, 64);
    if (part_k == 0 && lane == 0) s_dot[half] = dot * norm;
    __syncthreads();
    if (threadIdx.x == 0) {
      double* p = part + 2 * (size_t)(blockIdx.y * gridDim.x + blockIdx.x);
      p[0] = s_dot[0] + s_dot[1];
      p[1] = 0.0;
    }
  }
}

// The radial system of sine mode m, (lambda_m V_j + radial operator) y = f, by
// parallel cyclic reduction in FP64: one work group per mode, its row read
// and overwritten.  Each sweep eliminates the neighbours at distance s (the
// rows kept scaled to a unit diagonal), for s = 1, 2, 4, ... nj.
__global__ __launch_bounds__(SB) void k_modes_solve(CgOp o, float* __restrict__ f) {
  extern __shared__ double s_row[];  // a, c, d of the row's nj unknowns
  const int nj = o.nj, m = blockIdx.x;
  double *a = s_row, *c = a + nj, *d = c + nj;
  float* row = f + (size_t)m * nj;
  const double pi = 3.14159265358979323846;
  const double sh = sin(0.5 * pi * (m + 1) / (o.ni + 1));
  const double lam = 4.0 * sh * sh * o.g2 / (o.dx * o.dx);
  constexpr int PT = (PRE_NJ_MAX + SB - 1) / SB;  // unknowns per thread at most
  for (int j = threadIdx.x; j < nj; j += SB) {
    const double up = face_j(o, j), dn = j > 0 ? face_j(o, j - 1) : 0.0;
    const double ib = 1.0 / (lam * vol_j(o, j) + up + dn);
    a[j] = -dn * ib;
    c[j] = j + 1 < nj ? -up * ib : 0.0;  // (phi = 0 at r_max)
    d[j] = (double)row[j] * ib;
  }
  __syncthreads();
  for (int s = 1; s < nj; s *= 2) {
    double na[PT], nc[PT], nd[PT];
    int u = 0;
    for (int j = threadIdx.x; j < nj; j += SB, ++u) {
      const bool lo = j >= s, hi = j + s < nj;
      const double aj = a[j], cj = c[j];
      const double al = lo ? a[j - s] : 0.0, cl = lo ? c[j - s] : 0.0, dl = lo ? d[j - s] : 0.0;
      const double ah = hi ? a[j + s] : 0.0, ch = hi ? c[j + s] : 0.0, dh = hi ? d[j + s] : 0.0;
      const double ib = 1.0 / (1.0 - aj * cl - cj * ah);
      na[u] = -aj * al * ib;
      nc[u] = -cj * ch * ib;
      nd[u] = (d[j] - aj * dl - cj * dh) * ib;
    }
    __syncthreads();
    u = 0;
    for (int j = threadIdx.x; j < nj; j += SB, ++u) {
      a[j] = na[u];
      c[j] = nc[u];
      d[j] = nd[u];
    }
    __syncthreads();
  }
  for (int j = threadIdx.x; j < nj; j += SB) row[j] = (float)d[j];
}

// The vector kernels run PCG_BLOCKS groups at most, so that each group of the
// kernel that needs a sum adds up the partial sums by itself (in the same
// order): a launch of its own for that costs as much as the kernel.
constexpr int PCG_BLOCKS = 512;
static_assert(SB == 256, "cg_sum_parts is written for 256 threads");

// beta = r.z / r.z of the iteration before (rz[0], 0 in the first); p =
// |r| z + beta p (z was taken of r / |r|); this iteration's r.z to rz[1]
__global__ __launch_bounds__(SB) void k_pcg_direction(long long n, int np, CgVecs v, const float* __restrict__ z,
                                                      const double* __restrict__ rz_old, double* __restrict__ rz_new) {
  __shared__ double t[2];
  cg_sum_parts<2>(v.part, np, t);
  __syncthreads();
  const double old = *rz_old, norm = sqrt(v.s[CG_RR]);
  const double beta = old == 0.0 ? 0.0 : t[0] / old;
  if (blockIdx.x == 0 && threadIdx.x == 0) *rz_new = t[0];
  for (long long k = (long long)blockIdx.x * SB + threadIdx.x; k < n; k += (long long)gridDim.x * SB)
    v.p[k] = norm * (double)z[k] + (beta == 0.0 ? 0.0 : beta * v.p[k]);
}

// q = K p; partial sums of p.q
__global__ __launch_bounds__(SB) void k_pcg_apply(CgOp o, CgVecs v) {
  __shared__ double red[SB];
  double s[1] = {0.0};
  const double* p = v.p;
  for (long long k = (long long)blockIdx.x * SB + threadIdx.x; k < (long long)o.ni * o.nj;
       k += (long long)gridDim.x * SB) {
    const int i = (int)(k / o.nj), j = (int)(k - (long long)i * o.nj);
    const double pc = p[k];
    const double cx = vol_j(o, j) * o.g2 / (o.dx * o.dx);
    const double pl = i > 0 ? p[k - o.nj] : 0.0, pr = i < o.ni - 1 ? p[k + o.nj] : 0.0;
    const double pu = j < o.nj - 1 ? p[k + 1] : 0.0, pd = j > 0 ? p[k - 1] : 0.0;
    double q = cx * (2.0 * pc - pl - pr) + face_j(o, j) * (pc - pu);
    if (j > 0) q += face_j(o, j - 1) * (pc - pd);
    v.q[k] = q;
    s[0] += pc * q;
  }
  cg_block_sum<1>(s, red, v.part);
}

// alpha = r.z / p.q; x and r; partial sums of r.r in part[PCG_BLOCKS + b]
__global__ __launch_bounds__(SB) void k_pcg_update(long long n, CgVecs v, const double* __restrict__ rz) {
  __shared__ double red[SB];
  __shared__ double t[1];
  cg_sum_parts<1>(v.part, gridDim.x, t);
  __syncthreads();
  const double alpha = t[0] != 0.0 ? *rz / t[0] : 0.0;
  double s[1] = {0.0};
  for (long long k = (long long)blockIdx.x * SB + threadIdx.x; k < n; k += (long long)gridDim.x * SB) {
    v.x[k] += alpha * v.p[k];
    const double r = v.r[k] - alpha * v.q[k];
    v.r[k] = r;
    s[0] += r * r;
  }
  cg_block_sum<1>(s, red, v.part + PCG_BLOCKS);
}

// r.r of the update's partial sums
__global__ __launch_bounds__(256) void k_pcg_residual(int nb, CgVecs v) {
  __shared__ double t[1];
  cg_sum_parts<1>(v.part + PCG_BLOCKS, nb, t);
  if (threadIdx.x == 0) v.s[CG_RR] = t[0];
}

// E_x, E_r, B_theta (and Bbar_theta) of phi, added to the mode-0 grids
template <class R>
__global__ __launch_bounds__(SB) void k_bunch_fields(Geo g, Grids<R> f, CgOp o, double beta, CgVecs v) {
  const long long k = (long long)blockIdx.x * SB + threadIdx.x;
  const int nr1 = g.nr + 1;
  if (k >= (long long)(g.nx + 1) * nr1) return;
  const int i = (int)(k / nr1), j = (int)(k - (long long)i * nr1);
  auto phi = [&](int a, int b) -> double {  // zero on the x ends and at r_max
    if (a < 1 || a > o.ni || b < 0 || b >= o.nj) return 0.0;
    return v.x[(size_t)(a - 1) * o.nj + b];
  };
  const size_t at = (size_t)phys_col(g, i) * g.pitch + j;
  if (i <= g.nx - 1) {
    const double ex = -(phi(i + 1, j) - phi(i, j)) * o.g2 / o.dx;
    f.ex[at] = (R)((double)f.ex[at] + ex);
  }
  if (j <= g.nr - 1) {
    const double er = -(phi(i, j + 1) - phi(i, j)) / o.dr;
    f.er[at] = (R)((double)f.er[at] + er);
    if (i <= g.nx - 1) {
      const double er1 = -(phi(i + 1, j + 1) - phi(i + 1, j)) / o.dr;
      const double bt = beta * 0.5 * (er + er1);
      f.bt[at] = (R)((double)f.bt[at] + bt);
      f.btb[at] = (R)((double)f.btb[at] + bt);
    }
  }
}

long long cg_unknowns(int nx, int nr) { return (long long)(nx - 1) * nr; }
// the sine modes' sums: one per tile of the products
static int dst_tiles(int nx, int nr) { return ((nx - 1 + DT_M - 1) / DT_M) * ((nr + DT_N - 1) / DT_N); }
int cg_blocks(int nx, int nr) {
  return (int)std::max({(cg_unknowns(nx, nr) + SB - 1) / SB, (long long)dst_tiles(nx, nr), (long long)PCG_BLOCKS});
}
bool cg_sine_modes(int nx, int nr) { return nx <= PRE_NX_MAX && nr <= PRE_NJ_MAX; }

// The iterations with the sine-mode preconditioner from x = 0, r = b (whose
// square is bb); z and the modes share the second direction buffer.
static int solve_sine_modes(const CgOp& o, const CgVecs& v, double bb, double tol, int max_iter, hipStream_t st,
                            int* iters, double* rr_out) {
  const int nx = o.ni + 1;
  const long long n = (long long)o.ni * o.nj;
  const int nb = (int)std::min<long long>((n + SB - 1) / SB, PCG_BLOCKS);
  float* modes = reinterpret_cast<float*>(v.p2);
  float* z = modes + n;
  const dim3 grid((o.ni + DT_M - 1) / DT_M, (o.nj + DT_N - 1) / DT_N);
  const size_t lds_dst = dst_lds(nx), lds_row = 3 * (size_t)o.nj * sizeof(double);
  if (hipFuncSetAttribute((const void*)k_dst<double, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)lds_dst) != hipSuccess ||
      hipFuncSetAttribute((const void*)k_dst<float, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)lds_dst) != hipSuccess ||
      hipFuncSetAttribute((const void*)k_modes_solve, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_row) !=
          hipSuccess)
    return -1;
  hipLaunchKernelGGL(k_sine_table, dim3((2 * nx + SB - 1) / SB), dim3(SB), 0, st, nx, v.sine);
  const double stop = tol * tol * bb;
  double rr = bb, hs[CG_NS];
  int it = 0;
  while (it < max_iter && rr > stop) {
    hipLaunchKernelGGL((k_dst<double, false>), grid, dim3(DT_T), lds_dst, st, nx, o.nj, v.sine, v.r, modes, 1.0f,
                       v.s + CG_RR, nullptr, nullptr);
    hipLaunchKernelGGL(k_modes_solve, dim3(o.ni), dim3(SB), lds_row, st, o, modes);
    hipLaunchKernelGGL((k_dst<float, true>), grid, dim3(DT_T), lds_dst, st, nx, o.nj, v.sine, modes, z, 2.0f / nx,
                       v.s + CG_RR, v.r, v.part);
    double *rz = v.s + (it & 1 ? CG_RZ2 : CG_RZ), *rz_old = v.s + (it == 0 ? CG_ZERO : it & 1 ? CG_RZ : CG_RZ2);
    hipLaunchKernelGGL(k_pcg_direction, dim3(nb), dim3(SB), 0, st, n, (int)(grid.x * grid.y), v, z, rz_old, rz);
    hipLaunchKernelGGL(k_pcg_apply, dim3(nb), dim3(SB), 0, st, o, v);
    hipLaunchKernelGGL(k_pcg_update, dim3(nb), dim3(SB), 0, st, n, v, rz);
    hipLaunchKernelGGL(k_pcg_residual, dim3(1), dim3(256), 0, st, nb, v);
    ++it;
    if (hipMemcpyAsync(hs, v.s, sizeof(hs), hipMemcpyDeviceToHost, st) != hipSuccess) return -1;
    if (hipStreamSynchronize(st) != hipSuccess) return -1;
    rr = hs[CG_RR];
    if (!(rr == rr)) break;  // not a number: no iteration will bring it back
  }
  *iters = it;
  *rr_out = rr;
  return 0;
}

// the iterations with the diagonal as preconditioner
static int solve_diagonal(const CgOp& o, const CgVecs& v, double bb, double tol, int max_iter, hipStream_t st,
                          int* iters, double* rr_out) {
  const int nb = (int)(((long long)o.ni * o.nj + SB - 1) / SB);
  double rr = bb, hs[CG_NS];
  int it = 0;
  const double stop = tol * tol * bb;
  double* pa = v.p;   // direction of the previous iteration (zero at the start)
  double* pb = v.p2;  // the new one
  while (it < max_iter && rr > stop) {
    const int burst = std::min(CG_CHECK, max_iter - it);
    for (int k = 0; k < burst; ++k) {
      hipLaunchKernelGGL(k_cg_apply, dim3(nb), dim3(SB), 0, st, o, v, pa, pb);
      hipLaunchKernelGGL(k_cg_alpha, dim3(1), dim3(256), 0, st, nb, v);
      hipLaunchKernelGGL(k_cg_update, dim3(nb), dim3(SB), 0, st, o, v, pb);
      hipLaunchKernelGGL(k_cg_beta, dim3(1), dim3(256), 0, st, nb, v);
      std::swap(pa, pb);
    }
    it += burst;
    if (hipMemcpyAsync(hs, v.s, sizeof(hs), hipMemcpyDeviceToHost, st) != hipSuccess) return -1;
    if (hipStreamSynchronize(st) != hipSuccess) return -1;
    rr = hs[CG_RR];
  }
  *iters = it;
  *rr_out = rr;
  return 0;
}

template <class R>
int bunch_solve(const Geo& g, const Parts<R>& P, const Layout& L, int max_items, const Grids<R>& f,
                unsigned id_lo, unsigned id_hi, double beta, double tol, int max_iter, const CgVecs& v,
                hipStream_t st, int* iters, double* resid) {
  CgOp o;
  o.ni = g.nx - 1;
  o.nj = g.nr;
  o.g2 = 1.0 - beta * beta;
  o.dx = g.dx;
  o.dr = g.dr;
  const long long n = cg_unknowns(g.nx, g.nr);
  const int nb = (int)((n + SB - 1) / SB);
  hipLaunchKernelGGL(k_cg_zero, dim3(nb), dim3(SB), 0, st, v.r, n);
  hipLaunchKernelGGL(k_cg_idiag, dim3((o.nj + SB - 1) / SB), dim3(SB), 0, st, o, v);
  hipLaunchKernelGGL((k_bunch_charge<R>), dim3(max_items, Q_SPLIT), dim3(SB), 0, st, g, P, L, id_lo, id_hi, o, v.r);
  hipLaunchKernelGGL(k_cg_start, dim3(nb), dim3(SB), 0, st, o, v);
  hipLaunchKernelGGL(k_cg_init_scalars, dim3(1), dim3(256), 0, st, nb, v);
  double hs[CG_NS];
  if (hipMemcpyAsync(hs, v.s, sizeof(hs), hipMemcpyDeviceToHost, st) != hipSuccess) return -1;
  if (hipStreamSynchronize(st) != hipSuccess) return -1;
  const double bb = hs[CG_BB];
  *iters = 0;
  *resid = 0.0;
  if (bb == 0.0) return 0;  // no charge: nothing to add (x = 0)
  int it = 0;
  double rr = bb;
  if (cg_sine_modes(g.nx, g.nr)) {
    if (solve_sine_modes(o, v, bb, tol, max_iter, st, &it, &rr)) return -1;
  } else if (solve_diagonal(o, v, bb, tol, max_iter, st, &it, &rr)) {
    return -1;
  }
  *iters = it;
  *resid = std::sqrt(rr / bb);
  const long long nodes = (long long)(g.nx + 1) * (g.nr + 1);
  hipLaunchKernelGGL((k_bunch_fields<R>), dim3((unsigned)((nodes + SB - 1) / SB)), dim3(SB), 0, st, g, f, o, beta, v);
  return 0;
}

template int bunch_solve<float>(const Geo&, const Parts<float>&, const Layout&, int, const Grids<float>&, unsigned,
                                unsigned, double, double, int, const CgVecs&, hipStream_t, int*, double*);
template int bunch_solve<double>(const Geo&, const Parts<double>&, const Layout&, int, const Grids<double>&,
                                 unsigned, unsigned, double, double, int, const CgVecs&, hipStream_t, int*, double*);

}  // namespace envpic
