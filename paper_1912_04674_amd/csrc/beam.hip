// beam.hip -- injected-beam parameters of the particle set (Sec. 4, Table
// BeamParams of arXiv:1912.04674): peak of the electron energy spectrum,
// beam charge, relative energy spread and normalized transverse emittance
// sqrt(s_xx s_pp - s_xp^2), over the particles within two FWHM widths in
// energy around the spectrum peak.
//
// Definitions (the table gives the quantities only):
//   energy     gamma - 1 = |p|^2 / (1 + sqrt(1 + |p|^2)) of the momentum, FP64;
//   spectrum   charge histogram sum |q| w over nbins equal bins of
//              [e_lo, e_hi), summed as 64-bit fixed point (exact and
//              independent of the order of the atomics);
//   peak       the fullest bin (lowest on a tie), energy at its centre;
//   FWHM       first bin below half maximum on each side of the peak, the
//              crossing interpolated between bin centres; a side that stays
//              above ends at the range edge;
//   window     [E_peak - FWHM, E_peak + FWHM] within [e_lo, e_hi);
//   moments    weighted by w, centred (a pass for the means, one for the
//              second moments), FP64 tree sums per work item, then a
//              fixed-order sum over the items.
//
// Seven launches on the simulation's stream: clear; histogram (one work group
// per work item, LDS histogram flushed with integer atomics), which also
// leaves a bit per particle that lies in the range; peak (one work group); and
// for each moment pass a kernel per item, which reads only the particles
// whose bit is set, and a one-group fixed-order reduction.  The range is
// meant to hold a beam out of a plasma, so the moment passes are short (18 and
// 14 us where 1.4 % of 8.4 M particles are in range, latency; 48 and 47 when
// they read every record), and the histogram, bound by its 168 MB (28 us at
// the rate of a large copy), takes 29 to 31 us (43 before its loads were
// issued turns ahead).
#include <algorithm>

#include "common.hpp"
#include "elem.hpp"
#include "envpic.h"
#include "launch.hpp"

// the energy, bin and moment arithmetic is written out term by term; keep
// the compiler from fusing it into FMAs so the rounding is that of the
// expressions as written
#pragma clang fp contract(off)

namespace envpic {

constexpr int BG = 256;      // threads of the histogram kernel's groups
constexpr int BM = 512;      // threads of the moment kernels' groups
// Their groups: as many as the device holds at once, each taking every
// MOMENT_GROUPS-th item.  Most items hold no particle in range, and a group
// per item the layout may have costs 2 ns each to dispatch: 18 and 14 us instead
// of 21 and 16 (and 21 and 18 with 512 groups of 1024 threads).
constexpr int MOMENT_GROUPS = 1024;
constexpr int BPK = 1024;    // threads of the peak kernel
constexpr int NBM = BEAM_PARTS;  // partial sums per item in each moment pass

__device__ inline double kin_energy(double px, double py, double pz) {
  const double p2 = px * px + py * py + pz * pz;
  return p2 / (1.0 + sqrt(1.0 + p2));
}

__device__ inline int energy_bin(const BeamArgs& a, double e) {
  if (!(e >= a.e_lo && e < a.e_hi)) return -1;
  int k = (int)floor((e - a.e_lo) / a.de);
  return k < a.nbins - 1 ? k : a.nbins - 1;
}

__global__ __launch_bounds__(BG) void k_beam_clear(BeamScratch b, int nbins) {
  const int k = blockIdx.x * BG + threadIdx.x;
  if (k < nbins) b.hist[k] = 0;
  if (k < BEAM_STATE) b.st[k] = 0.0;
}

// The loads of BU turns are issued before any is used.  e <= p^2 / 2 (and
// half a part in 10^7 of room for the rounding) settles a particle below the
// range, which is most of a plasma, without the square root and the division.
constexpr int BU = 4;
template <class R>
__global__ __launch_bounds__(BG) void k_beam_hist(Parts<R> P, Layout L, BeamArgs a, BeamScratch b) {
  extern __shared__ long long h[];  // [nbins]
  const int item = blockIdx.x;
  if (item >= *L.n_items) return;
  for (int k = threadIdx.x; k < a.nbins; k += BG) h[k] = 0;
  __syncthreads();
  const int4 it = L.items[item];
  const int total = it.z + it.w;
  unsigned long long* bits = b.bits + (size_t)item * b.item_words;
  for (int k0 = 0; k0 < total; k0 += BU * BG) {
    unsigned cw[BU];
    R px[BU], py[BU], pz[BU], w[BU];
#pragma unroll
    for (int u = 0; u < BU; ++u) {
      const int p = item_slot(L, it, min(k0 + u * BG + (int)threadIdx.x, total - 1));
      cw[u] = P.cell[p];
      px[u] = P.px[p];
      py[u] = P.py[p];
      pz[u] = P.pz[p];
      w[u] = P.w[p];
    }
#pragma unroll
    for (int u = 0; u < BU; ++u) {
      const int k = k0 + u * BG + (int)threadIdx.x;
      const double x = (double)px[u], y = (double)py[u], z = (double)pz[u];
      int bin = -1;
      // (a momentum that is not a number takes the branch and no bin)
      if (k < total && cw[u] != kDead && !((x * x + y * y + z * z) * 0.50000005 < a.e_lo))
        bin = energy_bin(a, kin_energy(x, y, z));
      const unsigned long long in = __ballot(bin >= 0);
      if ((threadIdx.x & 63) == 0 && k < total) bits[k >> 6] = in;
      if (bin < 0) continue;
      // |q| w in fixed point (q = -1): the scale keeps every sum below 2^62
      const long long c = __double2ll_rn((double)w[u] * a.scale);
      atomicAdd((unsigned long long*)&h[bin], (unsigned long long)c);
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < a.nbins; k += BG)
    if (h[k] != 0) atomicAdd((unsigned long long*)&b.hist[k], (unsigned long long)h[k]);
}

// block reductions of the peak kernel
__device__ inline void argmax_block(long long v, int k, long long* sv, int* sk) {
  // value, then the lower index on a tie
  sv[threadIdx.x] = v;
  sk[threadIdx.x] = k;
  __syncthreads();
  for (int s = BPK / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      const long long v2 = sv[threadIdx.x + s];
      const int k2 = sk[threadIdx.x + s];
      if (v2 > sv[threadIdx.x] || (v2 == sv[threadIdx.x] && k2 < sk[threadIdx.x])) {
        sv[threadIdx.x] = v2;
        sk[threadIdx.x] = k2;
      }
    }
    __syncthreads();
  }
}
__device__ inline int reduce_idx(int k, bool take_max, int* sk) {
  sk[threadIdx.x] = k;
  __syncthreads();
  for (int s = BPK / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      const int k2 = sk[threadIdx.x + s];
      if (take_max ? k2 > sk[threadIdx.x] : k2 < sk[threadIdx.x]) sk[threadIdx.x] = k2;
    }
    __syncthreads();
  }
  const int r = sk[0];
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(BPK) void k_beam_peak(BeamArgs a, BeamScratch b) {
  __shared__ long long sv[BPK];
  __shared__ int sk[BPK];
  const int n = a.nbins;
  // the fullest bin, lowest index on a tie
  long long best = -1;
  int kbest = n;
  for (int k = threadIdx.x; k < n; k += BPK) {
    const long long v = (long long)b.hist[k];
    if (v > best) {  // strided in increasing k: the first of equal values stays
      best = v;
      kbest = k;
    }
  }
  argmax_block(best, kbest, sv, sk);
  const long long hmax = sv[0];
  const int kp = sk[0];
  __syncthreads();
  const double inv = 1.0 / a.scale;
  for (int k = threadIdx.x; k < n; k += BPK) b.hist_f[k] = (double)(long long)b.hist[k] * inv;
  if (hmax <= 0) {  // empty spectrum: nothing is selected, every output is zero
    if (threadIdx.x == 0) {
      b.st[BS_NONEMPTY] = 0.0;
      b.st[BS_LO] = 1.0;
      b.st[BS_HI] = -1.0;
    }
    return;
  }
  // first bin below half maximum on each side (2 H < H_max, exact integers)
  int kl = -1, kr = n;
  for (int k = threadIdx.x; k < n; k += BPK) {
    const bool below = 2 * (long long)b.hist[k] < hmax;
    if (below && k < kp && k > kl) kl = k;
    if (below && k > kp && k < kr) kr = k;
  }
  kl = reduce_idx(kl, true, sk);
  kr = reduce_idx(kr, false, sk);
  if (threadIdx.x == 0) {
    const double h = (double)hmax * inv, half = 0.5 * h;
    const double e_peak = a.e_lo + (kp + 0.5) * a.de;
    double left = a.e_lo, right = a.e_hi;
    if (kl >= 0) {
      const double hl = (double)(long long)b.hist[kl] * inv, hl1 = (double)(long long)b.hist[kl + 1] * inv;
      left = (a.e_lo + (kl + 0.5) * a.de) + (half - hl) / (hl1 - hl) * a.de;
    }
    if (kr < n) {
      const double hr = (double)(long long)b.hist[kr] * inv, hr0 = (double)(long long)b.hist[kr - 1] * inv;
      right = (a.e_lo + (kr - 1 + 0.5) * a.de) + (hr0 - half) / (hr0 - hr) * a.de;
    }
    const double fwhm = right - left;
    b.st[BS_NONEMPTY] = 1.0;
    b.st[BS_PEAK] = e_peak;
    b.st[BS_FWHM] = fwhm;
    b.st[BS_LO] = fmax(a.e_lo, e_peak - fwhm);
    b.st[BS_HI] = e_peak + fwhm;
  }
}

// PASS 1: sums of w, w E, w y, w z, w p_y, w p_z, count over the window and
// w over the whole spectrum range; PASS 2: centred second moments
// w dE^2, w dy^2, w dpy^2, w dy dpy, w dz^2, w dpz^2, w dz dpz
template <class R, int PASS>
__global__ __launch_bounds__(BM) void k_beam_moments(Geo g, Parts<R> P, Layout L, BeamArgs a, BeamScratch b) {
  __shared__ double red[BM / 64][NBM];
  const int n_items = *L.n_items;
  const double lo = b.st[BS_LO], hi = b.st[BS_HI];
  const double em = b.st[BS_EMEAN], ym = b.st[BS_YMEAN], zm = b.st[BS_ZMEAN];
  const double pym = b.st[BS_PYMEAN], pzm = b.st[BS_PZMEAN];
  for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
    double v[NBM] = {0, 0, 0, 0, 0, 0, 0, 0};
    const int4 it = L.items[item];
    const int words = (it.z + it.w + 63) >> 6;
    const unsigned long long* bits = b.bits + (size_t)item * b.item_words;
    // wavefront q takes every (BM / 64)-th word from q on; a lane holds one of
    // them, and the wavefront goes through those that are not zero
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bool any = false;
    for (int w0 = wave; w0 < words; w0 += 64 * (BM / 64)) {
      const int mine = w0 + lane * (BM / 64);
      const unsigned long long held = mine < words ? bits[mine] : 0ull;
      for (unsigned long long some = __ballot(held != 0ull); some; some &= some - 1) {
        any = true;
        const int from = __ffsll(some) - 1;
        const unsigned long long word = __shfl(held, from, 64);
        if ((word >> lane) & 1ull) {
          const int p = item_slot(L, it, (w0 + from * (BM / 64)) * 64 + lane);
          const unsigned cw = P.cell[p];
          const double px = P.px[p], py = P.py[p], pz = P.pz[p];
          const double e = kin_energy(px, py, pz);
          const double w = P.w[p];
          if (PASS == 1) v[7] += w;
          if (!(e >= lo && e <= hi)) continue;
          const double r = ((double)cell_jr(cw) + (double)P.fr[p]) * g.dr;
          double sn, cs;
          sincos_r((double)P.th[p], &sn, &cs);
          const double y = r * cs, z = r * sn;
          if (PASS == 1) {
            v[0] += w;
            v[1] += w * e;
            v[2] += w * y;
            v[3] += w * z;
            v[4] += w * py;
            v[5] += w * pz;
            v[6] += 1.0;
          } else {
            const double de = e - em, dy = y - ym, dz = z - zm, dpy = py - pym, dpz = pz - pzm;
            v[0] += w * de * de;
            v[1] += w * dy * dy;
            v[2] += w * dpy * dpy;
            v[3] += w * dy * dpy;
            v[4] += w * dz * dz;
            v[5] += w * dpz * dpz;
            v[6] += w * dz * dpz;
          }
        }
      }
    }
    // sums over the lanes (fixed order), then over the wavefronts
    if (any) {
#pragma unroll
      for (int k = 0; k < NBM; ++k)
        for (int o = 32; o >= 1; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
    }
    if (lane == 0)
      for (int k = 0; k < NBM; ++k) red[wave][k] = v[k];
    __syncthreads();
    if (threadIdx.x < NBM) {
      double t = 0.0;
      for (int q = 0; q < BM / 64; ++q) t += red[q][threadIdx.x];
      b.part[(size_t)item * NBM + threadIdx.x] = t;
    }
    __syncthreads();  // red is free again
  }
}

// fixed-order sum of the per-item partials, then the means (PASS 1) or the
// outputs (PASS 2).  One group of BR lanes per quantity, adjacent threads
// reading adjacent words.
constexpr int BR = 128;
template <int PASS>
__global__ __launch_bounds__(BR * NBM) void k_beam_reduce(Layout L, const int* __restrict__ err, BeamArgs a,
                                                          BeamScratch b) {
  __shared__ double lanes[BR][NBM];
  __shared__ double t[NBM];
  const int n_items = *L.n_items;
  const int q = threadIdx.x % NBM, l = threadIdx.x / NBM;
  double s = 0.0;
#pragma unroll 8
  for (int i = l; i < n_items; i += BR) s += b.part[(size_t)i * NBM + q];
  lanes[l][q] = s;
  __syncthreads();
  for (int h = BR / 2; h > 0; h >>= 1) {
    if (l < h) lanes[l][q] += lanes[l + h][q];
    __syncthreads();
  }
  if (l == 0) t[q] = lanes[0][q];
  __syncthreads();
  if (threadIdx.x != 0) return;
  double* st = b.st;
  if (PASS == 1) {
    const double W = t[0];
    st[BS_W] = W;
    st[BS_COUNT] = t[6];
    st[BS_QSPEC] = -t[7];
    if (W != 0.0) {
      st[BS_EMEAN] = t[1] / W;
      st[BS_YMEAN] = t[2] / W;
      st[BS_ZMEAN] = t[3] / W;
      st[BS_PYMEAN] = t[4] / W;
      st[BS_PZMEAN] = t[5] / W;
    }
    return;
  }
  double* out = b.out;
  for (int k = 0; k < ENVPIC_NBEAM; ++k) out[k] = 0.0;
  out[ENVPIC_NBEAM] = (double)*err;
  const double W = st[BS_W];
  if (st[BS_NONEMPTY] == 0.0 || W == 0.0) return;
  const double e_rms = sqrt(t[0] / W);
  const double syy = t[1] / W, spp = t[2] / W, syp = t[3] / W;
  const double szz = t[4] / W, sqq = t[5] / W, szq = t[6] / W;
  out[ENVPIC_B_PEAK] = st[BS_PEAK];
  out[ENVPIC_B_FWHM] = st[BS_FWHM];
  out[ENVPIC_B_CHARGE] = -W;
  out[ENVPIC_B_EMEAN] = st[BS_EMEAN];
  out[ENVPIC_B_ERMS] = e_rms;
  out[ENVPIC_B_SPREAD] = e_rms / st[BS_PEAK];
  out[ENVPIC_B_EMIT_Y] = sqrt(fmax(0.0, syy * spp - syp * syp));
  out[ENVPIC_B_EMIT_Z] = sqrt(fmax(0.0, szz * sqq - szq * szq));
  out[ENVPIC_B_COUNT] = st[BS_COUNT];
  out[ENVPIC_B_QSPEC] = st[BS_QSPEC];
  out[ENVPIC_B_WIN_LO] = st[BS_LO];
  out[ENVPIC_B_WIN_HI] = fmin(st[BS_HI], a.e_hi);
}

template <class R>
void launch_beam(const Geo& g, const Parts<R>& P, const Layout& L, int max_items, const int* err, const BeamArgs& a,
                 const BeamScratch& b, hipStream_t st) {
  const int nclr = (std::max(a.nbins, (int)BEAM_STATE) + BG - 1) / BG;
  const int mg = std::min(max_items, MOMENT_GROUPS);
  hipLaunchKernelGGL(k_beam_clear, dim3(nclr), dim3(BG), 0, st, b, a.nbins);
  hipLaunchKernelGGL((k_beam_hist<R>), dim3(max_items), dim3(BG), a.nbins * sizeof(long long), st, P, L, a, b);
  hipLaunchKernelGGL(k_beam_peak, dim3(1), dim3(BPK), 0, st, a, b);
  hipLaunchKernelGGL((k_beam_moments<R, 1>), dim3(mg), dim3(BM), 0, st, g, P, L, a, b);
  hipLaunchKernelGGL(k_beam_reduce<1>, dim3(1), dim3(BR * NBM), 0, st, L, err, a, b);
  hipLaunchKernelGGL((k_beam_moments<R, 2>), dim3(mg), dim3(BM), 0, st, g, P, L, a, b);
  hipLaunchKernelGGL(k_beam_reduce<2>, dim3(1), dim3(BR * NBM), 0, st, L, err, a, b);
}

template void launch_beam<float>(const Geo&, const Parts<float>&, const Layout&, int, const int*, const BeamArgs&,
                                 const BeamScratch&, hipStream_t);
template void launch_beam<double>(const Geo&, const Parts<double>&, const Layout&, int, const int*, const BeamArgs&,
                                  const BeamScratch&, hipStream_t);

}  // namespace envpic
