// export.hip -- state read back by the host as FP64: a field on its nodes of
// the window, and the particles in lab-frame Cartesian columns in ascending
// id order.  Converted and ordered on the device, in scratch memory that is
// free between steps, so the host only receives the columns.  An id's rank is
// the number of bits below its own in a bitmap of the ids (no sort: two passes
// over the ids and one over the records).  1 M particles take 0.2 ms here; the
// copy of their 60 MB to pageable host memory bounds the call (8 ms).
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"
#include "scan.hpp"

namespace envpic {

constexpr int EB = 256;            // threads per group
constexpr int EXPORT_WORDS = 16;   // words of the id bitmap per thread of a scan group

// ------------------------------------------------------------- fields --
// (nx+1) x (nr+1) nodes; the unused last column or row of a staggered field
// is zero; rows j <= 1 of the envelope come from the FP64 rows where held.
template <class R>
__global__ __launch_bounds__(EB) void k_export_field(Geo g, ExportField f, double* __restrict__ out) {
  const long long k = (long long)blockIdx.x * EB + threadIdx.x;
  const int nr1 = g.nr + 1;
  if (k >= (long long)(g.nx + 1) * nr1) return;
  const int i = (int)(k / nr1), j = (int)(k - (long long)i * nr1);
  const int pc = phys_col(g, i);
  const bool valid = (!f.dual_x || i <= g.nx - 1) && (!f.dual_r || j <= g.nr - 1);
  const size_t o = (size_t)pc * g.pitch + j;
  const R* src = static_cast<const R*>(f.ptr);
  if (f.cplx) {
    double2 v = make_double2(0.0, 0.0);
    if (f.rows && j <= 1)
      v = f.rows[pc * 2 + j];
    else if (valid)
      v = make_double2((double)src[2 * o], (double)src[2 * o + 1]);
    reinterpret_cast<double2*>(out)[k] = v;
  } else {
    out[k] = valid ? (double)src[o] : 0.0;
  }
}
template <class R> void launch_export_field(const Geo& g, const ExportField& f, double* out, hipStream_t st) {
  const long long nodes = (long long)(g.nx + 1) * (g.nr + 1);
  hipLaunchKernelGGL((k_export_field<R>), dim3((unsigned)((nodes + EB - 1) / EB)), dim3(EB), 0, st, g, f, out);
}
template void launch_export_field<float>(const Geo&, const ExportField&, double*, hipStream_t);
template void launch_export_field<double>(const Geo&, const ExportField&, double*, hipStream_t);

// ---------------------------------------------------------- particles --
struct ExportHead {
  unsigned n, id_min, id_max, duplicate;
};

__global__ void k_export_start(ExportHead* h) { *h = ExportHead{0u, ~0u, 0u, 0u}; }

// live particles and their range of ids
template <class R> __global__ __launch_bounds__(EB) void k_export_ids(Parts<R> P, Layout L, ExportHead* h) {
  __shared__ unsigned s_n, s_lo, s_hi;
  if ((int)blockIdx.x >= *L.n_items) return;
  const int4 it = L.items[blockIdx.x];
  if (threadIdx.x == 0) s_n = 0u, s_lo = ~0u, s_hi = 0u;
  __syncthreads();
  unsigned n = 0, lo = ~0u, hi = 0;
  for (int k = threadIdx.x; k < it.z + it.w; k += EB) {
    const int p = item_slot(L, it, k);
    if (P.cell[p] == kDead) continue;
    const unsigned id = P.id[p];
    n += 1;
    lo = min(lo, id);
    hi = max(hi, id);
  }
  atomicAdd(&s_n, n);
  atomicMin(&s_lo, lo);
  atomicMax(&s_hi, hi);
  __syncthreads();
  if (threadIdx.x == 0 && s_n > 0) {
    atomicAdd(&h->n, s_n);
    atomicMin(&h->id_min, s_lo);
    atomicMax(&h->id_max, s_hi);
  }
}

__global__ __launch_bounds__(EB) void k_export_clear(unsigned* bits, long long words) {
  const long long k = (long long)blockIdx.x * EB + threadIdx.x;
  if (k < words) bits[k] = 0u;
}

// a bit per id (from word0 on); two particles of one id are reported
template <class R>
__global__ __launch_bounds__(EB) void k_export_mark(Parts<R> P, Layout L, unsigned word0, unsigned* bits,
                                                    ExportHead* h) {
  if ((int)blockIdx.x >= *L.n_items) return;
  const int4 it = L.items[blockIdx.x];
  for (int k = threadIdx.x; k < it.z + it.w; k += EB) {
    const int p = item_slot(L, it, k);
    if (P.cell[p] == kDead) continue;
    const unsigned id = P.id[p], bit = 1u << (id & 31u);
    if (atomicOr(&bits[(id >> 5) - word0], bit) & bit) h->duplicate = 1u;
  }
}

// bits set per group of words, then (second launch) below each word: every
// group adds up the sums of the groups before it
__global__ __launch_bounds__(EB) void k_export_sums(const unsigned* __restrict__ bits, long long words, int* sums) {
  __shared__ long long s_w[EB / 64];
  const long long w0 = ((long long)blockIdx.x * EB + threadIdx.x) * EXPORT_WORDS;
  int c = 0;
  for (int q = 0; q < EXPORT_WORDS; ++q) c += w0 + q < words ? __popc(bits[w0 + q]) : 0;
  Pair total;
  block_scan<EB>(c, 0, s_w, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total.a;
}
__global__ __launch_bounds__(EB) void k_export_below(const unsigned* __restrict__ bits, long long words,
                                                     const int* __restrict__ sums, int* __restrict__ below) {
  __shared__ long long s_w[EB / 64];
  int before = 0;
  for (int b = threadIdx.x; b < (int)blockIdx.x; b += EB) before += sums[b];
  Pair total;
  block_scan<EB>(before, 0, s_w, &total);
  const long long w0 = ((long long)blockIdx.x * EB + threadIdx.x) * EXPORT_WORDS;
  int c = 0;
  for (int q = 0; q < EXPORT_WORDS; ++q) c += w0 + q < words ? __popc(bits[w0 + q]) : 0;
  int run = total.a;
  run += block_scan<EB>(c, 0, s_w, &total).a;
  for (int q = 0; q < EXPORT_WORDS; ++q) {
    if (w0 + q >= words) break;
    below[w0 + q] = run;
    run += __popc(bits[w0 + q]);
  }
}

// Columns [c0, c1) of x, y, z, px, py, pz, w, id of the particles, each of n
// words of 8 bytes (id: of 4), a particle at the rank of its id
template <class R>
__global__ __launch_bounds__(EB) void k_export_write(Geo g, Parts<R> P, Layout L, unsigned word0,
                                                     const unsigned* __restrict__ bits,
                                                     const int* __restrict__ below, unsigned n, int c0, int c1,
                                                     double* __restrict__ out) {
  if ((int)blockIdx.x >= *L.n_items) return;
  const int4 it = L.items[blockIdx.x];
  for (int k = threadIdx.x; k < it.z + it.w; k += EB) {
    const int p = item_slot(L, it, k);
    const unsigned cw = P.cell[p];
    if (cw == kDead) continue;
    const unsigned id = P.id[p], word = (id >> 5) - word0;
    const unsigned m = below[word] + __popc(bits[word] & ((1u << (id & 31u)) - 1u));
    if (m >= n) continue;  // (a duplicated id: the host discards this)
    double r = 0.0, sn = 0.0, cs = 0.0;
    if (c0 < 3 && c1 > 1) {
      r = ((double)cell_jr(cw) + (double)P.fr[p]) * g.dr;
      sincos((double)P.th[p], &sn, &cs);
    }
    for (int c = c0; c < c1; ++c) {
      double* col = out + (size_t)(c - c0) * n;
      if (c == 7) {
        reinterpret_cast<unsigned*>(col)[m] = id;
        continue;
      }
      double v;
      switch (c) {
        case 0: v = ((double)cell_ix(cw) + (double)P.fx[p]) * g.dx; break;
        case 1: v = r * cs; break;
        case 2: v = r * sn; break;
        case 3: v = (double)P.px[p]; break;
        case 4: v = (double)P.py[p]; break;
        case 5: v = (double)P.pz[p]; break;
        default: v = (double)P.w[p]; break;
      }
      col[m] = v;
    }
  }
}

// The number of live particles to *n and their columns to outs[0..6] and id
// (any of them may be null).  Returns 1 if the scratch memory cannot hold the
// ids' bitmap and a column or an id occurs twice (nothing was written: the
// host sorts), a negative number on a failure of the runtime.
template <class R>
int export_particles(const Geo& g, const Parts<R>& P, const Layout& L, int max_items, char* scratch, size_t bytes,
                     double* const* outs, uint32_t* ids, int64_t* n, hipStream_t st) {
  const auto up = [](size_t b) { return (b + 255) / 256 * 256; };
  if (bytes < 256) return 1;
  ExportHead* head = reinterpret_cast<ExportHead*>(scratch);
  ExportHead h{};
  const dim3 grid(max_items), block(EB);
  hipLaunchKernelGGL(k_export_start, dim3(1), dim3(1), 0, st, head);
  hipLaunchKernelGGL((k_export_ids<R>), grid, block, 0, st, P, L, head);
  if (hipMemcpyAsync(&h, head, sizeof h, hipMemcpyDeviceToHost, st) != hipSuccess) return -1;
  if (hipStreamSynchronize(st) != hipSuccess) return -1;
  *n = h.n;
  bool wanted = ids != nullptr;
  for (int c = 0; c < 7; ++c) wanted |= outs[c] != nullptr;
  if (h.n == 0 || !wanted) return 0;
  const unsigned word0 = h.id_min >> 5;
  const long long words = (long long)(h.id_max >> 5) - word0 + 1;
  const long long groups = (words + EB * EXPORT_WORDS - 1) / (EB * EXPORT_WORDS);
  size_t off = 256;
  unsigned* bits = reinterpret_cast<unsigned*>(scratch + off);
  off += up(words * sizeof(unsigned));
  int* below = reinterpret_cast<int*>(scratch + off);
  off += up(words * sizeof(int));
  int* sums = reinterpret_cast<int*>(scratch + off);
  off += up(groups * sizeof(int));
  const size_t column = (size_t)h.n * sizeof(double);
  if (off + column > bytes) return 1;
  const int fit = (int)std::min<size_t>(8, (bytes - off) / column);
  double* cols = reinterpret_cast<double*>(scratch + off);
  hipLaunchKernelGGL(k_export_clear, dim3((unsigned)((words + EB - 1) / EB)), block, 0, st, bits, words);
  hipLaunchKernelGGL((k_export_mark<R>), grid, block, 0, st, P, L, word0, bits, head);
  hipLaunchKernelGGL(k_export_sums, dim3((unsigned)groups), block, 0, st, bits, words, sums);
  hipLaunchKernelGGL(k_export_below, dim3((unsigned)groups), block, 0, st, bits, words, sums, below);
  for (int c0 = 0; c0 < 8; c0 += fit) {
    const int c1 = std::min(8, c0 + fit);
    hipLaunchKernelGGL((k_export_write<R>), grid, block, 0, st, g, P, L, word0, bits, below, h.n, c0, c1, cols);
    if (c0 == 0) {
      if (hipMemcpyAsync(&h, head, sizeof h, hipMemcpyDeviceToHost, st) != hipSuccess) return -1;
      if (hipStreamSynchronize(st) != hipSuccess) return -1;
      if (h.duplicate) return 1;
    }
    for (int c = c0; c < c1; ++c) {
      void* to = c == 7 ? (void*)ids : (void*)outs[c];
      const size_t b = c == 7 ? (size_t)h.n * sizeof(uint32_t) : column;
      if (to && hipMemcpyAsync(to, cols + (size_t)(c - c0) * h.n, b, hipMemcpyDeviceToHost, st) != hipSuccess)
        return -1;
    }
  }
  return hipStreamSynchronize(st) == hipSuccess ? 0 : -1;
}
template int export_particles<float>(const Geo&, const Parts<float>&, const Layout&, int, char*, size_t,
                                     double* const*, uint32_t*, int64_t*, hipStream_t);
template int export_particles<double>(const Geo&, const Parts<double>&, const Layout&, int, char*, size_t,
                                      double* const*, uint32_t*, int64_t*, hipStream_t);

}  // namespace envpic
