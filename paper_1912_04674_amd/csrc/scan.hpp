// scan.hpp -- the sort's scans (device side): per tile, the exclusive scan
// of its cells' counts into the per-cell cursors (work groups of the
// field-stage kernel); over all tiles, the scans of the tile totals into the
// next layout's segments and work items, or of the arrivals into the free
// slots and overflow ranges of an incremental sort (launched after it).
#pragma once
#include "common.hpp"

namespace envpic {

// Tile t's 16 x 16 cells (column-major, radius fastest) by 256 consecutive
// threads of the block (lt = 0..255, s: their 256 LDS ints): exclusive scan
// of the counts into the per-cell cursors, the total into hist[t], counts
// cleared.  Every thread of the block calls it (it synchronizes the block);
// inactive halves pass t < 0.
__device__ inline void cell_scan_tile(const Geo& g, int t, int lt, int* ccount, int* ccur, int* hist, int* s) {
  const bool active = t >= 0 && t < g.ntiles;
  int c = 0;
  size_t o = 0;
  bool valid = false;
  if (active) {
    const int tcx = t / g.ntr, tcr = t - (t / g.ntr) * g.ntr;
    const int a = lt / TR, b = lt - (lt / TR) * TR;
    const long long col = (long long)lab_tile(g, tcx) * TX + a;
    const int rel = (int)(col - g.shift), j = tcr * TR + b;
    valid = rel >= 0 && rel < g.nx && j < g.nr;
    o = valid ? (size_t)phys_col(g, rel) * g.pitch + j : 0;
    c = valid ? ccount[o] : 0;
  }
  s[lt] = c;
  __syncthreads();
  for (int off = 1; off < TX * TR; off <<= 1) {
    const int v = lt >= off ? s[lt - off] : 0;
    __syncthreads();
    s[lt] += v;
    __syncthreads();
  }
  if (valid) {
    ccur[o] = s[lt] - c;
    ccount[o] = 0;
  }
  if (active && lt == TX * TR - 1) hist[t] = s[lt];
}

// Exclusive scan of two non-negative sums per thread (in the halves of one
// word) over the NT threads of a block (NT a multiple of 64, at most 64
// wavefronts): shuffles inside each wavefront, then the wavefront totals
// through s_w (NT / 64 words).  Returns the sums of the lower threads' values;
// *total gets the block's.  Every thread calls it.
struct Pair {
  int a, b;
};
__device__ inline long long pack_pair(int a, int b) { return ((long long)a << 32) | (unsigned)b; }
template <int NT> __device__ inline Pair block_scan(int a, int b, long long* s_w, Pair* total) {
  const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
  const long long v = pack_pair(a, b);
  long long x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const long long y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) s_w[w] = x;
  __syncthreads();
  long long pre = 0, tot = 0;
  for (int k = 0; k < NT / 64; ++k) {
    const long long t = s_w[k];
    pre += k < w ? t : 0;
    tot += t;
  }
  __syncthreads();  // s_w is free again
  *total = Pair{(int)(tot >> 32), (int)tot};
  const long long e = pre + x - v;
  return Pair{(int)(e >> 32), (int)e};
}
// the block's sum of two values per thread, in every thread
template <int NT> __device__ inline Pair block_sum(int a, int b, long long* s_w) {
  Pair t;
  block_scan<NT>(a, b, s_w, &t);
  return t;
}
// The items (pending[0]) and slots past the used ones (pending[1]) of a
// column injected since the last scan join layout L, the layout in use: an
// item placed at the end of its tile's segment extends the segment's used
// slots (the items of one column lie in distinct tiles).  Every thread of
// the block calls it; the caller synchronizes before reading L.
__device__ inline void bump_pending(const Geo& g, Layout L, int* pending) {
  const int np = pending[0];
  if (np == 0) return;
  const int n0 = *L.n_items, seg_end = L.offsets[g.ntiles];  // (an injected item has no riders)
  for (int i = threadIdx.x; i < np; i += blockDim.x) {
    const int4 it = L.items[n0 + i];
    if (it.y < seg_end) L.ext[it.x] += it.z;
  }
  __syncthreads();  // every thread has read n_items and pending
  if (threadIdx.x == 0) {
    *L.n_items = n0 + np;
    *L.fill += pending[1];
    pending[0] = 0;
    pending[1] = 0;
  }
}

// Work items of v particles from slot st: ceil(v / chunk) items of
// item_share particles (the last holds the rest), written from items[em] on
// (none past max_em); returns their number.
__device__ inline int emit_items(const Geo& g, int4* items, int em, int max_em, int key, int st, int v,
                                 int capacity) {
  const int nm = (v + g.chunk - 1) / g.chunk, sh = item_share(v, g.chunk);
  for (int k = 0; k < nm; ++k) {
    const int lo = k * sh, hi = min(lo + sh, v);
    // items never reach past the buffer (an overflow is flagged by the caller)
    if (em + k < max_em)
      items[em + k] = (st + hi <= capacity) ? make_int4(key, st + lo, hi - lo, 0) : make_int4(key, 0, 0, 0);
  }
  return nm;
}

// whether the v particles of a tile's overflow range ride with the last work
// item of the n in its segment
__device__ inline bool overflow_rides(const Geo& g, int n, int v) { return n > 0 && v > 0 && v <= min(MAX_RIDERS, g.chunk / 2); }

// Slots a rebuilt layout holds for tile t of v particles: v, or a full tile
// when the tile lies in the `entering` tile columns ahead of a moving window
// (or in the one its front is in), which fill as columns are injected.
// Other tiles get no free slots: measured on the LWFA workload, free slots of
// 1/16 of each tile made the passes that stream the particles 5 % slower
// (their arrivals, rare, take overflow ranges instead).  `align` rounds the
// room up, so that the next segment starts at a multiple of it.
__device__ inline int seg_room(const Geo& g, int t, int v, int entering, int align) {
  int room = v;
  if (entering > 0) {
    const int tcx = t / g.ntr, tr = t - (t / g.ntr) * g.ntr;
    const int T = lab_tile(g, tcx), front = (int)(g.shift + g.nx - 1) / TX;  // (lab columns fit 20 bits)
    if (T >= front && T <= front + entering)
      room = max(v, TX * min(TR, g.nr - tr * TR) * g.ppc_x * g.ppc_r * g.ppc_t);
  }
  return round_slots(room, align);
}

// The tile totals in hist become layout `out` of the other buffer, the whole
// layout rebuilt, by one block of NT threads per NT tiles: the segment of a
// tile of v particles holds seg_room slots (the room for entering tiles, and
// the alignment of the segments, only when `reserve` slots past the segments
// stay free), and its particles form ceil(v / chunk) items.  hist stays (the
// kernels keep it current).  Flags when the particles plus the columns
// injected before the next sort would not fit.
template <int NT>
__device__ inline void full_layout(const Geo& g, const int* hist, Layout out, int capacity, int inj_max, int reserve,
                                   int entering, int max_items, int* err, int mode, long long* s_w) {
  const int nt = g.ntiles, first = blockIdx.x * NT, t = first + threadIdx.x;
  // over all tiles and over those before this block's: the segments' size
  // with and without the room for entering tiles, packed and aligned, and
  // the items
  int r[5] = {0, 0, 0, 0, 0}, q[5] = {0, 0, 0, 0, 0};
  for (int k = threadIdx.x; k < nt; k += NT) {
    const int v = hist[k];
    const int x[5] = {v, round_slots(v, SLOT_ALIGN), seg_room(g, k, v, entering, 1),
                      seg_room(g, k, v, entering, SLOT_ALIGN), (v + g.chunk - 1) / g.chunk};
    for (int e = 0; e < 5; ++e) {
      r[e] += x[e];
      q[e] += k < first ? x[e] : 0;
    }
  }
  const Pair none = block_sum<NT>(r[0], r[1], s_w), with = block_sum<NT>(r[2], r[3], s_w);
  const int ent = with.a <= capacity - reserve ? entering : 0;
  const Pair room = ent > 0 ? with : none;
  const int align = room.b <= capacity - reserve ? SLOT_ALIGN : 1;
  const int seg_end = align > 1 ? room.b : room.a;
  const int items = block_sum<NT>(r[4], 0, s_w).a;
  const int before = align > 1 ? (ent > 0 ? q[3] : q[1]) : (ent > 0 ? q[2] : q[0]);
  const Pair base = block_sum<NT>(before, q[4], s_w);
  // room kept for the columns injected before the next sort (one per step)
  const int item_cap = max_items - SORT_EVERY * g.ntr;
  const int v = t < nt ? hist[t] : 0;
  Pair tot;
  const Pair pre =
      block_scan<NT>(t < nt ? seg_room(g, t, v, ent, align) : 0, (v + g.chunk - 1) / g.chunk, s_w, &tot);
  if (t < nt) {
    const int st = base.a + pre.a;
    out.offsets[t] = st;
    out.ext[t] = v;
    out.cursor[t] = st;
    out.ovb[t] = 0;
    out.ovn[t] = 0;
    emit_items(g, out.items, base.b + pre.b, item_cap, t, st, v, capacity);
  }
  if (t == 0) {
    out.offsets[nt] = seg_end;
    *out.fill = seg_end;
    *out.n_items = min(items, item_cap);
    *out.mode = mode;
    if (items > item_cap) atomicOr(err, ERR_ITEMS);
    if (seg_end > capacity - SORT_EVERY * inj_max) atomicOr(err, ERR_CAPACITY);
  }
}

// Before a tile sort, by one block of NT threads per NT tiles: layout `out`
// of the same buffer as `in`, where only the particles that change tile move.
// arr[t] holds the arrivals of tile t (particles of other tiles' items whose
// cell is now in t, and every particle of t's items past the segments:
// injected columns, earlier overflows), hist[t] its particles after the sort.
// The arrivals fill the free slots at the end of t's segment, then a range of
// their own past the used slots (from ovb[t], ovn[t] of them).  When the
// overflow or the items would not fit, the layout is rebuilt as by
// full_layout instead (mode LAYOUT_FULL: the sort then scatters every
// particle).  arr_next, the arrivals of the next tile sort, is cleared (arr
// itself is still read by other blocks); stats[0] counts the incremental
// layouts, stats[1] the rebuilt ones.
template <int NT>
__device__ inline void move_layout(const Geo& g, const int* hist, const int* arr, int* arr_next, Layout in, Layout out,
                                   int capacity, int inj_max, int reserve, int entering, int max_items, int* err,
                                   int* stats, long long* s_w) {
  const int nt = g.ntiles, first = blockIdx.x * NT, t = first + threadIdx.x;
  const int seg_end = in.offsets[nt];
  const int fill0 = *in.fill;
  // arrivals of tile k: `tail` into its segment's free slots (e in use),
  // `ov` past the segments; `items` of both
  struct Plan {
    int e, tail, ov, items;
  };
  auto plan = [&](int k) {
    Plan p;
    const int a = arr[k];
    p.e = in.ext[k];
    p.tail = min(a, in.offsets[k + 1] - in.offsets[k] - p.e);
    p.ov = a - p.tail;
    p.items = (p.e + p.tail + g.chunk - 1) / g.chunk;
    if (!overflow_rides(g, p.e + p.tail, p.ov)) p.items += (p.ov + g.chunk - 1) / g.chunk;
    return p;
  };
  if (t < nt) arr_next[t] = 0;
  const Plan p = t < nt ? plan(t) : Plan{0, 0, 0, 0};
  Pair all, base{0, 0};
  const Pair pre = block_scan<NT>(p.ov, p.items, s_w, &all);
  if (nt > NT) {
    // all tiles, and those before this block's
    int ov = 0, m = 0, ov_before = 0, m_before = 0;
    for (int k = threadIdx.x; k < nt; k += NT) {
      const Plan x = plan(k);
      ov += x.ov;
      m += x.items;
      ov_before += k < first ? x.ov : 0;
      m_before += k < first ? x.items : 0;
    }
    all = block_sum<NT>(ov, m, s_w);
    base = block_sum<NT>(ov_before, m_before, s_w);
  }
  const int fill_new = fill0 + all.a;
  const int item_cap = max_items - SORT_EVERY * g.ntr;
  if (fill_new > capacity - SORT_EVERY * inj_max || all.b > item_cap) {
    // every thread of every block takes the same branch
    if (t == 0) stats[1] += 1;
    full_layout<NT>(g, hist, out, capacity, inj_max, reserve, entering, max_items, err, LAYOUT_FULL, s_w);
    return;
  }
  if (t < nt) {
    const int ob = fill0 + base.a + pre.a, n = p.e + p.tail, st = in.offsets[t];
    int em = base.b + pre.b;
    out.offsets[t] = st;
    out.ext[t] = n;
    out.cursor[t] = 0;
    out.ovb[t] = ob;
    out.ovn[t] = p.ov;
    em += emit_items(g, out.items, em, item_cap, t, st, n, capacity);
    if (overflow_rides(g, n, p.ov))
      out.items[em - 1].w = p.ov;
    else
      emit_items(g, out.items, em, item_cap, t, ob, p.ov, capacity);
  }
  if (t == 0) {
    out.offsets[nt] = seg_end;
    *out.fill = fill_new;
    *out.n_items = all.b;
    *out.mode = LAYOUT_MOVE;
    stats[0] += 1;
  }
}

// After a tile sort whose scan rebuilt the layout (LAYOUT_FULL), the sort
// wrote every particle into the other buffer: copy the used slots back (b of
// nb groups of 256 threads), so that the particles stay in the buffer they
// were in.  Nothing to do after an incremental sort.  Each lane moves four
// consecutive slots of every record array per pass with 16-byte accesses
// (the arrays start 256-byte aligned), so that enough bytes are in flight to
// stream at the copy rate; the slots past the last multiple of four go one
// by one.
template <class T> __device__ inline void copy4(T* to, const T* from, long long i) {
  static_assert(sizeof(T) == 4, "4-byte record arrays");
  *reinterpret_cast<uint4*>(to + i) = *reinterpret_cast<const uint4*>(from + i);
}
template <class R>
__device__ inline void settle_copy(const SettleArgs<R>& sa, int b, int nb) {
  if (*sa.L.mode != LAYOUT_FULL) return;
  const long long n = min((long long)*sa.L.fill, sa.cap);
  const long long n4 = n & ~3LL;
  if constexpr (sizeof(R) == 4) {
    for (long long i = ((long long)b * 256 + threadIdx.x) * 4; i < n4; i += (long long)nb * 256 * 4) {
      copy4(sa.to.cell, sa.from.cell, i);
      copy4(sa.to.fx, sa.from.fx, i);
      copy4(sa.to.fr, sa.from.fr, i);
      copy4(sa.to.th, sa.from.th, i);
      copy4(sa.to.px, sa.from.px, i);
      copy4(sa.to.py, sa.from.py, i);
      copy4(sa.to.pz, sa.from.pz, i);
      copy4(sa.to.w, sa.from.w, i);
      copy4(sa.to.id, sa.from.id, i);
    }
  }
  const long long i0 = sizeof(R) == 4 ? n4 : 0;
  for (long long i = i0 + (long long)b * 256 + threadIdx.x; i < n; i += (long long)nb * 256) {
    sa.to.cell[i] = sa.from.cell[i];
    sa.to.fx[i] = sa.from.fx[i];
    sa.to.fr[i] = sa.from.fr[i];
    sa.to.th[i] = sa.from.th[i];
    sa.to.px[i] = sa.from.px[i];
    sa.to.py[i] = sa.from.py[i];
    sa.to.pz[i] = sa.from.pz[i];
    sa.to.w[i] = sa.from.w[i];
    sa.to.id[i] = sa.from.id[i];
  }
}

}  // namespace envpic
