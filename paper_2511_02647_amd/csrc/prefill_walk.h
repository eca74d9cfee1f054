// Where a query tile's workgroup finds its segment and which KV tiles it walks: shared by the
// prefill kernels on the matrix cores.
//
// In launches with few tiles the host has listed them (tile_list in the argument block), and a workgroup reads its entry and its
// segment's two ends; otherwise it searches the segment tables.  A workgroup alone on its SIMDs takes 4 to 5 cycles per instruction,
// so what counts at the start of a short launch is how many there are, divisions by head counts included.
//
// The segment tables sit in the kernel-argument buffer, too.  Walking them entry by entry costs
// one scalar-cache miss after another while nothing else is in flight, so every lane
// fetches the entries of segment `lane` (and `lane + 64`) of all tables in one go and the
// searches run on ballots.  Entry 0 of every table is 0.
#pragma once

#include <climits>

#include "common.h"

namespace fedattn {

struct SegTab {
  int lo, hi;  // table[lane + 1], table[lane + 65]; INT_MAX past the last segment
};
__device__ __attribute__((always_inline)) inline SegTab load_seg_tab(const int32_t* t, int lane, int n_seg) {
  // the tables have kMaxP + 1 entries whatever N is: fetch first (nothing to wait for), select after
  const int lo = t[lane + 1], hi = t[lane + 65];
  SegTab r;
  r.lo = lane < n_seg ? lo : INT_MAX;
  r.hi = lane + 64 < n_seg ? hi : INT_MAX;
  return r;
}
// table[idx] for a wave-uniform idx in [0, N]
__device__ __attribute__((always_inline)) inline int seg_tab_at(const SegTab& t, int idx) {
  if (idx == 0) return 0;
  return idx <= 64 ? __builtin_amdgcn_readlane(t.lo, idx - 1) : __builtin_amdgcn_readlane(t.hi, idx - 65);
}
// number of segments s with x >= table[s + 1], i.e. the segment a cumulative index falls in
__device__ __attribute__((always_inline)) inline int seg_tab_find(const SegTab& t, int x, int n_seg) {
  int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(x >= t.lo));
  if (n_seg > 64) n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(x >= t.hi));
  return n;
}

// Workgroup -> (KV head, set of heads of its group, position in the launch): KV head fastest, so that the workgroups of one
// KV head share an XCD's L2 when there are 8 (round-robin dispatch over 8 XCDs).
struct WgPlace {
  int g, set, p;
};
__device__ __attribute__((always_inline)) inline WgPlace find_wg_place(const PrefillArgs& a) {
  // All arguments that stand before the tables are requested here, together: one by one where they are used, each is a round trip to the
  // scalar cache, some to memory, that nothing overlaps with (a sync block of 64 and 76 tokens, 8/8 heads of 128: 6.2 and 5.7 us).
  asm volatile("" ::"s"(a.q), "s"(a.k), "s"(a.v), "s"(a.keep_chunks), "s"(a.Hkv), "s"(a.kv_shift), "s"(a.set_shift), "s"(a.head_sets), "s"(a.group),
               "s"(a.n_listed), "s"(a.sync_override), "s"(a.q_tile_rows), "s"(a.causal), "s"(a.apart), "s"(a.seg.n));
  const unsigned id = blockIdx.x;
  const unsigned rest = a.kv_shift >= 0 ? id >> a.kv_shift : id / (unsigned)a.Hkv;
  const unsigned p = a.set_shift >= 0 ? rest >> a.set_shift : rest / (unsigned)a.head_sets;
  return WgPlace{(int)(id - rest * a.Hkv), (int)(rest - p * a.head_sets), (int)p};
}

// A query tile: its segment, the segment's ends, the tile's first row.
struct TilePlace {
  int n, seg_lo, seg_hi, q0;
};
// The host's list and the segments' ends, requested with the first instructions of the kernel: together with the other arguments one
// round trip to memory (entry, then segment, by scalar loads: two more, 0.3 us of a launch).
struct ListTab {
  uint32_t w[kMaxListedTiles / 128];   // word 64 x + lane
  SegTab seg;
};
__device__ __attribute__((always_inline)) inline ListTab load_list(const PrefillArgs& a, int lane) {
  ListTab t;
#pragma unroll
  for (int x = 0; x < kMaxListedTiles / 128; ++x) t.w[x] = a.tile_list[64 * x + lane];
  t.seg = load_seg_tab(a.seg.seg_off, lane, a.seg.n);
  return t;
}
// entry i
__device__ __attribute__((always_inline)) inline uint32_t list_entry(const ListTab& t, int i) {
  const int word = i >> 1, lane = word & 63;
  uint32_t w = __builtin_amdgcn_readlane(t.w[0], lane);
#pragma unroll
  for (int x = 1; x < kMaxListedTiles / 128; ++x) w = word >> 6 == x ? __builtin_amdgcn_readlane(t.w[x], lane) : w;
  return w >> (16 * (i & 1)) & 0xffffu;
}
__device__ __attribute__((always_inline)) inline TilePlace place_listed(const PrefillArgs& a, const ListTab& l, uint32_t e) {
  TilePlace t;
  t.n = e & 127;
  t.seg_lo = seg_tab_at(l.seg, t.n);
  t.seg_hi = seg_tab_at(l.seg, t.n + 1);
  t.q0 = t.seg_lo + (int)(e >> 7) * a.q_tile_rows;
  return t;
}
// tile of a launch without a list
__device__ __attribute__((always_inline)) inline TilePlace place_in_tables(const PrefillArgs& a, const SegTab& seg_tab, const SegTab& tile_tab, int tile) {
  TilePlace t;
  t.n = seg_tab_find(tile_tab, tile, a.seg.n);
  t.seg_lo = seg_tab_at(seg_tab, t.n);
  t.seg_hi = seg_tab_at(seg_tab, t.n + 1);
  t.q0 = t.seg_lo + (tile - seg_tab_at(tile_tab, t.n)) * a.q_tile_rows;
  return t;
}
// One tile per workgroup, longest walks first (split and fp32 kernels): tile of position p.
__device__ __attribute__((always_inline)) inline TilePlace place_heavy_first(const PrefillArgs& a, const ListTab& list, int p, bool is_sync, int lane) {
  if (a.n_listed > 0) return place_listed(a, list, list_entry(list, p));
  const int N = a.seg.n, T = a.n_q_tiles;
  const SegTab seg_tab = list.seg;
  const SegTab tile_tab = load_seg_tab(a.seg.tile_cum, lane, N);
  const SegTab order_tab = load_seg_tab(a.seg.pair_cum, lane, N);
  const int order_lo = a.seg_order[lane], order_hi = a.seg_order[lane + 64];
  const int rank = a.short_half_ascending && p >= (T + 1) / 2 ? T - 1 - (p - (T + 1) / 2) : p;  // 0: longest walk
  int tile;
  if (is_sync) {
    tile = T - 1 - rank;
  } else {
    const int s = seg_tab_find(order_tab, rank, N);
    const int n = s < 64 ? __builtin_amdgcn_readlane(order_lo, s) : __builtin_amdgcn_readlane(order_hi, s - 64);
    tile = seg_tab_at(tile_tab, n + 1) - 1 - (rank - seg_tab_at(order_tab, s));
  }
  return place_in_tables(a, seg_tab, tile_tab, tile);
}

// Where participant n's own K (kv = 0) or V matrix lies.
__device__ __attribute__((always_inline)) inline const uint16_t* own_matrix(const PrefillArgs& a, int n, int kv) {
  return reinterpret_cast<const uint16_t*>(a.own[2 * n + kv]);
}
// Tiles of the global sequence from matrices that lie apart.  A tile inside one segment is loaded as from one matrix, whose place is kept
// from tile to tile; in one that crosses an end every lane picks its row's matrix.
struct ApartRows {
  int ends;         // lane n: the end of participant n's segment, INT_MAX past the last
  int m, lo, hi;    // the segment the last tile began in
  const uint16_t *k, *v;

  __device__ __attribute__((always_inline)) void init(const PrefillArgs& a, int lane) {
    static_assert(kMaxApart < 64, "one participant per lane");
    ends = lane < a.seg.n ? a.seg.seg_off[lane + 1] : INT_MAX;
    lo = hi = 0;
  }
  __device__ __attribute__((always_inline)) void enter(const PrefillArgs& a, int g, int kv0) {
    if (kv0 >= lo && kv0 < hi) return;
    m = __builtin_popcountll(__builtin_amdgcn_ballot_w64(kv0 >= ends));
    lo = a.seg.seg_off[m];
    hi = a.seg.seg_off[m + 1];
    k = own_matrix(a, m, 0) + g * a.D;
    v = own_matrix(a, m, 1) + g * a.D;
  }
  template <bool IS_V, typename TL>
  __device__ __attribute__((always_inline)) void load(const PrefillArgs& a, const TL& tile_io, int g, int kv0, int len, uint32_t stage) const {
    const int64_t row_elems = tile_io.row_elems;
    const uint16_t* base = IS_V ? v : k;
    if (kv0 + len <= hi) {
      tile_io.template dma<IS_V>(base + kv0 * row_elems, stage, len);
      return;
    }
    if (kv0 + len <= a.seg.seg_off[m + 2]) {   // one end, as nearly always
      const uint16_t* next = own_matrix(a, m + 1, IS_V) + g * a.D;
      tile_io.template dma_rows<IS_V>(stage, len, [&](int row) __attribute__((always_inline)) {
        return (kv0 + row >= hi ? next : base) + (kv0 + row) * row_elems;
      });
      return;
    }
    tile_io.template dma_rows<IS_V>(stage, len, [&](int row) __attribute__((always_inline)) {
      const uint16_t* p = base;
      for (int x = m + 1; a.seg.seg_off[x] < kv0 + len; ++x) {
        const uint16_t* q = own_matrix(a, x, IS_V) + g * a.D;
        p = kv0 + row >= a.seg.seg_off[x] ? q : p;
      }
      return p + (kv0 + row) * row_elems;
    });
  }
};

// One query tile's walk through its KV tiles (all members wave-uniform): two runs of the
// kept-tile list (sparse exchange: remote participants before and after the own one), then a
// dense range [dlo, dhi).
struct KvWalk {
  int seg_hi, q0, la_n, lb0, n_list, dlo, dhi, nt;
};
__device__ __attribute__((always_inline)) inline KvWalk make_kv_walk(const PrefillArgs& a, const TilePlace& tp, bool is_sync, bool sparse) {
  const int N = a.seg.n, BM = a.q_tile_rows;
  const bool causal = a.causal != 0;
  KvWalk w;
  const int n = tp.n, seg_lo = tp.seg_lo;
  w.seg_hi = tp.seg_hi;
  w.q0 = tp.q0;
  const int i_last = min(w.q0 + BM, w.seg_hi) - 1;
  int la_n = 0, lb0 = 0, lb_n = 0;
  if (sparse) {
    la_n = a.kept_cum[n];
    if (!causal) {
      lb0 = a.kept_cum[n + 1];
      lb_n = a.kept_cum[N] - lb0;
    }
  }
  w.la_n = la_n;
  w.lb0 = lb0;
  w.n_list = la_n + lb_n;
  w.dlo = (is_sync && !sparse) ? 0 : seg_lo;
  w.dhi = causal ? i_last + 1 : ((is_sync && !sparse) ? a.total : w.seg_hi);
  w.nt = w.n_list + (w.dhi - w.dlo + kKvTile - 1) / kKvTile;  // >= 1: the tile has a row
  return w;
}
__device__ __attribute__((always_inline)) inline void kv_tile_desc(const PrefillArgs& a, const KvWalk& w, int it,
                                                                   int& kv0, int& len, bool& causal_tile) {
  if (it < w.n_list) {
    const int idx = it < w.la_n ? it : w.lb0 + (it - w.la_n);
    const int2 t = a.kept_tiles[idx];
    kv0 = __builtin_amdgcn_readfirstlane(t.x);
    len = __builtin_amdgcn_readfirstlane(t.y);
    causal_tile = false;
  } else {
    kv0 = w.dlo + kKvTile * (it - w.n_list);
    len = min(kKvTile, w.dhi - kv0);
    causal_tile = a.causal != 0;
  }
}

}  // namespace fedattn
