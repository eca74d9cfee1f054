// bf16 prefill attention on the gfx950 matrix cores: varlen, segment-aware,
// flash-style tiling with fp32 online softmax in registers.
//
// One workgroup = 4 wavefronts.  Each wavefront owns 32 query rows of one query
// head; the 4 wavefronts of a workgroup share one KV head (GQA head sharing: with
// a group of 4 query heads they are the 4 heads of the group on the same 32 rows,
// so every wave has the same KV range and nobody idles on the causal diagonal).
// KV tiles of 64 rows are staged through LDS once per workgroup.
//
// Both products run transposed so that the softmax row statistics stay inside a
// lane: S^T = K Q^T puts one query row in one lane (32 of the tile's 64 scores in
// its registers, the other 32 in lane^32), and O^T += V^T P^T consumes P^T straight
// from those registers as the MFMA B operand.  V is transposed on its way into LDS.
//
// Which KV tiles a query tile walks (Phase I / Phase II attention, causal mask of
// Section III-B, sparse KV exchange):
//   local block:  own segment, up to the diagonal;
//   sync block:   the global sequence from token 0 up to the diagonal;
//   sparse sync:  the kept 64-row tiles of the remote participants, then the own
//                 segment up to the diagonal.
// Tiles entirely above the diagonal or in other participants' segments of a local
// block are never visited; only diagonal and ragged tiles apply an element mask.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "mfma_tile.h"
#include "prefill_walk.h"
#include "row_walk.h"

namespace fedattn {

namespace {

// NG = 1: 4 wavefronts per workgroup (two or three workgroups share a CU when the grid is large
// enough, and one's matrix work overlaps the other's softmax: inside a wavefront the softmax
// sits between the two products that depend on it, and spreading it under the MFMAs of the
// neighbouring tiles instead measured slower).  Three wavefronts per SIMD where the registers allow
// it (head dimension up to 64: 8 x 2000 tokens, 32/8 heads, sync 1132 -> 1032 us against two).
// NG = 2, where the estimate of choose_prefill_launch takes it to be faster (few workgroups per
// CU): 8 wavefronts = two groups of 4 on the same query rows;
// group g takes the KV tiles j with j mod 2 == g through its own LDS stages and the two
// partial results are merged at the end (split-KV inside the workgroup).
// FOLD: the softmax scale (and the change to base 2) is folded into the Q operand and the
// reference value of the online softmax into the starting value of the score accumulation, so
// that a score comes out of the MFMAs ready for the exponential: one vector instruction less per
// score, a quarter of the softmax's (3-4 % of the kernel's time on the large workloads).  Folding
// the scale rounds q * scale to bf16 once more; the host asks for it only when the scale does not
// exceed 1/sqrt(D), where that rounding stays well below the rounding of the weights themselves.
// EXACT: the weights keep their fp32 precision in the second product (three bf16 parts each), for
// the head dimensions other than 64 and 128; DP is the head dimension padded to a multiple of 32.
// Its matrix work is (1 + 3) / 2 times that of the other kind: 8 x 2000 tokens, 32/8 heads, sync:
// 590 useful TFLOP/s at head dimension 96 (1160 at 128 without EXACT).  A local and a sync block of
// 4 x 1000..2500 tokens, 8/2 heads of 96: 190 us.
// APART: a dense sync block whose participants' matrices lie apart, its tiles loaded from where they are.
template <int DP, int NG, bool FOLD, bool EXACT, bool APART>
__global__ __launch_bounds__(256 * NG, DP > 128 ? 1 : DP > 64 ? 2 : 3) void prefill_mfma_kernel(PrefillArgs a) {
  using TL = KvTile<DP, 1, 4, kKvTile, EXACT>;
  const int D = EXACT ? a.D : DP;
  constexpr int KSTEPS = TL::KSTEPS, DT = TL::DT, TILEB = TL::TILEB;
  // Per group: K and V tiles double-buffered; the group's i-th tile lives in stage i&1.
  // Layout per group: K stage 0, K stage 1, V stage 0, V stage 1 (TILEB bytes each).
  extern __shared__ __attribute__((aligned(1024))) unsigned char kv_lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave_all >> 2;   // wavefront group (KV tile parity)
  const int wave = wave_all & 3;   // wavefront inside the group
  const int l32 = lane & 31;
  const int hf = lane >> 5;
  const lds_cptr lds0 = (lds_cptr)(lds_void_ptr)kv_lds + grp * 4 * TILEB;
  const uint32_t lds_base = lds_addr_of(kv_lds) + grp * 4 * TILEB;

  const int Hq = a.Hq, Hkv = a.Hkv;
  const int HS = a.heads_per_wg;
  const ListTab list = load_list(a, lane);
  // the tables of launches without a list with them: a second round trip there is 0.3 to 0.5 % of a launch of many rounds
  const SegTab tile_tab = load_seg_tab(a.seg.tile_cum, lane, a.seg.n);
  const SegTab pair_tab = load_seg_tab(a.seg.pair_cum, lane, a.seg.n);
  const int order_lo = a.seg_order[lane], order_hi = a.seg_order[lane + 64];
  asm volatile("" ::"v"(tile_tab.lo), "v"(pair_tab.lo), "v"(order_lo));   // not moved to where they are used
  const WgPlace wg = find_wg_place(a);
  const int g = wg.g, p = wg.p;
  const int block = blockIdx.y;

  const bool is_sync = a.sync_override >= 0 ? (a.sync_override != 0)
                                            : sync_block_rule(a.sync_interval, a.block_idx0 + block);
  const bool causal = a.causal != 0;
  const bool sparse = is_sync && a.keep_chunks != nullptr;

  // Causal work grows along the sequence (sync block) or along each segment (local
  // block); a workgroup takes one query tile, dispatched in an order that the host lays out or
  // longest walks first, or a heavy tile and then its light mirror image.
  TilePlace place_a, place_b;  // heavy tile, then its light partner
  bool two = false;            // there is one
  if (a.n_listed > 0) {
    if (a.listed_pairs) {
      place_a = place_listed(a, list, list_entry(list, 2 * p));
      const uint32_t e = list_entry(list, 2 * p + 1);
      two = e != kNoTile;
      place_b = place_listed(a, list, two ? e : 0);
    } else {
      place_a = place_b = place_listed(a, list, list_entry(list, p));
    }
    // small causal launch: the light half waits about a microsecond: its loads then queue behind those of the heavy
    // half, whose workgroups set the length of the launch (the light ones have time to spare)
    if (p >= a.late_from) __builtin_amdgcn_s_sleep(32);
  } else {
    const int N = a.seg.n, T = a.n_q_tiles;
    const SegTab seg_tab = list.seg;
    int tile_a, tile_b = -1;
    if (!causal) {
      if (p >= T) return;
      tile_a = T - 1 - p;
    } else if (a.one_tile_heavy_first) {
      // One tile per workgroup, dispatched heaviest first: in a launch of several rounds of workgroups
      // the short walks at the end of the list fill the gaps that equal-sized pairs would leave in
      // the last round, in a launch of one round each walk is half a pair's.  Sync block: work
      // grows with the position in the sequence.  Local block: the participants in order of
      // decreasing length, each one's tiles from its last to its first.
      if (p >= T) return;
      if (is_sync) {
        tile_a = T - 1 - p;
      } else {
        const int s = seg_tab_find(pair_tab, p, N);   // position in the length order
        const int pi = p - seg_tab_at(pair_tab, s);
        const int n = s < 64 ? __builtin_amdgcn_readlane(order_lo, s) : __builtin_amdgcn_readlane(order_hi, s - 64);
        tile_a = seg_tab_at(tile_tab, n + 1) - 1 - pi;
      }
    } else if (is_sync) {
      if (p >= (T + 1) / 2) return;
      tile_a = T - 1 - p;
      if (p < T - 1 - p) tile_b = p;
    } else {
      if (p >= seg_tab_at(pair_tab, N)) return;
      const int n = seg_tab_find(pair_tab, p, N);
      const int pi = p - seg_tab_at(pair_tab, n);
      const int t0 = seg_tab_at(tile_tab, n), tn = seg_tab_at(tile_tab, n + 1) - t0;
      tile_a = t0 + tn - 1 - pi;
      if (pi < tn - 1 - pi) tile_b = t0 + pi;
    }
    place_a = place_b = place_in_tables(a, seg_tab, tile_tab, tile_a);
    two = tile_b >= 0;
    if (two) place_b = place_in_tables(a, seg_tab, tile_tab, tile_b);
  }

  const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.q) + (int64_t)block * a.q_block_stride;
  const uint16_t* kp = reinterpret_cast<const uint16_t*>(a.k) + (int64_t)block * a.kv_block_stride + g * D;
  const uint16_t* vp = reinterpret_cast<const uint16_t*>(a.v) + (int64_t)block * a.kv_block_stride + g * D;
  const uint16_t* kp_list = reinterpret_cast<const uint16_t*>(a.k_list) + g * D;  // kept-tile list (one block)
  const uint16_t* vp_list = reinterpret_cast<const uint16_t*>(a.v_list) + g * D;
  uint16_t* op = reinterpret_cast<uint16_t*>(a.out) + (int64_t)block * a.q_block_stride;
  const float sc = a.scale * kLog2e;
  const int row_elems = Hkv * D;  // elements between consecutive KV rows in HBM

  TL tile_io;
  tile_io.init(lane, wave, row_elems, D / 8 - 1);

  // participants' matrices apart: with a sparse exchange the dense range of a walk is the own one's rows, which in a pair may be
  // two participants' (4 x 500 tokens, 32/8 heads of 128, a tenth of the 64-token chunks kept: 31.0 us from an aggregated copy, 29.0 in
  // pairs from where they are, 30.9 by the next best launch; 651, 1169 and 1628 tokens, 8/2 heads: 52.0 and 47.0 in pairs)
  const auto use_own_matrices = [&](int n) __attribute__((always_inline)) {
    asm volatile("");   // a branch around it, no lookup by every workgroup
    kp = own_matrix(a, n, 0) + g * D;
    vp = own_matrix(a, n, 1) + g * D;
  };
  if (!EXACT && a.apart) use_own_matrices(place_a.n);

  struct Walk : KvWalk {
    int row0w;  // first query row of this wavefront
  };
  const int wave_head = wave & (HS - 1), wave_rows = wave >> (HS >> 1);   // HS = 1, 2 or 4
  auto make_walk = [&](const TilePlace& tp, Walk& w) __attribute__((always_inline)) {
    static_cast<KvWalk&>(w) = make_kv_walk(a, tp, is_sync, sparse);
    w.row0w = w.q0 + kWaveRows * wave_rows;
  };
  // K and V tile `it` of walk w into the stage at byte offset st of this group
  ApartRows apart_rows;
  if constexpr (APART) apart_rows.init(a, lane);
  auto fetch_tile = [&](const Walk& w, int it, int st) __attribute__((always_inline)) {
    int kv0, len;
    bool ct;
    kv_tile_desc(a, w, it, kv0, len, ct);
    if constexpr (APART) {
      apart_rows.enter(a, g, kv0);
      apart_rows.template load<false>(a, tile_io, g, kv0, len, lds_base + st);
      apart_rows.template load<true>(a, tile_io, g, kv0, len, lds_base + 2 * TILEB + st);
      return;
    }
    const bool listed = it < w.n_list;
    tile_io.template dma<false>((listed ? kp_list : kp) + (int64_t)kv0 * row_elems, lds_base + st, len);
    tile_io.template dma<true>((listed ? vp_list : vp) + (int64_t)kv0 * row_elems, lds_base + 2 * TILEB + st, len);
  };
  const int head = g * a.group + wg.set * HS + wave_head;
  // Q fragments (B operand of S^T): lane (q row = l32, half hf) holds
  // Q[row][16*step + 8*hf .. +8].
  auto load_q = [&](const Walk& w, bf16x8 (&qf)[KSTEPS]) __attribute__((always_inline)) {
    const int row_ld = min(w.row0w + l32, w.seg_hi - 1);
    const uint16_t* qrow = qp + ((int64_t)row_ld * Hq + head) * D + 8 * hf;
#pragma unroll
    for (int st = 0; st < KSTEPS; ++st)
      qf[st] = __builtin_bit_cast(bf16x8, !EXACT || 16 * st + 8 * hf < D ? *reinterpret_cast<const u32x4*>(qrow + 16 * st)
                                                                         : u32x4{0u, 0u, 0u, 0u});
  };

  // The first walk's Q rows come through LDS instead: loaded as above, an instruction touches
  // 32 rows (32 bytes of each) and a launch of a few thousand tokens spends its first
  // microsecond in the address path.  Here the wavefront moves its 32 x D tile with whole-row
  // direct-to-LDS loads (4 rows of 2 D bytes per instruction) into the half of a K or V stage
  // that the first tile does not use, in the K tile's swizzled layout, and reads the fragments
  // back like K fragments.  Nobody else touches that half before the barrier below.
  constexpr int QINST = kWaveRows * TL::ROWB / 1024;  // load instructions per wavefront
  const int q_lds = (wave >> 1) * 2 * TILEB + TILEB + (wave & 1) * (TILEB / 2);  // byte offset in the group's stages
  auto fetch_q_lds = [&](const Walk& w) __attribute__((always_inline)) {
    const int rbase = min(w.row0w, w.seg_hi - 1);
    const uint16_t* qbase = qp + ((int64_t)rbase * Hq + head) * D;
#pragma unroll
    for (int i = 0; i < QINST; ++i) {
      const int sidx = i * 64 + lane;
      const int row = sidx / TL::CPR, cp = sidx % TL::CPR;
      const int row_ld = min(w.row0w + row, w.seg_hi - 1) - rbase;  // >= 0
      const int chunk = tile_io.stored_chunk(cp ^ TL::k_swizzle(row));
      const uint32_t off = (uint32_t)(row_ld * (Hq * D) + chunk * 8) * 2u;
      lds_dma_16(qbase, off, lds_base + q_lds + i * 1024);
    }
  };
  auto read_q_lds = [&](bf16x8 (&qf)[KSTEPS]) __attribute__((always_inline)) {
#pragma unroll
    for (int st = 0; st < KSTEPS; ++st)
      qf[st] = __builtin_bit_cast(
          bf16x8, *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(lds0 + (q_lds + tile_io.k_off[st])));
    if constexpr (EXACT) {   // the padded columns are zero
#pragma unroll
      for (int st = 0; st < KSTEPS; ++st)
        if (16 * st + 8 * hf >= D) qf[st] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
    }
  };

  // The workgroup's walks run as one pipeline: the stage parity carries on from the
  // first walk into the second, whose first tile and Q fragments are fetched while
  // the first walk finishes.
  Walk cur, nxt;
  make_walk(place_a, cur);
  bf16x8 qf[KSTEPS];
  fetch_q_lds(cur);
  if (grp < cur.nt) fetch_tile(cur, grp, 0);
  nxt = cur;
  unsigned warm = 0;
  if (two) {
    make_walk(place_b, nxt);
    // pull the second walk's Q rows into L2 now (one dword per 128-byte line)
    const int row_ld = min(nxt.row0w + l32, nxt.seg_hi - 1);
    warm = *reinterpret_cast<const unsigned*>(qp + ((int64_t)row_ld * Hq + head) * D + (hf * 64) % D);
  }
  // Small problems (all of a KV head's K and V fit in L2 with room to spare): the launch starts
  // with every workgroup asking HBM for its Q rows and first tile at once, and the later tiles
  // of the long walks would each be one more cold miss behind that burst.  Instead the K and V
  // rows of the workgroup's own query rows are requested now, one dword per 128-byte line; all
  // workgroups together cover every row, and the walks then find their tiles in L2.
  unsigned warm_k = 0;
  if (!EXACT && a.warm_kv && grp == 0) {
    constexpr int LPR = TL::ROWB / 128;  // 128-byte lines per K/V row
    const int sub = wave_head;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if ((i & (HS - 1)) != sub || (i >= 2 && !two)) continue;   // wave-uniform
      const Walk& w = i >= 2 ? nxt : cur;
      const int row = min(w.row0w + lane / LPR, w.seg_hi - 1);
      const uint16_t* base = (i & 1) ? vp : kp;
      warm_k += *reinterpret_cast<const unsigned*>(base + (int64_t)row * row_elems + (lane % LPR) * 64);
    }
  }
  int git = 0;  // iterations this workgroup has run: stage of an iteration = git & 1
  // EXACT: the wavefront's rows that came out not finite, per walk (in LDS: its registers are all in use)
  struct OddRows { uint32_t odd; int row0; };
  __shared__ OddRows odd_s[4][2];
  if (EXACT && grp == 0) odd_s[wave][0].odd = odd_s[wave][1].odd = 0;

  for (int part = 0;; ++part) {
    const bool more = part == 0 && two;
    const int my_row = cur.row0w + l32;
    f32x16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
    float m_run = -INFINITY;  // row maximum the accumulators refer to, log2 domain
    float l_run = 0.f;        // this lane's share of the row sum
    f32x16 neg_ref;           // FOLD: minus that reference (0 while there is none) in every element; else zeros
#pragma unroll
    for (int e = 0; e < 16; ++e) neg_ref[e] = 0.f;

    const int n_it = (cur.nt + NG - 1) / NG;  // iterations of the workgroup (uniform: they carry barriers)
    wait_vmcnt<0>();
    if (part == 0) {
      asm volatile("" ::"v"(warm), "v"(warm_k));
      read_q_lds(qf);  // this wavefront's own loads: landed with the wait above; the barrier waits for the reads
    }
    if constexpr (FOLD) {
#pragma unroll
      for (int st = 0; st < KSTEPS; ++st)
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[st][e] = (bf16_t)((float)qf[st][e] * sc);
    }
    __syncthreads();

    // ---- main loop: the group's i-th tile is computed from one stage while its next tile
    // (in the last iteration: the first tile of the next walk) streams into the other ---------
    for (int it = 0; it < n_it; ++it, ++git) {
      const int j = it * NG + grp;
      const int st_cur = (git & 1) * TILEB;
      const int st_nxt = TILEB - st_cur;
      if (it + 1 < n_it) {
        if (j + NG < cur.nt) fetch_tile(cur, j + NG, st_nxt);
      } else if (more) {  // last iteration of the first walk: start on the second walk
        if constexpr (NG == 2 && !EXACT && !APART)   // pairs of one block are of this kind
          if (a.apart) use_own_matrices(place_b.n);
        if (grp < nxt.nt) fetch_tile(nxt, grp, st_nxt);
      }

      if (j < cur.nt) {
        int kv0, len;
        bool causal_tile;
        kv_tile_desc(a, cur, j, kv0, len, causal_tile);
        f32x16 s_cur[2];
        tile_io.scores(lds0, st_cur, qf, neg_ref, s_cur);

        if (len < kKvTile || (causal_tile && kv0 + kKvTile - 1 > cur.row0w)) {
          // valid kv rows of this tile for this lane's query: [0, lim)
          int lim = len;
          if (causal_tile) lim = min(lim, my_row - kv0 + 1);
          mask_scores(s_cur, lim, hf);
        }

        if constexpr (EXACT) {
          const float m_use = softmax_max(s_cur, sc, m_run, l_run, o);
          softmax_exp_f32(s_cur, sc, m_use, l_run);
          tile_io.pv_f32(lds0, 2 * TILEB + st_cur, s_cur, o);
        } else {
          bf16x8 pb[4];
          if constexpr (FOLD) softmax_step_rel(s_cur, m_run, l_run, o, neg_ref, pb);
          else softmax_step(s_cur, sc, m_run, l_run, o, pb);
          tile_io.pv(lds0, 2 * TILEB + st_cur, pb, o);
        }
      }

      wait_vmcnt<0>();
      __syncthreads();
    }

    // This walk's Q fragments are dead: fetch the next walk's behind the epilogue.  With two
    // groups the hand-over barrier comes first (group 1 has nothing else to do after it;
    // group 0 loads once it has taken group 1's partial results over).
    if (NG == 1 && more) load_q(nxt, qf);

    if constexpr (NG == 2) {
      // ---- merge the two groups: group 1 hands (m, l, O) to group 0 through LDS.  The K and
      // V stages of the last iteration are free in both groups (the other stages may be
      // receiving the next walk's first tiles): wave w gets one of these four buffers.
      __shared__ float xml[4 * 128];
      const int st_free = ((git - 1) & 1) * TILEB;
      f32x4* xo = reinterpret_cast<f32x4*>(kv_lds + (wave >> 1) * 4 * TILEB + (wave & 1) * 2 * TILEB + st_free) + lane;
      float* xm = xml + wave * 128 + lane;
      if (grp == 1) {
        xm[0] = m_run;
        xm[64] = l_run;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq)
            xo[(4 * dt + vq) * 64] = f32x4{o[dt][4 * vq], o[dt][4 * vq + 1], o[dt][4 * vq + 2], o[dt][4 * vq + 3]};
      }
      // LDS-only hand-over: wait for the LDS writes, not for the loads in flight for the next walk
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
      if (grp == 1 && more) load_q(nxt, qf);
      if (grp == 0) {
        const float m1 = xm[0], l1 = xm[64];
        const float mm = fmaxf(m_run, m1);
        const float mu = (mm == -INFINITY) ? 0.f : mm;
        const float f0 = __builtin_amdgcn_exp2f(m_run - mu), f1 = __builtin_amdgcn_exp2f(m1 - mu);
        l_run = l_run * f0 + l1 * f1;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) {
            const f32x4 x = xo[(4 * dt + vq) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[dt][4 * vq + e] = o[dt][4 * vq + e] * f0 + x[e] * f1;
          }
        if (more) load_q(nxt, qf);
      }
    }

    // ---- normalise and write: the wave's 32 x D tile goes through a free LDS stage so
    // that every store instruction writes whole rows (a lane owns a row in registers, which
    // written directly would scatter 16-byte pieces over 32 rows per instruction) ----------
    const float l_tot = sum_across_halves(l_run);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    if (grp == 0) {
      constexpr int ROWB = TL::ROWB, CPR = TL::CPR;
      const int st_free = ((git - 1) & 1) * TILEB;
      unsigned char* stage = NG == 2 ? kv_lds + (wave >> 1) * 4 * TILEB + (wave & 1) * 2 * TILEB + st_free
                                     : kv_lds + (wave >> 1) * 2 * TILEB + st_free + (wave & 1) * (TILEB / 2);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          bf16x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = (bf16_t)(o[dt][4 * vq + e] * inv);
          const int c = 4 * dt + vq;
          *reinterpret_cast<u32x2*>(stage + l32 * ROWB + ((c ^ TL::k_swizzle(l32)) << 4) + 8 * hf) =
              __builtin_bit_cast(u32x2, w);
        }
      FiniteCheckBf16 fin;
#pragma unroll
      for (int kk = 0; kk < kWaveRows * CPR / 64; ++kk) {
        const int r = (kk * 64 + lane) / CPR, c = (kk * 64 + lane) % CPR;
        const u32x4 w = *reinterpret_cast<const u32x4*>(stage + r * ROWB + ((c ^ TL::k_swizzle(r)) << 4));
        if constexpr (EXACT) fin.add8(w);
        if (cur.row0w + r < cur.seg_hi && (!EXACT || 8 * c < D))
          // streaming store: the rows are not read again in this launch, and written through
          // now they are not left for the write-back at the end of the kernel
          __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(op + ((int64_t)(cur.row0w + r) * Hq + head) * D + 8 * c));
      }
      if constexpr (EXACT) {
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(fin.failed()) != 0, 0)) {   // which rows
          if (lane == 0) odd_s[wave][part].row0 = cur.row0w;
#pragma unroll 1
          for (int kk = 0; kk < kWaveRows * CPR / 64; ++kk) {
            const int r = (kk * 64 + lane) / CPR, c = (kk * 64 + lane) % CPR;
            FiniteCheckBf16 piece;
            piece.add8(*reinterpret_cast<const u32x4*>(stage + r * ROWB + ((c ^ TL::k_swizzle(r)) << 4)));
            if (cur.row0w + r < cur.seg_hi && 8 * c < D && piece.failed()) atomicOr(&odd_s[wave][part].odd, 1u << r);
          }
        }
      }
    }
    if (!more) break;
    cur = nxt;
  }
  if constexpr (EXACT) {
    if (grp == 0) {
#pragma unroll 1
      for (int part = 0; part < 2; ++part) {
        const uint32_t odd = __builtin_amdgcn_readfirstlane(odd_s[wave][part].odd);
        if (__builtin_expect(odd != 0, 0))
          redo_prefill_rows<uint16_t, 1>(__builtin_amdgcn_readfirstlane(odd_s[wave][part].row0), odd, head, [](int) { return true; });
      }
    }
  }
}

// ---- keep-lists of a sync block -----------------------------------------------------------------
// The attention kernels walk a list of kept 64-row KV tiles, participant after participant, with the
// number of kept tiles before each participant beside it.  Nothing here moves much data: what counts is
// the chain of dependent memory accesses, and the launches.

// This lane's share of the flags set in keep[0 .. nc).
__device__ inline int lane_flags(const uint8_t* keep, int nc, int lane) {
  int n = 0;
#pragma unroll 4
  for (int c = lane; c < nc; c += 64) n += keep[c] != 0 ? 1 : 0;
  return n;
}
__device__ inline int wave_sum_int(int x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// One wavefront: cnt[n] tiles of participant n (zero from N on) -> tiles of the participants before it, cnt[N] = all.
__device__ inline void sum_before(int (&cnt)[kMaxP + 1], int N, int lane, int32_t* kept_cum) {
  static_assert(kMaxP == 128, "two participants per lane");
  const int x0 = cnt[2 * lane], x1 = cnt[2 * lane + 1];
  int incl = x0 + x1;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  const int before = incl - x0 - x1;
  cnt[2 * lane] = before;
  cnt[2 * lane + 1] = before + x0;
  if (lane == 63) cnt[kMaxP] = incl;
  if (2 * lane <= N) kept_cum[2 * lane] = before;
  if (2 * lane + 1 <= N) kept_cum[2 * lane + 1] = before + x0;
  if (N == kMaxP && lane == 63) kept_cum[kMaxP] = incl;
}

// Keep chunks of whole tiles: the list of the kept tiles where they are, one wavefront per participant
// (16 participants of 64 chunks: 22 us with one thread each, 5 us now; a launch alone takes 4 in the same trace).
constexpr int kListWaves = 16;
__global__ __launch_bounds__(64 * kListWaves) void build_kept_tiles_kernel(PrefillArgs a, int2* kept_tiles, int32_t* kept_cum) {
  __shared__ int cnt[kMaxP + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int N = a.seg.n;
  const int tpc = a.chunk_tokens / kKvTile;   // tiles of a chunk; the last one of a participant may have fewer
  if (tid <= kMaxP) cnt[tid] = 0;
  __syncthreads();
  for (int n = wave; n < N; n += kListWaves) {
    const uint8_t* keep = a.keep_chunks + a.seg.chunk_cum[n];
    const int nc = a.seg.chunk_cum[n + 1] - a.seg.chunk_cum[n];
    int tiles = lane_flags(keep, nc, lane) * tpc;
    if (nc > 0 && lane == 0 && keep[nc - 1]) {
      const int len = a.seg.seg_off[n + 1] - a.seg.seg_off[n] - (nc - 1) * a.chunk_tokens;
      tiles -= tpc - (len + kKvTile - 1) / kKvTile;
    }
    tiles = wave_sum_int(tiles);
    if (lane == 0) cnt[n] = tiles;
  }
  __syncthreads();
  if (wave == 0) sum_before(cnt, N, lane, kept_cum);
  __syncthreads();
  for (int n = wave; n < N; n += kListWaves) {
    const int lo = a.seg.seg_off[n], hi = a.seg.seg_off[n + 1];
    const uint8_t* keep = a.keep_chunks + a.seg.chunk_cum[n];
    const int nc = a.seg.chunk_cum[n + 1] - a.seg.chunk_cum[n];
    int w0 = cnt[n];
    for (int c0 = 0; c0 < nc; c0 += 64) {
      const int c = c0 + lane;
      const bool flag = c < nc && keep[c] != 0;
      const unsigned long long set = __builtin_amdgcn_ballot_w64(flag);
      if (flag) {
        const int start = lo + c * a.chunk_tokens;
        const int clen = min(a.chunk_tokens, hi - start);
        int w = w0 + __builtin_popcountll(set & ((1ull << lane) - 1ull)) * tpc;
        for (int t = 0; t < clen; t += kKvTile) kept_tiles[w++] = make_int2(start + t, min(kKvTile, clen - t));
      }
      w0 += __builtin_popcountll(set) * tpc;
    }
  }
}

// Keep chunks finer than a tile (down to single tokens): each participant's kept rows are gathered
// into the front of its own segment of a packed K, V copy, so that the attention kernel still walks
// dense tiles.  Among remote rows only membership matters (a remote participant lies entirely before or
// entirely after the query in the global order), so packing loses nothing.
// Workgroup (x, m, z): rows [x span, (x + 1) span) of participant m, of K (z = 0) or V.  It counts the kept
// rows before its own by reading the participant's flags over again; span is at least a 64th of the longest
// segment, so that this stays a few reads per flag.  The workgroups of the last x write the tile list.
// (8 participants of 300..1500 rows of 1 KB, single tokens: a scan, a list and a gather kernel took
// 4.8 + 4.8 + 5.2 us under a profiler that shows 4 us for an empty one; now one launch.)
// Matrices that lie apart are read where they are: the copy holds kept rows only, and the attention kernels' workgroups read
// their own participant's rows there, too (an aggregated copy of all rows before it was a launch of its own: 8 participants of 300..1500 rows, 16/4 heads of 128, single tokens, 30 % kept: 103.6 -> 95.5 us).
constexpr int kPackThreads = 512;
__global__ __launch_bounds__(kPackThreads) void pack_kept_rows_kernel(PackArgs a) {
  constexpr int NW = kPackThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int N = a.n, row_vecs = a.row_vecs, span = a.span;
  if (blockIdx.x == gridDim.x - 1) {
    // packed rows of participant n: [seg_off[n], + kept rows), in tiles of 64 of which the last is ragged
    __shared__ int cnt[kMaxP + 1], rows[kMaxP];
    if (blockIdx.y != 0 || blockIdx.z != 0) return;
    if (tid <= kMaxP) cnt[tid] = 0;
    __syncthreads();
    for (int n = wave; n < N; n += NW) {
      const uint8_t* keep = a.keep_chunks + a.chunk_cum[n];
      const int nc = a.chunk_cum[n + 1] - a.chunk_cum[n];
      int kept = lane_flags(keep, nc, lane) * a.chunk_tokens;
      if (nc > 0 && lane == 0 && keep[nc - 1]) kept -= nc * a.chunk_tokens - (a.seg_off[n + 1] - a.seg_off[n]);
      kept = wave_sum_int(kept);
      if (lane == 0) {
        rows[n] = kept;
        cnt[n] = (kept + kKvTile - 1) / kKvTile;
      }
    }
    __syncthreads();
    if (wave == 0) sum_before(cnt, N, lane, a.kept_cum);
    __syncthreads();
    for (int n = wave; n < N; n += NW) {
      const int lo = a.seg_off[n];
      for (int i = lane; i * kKvTile < rows[n]; i += 64) a.kept_tiles[cnt[n] + i] = make_int2(lo + i * kKvTile, min(kKvTile, rows[n] - i * kKvTile));
    }
    return;
  }

  __shared__ int wave_cnt[NW];
  __shared__ int from[kPackThreads];   // kept rows of this round
  const int m = blockIdx.y;
  const int lo = a.seg_off[m], hi = a.seg_off[m + 1];
  const int64_t first64 = lo + (int64_t)blockIdx.x * span;
  if (first64 >= hi) return;
  const int first = (int)first64, last = min(first64 + span, (int64_t)hi);
  const uint8_t* keep = a.keep_chunks + a.chunk_cum[m];
  const uint4* __restrict__ src = reinterpret_cast<const uint4*>(a.apart ? a.own[2 * m + blockIdx.z] : blockIdx.z == 0 ? a.k : a.v);
  uint4* __restrict__ dst = blockIdx.z == 0 ? a.k_packed : a.v_packed;

  const int c_first = (first - lo) / a.chunk_tokens;   // chunk of the first row; those before it are whole
  int n = 0;
  for (int c = tid; c < c_first; c += kPackThreads) n += keep[c] != 0 ? 1 : 0;
  n = wave_sum_int(n);
  if (lane == 0) wave_cnt[wave] = n;
  __syncthreads();
  n = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) n += wave_cnt[w];
  int to = lo + n * a.chunk_tokens;   // packed row of the next kept one
  if (keep[c_first]) to += first - lo - c_first * a.chunk_tokens;

  for (int base = first; base < last; base += kPackThreads) {
    const int t = base + tid;
    const bool flag = t < last && keep[(t - lo) / a.chunk_tokens] != 0;
    const unsigned long long set = __builtin_amdgcn_ballot_w64(flag);
    __syncthreads();   // wave_cnt and from have been read
    if (lane == 0) wave_cnt[wave] = __builtin_popcountll(set);
    __syncthreads();
    int pos = __builtin_popcountll(set & ((1ull << lane) - 1ull)), kept = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      pos += w < wave ? wave_cnt[w] : 0;
      kept += wave_cnt[w];
    }
    if (flag) from[pos] = t;
    __syncthreads();
#pragma unroll 4
    for (int i = tid; i < kept * row_vecs; i += kPackThreads) {
      const int r = i / row_vecs, v = i - r * row_vecs;
      dst[(int64_t)(to + r) * row_vecs + v] = src[(int64_t)from[r] * row_vecs + v];
    }
    to += kept;
  }
}

}  // namespace

hipError_t launch_pack_kept_rows(PackArgs& a, hipStream_t s) {
  int max_len = 1;
  for (int n = 0; n < a.n; ++n) max_len = max(max_len, a.seg_off[n + 1] - a.seg_off[n]);
  a.span = (max_len - 1) / 4096 * 64 + 64;
  const dim3 grid((unsigned)((max_len - 1) / a.span + 2), (unsigned)a.n, 2);
  return launch_with(&pack_kept_rows_kernel, grid, dim3(kPackThreads), 0, s, a);
}

template <int DP, int NG, bool FOLD, bool EXACT, bool APART = false>
hipError_t launch_prefill_mfma_t(const PrefillArgs& a, dim3 grid, hipStream_t s) {
  constexpr int smem = NG * 4 * KvTile<DP, 1>::TILEB;
  static std::atomic<uint64_t> attr_done{0};
  hipError_t e0 = set_max_dynamic_lds_once(attr_done, reinterpret_cast<const void*>(&prefill_mfma_kernel<DP, NG, FOLD, EXACT, APART>), smem);
  if (e0 != hipSuccess) return e0;
  return launch_with(&prefill_mfma_kernel<DP, NG, FOLD, EXACT, APART>, grid, dim3(256 * NG), smem, s, a);
}

template <int DP>
hipError_t launch_prefill_exact(const PrefillArgs& a, bool wide, dim3 grid, hipStream_t s) {
  if constexpr (DP <= 128)
    if (wide) return launch_prefill_mfma_t<DP, 2, false, true>(a, grid, s);
  return launch_prefill_mfma_t<DP, 1, false, true>(a, grid, s);
}

hipError_t launch_prefill_mfma(PrefillArgs& a, int n_blocks, hipStream_t s) {
  if (a.n_q_tiles == 0 || n_blocks == 0) return hipSuccess;
  lay_out_heads(a);
  TileList list(a);
  a.late_from = INT32_MAX;
  // one block whose K and V of a KV head are at most 2 MB: the workgroups pull them into L2 up front
  a.warm_kv = (n_blocks == 1 && a.keep_chunks == nullptr && (int64_t)a.total * a.D * 4 <= (2 << 20)) ? 1 : 0;
  const int G = a.Hq / a.Hkv;
  const int per_tile = a.Hkv * (G / a.heads_per_wg);  // workgroups per query tile (or pair)
  // causal: query tiles are paired; a local block pairs inside each segment, which
  // needs at least as many workgroups as the sequence-wide pairing of a sync block
  dim3 grid((unsigned)((a.causal ? a.seg.pair_cum[a.seg.n] : a.n_q_tiles) * per_tile), (unsigned)n_blocks, 1);
  // scale folded into Q only up to the usual 1/sqrt(D): its rounding error grows with the scale
  const bool exact = a.D != 64 && a.D != 128;
  const bool fold = !exact && folds_scale(a.scale, a.D);
  // several blocks in one launch (local and sync ones mixed): pairs, in 8-wavefront workgroups where
  // there would be fewer than two 4-wavefront ones per CU
  bool wide = (int64_t)grid.x * grid.y < 2 * (int64_t)a.n_cus && a.D <= 128;
  if (n_blocks == 1) {
    const bool is_sync = a.sync_override >= 0 ? a.sync_override != 0 : sync_block_rule(a.sync_interval, a.block_idx0);
    const PrefillLaunch plan = launch_to_take(PrefillShape{a.seg.seg_off, a.seg.n, a.Hq, a.Hkv, a.D, a.causal != 0, a.keep_chunks != nullptr,
                                                                  a.heads_per_wg, a.q_tile_rows, a.n_cus}, is_sync);
    if (plan == kSplit) return launch_prefill_split(a, fold, s);
    wide = plan == kEight || plan == kEightPairs;
    if (a.apart && plan == kEightPairs) a.warm_kv = 0;   // it looks for a pair's rows in one participant's matrices
    if (plan == kFourOrdered) {
      // All workgroups are resident at once, two per CU.  Order: heavy half first, heaviest first;
      // then the light half, lightest first, so that the workgroups that come to share a CU
      // (index p and p + half, dispatched in order) carry about the same load together.
      struct Item { int n, t, work; };
      Item items[kMaxListedTiles];
      int cnt = 0;
      for (int n = 0; n < a.seg.n; ++n) {
        const int lo = a.seg.seg_off[n], hi = a.seg.seg_off[n + 1];
        for (int t = 0; t < list.tiles(n); ++t) {
          const int last = min(lo + (t + 1) * a.q_tile_rows, hi);  // one past the tile's last row
          items[cnt++] = Item{n, t, (last - (is_sync ? 0 : lo) + kKvTile - 1) / kKvTile};
        }
      }
      std::stable_sort(items, items + cnt, [](const Item& x, const Item& y) { return x.work > y.work; });
      const int half = (cnt + 1) / 2;
      for (int i = 0; i < cnt; ++i) list.put(i < half ? i : cnt - 1 - (i - half), TileList::entry(items[i].n, items[i].t));
      a.n_listed = cnt;
      a.late_from = half;
      grid.x = (unsigned)(cnt * per_tile);
    } else if (plan == kEightPairs) {
      if (TileList::fits(a, 2)) {   // at most as many pairs as tiles
        const int T = a.n_q_tiles;
        int cnt = 0;
        uint32_t all[kMaxListedTiles];
        for (int n = 0, i = 0; n < a.seg.n; ++n)
          for (int t = 0; t < list.tiles(n); ++t) all[i++] = TileList::entry(n, t);
        const auto pair_up = [&](int t0, int tn) {   // tiles [t0, t0 + tn): the last with the first and so on
          for (int i = 0; i < (tn + 1) / 2; ++i, ++cnt) {
            list.put(2 * cnt, all[t0 + tn - 1 - i]);
            list.put(2 * cnt + 1, i < tn - 1 - i ? all[t0 + i] : kNoTile);
          }
        };
        if (is_sync) pair_up(0, T);
        else for (int n = 0; n < a.seg.n; ++n) pair_up(a.seg.tile_cum[n], list.tiles(n));
        a.n_listed = cnt;
        a.listed_pairs = 1;
        grid.x = (unsigned)(cnt * per_tile);
      }
    } else {
      if (a.causal) a.one_tile_heavy_first = 1;
      if (a.causal && !is_sync) order_segments_by_length(a);
      grid.x = (unsigned)(a.n_q_tiles * per_tile);
      list_heavy_first(a, is_sync || !a.causal);
    }
  }
  if (exact) {
    switch ((a.D + 31) / 32) {
      case 1: return launch_prefill_exact<32>(a, wide, grid, s);
      case 2: return launch_prefill_exact<64>(a, wide, grid, s);
      case 3: return launch_prefill_exact<96>(a, wide, grid, s);
      case 4: return launch_prefill_exact<128>(a, wide, grid, s);
      case 5: return launch_prefill_exact<160>(a, wide, grid, s);
      case 6: return launch_prefill_exact<192>(a, wide, grid, s);
      case 7: return launch_prefill_exact<224>(a, wide, grid, s);
      default: return launch_prefill_exact<256>(a, wide, grid, s);
    }
  }
  if (a.apart && a.keep_chunks == nullptr) {   // scales that are folded only
    if (a.D == 128) return wide ? launch_prefill_mfma_t<128, 2, true, false, true>(a, grid, s) : launch_prefill_mfma_t<128, 1, true, false, true>(a, grid, s);
    return wide ? launch_prefill_mfma_t<64, 2, true, false, true>(a, grid, s) : launch_prefill_mfma_t<64, 1, true, false, true>(a, grid, s);
  }
  if (a.D == 128) {
    if (fold) return wide ? launch_prefill_mfma_t<128, 2, true, false>(a, grid, s) : launch_prefill_mfma_t<128, 1, true, false>(a, grid, s);
    return wide ? launch_prefill_mfma_t<128, 2, false, false>(a, grid, s) : launch_prefill_mfma_t<128, 1, false, false>(a, grid, s);
  }
  if (fold) return wide ? launch_prefill_mfma_t<64, 2, true, false>(a, grid, s) : launch_prefill_mfma_t<64, 1, true, false>(a, grid, s);
  return wide ? launch_prefill_mfma_t<64, 2, false, false>(a, grid, s) : launch_prefill_mfma_t<64, 1, false, false>(a, grid, s);
}

hipError_t launch_build_kept_tiles(const PrefillArgs& a, int2* kept_tiles, int32_t* kept_cum,
                                   hipStream_t s) {
  hipLaunchKernelGGL(build_kept_tiles_kernel, dim3(1), dim3(64 * kListWaves), 0, s, a, kept_tiles, kept_cum);
  return hipGetLastError();
}

}  // namespace fedattn
