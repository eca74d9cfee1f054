// bf16 prefill attention for launches too small to fill the chip with one workgroup per (32 query rows,
// KV head): here a workgroup is one query head's 32 rows, and its 8 wavefronts share the keys out among
// them.  Wavefront w walks the 32-key tiles w, w + 8, ... through LDS buffers of its own (no barrier in
// the walk), with the products and the online softmax of prefill_mfma.hip; the eight partial results
// meet in LDS at the end.
//
// A walk is eight times shorter than with 4-wavefront workgroups and there are four times as many
// workgroups (four heads per KV head), but every head loads K and V for itself: from about one
// workgroup per CU on the launch is bound by L2 -> LDS loads (128 KB per 256 keys and 32 rows at head
// dimension 128, 64 bytes per cycle and CU).  Sync blocks, before and after: 1000 tokens, 8 heads 26 -> 11 us;
// 4 x 448 tokens, 8/2 heads 36 -> 21; 4000 tokens, 4/1 heads 65 -> 37; 8 x 700 tokens, 4/1 heads of 64
// 60 -> 32.  With 64 query rows or two heads per wavefront (half the loads per row) a walk took twice as
// long: one wavefront per SIMD, nothing to cover its softmax.  Tiles double-buffered in LDS (one workgroup
// per CU instead of two at head dimension 64) measured 22 % slower with two workgroups' worth of work per CU.
#include <type_traits>

#include "common.h"
#include "half_tile.h"
#include "mfma_tile.h"
#include "prefill_walk.h"
#include "row_walk.h"

namespace fedattn {

namespace {

constexpr int kSplitWaves = 8;

// Waits that also keep the compiler from moving LDS accesses across them: a wavefront's buffers are its
// own here, so no barrier stands between the loads into them and the reads.
template <int N>
__device__ inline void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ inline void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// FOLD, EXACT, DP: as in prefill_mfma.hip
template <int DP, bool FOLD, bool EXACT, bool APART>
__global__ __launch_bounds__(64 * kSplitWaves, DP > 64 ? 2 : 4) void prefill_split_kernel(PrefillArgs a) {
  constexpr int KS = kSplitWaves;
  using TL = KvTile<DP, 1, 1, kSplitRows, EXACT>;
  constexpr int KSTEPS = TL::KSTEPS, DT = TL::DT, TILEB = TL::TILEB, ROWB = TL::ROWB, CPR = TL::CPR;
  constexpr int WAVEB = 2 * TILEB;           // a wavefront's share: K tile, V tile; in the end its partial result
  constexpr int NT = 64 * KS;
  extern __shared__ __attribute__((aligned(1024))) unsigned char kv_lds[];  // the shares, then the Q tile (in the end the output)
  __shared__ float ml_s[KS][2][64];
  __shared__ uint32_t odd_s;   // EXACT: rows that came out not finite
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hf = lane >> 5;
  unsigned char* own = kv_lds + wave * WAVEB;
  unsigned char* q_lds = kv_lds + KS * WAVEB;
  const lds_cptr lds0 = (lds_cptr)(lds_void_ptr)own;
  const uint32_t lds_base = lds_addr_of(own);

  const int Hq = a.Hq, Hkv = a.Hkv;
  const int D = EXACT ? a.D : DP;

  // workgroup -> (KV head, head of its group, query tile), longest walks first
  const ListTab list = load_list(a, lane);
  const WgPlace wg = find_wg_place(a);
  const int g = wg.g, head = g * a.group + wg.set;
  const bool is_sync = a.sync_override >= 0 ? (a.sync_override != 0) : sync_block_rule(a.sync_interval, a.block_idx0);
  const bool causal = a.causal != 0;
  const bool sparse = is_sync && a.keep_chunks != nullptr;
  const TilePlace place = place_heavy_first(a, list, wg.p, is_sync, lane);
  const KvWalk w = make_kv_walk(a, place, is_sync, sparse);
  const int row0 = w.q0;

  const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.q);
  const uint16_t* kp = reinterpret_cast<const uint16_t*>(a.k) + g * D;
  const uint16_t* vp = reinterpret_cast<const uint16_t*>(a.v) + g * D;
  const uint16_t* kp_list = reinterpret_cast<const uint16_t*>(a.k_list) + g * D;
  const uint16_t* vp_list = reinterpret_cast<const uint16_t*>(a.v_list) + g * D;
  if (!EXACT && a.apart) {   // matrices apart: the dense range is the own participant's rows
    asm volatile("");   // a branch: looked up by every workgroup and selected, they cost 0.25 us of a 6 us call
    kp = own_matrix(a, place.n, 0) + g * D;
    vp = own_matrix(a, place.n, 1) + g * D;
  }
  uint16_t* op = reinterpret_cast<uint16_t*>(a.out);
  const float sc = a.scale * kLog2e;
  const int row_elems = Hkv * D;
  TL tile_io;
  tile_io.init(lane, 0, row_elems, D / 8 - 1);

  // 32-key tiles of the walk: every listed 64-row tile is two (the second one may be empty), then the dense range
  const int n_list = 2 * w.n_list;
  const int nt = n_list + (w.dhi - w.dlo + kSplitRows - 1) / kSplitRows;
  struct Tile {
    const uint16_t *k, *v;   // first row to load
    int kv0, len, load_len;
    bool causal_tile;
  };
  auto tile_at = [&](int it) __attribute__((always_inline)) {
    Tile t;
    int first;
    if (it < n_list) {
      const int i2 = it >> 1;
      const int2 e = a.kept_tiles[i2 < w.la_n ? i2 : w.lb0 + (i2 - w.la_n)];
      const HalfTile h = half_of_tile(__builtin_amdgcn_readfirstlane(e.x), __builtin_amdgcn_readfirstlane(e.y), it & 1);
      t.kv0 = h.kv0;
      t.len = h.len;
      t.load_len = h.load_len;
      first = h.load0;
      t.causal_tile = false;
    } else {
      t.kv0 = first = w.dlo + kSplitRows * (it - n_list);
      t.len = t.load_len = min(w.dhi - t.kv0, kSplitRows);
      t.causal_tile = causal;
    }
    t.k = (it < n_list ? kp_list : kp) + (int64_t)first * row_elems;
    t.v = (it < n_list ? vp_list : vp) + (int64_t)first * row_elems;
    return t;
  };

  ApartRows apart_rows;
  if constexpr (APART) apart_rows.init(a, lane);
  auto load_k = [&](const Tile& t) __attribute__((always_inline)) {
    if constexpr (APART) apart_rows.enter(a, g, t.kv0);
    if constexpr (APART) apart_rows.template load<false>(a, tile_io, g, t.kv0, t.load_len, lds_base);
    else tile_io.template dma<false>(t.k, lds_base, t.load_len);
  };
  auto load_v = [&](const Tile& t) __attribute__((always_inline)) {
    if constexpr (APART) apart_rows.template load<true>(a, tile_io, g, t.kv0, t.load_len, lds_base + TILEB);   // of the tile K was loaded of last
    else tile_io.template dma<true>(t.v, lds_base + TILEB, t.load_len);
  };

  // Q tile (whole rows, K's swizzled layout): the wavefronts share the loads out among them
  constexpr int QTILEB = kWaveRows * ROWB;
#pragma unroll
  for (int i0 = 0; i0 < QTILEB / 1024; i0 += KS) {
    const int i = i0 + wave;
    if (i < QTILEB / 1024) {
      const int sidx = i * 64 + lane;
      const int row = sidx / CPR, chunk = tile_io.stored_chunk((sidx % CPR) ^ TL::k_swizzle(row));
      const int row_ld = min(row0 + row, w.seg_hi - 1);
      lds_dma_16(qp + ((int64_t)row0 * Hq + head) * D, (uint32_t)((row_ld - row0) * (Hq * D) + chunk * 8) * 2u,
                 lds_addr_of(q_lds) + i * 1024);
    }
  }
  Tile cur = tile_at(min(wave, nt - 1));
  if (wave < nt) {
    load_k(cur);
    load_v(cur);
    wait_loads<2 * TL::IPW>();
  } else {
    wait_loads<0>();
  }
  __syncthreads();
  bf16x8 qf[KSTEPS];
#pragma unroll
  for (int st = 0; st < KSTEPS; ++st) {
    qf[st] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(q_lds + tile_io.k_off[st]));
    if constexpr (EXACT)
      if (16 * st + 8 * hf >= D) qf[st] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
    if constexpr (FOLD) {
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[st][e] = (bf16_t)((float)qf[st][e] * sc);
    }
  }

  f32x16 o[DT];
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt][e] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  float neg_ref = 0.f;   // minus the reference value of the scores (FOLD)

  // One tile.  K of the next tile streams in under the softmax and the second product, V of the next
  // tile under the next tile's first product and softmax.
  auto step = [&](auto more, const Tile& t, const Tile& nx) __attribute__((always_inline)) {
    constexpr bool MORE = decltype(more)::value;
    wait_loads<TL::IPW>();                       // K (V was requested after it)
    f32x16 s[1];
    bf16x8 kf[KSTEPS];
#pragma unroll
    for (int st = 0; st < KSTEPS; ++st)
      kf[st] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(
                                              lds0 + tile_io.k_off[st]));
    set_ref(s[0], neg_ref);
#pragma unroll
    for (int st = 0; st < KSTEPS; ++st) s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[st], qf[st], s[0], 0, 0, 0);
    if constexpr (MORE) {
      wait_lds_reads();
      load_k(nx);
    }
    if (t.len < kSplitRows || (t.causal_tile && t.kv0 + kSplitRows - 1 > row0)) {
      int lim = t.len;
      if (t.causal_tile) lim = min(lim, row0 + l32 - t.kv0 + 1);
      mask_scores(s, lim, hf);
    }
    bf16x8 pb[2];
    if constexpr (EXACT) {
      const float m_use = softmax_max(s, sc, m_run, l_run, o);
      softmax_exp_f32(s, sc, m_use, l_run);
    } else if constexpr (FOLD) {
      softmax_step_rel(s, m_run, l_run, o, neg_ref, pb);
    } else {
      softmax_step(s, sc, m_run, l_run, o, pb);
    }
    if constexpr (MORE) wait_loads<TL::IPW>();   // V (the next K was requested after it)
    else wait_loads<0>();
    bf16x8 vf[2][DT];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) vf[kk][dt] = tile_io.v_operand(lds0, TILEB, kk, dt);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      bf16x8 part[3];
      if constexpr (EXACT) {
        float pr[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) pr[e] = s[0][8 * kk + e];
        split_weights(pr, part);
      }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        if constexpr (EXACT) {
#pragma unroll
          for (int t3 = 2; t3 >= 0; --t3) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kk][dt], part[t3], o[dt], 0, 0, 0);
        } else {
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kk][dt], pb[kk], o[dt], 0, 0, 0);
        }
      }
    }
    if constexpr (MORE) {
      wait_lds_reads();
      load_v(nx);
    }
  };
  if (wave < nt) {
    for (int it = wave + KS; it < nt; it += KS) {
      const Tile nx = tile_at(it);
      step(std::true_type{}, cur, nx);
      cur = nx;
    }
    step(std::false_type{}, cur, cur);
  }

  // ---- merge: every wavefront hands (m, l, O) over in its own LDS share, then takes every KS-th
  // quarter of a 32-column slice of the output ------------------------------------------------------
  static_assert(DT * 4096 <= WAVEB, "the merge reuses the tiles");
  f32x4* xo = reinterpret_cast<f32x4*>(own) + lane;
  if (EXACT && tid == 0) odd_s = 0;
  ml_s[wave][0][lane] = m_run;
  ml_s[wave][1][lane] = sum_across_halves(l_run);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int vq = 0; vq < 4; ++vq)
      xo[(4 * dt + vq) * 64] = f32x4{o[dt][4 * vq], o[dt][4 * vq + 1], o[dt][4 * vq + 2], o[dt][4 * vq + 3]};
  __syncthreads();
  float mm = -INFINITY, den = 0.f, f[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) mm = fmaxf(mm, ml_s[k][0][lane]);
  const float mu = (mm == -INFINITY) ? 0.f : mm;
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    f[k] = __builtin_amdgcn_exp2f(ml_s[k][0][lane] - mu);
    den = fmaf(ml_s[k][1][lane], f[k], den);
  }
  const float inv = den > 0.f ? 1.f / den : 0.f;
  FiniteCheck fin;
#pragma unroll
  for (int c = wave; c < 4 * DT; c += KS) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < KS; ++k) acc += *(reinterpret_cast<const f32x4*>(kv_lds + k * WAVEB) + lane + c * 64) * f[k];
    if (EXACT && 8 * c < D) fin.add4(acc * inv);
    const bf16x4 b = {(bf16_t)(acc[0] * inv), (bf16_t)(acc[1] * inv), (bf16_t)(acc[2] * inv), (bf16_t)(acc[3] * inv)};
    *reinterpret_cast<u32x2*>(q_lds + l32 * ROWB + ((c ^ TL::k_swizzle(l32)) << 4) + 8 * hf) = __builtin_bit_cast(u32x2, b);
  }
  if constexpr (EXACT) {
    const uint64_t lanes = __builtin_amdgcn_ballot_w64(fin.failed() && row0 + l32 < w.seg_hi);
    if (lanes != 0 && lane == 0) atomicOr(&odd_s, (uint32_t)lanes | (uint32_t)(lanes >> 32));
  }
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < (kWaveRows * CPR + NT - 1) / NT; ++kk) {
    const int idx = kk * NT + tid;
    const int r = idx / CPR, c = idx % CPR;
    if (r < kWaveRows && row0 + r < w.seg_hi && (!EXACT || 8 * c < D))
      __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(q_lds + r * ROWB + ((c ^ TL::k_swizzle(r)) << 4)),
                                  reinterpret_cast<u32x4*>(op + ((int64_t)(row0 + r) * Hq + head) * D + 8 * c));
  }
  if constexpr (EXACT) {
    const uint32_t odd = __builtin_amdgcn_readfirstlane(odd_s);
    if (__builtin_expect(odd != 0, 0)) redo_prefill_rows<uint16_t, KS>(row0, odd, head, [](int) { return true; });
  }
}

template <int DP, bool FOLD, bool EXACT, bool APART = false>
hipError_t launch_split_t(const PrefillArgs& a, hipStream_t s) {
  constexpr int smem = (2 * kSplitWaves + 1) * KvTile<DP, 1, 1, kSplitRows>::TILEB;
  static std::atomic<uint64_t> attr_done{0};
  hipError_t e = set_max_dynamic_lds_once(attr_done, reinterpret_cast<const void*>(&prefill_split_kernel<DP, FOLD, EXACT, APART>), smem);
  if (e != hipSuccess) return e;
  dim3 grid((unsigned)(a.n_q_tiles * a.Hq));
  return launch_with(&prefill_split_kernel<DP, FOLD, EXACT, APART>, grid, dim3(64 * kSplitWaves), smem, s, a);
}

}  // namespace

// one block; head dimension at most 128
hipError_t launch_prefill_split(PrefillArgs& a, bool fold, hipStream_t s) {
  lay_out_query_tiles(a, kWaveRows);
  a.heads_per_wg = 1;
  lay_out_heads(a);
  order_segments_by_length(a);
  a.short_half_ascending = (int64_t)a.n_q_tiles * a.Hq <= 2 * (int64_t)a.n_cus ? 1 : 0;
  list_heavy_first(a, a.sync_override >= 0 ? a.sync_override != 0 : sync_block_rule(a.sync_interval, a.block_idx0));
  if (a.apart && a.keep_chunks == nullptr) {
    return a.D == 128 ? launch_split_t<128, true, false, true>(a, s) : launch_split_t<64, true, false, true>(a, s);
  }
  if (a.D == 128) return fold ? launch_split_t<128, true, false>(a, s) : launch_split_t<128, false, false>(a, s);
  if (a.D == 64) return fold ? launch_split_t<64, true, false>(a, s) : launch_split_t<64, false, false>(a, s);
  if (a.D <= 32) return launch_split_t<32, false, true>(a, s);
  if (a.D <= 64) return launch_split_t<64, false, true>(a, s);
  if (a.D <= 96) return launch_split_t<96, false, true>(a, s);
  return launch_split_t<128, false, true>(a, s);
}

}  // namespace fedattn
