// fp32 prefill attention on the matrix cores: fp32 operands, fp32 products and sums
// (v_mfma_f32_16x16x4_f32), the same walks over KV tiles as the bf16 kernel.
//
// Both products run transposed: S^T = K Q^T leaves the scores of one query in one lane group
// (query = lane mod 16, the 4 lanes kg = lane / 16 hold keys 4 kg .. 4 kg + 3 of each 16-key
// sub-tile), and element e of those registers is, as it stands, the B operand of the e-th
// k-step of O^T += V^T P^T (k-slot kg = key 4 kg + e).
//
// Bound by the fp32 matrix rate (256 FLOP per cycle and CU, 157 TFLOP/s; a library fp32 GEMM reaches
// 154 here): a 64-key tile costs a CU 16 000 cycles of matrix work against 64 KB of tile loads, so one
// stage of K and one of V suffice and two 4-wavefront workgroups per CU cover each other's softmax.
// 4 participants of 100..900 tokens, 8/2 heads of 128, a local and a sync block: 2057 us on the
// wavefront-per-row kernel, 120 us here; 8 x 2000 tokens, 32/8 heads, sync: 137 TFLOP/s.
#include "common.h"
#include "mfma_tile.h"
#include "prefill_walk.h"
#include "row_walk.h"

namespace fedattn {

namespace {

// DP: head dimension padded to the instantiated size (Q is zero there, K and V re-read a valid
//     chunk, so a padded product is 0 * finite).
// NQ: 16-row query sub-tiles per wavefront (each K and V operand read from LDS feeds NQ MFMAs).
// KS: wavefronts that split the keys of a tile among them (they share the query rows and are
//     merged at the end); 4 / KS wavefronts hold different query rows or heads.
template <int DP, int NQ, int KS>
__global__ __launch_bounds__(256, DP > 128 ? 1 : 2) void prefill_f32_kernel(PrefillArgs a) {
  constexpr int CH = DP / 4;               // 16-byte chunks per row
  constexpr int ROWB = DP * 4;
  constexpr int TILEB = kKvTile * ROWB;    // one K or V tile
  constexpr int IPW = TILEB / 1024 / 4;    // direct-to-LDS loads per wavefront and tile
  constexpr int DS = DP / 16;              // 16-wide slices of the head dimension
  constexpr int KPW = kKvTile / KS;        // keys of a tile that a wavefront works on
  constexpr int NK = KPW / 16;
  constexpr int QG = 4 / KS;
  static_assert(KS == 1 || 4 * NQ * DS * 1024 <= 2 * TILEB, "the merge reuses the K and V stages");
  extern __shared__ __attribute__((aligned(1024))) unsigned char kv_lds[];  // K tile, then V tile
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kg = lane >> 4;
  const int ks = wave % KS, qg = wave / KS;
  const lds_cptr lds0 = (lds_cptr)(lds_void_ptr)kv_lds;
  const uint32_t lds_base = lds_addr_of(kv_lds);

  const int Hq = a.Hq, Hkv = a.Hkv, D = a.D;
  const int G = Hq / Hkv;
  const int HS = a.heads_per_wg, HG = G / HS;
  const int N = a.seg.n, T = a.n_q_tiles;
  const SegTab seg_tab = load_seg_tab(a.seg.seg_off, lane, N);
  const SegTab tile_tab = load_seg_tab(a.seg.tile_cum, lane, N);
  const SegTab order_tab = load_seg_tab(a.seg.pair_cum, lane, N);
  const int order_lo = a.seg_order[lane], order_hi = a.seg_order[lane + 64];

  // workgroup -> (KV head, head subgroup, query tile): KV head fastest, so that the workgroups of
  // one KV head share an XCD's L2 when there are 8; longest walks first (sync block: from the end
  // of the sequence; local block: participants by decreasing length, each from its last tile)
  const int g = blockIdx.x % Hkv;
  const int rest = blockIdx.x / Hkv;
  const int hsub = rest % HG;
  const int p = rest / HG;
  const int block = blockIdx.y;
  const bool is_sync = a.sync_override >= 0 ? (a.sync_override != 0)
                                            : sync_block_rule(a.sync_interval, a.block_idx0 + block);
  const bool sparse = is_sync && a.keep_chunks != nullptr;
  const int rank = a.short_half_ascending && p >= (T + 1) / 2 ? T - 1 - (p - (T + 1) / 2) : p;  // 0: longest walk
  int tile;
  if (is_sync) {
    tile = T - 1 - rank;
  } else {
    const int s = seg_tab_find(order_tab, rank, N);
    const int n = s < 64 ? __builtin_amdgcn_readlane(order_lo, s) : __builtin_amdgcn_readlane(order_hi, s - 64);
    tile = seg_tab_at(tile_tab, n + 1) - 1 - (rank - seg_tab_at(order_tab, s));
  }
  const KvWalk w = make_kv_walk(a, seg_tab, tile_tab, tile, is_sync, sparse);
  const int row0 = w.q0 + 16 * NQ * (qg / HS);   // this wavefront's first query row
  const int head = g * G + hsub * HS + qg % HS;

  const float* qp = reinterpret_cast<const float*>(a.q) + (int64_t)block * a.q_block_stride;
  const float* kp = reinterpret_cast<const float*>(a.k) + (int64_t)block * a.kv_block_stride + g * D;
  const float* vp = reinterpret_cast<const float*>(a.v) + (int64_t)block * a.kv_block_stride + g * D;
  const float* kp_list = reinterpret_cast<const float*>(a.k_list) + g * D;
  const float* vp_list = reinterpret_cast<const float*>(a.v_list) + g * D;
  float* op = reinterpret_cast<float*>(a.out) + (int64_t)block * a.q_block_stride;
  const int row_elems = Hkv * D;
  const int last_chunk = D / 4 - 1;

  // K or V tile -> LDS; slot (row, cp) receives chunk cp ^ (row mod 8)
  auto fetch = [&](const float* base, const float* list_base, int it, uint32_t stage) __attribute__((always_inline)) {
    int kv0, len;
    bool ct;
    kv_tile_desc(a, w, it, kv0, len, ct);
    const float* t = (it < w.n_list ? list_base : base) + (int64_t)kv0 * row_elems;
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int sidx = (wave * IPW + i) * 64 + lane;
      const int row = sidx / CH, chunk = min((sidx % CH) ^ (row & 7), last_chunk);
      lds_dma_16(t, (uint32_t)(min(row, len - 1) * row_elems + chunk * 4) * 4u, stage + (wave * IPW + i) * 1024);
    }
  };

  fetch(kp, kp_list, 0, lds_base);
  fetch(vp, vp_list, 0, lds_base + TILEB);

  // Q (B operand of S^T): lane (query l16, kg) holds Q[query][16 s + 4 kg .. +4]
  f32x4 q[NQ][DS];
#pragma unroll
  for (int iq = 0; iq < NQ; ++iq) {
    const float* qrow = qp + ((int64_t)min(row0 + 16 * iq + l16, w.seg_hi - 1) * Hq + head) * D + 4 * kg;
#pragma unroll
    for (int s = 0; s < DS; ++s)
      q[iq][s] = 16 * s + 4 * kg < D ? *reinterpret_cast<const f32x4*>(qrow + 16 * s) : f32x4{0.f, 0.f, 0.f, 0.f};
  }

  const int k_addr = (ks * KPW + l16) * ROWB;
  const int k_swz = l16 & 7;
  // V operand of k-step e: row 4 kg + e of the sub-tile, element 16 dt + l16, i.e. chunk
  // 4 dt + l16 / 4 in slot (chunk ^ (4 (kg mod 2) + e))
  int v_addr[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v_addr[e] = TILEB + (ks * KPW + 4 * kg + e) * ROWB + (((l16 >> 2) ^ e) << 4) + (l16 & 3) * 4;
  const int v_half = (kg & 1) * 64;

  f32x4 o[NQ][DS];
  float m_run[NQ], l_run[NQ];
#pragma unroll
  for (int iq = 0; iq < NQ; ++iq) {
    m_run[iq] = -INFINITY;
    l_run[iq] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DS; ++dt) o[iq][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float sc = a.scale * kLog2e;
  const int row_last = min(row0 + 16 * NQ, w.seg_hi) - 1;

  // K of the next tile streams in under this tile's second product, V of the next tile under its
  // first product; one stage of each is enough because a product takes thousands of cycles.
  for (int j = 0; j < w.nt; ++j) {
    int kv0, len;
    bool causal_tile;
    kv_tile_desc(a, w, j, kv0, len, causal_tile);
    const int key0 = ks * KPW;
    // keys this wavefront has to look at in the tile (none past the diagonal or the tile's end)
    const bool active = key0 < len && (!causal_tile || kv0 + key0 <= row_last);
    wait_vmcnt<0>();   // K tile j (issued before the second product of tile j - 1)
    __syncthreads();   // everyone's part of it; and everyone is done with V tile j - 1
    if (j > 0) fetch(vp, vp_list, j, lds_base + TILEB);

    f32x4 s[NK][NQ];
    if (active) {
#pragma unroll
      for (int nk = 0; nk < NK; ++nk)
#pragma unroll
        for (int iq = 0; iq < NQ; ++iq) s[nk][iq] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < DS; ++st) {
        f32x4 kf[NK];
#pragma unroll
        for (int nk = 0; nk < NK; ++nk)
          kf[nk] = *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(
              lds0 + (k_addr + 16 * nk * ROWB + (((4 * st + kg) ^ k_swz) << 4)));
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int nk = 0; nk < NK; ++nk)
#pragma unroll
            for (int iq = 0; iq < NQ; ++iq)
              s[nk][iq] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[nk][e], q[iq][st][e], s[nk][iq], 0, 0, 0);
      }
    }
    wait_vmcnt<0>();   // V tile j
    __syncthreads();   // everyone's part of it; and everyone is done with K tile j
    if (j + 1 < w.nt) fetch(kp, kp_list, j + 1, lds_base);
    if (!active) continue;

    if (key0 + KPW > len || (causal_tile && kv0 + key0 + KPW - 1 > row0)) {
#pragma unroll
      for (int iq = 0; iq < NQ; ++iq) {
        int lim = len;
        if (causal_tile) lim = min(lim, row0 + 16 * iq + l16 - kv0 + 1);
        lim -= key0 + 4 * kg;
#pragma unroll
        for (int nk = 0; nk < NK; ++nk)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (16 * nk + e >= lim) s[nk][iq][e] = -INFINITY;
      }
    }
#pragma unroll
    for (int iq = 0; iq < NQ; ++iq) {
      float mx = s[0][iq][0];
#pragma unroll
      for (int nk = 0; nk < NK; ++nk)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = fmaxf(mx, s[nk][iq][e]);
      const float m_cand = max_over_kgroups(mx) * sc;
      if (__builtin_amdgcn_ballot_w64(m_cand > m_run[iq] + kRescaleThreshold) != 0) {
        const float m_new = fmaxf(m_run[iq], m_cand);
        const float alpha = __builtin_amdgcn_exp2f(m_run[iq] - ((m_new == -INFINITY) ? 0.f : m_new));
        m_run[iq] = m_new;
        l_run[iq] *= alpha;
#pragma unroll
        for (int dt = 0; dt < DS; ++dt) o[iq][dt] *= alpha;
      }
      const float m_use = (m_run[iq] == -INFINITY) ? 0.f : m_run[iq];
#pragma unroll
      for (int nk = 0; nk < NK; ++nk) {
#pragma unroll
        for (int e = 0; e < 4; ++e) s[nk][iq][e] = __builtin_amdgcn_exp2f(fmaf(s[nk][iq][e], sc, -m_use));
        l_run[iq] += (s[nk][iq][0] + s[nk][iq][1]) + (s[nk][iq][2] + s[nk][iq][3]);
      }
    }
#pragma unroll
    for (int nk = 0; nk < NK; ++nk)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int dt = 0; dt < DS; ++dt) {
          const float vf = *reinterpret_cast<const __attribute__((address_space(3))) float*>(
              lds0 + (v_addr[e] + 16 * nk * ROWB + (dt >> 1) * 128 + ((dt & 1) ? 64 - v_half : v_half)));
#pragma unroll
          for (int iq = 0; iq < NQ; ++iq)
            o[iq][dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf, s[nk][iq][e], o[iq][dt], 0, 0, 0);
        }
  }

#pragma unroll
  for (int iq = 0; iq < NQ; ++iq) l_run[iq] = sum_over_kgroups(l_run[iq]);
  uint32_t odd = 0;   // rows that came out not finite: bit 16 iq + l16
  auto look = [&](int iq, bool nan) __attribute__((always_inline)) {
    const uint64_t lanes = __builtin_amdgcn_ballot_w64(nan);
    const uint32_t both = (uint32_t)lanes | (uint32_t)(lanes >> 32);
    odd |= ((both | both >> 16) & 0xffffu) << (16 * iq);
  };
  if constexpr (KS == 1) {
#pragma unroll
    for (int iq = 0; iq < NQ; ++iq) {
      const int row = row0 + 16 * iq + l16;
      const float inv = l_run[iq] > 0.f ? 1.f / l_run[iq] : 0.f;
      FiniteCheck fin;
      float* orow = op + ((int64_t)row * Hq + head) * D + 4 * kg;
      const bool mine = row < w.seg_hi;
#pragma unroll
      for (int dt = 0; dt < DS; ++dt) {
        const f32x4 x = o[iq][dt] * inv;
        if (16 * dt + 4 * kg < D) {
          fin.add4(x);
          if (mine) __builtin_nontemporal_store(x, reinterpret_cast<f32x4*>(orow + 16 * dt));
        }
      }
      look(iq, mine && fin.failed());
    }
  } else {
    // merge the KS wavefronts of a query group through LDS, each taking every KS-th slice of the head dimension
    __shared__ float ml_s[4][NQ][2][16];
    __syncthreads();   // everyone is done with the tiles
    f32x4* xo = reinterpret_cast<f32x4*>(kv_lds) + lane;
#pragma unroll
    for (int iq = 0; iq < NQ; ++iq) {
      if (kg == 0) {
        ml_s[wave][iq][0][l16] = m_run[iq];
        ml_s[wave][iq][1][l16] = l_run[iq];
      }
#pragma unroll
      for (int dt = 0; dt < DS; ++dt) xo[((wave * NQ + iq) * DS + dt) * 64] = o[iq][dt];
    }
    __syncthreads();
#pragma unroll
    for (int iq = 0; iq < NQ; ++iq) {
      float mm = -INFINITY, den = 0.f, f[KS];
#pragma unroll
      for (int k = 0; k < KS; ++k) mm = fmaxf(mm, ml_s[qg * KS + k][iq][0][l16]);
      const float mu = (mm == -INFINITY) ? 0.f : mm;
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        f[k] = __builtin_amdgcn_exp2f(ml_s[qg * KS + k][iq][0][l16] - mu);
        den = fmaf(ml_s[qg * KS + k][iq][1][l16], f[k], den);
      }
      const int row = row0 + 16 * iq + l16;
      const float inv = den > 0.f ? 1.f / den : 0.f;
      float* orow = op + ((int64_t)row * Hq + head) * D + 4 * kg;
      const bool mine = row < w.seg_hi;
      FiniteCheck fin;
      for (int dt = ks; dt < DS; dt += KS) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KS; ++k) acc += xo[(((qg * KS + k) * NQ + iq) * DS + dt) * 64] * f[k];
        acc *= inv;
        if (16 * dt + 4 * kg < D) {
          fin.add4(acc);
          if (mine) __builtin_nontemporal_store(acc, reinterpret_cast<f32x4*>(orow + 16 * dt));
        }
      }
      look(iq, mine && fin.failed());
    }
  }
  if (__builtin_expect(odd != 0, 0))   // a wavefront wrote the slices ks, ks + KS, ... of its rows
    redo_prefill_rows<float, 1>(row0, odd, head, [&](int d) { return KS == 1 || (d >> 4) % KS == ks; });
}

template <int DP, int NQ, int KS>
hipError_t launch_prefill_f32_t(const PrefillArgs& a, int n_blocks, hipStream_t s) {
  constexpr int smem = 2 * kKvTile * DP * 4;
  static std::atomic<uint64_t> attr_done{0};
  hipError_t e = set_max_dynamic_lds_once(attr_done, reinterpret_cast<const void*>(&prefill_f32_kernel<DP, NQ, KS>), smem);
  if (e != hipSuccess) return e;
  dim3 grid((unsigned)(a.n_q_tiles * a.Hkv * (a.Hq / a.Hkv / a.heads_per_wg)), (unsigned)n_blocks);
  hipLaunchKernelGGL((prefill_f32_kernel<DP, NQ, KS>), grid, dim3(256), smem, s, a);
  return hipGetLastError();
}

template <int DP>
hipError_t launch_prefill_f32_d(PrefillArgs& a, int n_blocks, hipStream_t s) {
  constexpr int NQ = DP > 128 ? 1 : 2;
  const F32Launch plan = choose_f32_launch(a.seg.seg_off, a.seg.n, a.Hq, a.Hkv, a.D, n_blocks, a.n_cus);
  a.heads_per_wg = plan == kF32Shared ? heads_in_common(a.Hq / a.Hkv) : 1;
  lay_out_query_tiles(a, plan == kF32Narrow ? 16 : 16 * NQ * (4 / (plan == kF32Shared ? a.heads_per_wg : 4)));
  const int64_t wgs = (int64_t)a.n_q_tiles * a.Hkv * (a.Hq / a.Hkv / a.heads_per_wg) * n_blocks;
  if (wgs / n_blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  a.short_half_ascending = wgs <= 2 * (int64_t)a.n_cus ? 1 : 0;
  order_segments_by_length(a);
  if (plan == kF32Shared) return launch_prefill_f32_t<DP, NQ, 1>(a, n_blocks, s);
  return plan == kF32Narrow ? launch_prefill_f32_t<DP, 1, 4>(a, n_blocks, s) : launch_prefill_f32_t<DP, NQ, 4>(a, n_blocks, s);
}

}  // namespace

hipError_t launch_prefill_f32(const PrefillArgs& a_in, int n_blocks, hipStream_t s) {
  PrefillArgs a = a_in;
  if (a.D <= 32) return launch_prefill_f32_d<32>(a, n_blocks, s);
  if (a.D <= 64) return launch_prefill_f32_d<64>(a, n_blocks, s);
  if (a.D <= 96) return launch_prefill_f32_d<96>(a, n_blocks, s);
  if (a.D <= 128) return launch_prefill_f32_d<128>(a, n_blocks, s);
  if (a.D <= 192) return launch_prefill_f32_d<192>(a, n_blocks, s);
  return launch_prefill_f32_d<256>(a, n_blocks, s);
}

}  // namespace fedattn
