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
// 8 x 2000 tokens, 32/8 heads, sync: 137 TFLOP/s.
// This kernel takes blocks that fill the chip with workgroups whose wavefronts share K and V tiles (KS = 1), and, with
// KS = 4, head dimensions above 128; the others run prefill_f32_keys_kernel below.
#include <type_traits>

#include "common.h"
#include "mfma_tile.h"
#include "prefill_walk.h"
#include "row_walk.h"

namespace fedattn {

namespace {

// Waits that also keep the compiler from moving memory accesses across them.
template <int N>
__device__ inline void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

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
  const int HS = a.heads_per_wg;

  // longest walks first (sync block: from the end of the sequence; local block: participants by
  // decreasing length, each from its last tile)
  const ListTab list = load_list(a, lane);
  const WgPlace wg = find_wg_place(a);
  const int g = wg.g;
  const int block = blockIdx.y;
  const bool is_sync = a.sync_override >= 0 ? (a.sync_override != 0)
                                            : sync_block_rule(a.sync_interval, a.block_idx0 + block);
  const bool sparse = is_sync && a.keep_chunks != nullptr;
  const KvWalk w = make_kv_walk(a, place_heavy_first(a, list, wg.p, is_sync, lane), is_sync, sparse);
  const int row0 = w.q0 + 16 * NQ * (qg / HS);   // this wavefront's first query row
  const int head = g * a.group + wg.set * HS + qg % HS;

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

// Tiles whose keys the 4 wavefronts share out (head dimensions up to 128): 16 query rows of one head; wavefront w walks the 16-key
// slices w, w + 4, ...  No K or V element is used by two wavefronts: V comes straight into the registers that feed the
// MFMAs, K, whose operand layout would take 16 bytes from each of 16 rows per quarter of a load, passes through LDS buffers that
// are the wavefront's own, so no barrier stands in the walk.  K of the next slice is in flight while one is worked on.
// V arrives in 16-byte pieces: lane l16 holds elements 64 c + 4 l16 + j of a row (and 64 C4 + 2 l16 + j of the last 32 where the
// padded head dimension is an odd multiple of 32), so O^T tile (c, j) has element 64 c + 4 i + j as its row i.
//
// Bound by the SIMDs: next to an fp32 MFMA the vector ALU runs, for the same wavefront, hardly at all (a loop of one MFMA and n v_fma_f32
// takes 32 + 5.3 n cycles) and for two that share a SIMD about half the time.  So what counts beside the 64 MFMAs of a slice is the
// number of vector instructions: 130 with the loads' addresses worked out per slice, about 40 with those of full slices kept.
// Bidirectional, 1024 tokens, 8 heads of 128 (2 workgroups per CU), us: keys of a 64-row tile staged for all four wavefronts,
// as in prefill_f32_kernel, 47.2; K and V into registers 48.1 (K's loads at a quarter of their rate); K through LDS 45.7; addresses kept 41.8.
// Wavefronts that share a SIMD get different priorities: with equal ones they reach their softmax together and neither covers the other's
// (4 participants of 100..900 tokens, 8/2 heads of 128, a local and a sync block: 117.7 -> 110.3 us; all of the above 120 -> 104).
// Two query sub-tiles per wavefront (32 rows per workgroup): 2 to 17 % slower in ten layouts of 1 x 1024 to 8 x 1000 tokens but one,
// bidirectional with 16 heads, 4 % faster.
// SHORT: a block whose listed tiles may be short (launch_prefill_f32_d).
template <int DP, bool SHORT>
__global__ __launch_bounds__(256, SHORT && DP == 96 ? 3 : 2) void prefill_f32_keys_kernel(PrefillArgs a) {
  constexpr int DS = DP / 16;              // 16-wide slices of the head dimension
  constexpr int C4 = DP / 64, C2 = DP % 64 / 32;
  constexpr int CH = DP / 4;               // 16-byte chunks per row
  constexpr int ROWB = DP * 4, SLICEB = 16 * ROWB;
  constexpr int UNIT = 4 * 17;             // 16-byte pieces of a merge unit: 4 groups of 16 lanes, padded (conflict-free by rows and by pieces)
  extern __shared__ __attribute__((aligned(1024))) unsigned char keys_lds[];   // [wave][2] K slices, in the end [wave][DS] merge units
  __shared__ float ml_s[4][2][16];
  __shared__ uint32_t odd_s;               // rows that came out not finite
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kg = lane >> 4;
  const lds_cptr lds0 = (lds_cptr)(lds_void_ptr)(keys_lds + wave * 2 * SLICEB);
  const uint32_t lds_base = lds_addr_of(keys_lds) + wave * 2 * SLICEB;

  const int Hq = a.Hq, Hkv = a.Hkv, D = a.D;

  // workgroup -> (KV head, head of its group, query tile), in the order of prefill_f32_kernel
  const ListTab list = load_list(a, lane);
  const WgPlace wg = find_wg_place(a);
  const int g = wg.g, head = g * a.group + wg.set;
  const int block = blockIdx.y;
  const bool is_sync = a.sync_override >= 0 ? (a.sync_override != 0)
                                            : sync_block_rule(a.sync_interval, a.block_idx0 + block);
  const bool causal = a.causal != 0;
  const bool sparse = is_sync && a.keep_chunks != nullptr;
  const KvWalk w = make_kv_walk(a, place_heavy_first(a, list, wg.p, is_sync, lane), is_sync, sparse);
  const int row0 = w.q0;

  const float* qp = reinterpret_cast<const float*>(a.q) + (int64_t)block * a.q_block_stride;
  const float* kp = reinterpret_cast<const float*>(a.k) + (int64_t)block * a.kv_block_stride + g * D;
  const float* vp = reinterpret_cast<const float*>(a.v) + (int64_t)block * a.kv_block_stride + g * D;
  const float* kp_list = reinterpret_cast<const float*>(a.k_list) + g * D;
  const float* vp_list = reinterpret_cast<const float*>(a.v_list) + g * D;
  float* op = reinterpret_cast<float*>(a.out) + (int64_t)block * a.q_block_stride;
  const int row_elems = Hkv * D;

  // 16-key slices of the walk: four per listed 64-row tile (the last ones may be empty), then the dense range
  const int n_list = 4 * w.n_list;
  const int ns = n_list + (w.dhi - w.dlo + 15) / 16;
  struct Slice {
    const float *k, *v;    // first row to load
    int kv0, len, load_len;
    bool causal_slice;
  };
  auto slice_at = [&](int i) __attribute__((always_inline)) {
    Slice t;
    int first;
    if (i < n_list) {
      const int i4 = i >> 2, off = 16 * (i & 3);
      const int2 e = a.kept_tiles[i4 < w.la_n ? i4 : w.lb0 + (i4 - w.la_n)];
      const int lo = __builtin_amdgcn_readfirstlane(e.x), left = __builtin_amdgcn_readfirstlane(e.y) - off;
      t.kv0 = lo + off;
      t.len = min(max(left, 0), 16);
      first = left > 0 ? t.kv0 : lo;       // an empty slice loads the tile's first row, unseen
      t.load_len = max(t.len, 1);
      t.causal_slice = false;
    } else {
      t.kv0 = first = w.dlo + 16 * (i - n_list);
      t.len = t.load_len = min(w.dhi - t.kv0, 16);
      t.causal_slice = causal;
    }
    t.k = (i < n_list ? kp_list : kp) + (int64_t)first * row_elems;
    t.v = (i < n_list ? vp_list : vp) + (int64_t)first * row_elems;
    return t;
  };
  // SHORT: slices without rows are left out.  One slice of every listed tile, if the tile has that many rows, another one from tile to tile,
  // then every fourth of the dense range.
  int2 tile = make_int2(0, 0);   // lane i: tile 64 x + i of the walk's list
  uint64_t tiles_left = 0;       // those of them whose slice is still to be walked
  int listed = 0;                // tiles looked at
  int dense = w.dlo + 16 * wave;
  auto next_slice = [&](Slice& t) __attribute__((always_inline)) {
    while (tiles_left == 0 && listed < w.n_list) {
      const int i = listed + lane;
      tile = make_int2(0, 0);
      if (i < w.n_list) tile = a.kept_tiles[i < w.la_n ? i : w.lb0 + (i - w.la_n)];
      tiles_left = __builtin_amdgcn_ballot_w64(tile.y > 16 * ((wave + lane) & 3));
      listed += 64;
    }
    const bool from_list = tiles_left != 0;
    if (from_list) {
      const int i = __builtin_ctzll(tiles_left), off = 16 * ((wave + i) & 3);
      tiles_left &= tiles_left - 1;
      t.kv0 = __builtin_amdgcn_readlane(tile.x, i) + off;
      t.len = min(__builtin_amdgcn_readlane(tile.y, i) - off, 16);
    } else {
      if (dense >= w.dhi) return false;
      t.kv0 = dense;
      t.len = min(w.dhi - dense, 16);
      dense += 64;
    }
    t.load_len = t.len;
    t.causal_slice = causal && !from_list;
    t.k = (from_list ? kp_list : kp) + (int64_t)t.kv0 * row_elems;
    t.v = (from_list ? vp_list : vp) + (int64_t)t.kv0 * row_elems;
    return true;
  };

  // Rows of K and V are D <= DP long: pieces past the end re-read the last one (K meets a zero of Q there, V makes
  // outputs that are not stored).
  // Offsets of a full slice are worked out once: next to fp32 MFMAs every vector instruction counts (above).
  // K slice -> this wavefront's LDS buffer; slot (row, cp) receives chunk cp ^ (row mod 8)
  constexpr int KINST = SLICEB / 1024;
  auto k_slot = [&](int i, int rows) __attribute__((always_inline)) {
    const int row = (i * 64 + lane) / CH, chunk = min(((i * 64 + lane) % CH) ^ (row & 7), D / 4 - 1);
    return (uint32_t)(min(row, rows - 1) * row_elems + chunk * 4) * 4u;
  };
  // piece c of V row 4 kg + e; c = C4: the last 32 elements
  auto v_slot = [&](int e, int c, int rows) __attribute__((always_inline)) {
    return (uint32_t)(min(4 * kg + e, rows - 1) * row_elems + (c < C4 ? min(64 * c + 4 * l16, D - 4) : min(64 * C4 + 2 * l16, D - 2))) * 4u;
  };
  uint32_t k_full[KINST], v_full[4][C4 + C2];
#pragma unroll
  for (int i = 0; i < KINST; ++i) k_full[i] = k_slot(i, 16);
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int c = 0; c < C4 + C2; ++c) v_full[e][c] = v_slot(e, c, 16);
  auto fetch_k = [&](const Slice& t, int b) __attribute__((always_inline)) {
    if (t.load_len == 16) {
#pragma unroll
      for (int i = 0; i < KINST; ++i) lds_dma_16(t.k, k_full[i], lds_base + b * SLICEB + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < KINST; ++i) lds_dma_16(t.k, k_slot(i, t.load_len), lds_base + b * SLICEB + i * 1024);
    }
  };
  f32x4 v4[4][C4 == 0 ? 1 : C4];
  f32x2 v2[4];
  auto load_v = [&](const Slice& t) __attribute__((always_inline)) {
    const char* base = reinterpret_cast<const char*>(t.v);
    uint32_t at[4][C4 + C2];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < C4 + C2; ++c) at[e][c] = v_full[e][c];
    if (t.load_len < 16) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < C4 + C2; ++c) at[e][c] = v_slot(e, c, t.load_len);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int c = 0; c < C4; ++c) v4[e][c] = *reinterpret_cast<const f32x4*>(base + at[e][c]);
      if constexpr (C2 != 0) v2[e] = *reinterpret_cast<const f32x2*>(base + at[e][C4]);
    }
  };
  constexpr int VLOADS = 4 * (C4 + C2);
  int k_off[DS];   // LDS -> A operand of S^T: chunk 4 st + kg of row l16
#pragma unroll
  for (int st = 0; st < DS; ++st) k_off[st] = l16 * ROWB + (((4 * st + kg) ^ (l16 & 7)) << 4);

  Slice cur;
  bool any = true;
  if constexpr (SHORT) {   // ahead of Q, which the list's arrival would wait for
    any = next_slice(cur);
    if (any) fetch_k(cur, 0);
  }

  // Q (B operand of S^T): lane (query l16, kg) holds Q[query][16 s + 4 kg .. +4]
  f32x4 q[DS];
  const float* qrow = qp + ((int64_t)min(row0 + l16, w.seg_hi - 1) * Hq + head) * D;
#pragma unroll
  for (int s = 0; s < DS; ++s) {
    const int d = 16 * s + 4 * kg;
    q[s] = *reinterpret_cast<const f32x4*>(qrow + (s < DS - 2 ? d : min(d, D - 4)));
  }
  if constexpr (!SHORT) {
    cur = slice_at(min(wave, ns - 1));
    fetch_k(cur, 0);
  }

  f32x4 o[DS];
  float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
  for (int dt = 0; dt < DS; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float sc = a.scale * kLog2e;
#pragma unroll
  for (int s = DS - 2; s < DS; ++s)
    if (16 * s + 4 * kg >= D) q[s] = f32x4{0.f, 0.f, 0.f, 0.f};

  // One slice, in K buffer b.  K of the next slice and V of this one are requested first; V, the younger of the two, is
  // waited for behind the softmax, and K of this slice, which is older than both, here.
  auto step = [&](auto more, auto buffer, const Slice& cur, const Slice& nxt) __attribute__((always_inline)) {
    constexpr bool MORE = decltype(more)::value;
    constexpr int b = decltype(buffer)::value;
    if constexpr (MORE) fetch_k(nxt, b ^ 1);
    load_v(cur);
    wait_loads<(MORE ? KINST : 0) + VLOADS>();
    f32x4 kf[DS];
#pragma unroll
    for (int st = 0; st < DS; ++st)
      kf[st] = *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(lds0 + (k_off[st] + b * SLICEB));
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < DS; ++st)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[st][e], q[st][e], s, 0, 0, 0);
    if (cur.len < 16 || (cur.causal_slice && cur.kv0 + 15 > row0)) {
      int lim = cur.len;
      if (cur.causal_slice) lim = min(lim, row0 + l16 - cur.kv0 + 1);
      lim -= 4 * kg;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e >= lim) s[e] = -INFINITY;
    }
    const float m_cand = max_over_kgroups(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))) * sc;
    if (__builtin_amdgcn_ballot_w64(m_cand > m_run + kRescaleThreshold) != 0) {
      const float m_new = fmaxf(m_run, m_cand);
      const float alpha = __builtin_amdgcn_exp2f(m_run - ((m_new == -INFINITY) ? 0.f : m_new));
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < DS; ++dt) o[dt] *= alpha;
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = __builtin_amdgcn_exp2f(fmaf(s[e], sc, -m_use));
    l_run += (s[0] + s[1]) + (s[2] + s[3]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int c = 0; c < C4; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) o[4 * c + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v4[e][c][j], s[e], o[4 * c + j], 0, 0, 0);
      if constexpr (C2 != 0)
#pragma unroll
        for (int j = 0; j < 2; ++j) o[4 * C4 + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v2[e][j], s[e], o[4 * C4 + j], 0, 0, 0);
    }
  };
  priority_by_slot();
  using std::true_type;
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  if constexpr (SHORT) {
    Slice nxt;
    while (any) {
      if (!next_slice(nxt)) {
        step(std::false_type{}, B0{}, cur, cur);
        break;
      }
      step(true_type{}, B0{}, cur, nxt);
      if (!next_slice(cur)) {
        step(std::false_type{}, B1{}, nxt, nxt);
        break;
      }
      step(true_type{}, B1{}, nxt, cur);
    }
  } else if (wave < ns) {
    int i = wave + 4;
    for (; i + 4 < ns; i += 8) {
      const Slice n1 = slice_at(i), n2 = slice_at(i + 4);
      step(true_type{}, B0{}, cur, n1);
      step(true_type{}, B1{}, n1, n2);
      cur = n2;
    }
    if (i < ns) {
      const Slice n1 = slice_at(i);
      step(true_type{}, B0{}, cur, n1);
      step(std::false_type{}, B1{}, n1, n1);
    } else {
      step(std::false_type{}, B0{}, cur, cur);
    }
  }
  wait_loads<0>();
  lds_barrier();   // the merge reuses the K buffers

  // ---- merge: unit u of a wavefront holds, at piece 17 kg + l16, the four elements from d = 64 (u / 4) + 16 kg + 4 (u mod 4)
  // on (last 32: 64 C4 + 8 kg + 4 (u mod 4)) of row l16; then every thread takes whole pieces of output rows ----------------------
  f32x4* const units = reinterpret_cast<f32x4*>(keys_lds);
  if (tid == 0) odd_s = 0;
  const float l = sum_over_kgroups(l_run);
  if (kg == 0) {
    ml_s[wave][0][l16] = m_run;
    ml_s[wave][1][l16] = l;
  }
  f32x4* const xo = units + wave * DS * UNIT + 17 * kg + l16;
#pragma unroll
  for (int c = 0; c < C4; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) xo[(4 * c + r) * UNIT] = f32x4{o[4 * c][r], o[4 * c + 1][r], o[4 * c + 2][r], o[4 * c + 3][r]};
  if constexpr (C2 != 0)
#pragma unroll
    for (int r = 0; r < 2; ++r)
      xo[(4 * C4 + r) * UNIT] = f32x4{o[4 * C4][2 * r], o[4 * C4 + 1][2 * r], o[4 * C4][2 * r + 1], o[4 * C4 + 1][2 * r + 1]};
  lds_barrier();
  const int D4 = D / 4;
  for (int idx = tid; idx < 16 * D4; idx += 256) {
    const int r = idx / D4, d4 = idx - r * D4;
    const bool tail = C2 != 0 && d4 >= 16 * C4;
    const int u = 4 * (d4 >> 4) + (tail ? d4 & 1 : d4 & 3), k = tail ? (d4 & 15) >> 1 : (d4 & 15) >> 2;
    float mm = -INFINITY, den = 0.f;
#pragma unroll
    for (int x = 0; x < 4; ++x) mm = fmaxf(mm, ml_s[x][0][r]);
    const float mu = (mm == -INFINITY) ? 0.f : mm;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const float f = __builtin_amdgcn_exp2f(ml_s[x][0][r] - mu);
      den = fmaf(ml_s[x][1][r], f, den);
      acc += units[(x * DS + u) * UNIT + 17 * k + r] * f;
    }
    acc *= den > 0.f ? 1.f / den : 0.f;
    if (row0 + r < w.seg_hi) {
      __builtin_nontemporal_store(acc, reinterpret_cast<f32x4*>(op + ((int64_t)(row0 + r) * Hq + head) * D + 4 * d4));
      FiniteCheck fin;
      fin.add4(acc);
      if (fin.failed()) atomicOr(&odd_s, 1u << r);
    }
  }
  lds_barrier();
  const uint32_t odd = __builtin_amdgcn_readfirstlane(odd_s);
  if (__builtin_expect(odd != 0, 0)) redo_prefill_rows<float, 4>(row0, odd, head, [](int) { return true; });
}

template <int DP, int NQ, int KS>
hipError_t launch_prefill_f32_t(const PrefillArgs& a, int n_blocks, hipStream_t s) {
  constexpr int smem = 2 * kKvTile * DP * 4;
  static std::atomic<uint64_t> attr_done{0};
  hipError_t e = set_max_dynamic_lds_once(attr_done, reinterpret_cast<const void*>(&prefill_f32_kernel<DP, NQ, KS>), smem);
  if (e != hipSuccess) return e;
  dim3 grid((unsigned)(a.n_q_tiles * a.Hkv * (a.Hq / a.Hkv / a.heads_per_wg)), (unsigned)n_blocks);
  return launch_with(&prefill_f32_kernel<DP, NQ, KS>, grid, dim3(256), smem, s, a);
}

template <int DP, bool SHORT>
hipError_t launch_prefill_f32_keys(const PrefillArgs& a, int n_blocks, hipStream_t s) {
  constexpr int merge = 4 * (DP / 16) * 4 * 17 * 16, keys = 4 * 2 * 16 * DP * 4;
  constexpr int smem = merge > keys ? merge : keys;
  static std::atomic<uint64_t> attr_done{0};
  hipError_t e = set_max_dynamic_lds_once(attr_done, reinterpret_cast<const void*>(&prefill_f32_keys_kernel<DP, SHORT>), smem);
  if (e != hipSuccess) return e;
  dim3 grid((unsigned)(a.n_q_tiles * a.Hq), (unsigned)n_blocks);
  return launch_with(&prefill_f32_keys_kernel<DP, SHORT>, grid, dim3(256), smem, s, a);
}

template <int DP>
hipError_t launch_prefill_f32_d(PrefillArgs& a, int n_blocks, hipStream_t s) {
  constexpr int NQ = DP > 128 ? 1 : 2;
  const bool shared = f32_heads_shared(a.seg.seg_off, a.seg.n, a.Hq, a.Hkv, a.D, n_blocks, a.n_cus);
  a.heads_per_wg = shared ? heads_in_common(a.Hq / a.Hkv) : 1;
  lay_out_query_tiles(a, shared ? 16 * NQ * (4 / a.heads_per_wg) : 16);
  const int64_t wgs = (int64_t)a.n_q_tiles * a.Hkv * (a.Hq / a.Hkv / a.heads_per_wg) * n_blocks;
  if (wgs / n_blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  // All workgroups resident at once: the shorter half in ascending order, so that those that come to share a CU carry about the same
  // load together (1000 tokens, 8/2 heads of 128: 26.8 us, longest first throughout 33.1; 4 x 448, 4/1 heads: 44.2 and 52.4).
  a.short_half_ascending = wgs <= 2 * (int64_t)a.n_cus ? 1 : 0;
  lay_out_heads(a);
  order_segments_by_length(a);
  // blocks of one launch may be of both kinds
  if (n_blocks == 1) list_heavy_first(a, a.sync_override >= 0 ? a.sync_override != 0 : sync_block_rule(a.sync_interval, a.block_idx0));
  if (shared) return launch_prefill_f32_t<DP, NQ, 1>(a, n_blocks, s);
  if constexpr (DP <= 128) {
    // Every participant's list ends with a tile of few rows, or is one: where participants are many, most slices of the listed tiles are
    // empty.  Leaving them out costs 0.4 us a launch.  All slices walked and empty ones left out, us, 16/4 heads of 128: single tokens, a
    // tenth kept, 23 x 17..27 tokens, 32 heads 88.8 and 42.0 (keys of a tile staged for all wavefronts 66), 20 x 100 2.0 times
    // faster, 4 x 100 1.15, 3 x 100 1.15 and 3 x 200 0.95, 2 x 100 0.94; 64-token chunks, 30 % kept, 20 x 100 1.03, 6 x 100 1.06, 6 x 50 and 4 x 100 0.95.
    const bool short_tiles = a.keep_chunks != nullptr && a.seg.n >= (a.chunk_tokens < kKvTile ? 4 : 8);
    return short_tiles ? launch_prefill_f32_keys<DP, true>(a, n_blocks, s) : launch_prefill_f32_keys<DP, false>(a, n_blocks, s);
  } else {
    return launch_prefill_f32_t<DP, 1, 4>(a, n_blocks, s);
  }
}

}  // namespace

hipError_t launch_prefill_f32(PrefillArgs& a, int n_blocks, hipStream_t s) {
  if (a.D <= 32) return launch_prefill_f32_d<32>(a, n_blocks, s);
  if (a.D <= 64) return launch_prefill_f32_d<64>(a, n_blocks, s);
  if (a.D <= 96) return launch_prefill_f32_d<96>(a, n_blocks, s);
  if (a.D <= 128) return launch_prefill_f32_d<128>(a, n_blocks, s);
  if (a.D <= 192) return launch_prefill_f32_d<192>(a, n_blocks, s);
  return launch_prefill_f32_d<256>(a, n_blocks, s);
}

}  // namespace fedattn
