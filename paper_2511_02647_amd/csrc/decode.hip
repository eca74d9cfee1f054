// Decode attention (Section IV-C): one new query per participant over the block's
// KV cache; bandwidth-bound, so the cache is streamed exactly once.
//
// Split-KV: a workgroup takes one chunk of one participant's cache segment for
// one KV head and ALL query rows that may see it - the G query heads of that
// participant in a local block, the N*G rows of all participants in a sync block
// (the aggregated cache is read once for everybody).  The chunk streams through an
// LDS ring of 64-row K/V tiles filled by direct HBM -> LDS loads: three stages, two tiles in
// flight, where every CU has at most one workgroup, else (head dimensions padded to 96 or 128) two
// stages, so that more workgroups are resident.  Every wavefront works on
// every tile: wavefront w takes tile rows 16w..16w+15 against all query columns,
// S^T[kv][q] = K Q^T on v_mfma_f32_16x16x32_bf16 and O^T[d][q] += V^T P^T on
// v_mfma_f32_16x16x16_bf16, whose k-slots are exactly the 4 rows per lane that the
// first product leaves in a lane, with V^T operands from transposing LDS reads.  Each
// wavefront keeps its own online softmax per query column; the wavefronts are merged
// at the end, and the chunks by the workgroup that finishes last (few columns and chunks) or
// by a second small kernel:
//   o = sum_c O_c 2^(m_c - m) / sum_c l_c 2^(m_c - m).
#include "common.h"
#include "decode_walk.h"
#include "mfma_tile.h"
#include "row_walk.h"

namespace fedattn {

namespace {

// Three stages of 64-row K/V tiles (96 KB per workgroup, two tiles in flight while one is
// worked on): measured against four stages (three in flight), the deeper ring only lengthens
// the queue in front of the memory system; a block-step of 16 x 1152 rows takes 17.4 instead
// of 18.0 us.  Launches of more workgroups than CUs: launch_stream_mode.
// (Rows of more than 192 elements: two, three do not fit LDS.)
template <int D>
constexpr int decode_stages() { return D > 192 ? 2 : 3; }

template <int D, int STAGES>
constexpr int decode_smem_bytes() { return STAGES * 2 * KvTile<D, 0>::TILEB; }

// COLSPLIT = false (at most 16 query columns, e.g. the G heads of one participant in a
// local block): 4 wavefronts, wavefront w takes tile rows 16w..16w+15; they are merged
// through LDS at the end.  COLSPLIT = true (up to 64 query columns, sync blocks): 8
// wavefronts (two per SIMD, so that one's LDS and MFMA latencies hide behind the other);
// wavefront w takes query columns 16 (w mod 4).. against tile rows 32 (w / 4)..+31.  Its two
// 16-row sub-tiles fill the 8 k-slots per lane of one v_mfma_f32_16x16x32_bf16 in the second
// product (slot e < 4: row 4 kg + e of the first sub-tile, e >= 4: of the second), which
// halves its MFMA count.  The two row halves of a column block are merged through LDS.
// EXACT (head dimensions other than 64 and 128, padded to DP): the weights keep their fp32 precision
// in the second product, as three bf16 parts each (one participant of 62..207 rows to eight of 1500,
// bf16: 5 to 14 times faster than one wavefront per participant and head).
template <int DP, bool COLSPLIT, bool EXACT, bool PIECES, int STAGES>
__global__ __launch_bounds__(COLSPLIT ? 512 : 256, 1) void decode_stream_kernel(DecodeArgs a) {
  constexpr int NW = COLSPLIT ? 8 : 4;
  using TL = KvTile<DP, 0, NW, kKvTile, EXACT>;
  const int D = EXACT ? a.D : DP;
  constexpr int KS = DP / 32;                // k-steps of S^T (16x16x32)
  constexpr int DT = DP / 16;                // 16-row tiles of O^T along head_dim
  constexpr int ROWB = TL::ROWB, TILEB = TL::TILEB, IPW = TL::IPW;
  constexpr int RSUB = COLSPLIT ? 2 : 1;     // 16-row sub-tiles a wavefront processes per tile
  constexpr int QCOLS = COLSPLIT ? 64 : 16;  // query columns per workgroup
  constexpr int OPAD = DP + 4;               // floats per row of the merge buffer
  // stage s: K tile at s*2*TILEB, V tile at s*2*TILEB + TILEB; after the stream the
  // ring is reused as the merge buffer (row split only)
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  __shared__ float m_s[4][16];
  __shared__ float l_s[4][16];
  const lds_cptr lds0 = (lds_cptr)(lds_void_ptr)smem;
  const uint32_t lds_base = lds_addr_of(smem);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15;
  const int kg = lane >> 4;

  // block of a fused launch: its q/out, caches and workspace slice
  const int bz = blockIdx.z;
  const int64_t blk = a.block_list[bz];
  const unsigned char* q_ptr = reinterpret_cast<const unsigned char*>(a.q) + blk * a.q_block_bytes;
  unsigned char* out_ptr = reinterpret_cast<unsigned char*>(a.out) + blk * a.q_block_bytes;
  const unsigned char* k_ptr = reinterpret_cast<const unsigned char*>(a.k_cache) + blk * a.cache_block_bytes;
  const unsigned char* v_ptr = reinterpret_cast<const unsigned char*>(a.v_cache) + blk * a.cache_block_bytes;
  float* part_o = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(a.part_o) + bz * a.slice_bytes);
  float* part_ml = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(a.part_ml) + bz * a.slice_bytes);
  uint64_t* counters = reinterpret_cast<uint64_t*>(reinterpret_cast<unsigned char*>(a.counters) + bz * a.slice_bytes);

  const int Hq = a.Hq, Hkv = a.Hkv;
  const int G = Hq / Hkv;
  const DecodePiece pc = decode_piece<PIECES>(a);
  const int g = pc.g0 + blockIdx.x % pc.n_g;
  const int gc = blockIdx.x / pc.n_g;  // chunk index over all segments
  const int rh = COLSPLIT ? wave >> 2 : 0;   // row half of the tile (column split only)
  const int cb = pc.col0 + blockIdx.y * QCOLS + (COLSPLIT ? 16 * (wave & 3) : 0);  // first query column of this wavefront
  const int col_end = pc.col0 + pc.n_cols;

  const DecodeChunk ch = find_decode_chunk(a, gc, lane);
  const int m = ch.m;
  const int own_len = ch.own_len, rem_len = ch.rem_len, seg_row0 = ch.seg_row0;
  const int r_lo = ch.r_lo, r_hi = ch.r_hi, min_limit = ch.min_limit;
  const bool sync = a.is_sync != 0;
  const int nt = (r_hi - r_lo + kKvTile - 1) / kKvTile;
  const int row_elems = Hkv * D;

  const uint16_t* kbase = reinterpret_cast<const uint16_t*>(k_ptr) + ((int64_t)(seg_row0 + r_lo) * Hkv + g) * D;
  const uint16_t* vbase = reinterpret_cast<const uint16_t*>(v_ptr) + ((int64_t)(seg_row0 + r_lo) * Hkv + g) * D;

  TL tile_io;
  tile_io.init(lane, wave, row_elems, D / 8 - 1);

  // this lane's query column -> (participant, head); columns past the end are zero
  // rows: local block, column = head inside the KV group; sync block, column =
  // participant * G + head inside the group.  The loads are written out (like the tile
  // loads) so that the compiler's own wait for them does not drain the tile ring; they
  // are issued before any tile load, so the first tile wait below covers them.
  const int col = cb + l16;
  const bool col_ok = col < col_end;
  const bool wave_has_cols = cb < col_end;  // wave-uniform
  const int col_part = col_ok ? (sync ? col / G : m) : 0;
  const int col_head = col_ok ? g * G + (sync ? col % G : col) : 0;
  const int limit = col_ok ? (col_part == m ? own_len : rem_len) : 0;  // visible rows of this segment
  u32x4 qw[KS];  // B operand of S^T: Q[col][32 st + 8 kg .. +8]
  {
    const uint16_t* qrow = reinterpret_cast<const uint16_t*>(q_ptr) + ((int64_t)col_part * Hq + col_head) * D;
#pragma unroll
    for (int st = 0; st < KS; ++st) {
      const int d0 = EXACT ? min(32 * st + 8 * kg, D - 8) : 32 * st + 8 * kg;
      asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(qw[st]) : "v"(qrow + d0) : "memory");
    }
  }

  auto issue = [&](int t) __attribute__((always_inline)) {
    const int len = min(kKvTile, r_hi - r_lo - kKvTile * t);
    const uint32_t stage = lds_base + (t % STAGES) * 2 * TILEB;
    // every cache row is read once: the local-block kernel streams them past the caches (19.2
    // against 20.7 us per block-step at 16 x 1152 rows; no gain in the column-split kernel)
    tile_io.template dma<false, !COLSPLIT>(kbase + (int64_t)t * kKvTile * row_elems, stage, len);
    tile_io.template dma<true, !COLSPLIT>(vbase + (int64_t)t * kKvTile * row_elems, stage + TILEB, len);
  };
#pragma unroll
  for (int t = 0; t < STAGES - 1; ++t)
    if (t < nt) issue(t);
  // The chunk counter is requested here, behind the first tiles (ahead of them it cost 0.4 us of an 18 us
  // launch), and looked at after the stream.
  const MergeSet ms = merge_set(a, ch, g, counters);
  const bool set_up = !COLSPLIT && a.merge_in_kernel && ms.count > 1 && a.ticket != 0;
  uint64_t cnt_found = 0;
  if (set_up) cnt_found = __hip_atomic_load(ms.cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  // LDS -> A operand of S^T: lane (row l16 of a 16-row sub-tile, k-group kg) reads chunk
  // 4 st + kg; the sub-tile's first row goes in the address as a multiple of 16 rows,
  // which leaves the swizzle term unchanged
  int k_off[KS];
#pragma unroll
  for (int st = 0; st < KS; ++st) k_off[st] = l16 * ROWB + (((4 * st + kg) ^ TL::k_swizzle(l16)) * 16);
  // LDS -> A operand of O^T: transposing 8-byte reads; lane i = 4 e + c of a 16-lane group
  // supplies the address of V[sub-tile row 4 kg + e][16 dt + 4 c ..] and receives
  // V[sub-tile rows 4 kg + 0..3][16 dt + i]
  int v_off[DT];
  {
    const int vrow = 4 * kg + (l16 >> 2);
    const int fv = TL::v_swizzle(vrow);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) v_off[dt] = vrow * ROWB + (((2 * dt + ((l16 & 3) >> 1)) ^ fv) * 16) + (l16 & 1) * 8;
  }

  f32x4 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const float sc = a.scale * kLog2e;

  for (int t = 0; t < nt; ++t) {
    // this wavefront's part of tile t has landed once at most the loads of the tiles
    // issued after it are outstanding (the query loads are older still)
    // (the counter's load is allowed for where it matters, before the first tile)
    const int after = min(nt, t + STAGES - 1) - (t + 1);
    if (t == 0 && set_up && after == 1)
      wait_vmcnt<2 * IPW + 1>();
    else if (after >= 2)
      wait_vmcnt<2 * 2 * IPW>();
    else if (after == 1)
      wait_vmcnt<2 * IPW>();
    else
      wait_vmcnt<0>();
    __syncthreads();  // tile t is complete in LDS, and everyone is done with tile t-1
#pragma unroll
    for (int st = 0; st < KS; ++st) {
      asm volatile("" : "+v"(qw[st]));  // the query loads have landed by now
      if (EXACT && 32 * st + 8 * kg >= D) qw[st] = u32x4{0u, 0u, 0u, 0u};  // padded columns
    }
    if (t + STAGES - 1 < nt) issue(t + STAGES - 1);  // into the stage tile t-1 used
    if (COLSPLIT && !wave_has_cols) continue;

    const int kb = (t % STAGES) * 2 * TILEB;
    // ---- S^T: element e of s[rs] = sub-tile row 4 kg + e, query column l16 --------------------
    f32x4 s[RSUB];
#pragma unroll
    for (int rs = 0; rs < RSUB; ++rs) {
      s[rs] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int sub = (COLSPLIT ? 2 * rh + rs : wave) * 16 * ROWB;
#pragma unroll
      for (int st = 0; st < KS; ++st) {
        const bf16x8 kf = __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(lds0 + (kb + sub + k_off[st])));
        s[rs] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, __builtin_bit_cast(bf16x8, qw[st]), s[rs], 0, 0, 0);
      }
    }
    if (r_lo + kKvTile * (t + 1) > min_limit) {
#pragma unroll
      for (int rs = 0; rs < RSUB; ++rs) {
        const int row0 = r_lo + kKvTile * t + 16 * (COLSPLIT ? 2 * rh + rs : wave) + 4 * kg;  // cache row of element 0
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (row0 + e >= limit) s[rs][e] = -INFINITY;
      }
    }

    // ---- online softmax of the query column (log2 domain, lazy rescale) -----------------------
    float mx = -INFINITY;
#pragma unroll
    for (int rs = 0; rs < RSUB; ++rs) mx = fmaxf(mx, fmaxf(fmaxf(s[rs][0], s[rs][1]), fmaxf(s[rs][2], s[rs][3])));
    const float m_cand = max_over_kgroups(mx) * sc;
    if (__builtin_amdgcn_ballot_w64(m_cand > m_run + kRescaleThreshold) != 0) {
      const float m_new = fmaxf(m_run, m_cand);
      const float m_ref = (m_new == -INFINITY) ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_ref);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
    constexpr int PARTS = EXACT ? 3 : 1;
    s16x4 pb[PARTS][RSUB];
#pragma unroll
    for (int rs = 0; rs < RSUB; ++rs) {
      float p[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(s[rs][e], sc, -m_use));
      l_run += (p[0] + p[1]) + (p[2] + p[3]);
      if constexpr (EXACT) {
        bf16x4 part[3];
        split_weights(p, part);
#pragma unroll
        for (int t3 = 0; t3 < 3; ++t3) pb[t3][rs] = __builtin_bit_cast(s16x4, part[t3]);
      } else {
        const bf16x4 pv4 = {(bf16_t)p[0], (bf16_t)p[1], (bf16_t)p[2], (bf16_t)p[3]};
        pb[0][rs] = __builtin_bit_cast(s16x4, pv4);
      }
    }

    // ---- O^T[d][q] += V^T P^T -----------------------------------------------------------------
    if constexpr (COLSPLIT) {
      // both sub-tiles in one 16x16x32 MFMA: k-slot 8 kg + e = row 4 kg + (e mod 4) of sub-tile e / 4
      const int sub = 2 * rh * 16 * ROWB;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(lds0 + (kb + TILEB + sub + v_off[dt])));
        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(lds0 + (kb + TILEB + sub + 16 * ROWB + v_off[dt])));
        const s16x8 vv = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
        for (int t3 = PARTS - 1; t3 >= 0; --t3) {
          const s16x8 pp = __builtin_shufflevector(pb[t3][0], pb[t3][1], 0, 1, 2, 3, 4, 5, 6, 7);
          o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vv), __builtin_bit_cast(bf16x8, pp),
                                                          o[dt], 0, 0, 0);
        }
      }
    } else {
      // k-slot 4 kg + e of the 16x16x16 MFMA = sub-tile row 4 kg + e
      const int sub = wave * 16 * ROWB;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const s16x4 vf = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(lds0 + (kb + TILEB + sub + v_off[dt])));
#pragma unroll
        for (int t3 = PARTS - 1; t3 >= 0; --t3) o[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf, pb[t3][0], o[dt], 0, 0, 0);
      }
    }
  }

  asm volatile("" : "+v"(cnt_found));   // its wait belongs here: behind the exchange it would wait for that, too
  if (set_up) claim_counter(ms, cnt_found, a.ticket);
  l_run = sum_over_kgroups(l_run);
  if constexpr (COLSPLIT) {
    // ---- merge the two row halves of a column block: half 1 hands (m, l, O) to half 0 -------
    __syncthreads();  // every wavefront is done with the tile ring
    f32x4* xo = reinterpret_cast<f32x4*>(smem) + (wave & 3) * (DT * 64) + lane;         // [DT][64 lanes]
    float* xml = reinterpret_cast<float*>(smem + 4 * DT * 64 * 16) + (wave & 3) * 128 + lane;  // m, l per lane
    if (rh == 1) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) xo[dt * 64] = o[dt];
      xml[0] = m_run;
      xml[64] = l_run;
    }
    __syncthreads();
    if (rh == 0) {
      const float m1 = xml[0], l1 = xml[64];
      const float mm = fmaxf(m_run, m1);
      const float mu = (mm == -INFINITY) ? 0.f : mm;
      const float f0 = __builtin_amdgcn_exp2f(m_run - mu), f1 = __builtin_amdgcn_exp2f(m1 - mu);
      m_run = mm;
      l_run = l_run * f0 + l1 * f1;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt] = o[dt] * f0 + xo[dt * 64] * f1;
    }
    // half 0 owns the merged 16 columns: write the partial straight from registers
    if (rh == 0 && col_ok) {
      const int64_t prow = partial_row(a, pc, g, gc, col);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        if (!EXACT || 16 * dt + 4 * kg < D) *reinterpret_cast<f32x4*>(part_o + prow * D + 16 * dt + 4 * kg) = o[dt];
      if (kg == 0) {
        part_ml[prow * 2] = m_run;
        part_ml[prow * 2 + 1] = l_run;
      }
    }
  } else {
    // ---- merge the 4 wavefronts (each saw a quarter of the rows) ----------------------------
    __shared__ uint32_t odd_s;   // EXACT: output columns that came out not finite
    if (EXACT && tid == 0) odd_s = 0;
    if (kg == 0) m_s[wave][l16] = m_run;
    __syncthreads();  // also: every wavefront is done with the tile ring
    const float mm = fmaxf(fmaxf(m_s[0][l16], m_s[1][l16]), fmaxf(m_s[2][l16], m_s[3][l16]));
    const float mu = (mm == -INFINITY) ? 0.f : mm;
    const float f = __builtin_amdgcn_exp2f(m_run - mu);
    if (kg == 0) l_s[wave][l16] = l_run * f;
    float* o_s = reinterpret_cast<float*>(smem) + wave * (16 * OPAD);  // one region per wavefront
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<f32x4*>(o_s + l16 * OPAD + 16 * dt + 4 * kg) = o[dt] * f;
    __syncthreads();
    const int64_t prow0 = partial_row(a, pc, g, gc, 0);   // at most 16 columns: one workgroup per chunk
    const float* o_all = reinterpret_cast<const float*>(smem);
    uint16_t* out = reinterpret_cast<uint16_t*>(out_ptr);
    const bool only = a.merge_in_kernel && ms.count == 1;   // nothing to merge: normalise and write the output rows
    for (int idx = tid; idx < a.cols * (D / 4); idx += 256) {
      const int cl = idx / (D / 4), d4 = idx % (D / 4);
      const float* src = o_all + cl * OPAD + 4 * d4;
      const f32x4 v0 = *reinterpret_cast<const f32x4*>(src);
      const f32x4 v1 = *reinterpret_cast<const f32x4*>(src + 16 * OPAD);
      const f32x4 v2 = *reinterpret_cast<const f32x4*>(src + 32 * OPAD);
      const f32x4 v3 = *reinterpret_cast<const f32x4*>(src + 48 * OPAD);
      const f32x4 sum = (v0 + v1) + (v2 + v3);
      if (only) {
        const float den = l_s[0][cl] + l_s[1][cl] + l_s[2][cl] + l_s[3][cl];
        const f32x4 res = sum * (den > 0.f ? 1.f / den : 0.f);
        store_out4(out + decode_out_row(a, g, m, cl) * D + 4 * d4, res);
        if constexpr (EXACT) note_nonfinite(res, cl, &odd_s);
      } else {
        float* dst = part_o + (prow0 + cl) * D + 4 * d4;
        store_pair_agent(dst, sum[0], sum[1]);
        store_pair_agent(dst + 2, sum[2], sum[3]);
      }
    }
    if (only) {
      if constexpr (EXACT) {
        lds_barrier();
        if (__builtin_expect(odd_s != 0, 0)) redo_decode_columns<uint16_t, 4>(q_ptr, k_ptr, v_ptr, out_ptr, g, m, 0, odd_s);
      }
      return;
    }
    if (tid < a.cols)
      store_pair_agent(part_ml + (prow0 + tid) * 2, fmaxf(fmaxf(m_s[0][tid], m_s[1][tid]), fmaxf(m_s[2][tid], m_s[3][tid])),
                       l_s[0][tid] + l_s[1][tid] + l_s[2][tid] + l_s[3][tid]);
    if (a.merge_in_kernel) merge_if_last<uint16_t, EXACT>(a, ms, g, m, D, part_o, part_ml, out, q_ptr, k_ptr, v_ptr);
  }
}

// Merges the chunk partials of one query column (of one participant) and KV head and writes the output row:
//   o = sum_c O_c 2^(m_c - m) / sum_c l_c 2^(m_c - m),  m = max_c m_c.
// A chain of memory round trips: per kCombineAtOnce chunks one, in which every thread requests its partial O
// rows and the first wavefront the chunks' (m, l) before anything is known about the weights.  At least
// D/4 x 4 threads: thread (cg, d4) sums 4 head-dim elements over the chunks c = cg (mod 4); the 4 chunk groups
// meet in LDS.  (With a serial sum of the l, three barriers and, beyond 64 chunks, two passes over them, a sync
// block of 16 x 300..1000 rows, 8/4 heads of 64 took 12.4 instead of 11.2 us, of 1 x 8192 rows, 8/2 heads 11.9 instead of 11.3.)
template <typename T, bool PIECES>
__global__ __launch_bounds__(256) void decode_combine_kernel(DecodeArgs a) {
  constexpr int CG = 4;
  static_assert(kCombineAtOnce == 64 && kCombineAtOnce == 16 * CG, "one chunk per lane, 16 partial rows per thread");
  __shared__ float w_s[2][64];
  __shared__ float alpha_s[2], den_s;
  __shared__ f32x4 acc_s[CG][64];
  const DecodePiece pc = decode_piece<PIECES>(a);
  const int m = blockIdx.x / (pc.n_g * pc.n_cols);   // participant of a local block (0 in a sync block)
  const int r = blockIdx.x % (pc.n_g * pc.n_cols);
  const int g = pc.g0 + r / pc.n_cols, col = pc.col0 + r % pc.n_cols;
  const int c0 = a.is_sync ? 0 : a.chunk_cum[m];
  const int c1 = a.is_sync ? a.n_chunks : a.chunk_cum[m + 1];
  const int tid = threadIdx.x;
  const int D = a.D, D4 = D / 4;
  const int d4 = tid % D4, cg = tid / D4;  // blockDim: whole wavefronts, at least D4 * CG
  // block of a fused launch
  const int bz = blockIdx.y;
  unsigned char* out_ptr = reinterpret_cast<unsigned char*>(a.out) + (int64_t)a.block_list[bz] * a.q_block_bytes;
  const float* part_o = reinterpret_cast<const float*>(reinterpret_cast<const unsigned char*>(a.part_o) + bz * a.slice_bytes);
  const float* part_ml = reinterpret_cast<const float*>(reinterpret_cast<const unsigned char*>(a.part_ml) + bz * a.slice_bytes);
  const int64_t row0 = partial_row(a, pc, g, 0, col);
  const int64_t cstride = pc.n_cols;       // partial rows between consecutive chunks

  float m_run = -INFINITY, den = 0.f;      // first wavefront
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  int buf = 0;                             // the batch after the next one writes only when everyone is past the next barrier
  for (int cb = c0; cb < c1; cb += kCombineAtOnce, buf ^= 1) {
    const int nb = min(kCombineAtOnce, c1 - cb);
    const int nb_o = cg < CG ? nb : 0;     // chunks whose O rows this thread sums (every CG-th from cg on)
    const float* po = part_o + (row0 + cb * cstride) * D + 4 * d4;
    f32x4 part[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int i = cg + CG * u;
      part[u] = i < nb_o ? *reinterpret_cast<const f32x4*>(po + i * cstride * D) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (tid < 64) {
      f32x2 ml = {-INFINITY, 0.f};
      if (tid < nb) ml = *reinterpret_cast<const f32x2*>(part_ml + (row0 + (cb + tid) * cstride) * 2);
      const float m_new = fmaxf(m_run, wave_max(ml[0]));
      const float mu = (m_new == -INFINITY) ? 0.f : m_new;
      const float w = __builtin_amdgcn_exp2f(ml[0] - mu);
      const float alpha = __builtin_amdgcn_exp2f(m_run - mu);
      w_s[buf][tid] = w;
      if (tid == 0) alpha_s[buf] = alpha;
      den = den * alpha + wave_sum(ml[1] * w);
      if (tid == 0) den_s = den;
      m_run = m_new;
    }
    __syncthreads();
    acc *= alpha_s[buf];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int i = cg + CG * u;
      if (i < nb_o) acc += part[u] * w_s[buf][i];
    }
  }
  if (cg < CG) acc_s[cg][d4] = acc;
  __syncthreads();
  bool odd = false;
  if (cg == 0) {
    const float dn = c1 > c0 ? den_s : 0.f;
    const f32x4 sum = (acc_s[0][d4] + acc_s[1][d4]) + (acc_s[2][d4] + acc_s[3][d4]);
    T* out = reinterpret_cast<T*>(out_ptr) + decode_out_row(a, g, m, col) * D + 4 * d4;
    const f32x4 res = sum * (dn > 0.f ? 1.f / dn : 0.f);
    store_out4(out, res);
    // second look (row_walk.h); these threads are lanes of the first wavefront
    FiniteCheck fin;
    fin.add4(res);
    odd = fin.failed() && (sizeof(T) == 4 || (D != 64 && D != 128));
  }
  if (__builtin_expect(tid < 64 && __builtin_amdgcn_ballot_w64(odd) != 0, 0)) {
    const int64_t blk = a.block_list[bz];
    redo_decode_columns<T, 1>(reinterpret_cast<const unsigned char*>(a.q) + blk * a.q_block_bytes,
                              reinterpret_cast<const unsigned char*>(a.k_cache) + blk * a.cache_block_bytes,
                              reinterpret_cast<const unsigned char*>(a.v_cache) + blk * a.cache_block_bytes, out_ptr, g, m, col, 1u);
  }
}

// General decode kernel (plain ALU, fp32 arithmetic, any head_dim up to 256, fp32 or
// bf16 storage): one wavefront per (participant, query head), no split and no workspace.  It takes
// the calls that come without one; with one the split kernels are up to 70 times faster (fp32 sync
// block of 32 x 300..900 rows, 32/8 heads of 128: 14.8 ms here, 0.21 ms split).
template <typename T>
__global__ __launch_bounds__(64) void decode_rows_kernel(DecodeArgs a) {
  __shared__ float qs[256];
  const int n = blockIdx.x / a.Hq, h = blockIdx.x % a.Hq;
  const T* q = reinterpret_cast<const T*>(a.q) + ((int64_t)n * a.Hq + h) * a.D;
  for (int d = threadIdx.x; d < a.D; d += 64) qs[d] = RowLoad<T>::at(q + d);
  __syncthreads();
  decode_row(a, reinterpret_cast<const T*>(a.k_cache), reinterpret_cast<const T*>(a.v_cache), reinterpret_cast<T*>(a.out), n, h,
             [&](int d) { return qs[d]; });
}

// Query columns of a launch's KV heads, and those heads.
int launch_cols(const DecodeArgs& a, bool pieces) { return pieces ? a.n_cols : a.cols; }
int launch_heads(const DecodeArgs& a, bool pieces) { return pieces ? a.n_g : a.Hkv; }

template <int DP, bool COLSPLIT, bool EXACT, bool PIECES, int STAGES>
hipError_t launch_stream_stages(const DecodeArgs& a, dim3 grid, hipStream_t s) {
  static std::atomic<uint64_t> attr_done{0};
  constexpr int smem = decode_smem_bytes<DP, STAGES>();
  const auto kernel = &decode_stream_kernel<DP, COLSPLIT, EXACT, PIECES, STAGES>;
  hipError_t e0 = set_max_dynamic_lds_once(attr_done, reinterpret_cast<const void*>(kernel), smem);
  if (e0 != hipSuccess) return e0;
  return launch_with(kernel, grid, dim3(COLSPLIT ? 512 : 256), smem, s, a);
}

template <int DP, bool COLSPLIT, bool EXACT, bool PIECES = false>
hipError_t launch_stream_mode(const DecodeArgs& a, int n_z, hipStream_t s) {
  const int qcols = COLSPLIT ? 64 : 16;
  dim3 grid((unsigned)(a.n_chunks * launch_heads(a, PIECES)), (unsigned)((launch_cols(a, PIECES) + qcols - 1) / qcols), (unsigned)n_z);
  // More than one workgroup per CU: a third stage would keep the second one off the CU until the first has ended, and with
  // two resident one streams while the other starts or merges (6 blocks of 16 x 1152 rows, 32/8 heads, in one
  // launch: 92 us with three stages, 84 with two).  Padded to 96, where two with three stages do fit a CU, three with two are
  // faster, too (2 and 4 blocks of 1427 and 1517 rows, 8/8 heads of 96: 16.7 and 28.8 us with three, 9.8 and 14.0 with two; a launch per
  // block 17.4 and 35).
  if constexpr (DP == 96 || DP == 128)
    if ((int64_t)grid.x * grid.y * grid.z > a.n_cus) return launch_stream_stages<DP, COLSPLIT, EXACT, PIECES, 2>(a, grid, s);
  return launch_stream_stages<DP, COLSPLIT, EXACT, PIECES, decode_stages<DP>()>(a, grid, s);
}

// D: 64 or 128
template <int D>
hipError_t launch_stream(const DecodeArgs& a, int n_z, hipStream_t s) {
  return a.cols <= 16 ? launch_stream_mode<D, false, false>(a, n_z, s) : launch_stream_mode<D, true, false>(a, n_z, s);
}

// other head dimensions, at most DP (8 wavefronts share a tile's loads evenly from multiples of 64 on)
template <int DP>
hipError_t launch_stream_exact(const DecodeArgs& a, bool pieces, int n_z, hipStream_t s) {
  constexpr int DW = (DP + 63) / 64 * 64;
  if (pieces) return launch_stream_mode<DW, true, true, true>(a, n_z, s);
  return a.cols <= 16 ? launch_stream_mode<DP, false, true>(a, n_z, s) : launch_stream_mode<DW, true, true>(a, n_z, s);
}

template <typename T>
hipError_t launch_decode_combine(const DecodeArgs& a, bool pieces, int n_z, hipStream_t s) {
  const dim3 grid((unsigned)((a.is_sync ? 1 : a.N) * launch_heads(a, pieces) * launch_cols(a, pieces)), (unsigned)n_z);
  const dim3 block((unsigned)((a.D + 63) / 64 * 64));
  return launch_with(pieces ? &decode_combine_kernel<T, true> : &decode_combine_kernel<T, false>, grid, block, 0, s, a);
}

}  // namespace

// n_z > 1: the blocks a.block_list[0 .. n_z) in one launch (split kernels only)
hipError_t launch_decode(const DecodeArgs& a, int dtype, bool split, int n_z, hipStream_t s) {
  if (a.N == 0 || n_z == 0) return hipSuccess;
  if (!split) {
    if (n_z != 1) return hipErrorInvalidValue;
    dim3 grid((unsigned)(a.N * a.Hq));
    if (dtype == FEDATTN_F32)
      hipLaunchKernelGGL(decode_rows_kernel<float>, grid, dim3(64), 0, s, a);
    else
      hipLaunchKernelGGL(decode_rows_kernel<uint16_t>, grid, dim3(64), 0, s, a);
    return hipGetLastError();
  }
  const bool pieces = a.n_g < a.Hkv || a.n_cols < a.cols;
  if (a.n_chunks > 0) {
    hipError_t e;
    if (dtype == FEDATTN_F32) e = launch_decode_f32(a, pieces, n_z, s);
    else if (a.D == 128) e = launch_stream<128>(a, n_z, s);
    else if (a.D == 64) e = launch_stream<64>(a, n_z, s);
    else switch ((a.D + 31) / 32) {
      case 1: e = launch_stream_exact<32>(a, pieces, n_z, s); break;
      case 2: e = launch_stream_exact<64>(a, pieces, n_z, s); break;
      case 3: e = launch_stream_exact<96>(a, pieces, n_z, s); break;
      case 4: e = launch_stream_exact<128>(a, pieces, n_z, s); break;
      case 5: e = launch_stream_exact<160>(a, pieces, n_z, s); break;
      case 6: e = launch_stream_exact<192>(a, pieces, n_z, s); break;
      case 7: e = launch_stream_exact<224>(a, pieces, n_z, s); break;
      default: e = launch_stream_exact<256>(a, pieces, n_z, s);
    }
    if (e != hipSuccess) return e;
  }
  if (a.merge_in_kernel) return hipSuccess;
  return dtype == FEDATTN_F32 ? launch_decode_combine<float>(a, pieces, n_z, s) : launch_decode_combine<uint16_t>(a, pieces, n_z, s);
}

}  // namespace fedattn
