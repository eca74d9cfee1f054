// What the split-KV decode kernels share: which piece of which cache segment a workgroup streams, and the
// merge of the chunks inside the launch.
#pragma once

#include "common.h"
#include "mfma_tile.h"
#include "row_walk.h"

namespace fedattn {

struct DecodeChunk {
  int m;                // segment (participant) the chunk belongs to
  int chunk0;           // first chunk of that segment
  int n_seg_chunks;     // its number of chunks
  int own_len, rem_len; // rows its own query sees, rows the other participants' queries see
  int seg_row0;         // first cache row of the segment
  int r_lo, r_hi;       // rows of the segment that this chunk holds
  int min_limit;        // rows below this are visible to every query column
};

// The segment tables sit in the kernel-argument buffer; a walk over them would take one
// scalar-cache miss after another before the first cache row is requested.  Every lane
// fetches the entries of segments `lane` and `lane + 64` at once, the chunk's segment is
// found with ballots and its entries are read out of the lanes that hold them.
__device__ __attribute__((always_inline)) inline DecodeChunk find_decode_chunk(const DecodeArgs& a, int gc, int lane) {
  const int N = a.N;
  const int ck_lo = a.chunk_cum[lane + 1], ck_hi = a.chunk_cum[lane + 65];
  const int sl_lo = a.seg_lens[lane], sl_hi = a.seg_lens[lane + 64];
  const int rl_lo = a.remote_lens[lane], rl_hi = a.remote_lens[lane + 64];
  const int so_lo = a.seg_off[lane], so_hi = a.seg_off[lane + 64];
  int m = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < N && gc >= ck_lo));
  if (N > 64) m += __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane + 64 < N && gc >= ck_hi));
  auto pick = [&](int lo, int hi, int idx) __attribute__((always_inline)) {
    return idx < 64 ? __builtin_amdgcn_readlane(lo, idx) : __builtin_amdgcn_readlane(hi, idx - 64);
  };
  DecodeChunk c;
  c.m = m;
  c.chunk0 = m == 0 ? 0 : pick(ck_lo, ck_hi, m - 1);
  c.n_seg_chunks = pick(ck_lo, ck_hi, m) - c.chunk0;
  c.own_len = pick(sl_lo, sl_hi, m);
  c.rem_len = a.has_remote ? pick(rl_lo, rl_hi, m) : c.own_len;
  c.seg_row0 = pick(so_lo, so_hi, m);
  const int rows_end = a.is_sync ? max(c.own_len, c.rem_len) : c.own_len;
  c.min_limit = a.is_sync ? min(c.own_len, c.rem_len) : c.own_len;
  c.r_lo = (gc - c.chunk0) * a.chunk_rows;
  c.r_hi = min(c.r_lo + a.chunk_rows, rows_end);
  return c;
}

// ---- merge inside the launch (at most 16 query columns, one workgroup per chunk and KV head) --------
// Chunks whose partials are merged into the same output rows: those of a segment (local block) or all
// (sync block).  The workgroup that finishes the last of them merges.  Their counter holds (ticket of the
// call) << 16 | chunks counted in, and every launch leaves it at zero.  What it holds before a call does not
// matter: in a call's first launch of a kind (ticket set) the first workgroups put the ticket there.
struct MergeSet {
  int first, count;
  uint64_t* cnt;
};
__device__ __attribute__((always_inline)) inline MergeSet merge_set(const DecodeArgs& a, const DecodeChunk& ch, int g, uint64_t* counters) {
  MergeSet s;
  s.first = a.is_sync ? 0 : ch.chunk0;
  s.count = a.is_sync ? a.n_chunks : ch.n_seg_chunks;
  s.cnt = counters + g * a.N + (a.is_sync ? 0 : ch.m);
  return s;
}

// Not this call's yet: make it so.  The exchange fails only if another workgroup of the set came
// first, and it has completed (with the partial stores) before this workgroup counts itself in.
__device__ __attribute__((always_inline)) inline void claim_counter(const MergeSet& s, uint64_t found, uint64_t ticket) {
  if (threadIdx.x == 0 && found >> 16 != ticket)
    (void)__hip_atomic_compare_exchange_strong(s.cnt, &found, ticket << 16, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What a launch works on: all KV heads and query columns, or a piece of them.
struct DecodePiece {
  int g0, n_g, col0, n_cols;
};
template <bool PIECES>
__device__ __attribute__((always_inline)) inline DecodePiece decode_piece(const DecodeArgs& a) {
  return PIECES ? DecodePiece{a.g0, a.n_g, a.col0, a.n_cols} : DecodePiece{0, a.Hkv, 0, a.cols};
}
// Row of the partials that chunk gc leaves for query column col of KV head g.
__device__ __attribute__((always_inline)) inline int64_t partial_row(const DecodeArgs& a, const DecodePiece& p, int g, int gc, int col) {
  return ((int64_t)(g - p.g0) * a.n_chunks + gc) * p.n_cols + (col - p.col0);
}

// Output row of query column col: local block, head col of participant m's KV group; sync block, head
// col mod G of participant col / G.
__device__ __attribute__((always_inline)) inline int64_t decode_out_row(const DecodeArgs& a, int g, int m, int col) {
  const int G = a.Hq / a.Hkv;
  return a.is_sync ? (int64_t)(col / G) * a.Hq + g * G + col % G : (int64_t)m * a.Hq + g * G + col;
}

template <typename T>
__device__ __attribute__((always_inline)) inline void store_out4(T* p, const f32x4& v) {
  if constexpr (sizeof(T) == 2) {
    const bf16x4 w = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
    *reinterpret_cast<u32x2*>(p) = __builtin_bit_cast(u32x2, w);
  } else {
    *reinterpret_cast<f32x4*>(p) = v;
  }
}

// Sets bit cl of *odd if one of the four values is not finite.
__device__ __attribute__((always_inline)) inline void note_nonfinite(const f32x4& v, int cl, uint32_t* odd) {
  FiniteCheck fin;
  fin.add4(v);
  if (fin.failed()) atomicOr(odd, 1u << cl);
}

// Two floats at an 8-byte aligned address, coherent at the device.
__device__ inline void store_pair_agent(float* p, float x, float y) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), __builtin_bit_cast(uint64_t, f32x2{x, y}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline f32x2 load_pair_agent(const float* p) {
  return __builtin_bit_cast(f32x2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Counts the workgroup in; the one that finds all others of the set counted in merges their partials.
// The partials travel between workgroups inside one launch, so they are written (by the caller, with
// store_pair_agent) and read with device-scope atomic accesses (coherent at the device whatever caches sit
// in between) rather than with plain accesses plus cache-wide write-back and invalidate fences, which
// cost far more than the few KB exchanged here.  A workgroup counts itself in only after all its partial
// stores have completed (vmcnt = 0 in every wavefront, then the barrier).
// All partials of kMergeBatch chunks are requested before the first is looked at: one round trip to memory
// for them together (one chunk at a time, for the maximum and again for the sum, it was two per chunk).
// REDO: with a second look at columns that come out not finite (row_walk.h); q, k, v: the block's own.
template <typename T, bool REDO>
__device__ __attribute__((always_inline)) inline void merge_if_last(const DecodeArgs& a, const MergeSet& s, int g, int m, int D,
                                                                    const float* part_o, const float* part_ml, T* out, const void* q,
                                                                    const void* k, const void* v) {
  __shared__ int last_s;
  __shared__ uint32_t odd_s;
  const int tid = threadIdx.x;
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  wait_vmcnt<0>();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __syncthreads();
  if (tid == 0) {
    const uint64_t seen = __hip_atomic_fetch_add(s.cnt, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int last = (int)(seen & 0xffff) == s.count - 1;
    // left at zero: a launch replayed from a graph comes with the same ticket, and the call's later ones without
    if (last) __hip_atomic_store(s.cnt, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last_s = last;
    odd_s = 0;
  }
  __syncthreads();
  if (!last_s) return;
  const int64_t row0 = ((int64_t)g * a.n_chunks + s.first) * a.cols;   // first chunk, column 0
  const int64_t cstride = a.cols;                                      // partial rows between chunks
  for (int idx = tid; idx < a.cols * (D / 4); idx += 256) {
    const int cl = idx / (D / 4), d4 = idx % (D / 4);
    const float* ml = part_ml + (row0 + cl) * 2;
    const float* po = part_o + (row0 + cl) * D + 4 * d4;
    float mm = -INFINITY, den = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < s.count; c0 += kMergeBatch) {
      const int nb = min(kMergeBatch, s.count - c0);
      f32x2 mls[kMergeBatch], lo[kMergeBatch], hi[kMergeBatch];
#pragma unroll
      for (int u = 0; u < kMergeBatch; ++u) {
        mls[u] = f32x2{-INFINITY, 0.f};
        lo[u] = hi[u] = f32x2{0.f, 0.f};
        if (u < nb) {
          mls[u] = load_pair_agent(ml + (c0 + u) * cstride * 2);
          lo[u] = load_pair_agent(po + (c0 + u) * cstride * D);
          hi[u] = load_pair_agent(po + (c0 + u) * cstride * D + 2);
        }
      }
      float m_new = mm;
#pragma unroll
      for (int u = 0; u < kMergeBatch; ++u) m_new = fmaxf(m_new, mls[u][0]);
      const float mu = (m_new == -INFINITY) ? 0.f : m_new;
      const float before = __builtin_amdgcn_exp2f(mm - mu);
      mm = m_new;
      den *= before;
      acc *= before;
#pragma unroll
      for (int u = 0; u < kMergeBatch; ++u) {
        const float w = __builtin_amdgcn_exp2f(mls[u][0] - mu);
        den = fmaf(mls[u][1], w, den);
        acc[0] = fmaf(lo[u][0], w, acc[0]);
        acc[1] = fmaf(lo[u][1], w, acc[1]);
        acc[2] = fmaf(hi[u][0], w, acc[2]);
        acc[3] = fmaf(hi[u][1], w, acc[3]);
      }
    }
    acc *= den > 0.f ? 1.f / den : 0.f;
    store_out4(out + decode_out_row(a, g, m, cl) * D + 4 * d4, acc);
    if constexpr (REDO) note_nonfinite(acc, cl, &odd_s);
  }
  if constexpr (REDO) {
    lds_barrier();
    if (__builtin_expect(odd_s != 0, 0)) redo_decode_columns<T, 4>(q, k, v, out, g, m, 0, odd_s);
  }
}

}  // namespace fedattn
