// Attention of one output row by one wavefront, key by key (plain ALU, fp32 arithmetic): the general
// kernels, and the rows that the fp32 and full-precision tile kernels do over.
//
// Doing rows over.  The tile kernels multiply a masked key's weight, zero, with its V row, and a padded Q
// column, zero, with an element of its K row; a NaN or an infinity there turns rows into NaN that do not see it.
// They look at their results (about one instruction per element of a walk's or chunk's output, none per tile: 0 to 1 %
// of a launch, 3 % at 4 x 300..400 tokens, 8/2 heads of 120; finding such values in the tiles costs every tile), and a row that is
// not finite is computed here instead, unless nothing but what it sees can have made it so.  bf16 with head
// dimension 64 and 128 has no such second look.
#pragma once

#include "common.h"
#include "mfma_tile.h"

namespace fedattn {

template <typename T>
struct RowLoad;

template <>
struct RowLoad<float> {
  // dot of a vector (element d: q(d)) with a row in memory
  template <typename Q>
  static __device__ inline float dot(const Q& q, const float* row, int D) {
    float acc = 0.f;
    for (int d = 0; d < D; d += 4) {
      const float4 kv = *reinterpret_cast<const float4*>(row + d);
      acc = fmaf(q(d + 0), kv.x, acc);
      acc = fmaf(q(d + 1), kv.y, acc);
      acc = fmaf(q(d + 2), kv.z, acc);
      acc = fmaf(q(d + 3), kv.w, acc);
    }
    return acc;
  }
  static __device__ inline float at(const float* p) { return *p; }
  static __device__ inline void store(float* p, float x) { *p = x; }
  // whether the four bytes hold an infinity or a NaN, an infinity
  static __device__ inline bool nonfinite(uint32_t u) { return (u & 0x7fffffffu) >= 0x7f800000u; }
  static __device__ inline bool infinite(uint32_t u) { return (u & 0x7fffffffu) == 0x7f800000u; }
};

template <>
struct RowLoad<uint16_t> {
  template <typename Q>
  static __device__ inline float dot(const Q& q, const uint16_t* row, int D) {
    float acc = 0.f;
    for (int d = 0; d < D; d += 8) {
      const uint4 w = *reinterpret_cast<const uint4*>(row + d);
      const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc = fmaf(q(d + 2 * e), __uint_as_float(u[e] << 16), acc);
        acc = fmaf(q(d + 2 * e + 1), __uint_as_float(u[e] & 0xFFFF0000u), acc);
      }
    }
    return acc;
  }
  static __device__ inline float at(const uint16_t* p) { return bf16_bits_to_f32(*p); }
  static __device__ inline void store(uint16_t* p, float x) { *p = f32_to_bf16_bits(x); }
  static __device__ inline bool nonfinite(uint32_t u) { return (u & 0x7f80u) == 0x7f80u || (u & 0x7f800000u) == 0x7f800000u; }
  static __device__ inline bool infinite(uint32_t u) { return (u & 0x7fffu) == 0x7f80u || (u & 0x7fff0000u) == 0x7f800000u; }
};

__device__ __attribute__((always_inline)) inline float lane_value(float x, int lane) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), lane));
}

// The kernel's first argument, read anew: code that hardly ever runs takes it from here, so that nothing it needs
// is held in registers through the tile loops.
template <typename Args>
__device__ __attribute__((always_inline)) inline const Args& argument_again() {
  auto p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const Args*)(const __attribute__((address_space(4))) Args*)p;
}

// Looks for values that are not finite; four chains, so that a look costs their number in instructions, not in latencies.
struct FiniteCheck {
  float t[4] = {0.f, 0.f, 0.f, 0.f};   // NaN once something was not finite
  __device__ __attribute__((always_inline)) void add(int chain, float x) { t[chain & 3] = fmaf(x, 0.f, t[chain & 3]); }
  __device__ __attribute__((always_inline)) void add4(const f32x4& x) {
#pragma unroll
    for (int e = 0; e < 4; ++e) add(e, x[e]);
  }
  __device__ __attribute__((always_inline)) bool failed() const {
    const float s = (t[0] + t[1]) + (t[2] + t[3]);
    return s != s;
  }
};
// The same for bf16 values, two to a word: an exponent of ones carries into the sign's place.
struct FiniteCheckBf16 {
  uint32_t t = 0;
  __device__ __attribute__((always_inline)) void add8(const u32x4& w) {
#pragma unroll
    for (int e = 0; e < 4; ++e) t |= (w[e] & 0x7f807f80u) + 0x00800080u;
  }
  __device__ __attribute__((always_inline)) bool failed() const { return (t & 0x80008000u) != 0; }
};
// Orders LDS accesses of a workgroup as __syncthreads() does, without waiting for stores to memory.
__device__ __attribute__((always_inline)) inline void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Whether an element of rows [lo, hi) of one KV head is not finite; `rows` is row 0 of that head.
template <typename T>
__device__ inline bool rows_nonfinite(const T* rows, int lo, int hi, int row_elems, int D) {
  const int per_row = D * (int)sizeof(T) / 16, at_once = 64 / per_row;   // at most 64 pieces of 16 bytes per row
  const int lane = threadIdx.x & 63;
  const T* piece = rows + lane % per_row * (16 / (int)sizeof(T));
  bool bad = false;
  if (lane / per_row < at_once)
    for (int64_t r = lo + lane / per_row; r < hi; r += at_once) {
      const uint4 w = *reinterpret_cast<const uint4*>(piece + r * row_elems);
      bad = bad || RowLoad<T>::nonfinite(w.x) || RowLoad<T>::nonfinite(w.y) || RowLoad<T>::nonfinite(w.z) || RowLoad<T>::nonfinite(w.w);
    }
  return __builtin_amdgcn_ballot_w64(bad) != 0;
}
// Whether the last 16 bytes of one of these rows, which a padded tile repeats, hold an infinity.  (Head dimensions that are
// multiples of 64 are not padded; others may not be either.)
template <typename T>
__device__ inline bool padding_infinite(const T* rows, int lo, int hi, int row_elems, int D) {
  if (D % 64 == 0) return false;
  bool bad = false;
  for (int j = lo + (threadIdx.x & 63); j < hi; j += 64) {
    const uint4 w = *reinterpret_cast<const uint4*>(rows + (int64_t)j * row_elems + D - 16 / (int)sizeof(T));
    bad = bad || RowLoad<T>::infinite(w.x) || RowLoad<T>::infinite(w.y) || RowLoad<T>::infinite(w.z) || RowLoad<T>::infinite(w.w);
  }
  return __builtin_amdgcn_ballot_w64(bad) != 0;
}

// Row i of query head h.  Visibility of key j (Section III-B causal mask; Phase I / Phase II; adaptive KV
// aggregation): own segment always, remote segments only in a sync block and only in chunks flagged as
// exchanged, and j <= i when causal.  q(d): element d of the query; want(d): whether to write element d.
// A step of 256 keys without a score above minus infinity is passed over, with SEE_NAN only if none of them is a NaN.
template <typename T, bool SEE_NAN, typename Q, typename Want>
__device__ __attribute__((always_inline)) inline void prefill_row(const PrefillArgs& a, int block, bool is_sync, int i, int h, const Q& q,
                                                                  const Want& want) {
  const int lane = threadIdx.x & 63;
  const int D = a.D;
  const int g = h / (a.Hq / a.Hkv);
  const T* k = reinterpret_cast<const T*>(a.k) + (int64_t)block * a.kv_block_stride;
  const T* v = reinterpret_cast<const T*>(a.v) + (int64_t)block * a.kv_block_stride;
  T* out = reinterpret_cast<T*>(a.out) + (int64_t)block * a.q_block_stride;
  int n = 0;
  while (n + 1 < a.seg.n && i >= a.seg.seg_off[n + 1]) ++n;

  float m_run = -INFINITY, l_run = 0.f;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int m = 0; m < a.seg.n; ++m) {
    const int lo = a.seg.seg_off[m];
    int hi = a.seg.seg_off[m + 1];
    if (m != n && !is_sync) continue;
    if (a.causal && hi > i + 1) hi = i + 1;
    if (lo >= hi) continue;
    const bool filter = (m != n) && a.keep_chunks != nullptr;
    const uint8_t* keep = filter ? a.keep_chunks + a.seg.chunk_cum[m] : nullptr;

    for (int base = lo; base < hi; base += 256) {
      float s[4];
      float tmax = -INFINITY;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int j = base + lane + 64 * t;
        bool vis = j < hi;
        if (vis && filter) vis = keep[(j - lo) / a.chunk_tokens] != 0;
        s[t] = vis ? a.scale * RowLoad<T>::dot(q, k + ((int64_t)j * a.Hkv + g) * D, D) : -INFINITY;
        tmax = fmaxf(tmax, s[t]);
      }
      tmax = wave_max(tmax);
      bool seen = tmax != -INFINITY;   // wave-uniform
      if constexpr (SEE_NAN)
        seen = seen || __builtin_amdgcn_ballot_w64(s[0] != s[0] || s[1] != s[1] || s[2] != s[2] || s[3] != s[3]) != 0;
      if (!seen) continue;
      const float m_new = fmaxf(m_run, tmax);
      const float alpha = expf(m_run - m_new);  // exp(-inf) = 0 on the first visible step
      float psum = 0.f;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        s[t] = expf(s[t] - m_new);  // masked keys: exp(-inf) = 0
        psum += s[t];
      }
      l_run = l_run * alpha + wave_sum(psum);
      m_run = m_new;
#pragma unroll
      for (int dd = 0; dd < 4; ++dd) acc[dd] *= alpha;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int cnt = min(64, hi - base - 64 * t);
        for (int jj = 0; jj < cnt; ++jj) {
          const float p = lane_value(s[t], jj);
          if (p == 0.f) continue;  // wave-uniform
          const T* vrow = v + ((int64_t)(base + 64 * t + jj) * a.Hkv + g) * D;
#pragma unroll
          for (int dd = 0; dd < 4; ++dd) {
            const int d = lane + 64 * dd;
            if (d < D) acc[dd] = fmaf(p, RowLoad<T>::at(vrow + d), acc[dd]);
          }
        }
      }
    }
  }
  const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
#pragma unroll
  for (int dd = 0; dd < 4; ++dd) {
    const int d = lane + 64 * dd;
    if (d < D && want(d)) RowLoad<T>::store(out + ((int64_t)i * a.Hq + h) * D + d, acc[dd] * inv);
  }
}

// A tile kernel's second look, after it has written its rows: row0 + (set bits of `rows`) of query head h, of one
// query tile, came out not finite.  They are done over if the keys after row0 that share a query tile with it (at most
// kMaxTileRows) have something not finite in V, or the padding of a key holds an infinity.  Called by the
// wavefront that wrote them, or by all wavefronts of a workgroup with the same rows (WAVES > 1), which then share them out.
// It finds out everything else by itself, so that the tile kernels keep nothing in registers for it.
constexpr int kMaxTileRows = 4 * kWaveRows;
template <typename T, int WAVES, typename Want>
__device__ __attribute__((always_inline)) inline void redo_prefill_rows(int row0, uint32_t rows, int h, const Want& want) {
  const PrefillArgs& a = argument_again<PrefillArgs>();
  const int block = blockIdx.y;
  const bool is_sync = a.sync_override >= 0 ? (a.sync_override != 0) : sync_block_rule(a.sync_interval, a.block_idx0 + block);
  const int row_elems = a.Hkv * a.D;
  const int64_t at = (int64_t)block * a.kv_block_stride + h / (a.Hq / a.Hkv) * a.D;
  const T *k = reinterpret_cast<const T*>(a.k) + at, *v = reinterpret_cast<const T*>(a.v) + at;
  int n = 0;
  while (n + 1 < a.seg.n && row0 >= a.seg.seg_off[n + 1]) ++n;
  const int seg_lo = a.seg.seg_off[n], seg_hi = a.seg.seg_off[n + 1];
  const bool spoilt = (a.causal && rows_nonfinite(v, row0 + 1, min(row0 + kMaxTileRows, seg_hi), row_elems, a.D)) ||
                      padding_infinite(k, is_sync ? 0 : seg_lo, is_sync ? a.total : seg_hi, row_elems, a.D);
  if (!spoilt) return;
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): what this wavefront wrote has arrived
  if constexpr (WAVES > 1) __syncthreads();
  int turn = 0;
#pragma unroll 1
  for (; rows != 0; rows &= rows - 1, ++turn) {
    if (WAVES > 1 && turn % WAVES != (int)(threadIdx.x >> 6)) continue;
    const int i = row0 + __builtin_ctz(rows);
    const T* q = reinterpret_cast<const T*>(a.q) + (int64_t)block * a.q_block_stride + ((int64_t)i * a.Hq + h) * a.D;
    prefill_row<T, true>(a, block, is_sync, i, h, [&](int d) { return RowLoad<T>::at(q + d); }, want);
  }
}

// Row of participant n and query head h of a decoding step; q_ptr .. out_ptr: the block's own.
template <typename T, typename Q>
__device__ __attribute__((always_inline)) inline void decode_row(const DecodeArgs& a, const T* kc, const T* vc, T* out_ptr, int n, int h,
                                                                 const Q& q) {
  const int lane = threadIdx.x & 63;
  const int g = h / (a.Hq / a.Hkv);
  const int D = a.D;
  float m_run = -INFINITY, l_run = 0.f;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int m = 0; m < a.N; ++m) {
    int len;
    if (m == n) len = a.seg_lens[m];
    else if (!a.is_sync) len = 0;
    else len = a.has_remote ? a.remote_lens[m] : a.seg_lens[m];
    for (int base = 0; base < len; base += 64) {
      const int r = base + lane;
      float s = -INFINITY;
      if (r < len) s = a.scale * RowLoad<T>::dot(q, kc + ((int64_t)(a.seg_off[m] + r) * a.Hkv + g) * D, D);
      const float m_new = fmaxf(m_run, wave_max(s));
      const float alpha = expf(m_run - m_new);
      const float p = expf(s - m_new);
      l_run = l_run * alpha + wave_sum(p);
      m_run = m_new;
#pragma unroll
      for (int dd = 0; dd < 4; ++dd) acc[dd] *= alpha;
      const int cnt = min(64, len - base);
      for (int jj = 0; jj < cnt; ++jj) {
        const float pj = lane_value(p, jj);
        const T* vrow = vc + ((int64_t)(a.seg_off[m] + base + jj) * a.Hkv + g) * D;
#pragma unroll
        for (int dd = 0; dd < 4; ++dd) {
          const int d = lane + 64 * dd;
          if (d < D) acc[dd] = fmaf(pj, RowLoad<T>::at(vrow + d), acc[dd]);
        }
      }
    }
  }
  const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
  T* out = out_ptr + ((int64_t)n * a.Hq + h) * D;
#pragma unroll
  for (int dd = 0; dd < 4; ++dd) {
    const int d = lane + 64 * dd;
    if (d < D) RowLoad<T>::store(out + d, acc[dd] * inv);
  }
}

// The split kernels' second look at output columns of KV head g (participant m's in a local block) that came out not
// finite, col0 + (set bits of `cols`), after they are written: by the wavefront that wrote them, or by all wavefronts of a
// workgroup (WAVES > 1).  They are done over if there is something not finite in V in a row that only some columns see.
template <typename T, int WAVES>
__device__ __attribute__((always_inline)) inline void redo_decode_columns(const void* q_ptr, const void* k_ptr, const void* v_ptr, void* out, int g, int m,
                                                                          int col0, uint32_t cols) {
  const DecodeArgs& a = argument_again<DecodeArgs>();
  const T *k = reinterpret_cast<const T*>(k_ptr), *v = reinterpret_cast<const T*>(v_ptr);
  const int D = a.D, G = a.Hq / a.Hkv, row_elems = a.Hkv * D;
  bool spoilt = false;
#pragma unroll 1
  for (int n = 0; n < a.N && !spoilt; ++n) {
    if (!a.is_sync && n != m) continue;
    const int own = a.seg_lens[n], rem = a.is_sync && a.has_remote ? a.remote_lens[n] : own, at = a.seg_off[n];
    spoilt = rows_nonfinite(v + g * D, at + min(own, rem), at + max(own, rem), row_elems, D) ||
             padding_infinite(k + g * D, at, at + max(own, rem), row_elems, D);
  }
  if (!spoilt) return;   // the same for all wavefronts
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): what this wavefront wrote has arrived
  if constexpr (WAVES > 1) __syncthreads();
  int turn = 0;
#pragma unroll 1
  for (; cols != 0; cols &= cols - 1, ++turn) {
    if (WAVES > 1 && turn % WAVES != (int)(threadIdx.x >> 6)) continue;
    const int col = col0 + __builtin_ctz(cols);
    const int n = a.is_sync ? col / G : m, h = g * G + (a.is_sync ? col % G : col);
    const T* q = reinterpret_cast<const T*>(q_ptr) + ((int64_t)n * a.Hq + h) * D;
    decode_row(a, k, v, reinterpret_cast<T*>(out), n, h, [&](int d) { return RowLoad<T>::at(q + d); });
  }
}

}  // namespace fedattn
