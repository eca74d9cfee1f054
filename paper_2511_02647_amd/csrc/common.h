// Shared declarations of the FedAttn HIP library (gfx950 only): kernel argument
// blocks, launcher prototypes and small device helpers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>

#include "fedattn.h"
#include "launch_choice.h"

namespace fedattn {

constexpr int kMaxP = FEDATTN_MAX_PARTICIPANTS;
static_assert(kMaxP == kMaxSegments, "the launch rules hold one entry per participant");
constexpr int kMaxFusedBlocks = 64;    // blocks of one fused decode launch
constexpr int kMaxApart = 31;          // participants whose matrices a sync block reads where they are (what fits the argument block)
constexpr int kMergeBatch = 8;         // chunks whose partials a decode merge has in flight at once

// Segment layout of the global sequence, passed by value in the kernel arguments
// (read with scalar loads; no device copy of host arrays is needed).
struct SegLayout {
  int32_t n;                    // N participants
  int32_t seg_off[kMaxP + 1];   // token offsets, seg_off[N] = total
  int32_t tile_cum[kMaxP + 1];  // cumulative count of query tiles (tiles never straddle segments)
  int32_t chunk_cum[kMaxP + 1]; // cumulative count of keep-list chunks
  int32_t pair_cum[kMaxP + 1];  // cumulative count of query-tile pairs, tiles paired inside each segment
};

struct PrefillArgs {
  const void* q;
  const void* k;
  const void* v;
  void* out;
  int64_t q_block_stride;   // elements between consecutive blocks (batched launch)
  int64_t kv_block_stride;
  const uint8_t* keep_chunks;   // device, or nullptr
  const void* k_list;           // K, V the kept-tile list refers to: k, v themselves when the keep chunks
  const void* v_list;           // are whole tiles, else the packed copies of the kept rows (workspace)
  const int2* kept_tiles;       // device (workspace): (first row, valid rows) of kept 64-row tiles
  const int32_t* kept_cum;      // device (workspace): kept tiles of participants < n, [N+1]
  int32_t chunk_tokens;
  int32_t total;
  int32_t Hq, Hkv, D;
  int32_t block_idx0;
  int32_t sync_interval;
  int32_t sync_override;    // -1 rule, 0 local, 1 sync
  int32_t causal;
  int32_t heads_per_wg;     // query heads of one KV group handled by one workgroup: 1, 2 or 4
  int32_t group;            // Hq / Hkv
  int32_t head_sets;        // workgroups per query tile and KV head: group / heads_per_wg
  int32_t kv_shift, set_shift;   // log2 of Hkv and head_sets, -1 where they are not powers of two
  int32_t q_tile_rows;      // MFMA kernel: query rows per workgroup
  int32_t n_q_tiles;
  int32_t n_cus;            // compute units of the device (launch shape heuristics)
  float scale;              // softmax scale
  int32_t n_listed;         // > 0: the host has listed the query tiles of the workgroups (tile_list); else they are worked out
  int32_t listed_pairs;     // MFMA kernel: workgroup p takes the tiles 2 p and 2 p + 1 of the list, else tile p
  int32_t late_from;        // MFMA kernel: listed workgroups from here on start a little later
  int32_t warm_kv;          // MFMA kernel: every workgroup pulls the K, V rows of its own query rows into L2 first
  int32_t one_tile_heavy_first;  // MFMA kernel, causal launch of several rounds of workgroups: one query tile per
                                 // workgroup, heaviest first (seg.pair_cum then counts tiles in seg_order's order)
  int32_t short_half_ascending;  // split and fp32 kernels: workgroups of the shorter half of the walks in ascending order
  int32_t apart;                 // bf16 with D = 64 or 128, sync blocks: the participants' matrices are not in k and v but where `own` says
  const void* own[2 * kMaxApart];   // entries 2 n and 2 n + 1: global row r of K and V is at entry + r rows
  SegLayout seg;
  uint32_t tile_list[kMaxListedTiles / 2];   // two entries each: segment | tile inside the segment << 7; kNoTile: none
  uint8_t seg_order[kMaxP];      // participants by decreasing length (local blocks of a heavy-first launch)
};

constexpr uint32_t kNoTile = 0xffff;
static_assert(kMaxP <= 128 && kMaxListedTiles <= 512, "a list entry has 7 bits for the segment and 9 for its tile");
static_assert(sizeof(PrefillArgs) <= 4096, "kernel arguments are limited to 4 KB");

// Packing of the kept rows of a sync block.
struct PackArgs {
  const uint8_t* keep_chunks;
  int32_t chunk_tokens, n;
  int32_t row_vecs, span;       // 16-byte pieces of a row; rows per workgroup
  uint4 *k_packed, *v_packed;
  int2* kept_tiles;
  int32_t* kept_cum;
  const void* k;                // rows of all participants back to back, or, with `apart` set,
  const void* v;                // nothing: every participant's matrices on their own
  int32_t apart;
  const void* own[2 * kMaxApart];   // see PrefillArgs
  int32_t seg_off[kMaxP + 1];
  int32_t chunk_cum[kMaxP + 1];
};

struct DecodeArgs {
  const void* q;
  const void* k_cache;
  const void* v_cache;
  void* out;
  float* part_o;            // [Hkv, n_chunks, cols, D] fp32: sum_j p_j v_j with p_j = 2^(s_j - m), unnormalised
  float* part_ml;           // [Hkv, n_chunks, cols, 2] (m in log2 domain, l)
  uint64_t* counters;       // [Hkv, N] chunks counted in per (KV head, segment), sync block: [Hkv, 0]; zero after a launch
  uint64_t ticket;          // a call's first launch of a kind (local / sync): the call's number, 48 bits, marks the counters as set up; later ones: 0
  int32_t merge_in_kernel;  // the split kernel writes the output rows itself (no combine launch)
  int32_t N, Hq, Hkv, D;
  int32_t n_cus;            // compute units of the device (launch shape heuristics)
  int32_t is_sync;
  int32_t chunk_rows;       // cache rows per workgroup
  int32_t n_chunks;         // total chunks over all segments
  int32_t cols;             // query columns per KV head: G (local) or N*G (sync)
  int32_t has_remote;       // remote_lens given
  float scale;
  // several blocks in one launch (grid z, or y for the combine): block z is block_list[z]
  // blocks of q_block_bytes / cache_block_bytes away from q, out and the caches, and works in its own slice
  // of the workspace (slice_bytes apart, partials and counters laid out alike in every slice of a kind)
  int64_t q_block_bytes;
  int64_t cache_block_bytes;
  int64_t slice_bytes;
  uint16_t block_list[kMaxFusedBlocks];
  int32_t seg_off[kMaxP + 1];
  int32_t seg_lens[kMaxP];
  int32_t remote_lens[kMaxP];
  int32_t chunk_cum[kMaxP + 1];
  // A block whose partials do not fit the workspace runs in pieces (launches with PIECES): KV heads
  // [g0, g0 + n_g) and query columns [col0, col0 + n_cols), which then take the place of Hkv and cols in the partials.
  // (At the end: next to `cols`, and read by every launch, they cost calls of a few hundred rows 0.7 us.)
  int32_t g0, n_g, col0, n_cols;
};

struct AggregateArgs {
  const void* k_local[kMaxP];
  const void* v_local[kMaxP];
  void* k_global;
  void* v_global;
  int32_t seg_off[kMaxP + 1];
  int32_t n;
  int32_t row_bytes;        // Hkv * D * element size, multiple of 16
};

// Host side: cuts every segment into query tiles of `rows` rows (tiles never straddle segments).
inline void lay_out_query_tiles(PrefillArgs& a, int rows) {
  a.q_tile_rows = rows;
  int32_t tiles = 0, pairs = 0;
  for (int n = 0; n <= a.seg.n; ++n) {
    a.seg.tile_cum[n] = tiles;
    a.seg.pair_cum[n] = pairs;
    if (n == a.seg.n) break;
    const int32_t tn = (int32_t)(((int64_t)a.seg.seg_off[n + 1] - a.seg.seg_off[n] + rows - 1) / rows);
    tiles += tn;
    pairs += (tn + 1) / 2;
  }
  a.n_q_tiles = tiles;
}

// Host side: seg_order = participants by decreasing number of query tiles, pair_cum = cumulative
// number of query tiles in that order.
inline void order_segments_by_length(PrefillArgs& a) {
  const int N = a.seg.n;
  int order[kMaxP];
  for (int n = 0; n < N; ++n) order[n] = n;
  std::stable_sort(order, order + N, [&](int x, int y) {
    return a.seg.tile_cum[x + 1] - a.seg.tile_cum[x] > a.seg.tile_cum[y + 1] - a.seg.tile_cum[y];
  });
  int run = 0;
  for (int i = 0; i < N; ++i) {
    a.seg_order[i] = (uint8_t)order[i];
    a.seg.pair_cum[i] = run;
    run += a.seg.tile_cum[order[i] + 1] - a.seg.tile_cum[order[i]];
  }
  a.seg.pair_cum[N] = run;
}

// Host side: what the workgroups' place in a launch is found with (heads_per_wg is final).
inline int log2_or_none(int x) {
  int s = 0;
  while ((1 << s) < x) ++s;
  return (1 << s) == x ? s : -1;
}
inline void lay_out_heads(PrefillArgs& a) {
  a.group = a.Hq / a.Hkv;
  a.head_sets = a.group / a.heads_per_wg;
  a.kv_shift = log2_or_none(a.Hkv);
  a.set_shift = log2_or_none(a.head_sets);
}

// Host side: the list of query tiles that the workgroups of a launch of one block take.  A workgroup without a list finds its
// tile in the segment tables, 0.3 to 0.4 us before its first load.  Without and with a list, us: 39 and 22 tokens, 6/2 heads of 64 4.45 and 4.02, 64 and
// 76 tokens, 8/8 heads of 128 6.03 and 5.72, 4 x 100..900 tokens, 8/2 heads of 96, two launches 38.9 and 37.7, 4 x 512, 32/8 heads of 128, four
// launches 94.5 and 94.2.  kMaxListedTiles is what fits beside the tables in the argument block; launches with more tiles have several
// rounds of workgroups, whose starts hide behind one another (16 x 4096 tokens: no difference).
struct TileList {
  PrefillArgs& a;
  explicit TileList(PrefillArgs& args) : a(args) { a.n_listed = 0; }
  static bool fits(const PrefillArgs& a, int per_wg) { return (int64_t)a.n_q_tiles * per_wg <= kMaxListedTiles; }
  void put(int i, uint32_t e) {
    a.tile_list[i >> 1] = (i & 1) ? (a.tile_list[i >> 1] & 0xffffu) | e << 16 : (a.tile_list[i >> 1] & 0xffff0000u) | e;
  }
  static uint32_t entry(int n, int t) { return (uint32_t)(n | t << 7); }
  int tiles(int n) const { return a.seg.tile_cum[n + 1] - a.seg.tile_cum[n]; }
};

// Longest walks first: sync block from the end of the sequence; local block the participants in seg_order, each from its last tile.
inline void list_heavy_first(PrefillArgs& a, bool is_sync) {
  TileList l(a);
  if (!TileList::fits(a, 1)) return;
  const int N = a.seg.n, T = a.n_q_tiles, half = a.short_half_ascending ? (T + 1) / 2 : T;
  int i = 0;
  for (int x = 0; x < N; ++x) {
    const int n = is_sync ? N - 1 - x : a.seg_order[x];
    for (int t = l.tiles(n) - 1; t >= 0; --t, ++i) l.put(i < half ? i : T - 1 - (i - half), TileList::entry(n, t));
  }
  a.n_listed = T;
}

// Host-side launchers (one per kernel family); each returns the hipError_t of the launch.  Those that take the block
// for writing finish it: a caller has no use for it afterwards.
hipError_t launch_prefill_generic(const PrefillArgs& a, int n_blocks, int dtype, hipStream_t s);
hipError_t launch_prefill_mfma(PrefillArgs& a, int n_blocks, hipStream_t s);
hipError_t launch_prefill_split(PrefillArgs& a, bool fold, hipStream_t s);
hipError_t launch_prefill_f32(PrefillArgs& a, int n_blocks, hipStream_t s);
hipError_t launch_build_kept_tiles(const PrefillArgs& a, int2* kept_tiles, int32_t* kept_cum,
                                   hipStream_t s);
hipError_t launch_pack_kept_rows(PackArgs& a, hipStream_t s);
hipError_t launch_decode(const DecodeArgs& a, int dtype, bool split, int n_z, hipStream_t s);
hipError_t launch_decode_f32(const DecodeArgs& a, bool pieces, int n_z, hipStream_t s);
hipError_t launch_aggregate(const AggregateArgs& a, hipStream_t s);
hipError_t launch_rmsnorm(const float* x, void* out, int64_t rows, int d_model, float eps, hipStream_t s);
hipError_t launch_residual_add_rmsnorm(float* x, const void* y, void* out, int64_t rows, int d_model, float eps,
                                       hipStream_t s);
hipError_t launch_rope_split(const void* qkv, const int32_t* pos, void* q, void* k, void* v, int64_t tokens, int Hq,
                             int Hkv, int D, float theta, hipStream_t s);
hipError_t launch_swiglu(const void* gate_up, void* out, int64_t rows, int F, hipStream_t s);
hipError_t launch_residual_add(float* x, const void* y, int64_t n, hipStream_t s);
hipError_t launch_stream_probe(const void* src, int64_t bytes, int n_wgs, int pattern, float* sink, hipStream_t s);
hipError_t launch_mfma_probe(float* sink, int n_wgs, int iters, hipStream_t s);

// One launch with its argument block where it is: the launch syntax copies the block (up to 4 KB) once more on the way.
template <typename Args>
inline hipError_t launch_with(void (*kernel)(Args), dim3 grid, dim3 block, int smem, hipStream_t s, const Args& a) {
  void* args[] = {const_cast<Args*>(&a)};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, args, (size_t)smem, s);
  return e == hipSuccess ? hipSuccess : (void(hipGetLastError()), e);   // reported here, not by the next caller's look
}

// A kernel's dynamic-LDS limit is a per-device attribute: set it the first time the kernel is
// launched on a device (`done` holds one bit per device; setting it twice is harmless).
inline hipError_t set_max_dynamic_lds_once(std::atomic<uint64_t>& done, const void* kernel, int bytes) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = (dev >= 0 && dev < 64) ? (1ull << dev) : 0;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_release);
  return e;
}

// Algorithm 1: block m = Ht + h (1-based) is the global-attention block iff h = H.
__host__ __device__ inline bool sync_block_rule(int32_t H, int32_t block_idx) {
  return H >= 1 && ((block_idx + 1) % H) == 0;
}

#if defined(__HIPCC__)
typedef __bf16 bf16_t;
typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ inline float bf16_bits_to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// round-to-nearest-even float -> bf16 (hardware conversion on gfx950)
__device__ inline uint16_t f32_to_bf16_bits(float f) {
  bf16_t b = (bf16_t)f;
  return __builtin_bit_cast(uint16_t, b);
}

__device__ inline float wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}
__device__ inline float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
#endif

}  // namespace fedattn
