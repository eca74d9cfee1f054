// C ABI of the FedAttn library: argument validation, the sync-block rule of
// Algorithm 1, kernel selection and launch.  No device memory is allocated here
// and nothing is kept between calls.
#include <math.h>
#include <stdarg.h>
#include <stddef.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <chrono>
#include <mutex>

#include "common.h"

using namespace fedattn;

namespace {

thread_local char g_err[512] = "";

fedattn_status fail(fedattn_status st, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return st;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

fedattn_status check_params(const fedattn_params* p) {
  if (!p) return fail(FEDATTN_EINVAL, "params is NULL");
  if (p->n_participants < 1 || p->n_participants > FEDATTN_MAX_PARTICIPANTS)
    return fail(FEDATTN_EINVAL, "n_participants %d outside 1..%d", p->n_participants, FEDATTN_MAX_PARTICIPANTS);
  if (p->n_q_heads < 1 || p->n_kv_heads < 1 || p->n_q_heads % p->n_kv_heads != 0)
    return fail(FEDATTN_EINVAL, "n_q_heads %d must be a positive multiple of n_kv_heads %d", p->n_q_heads,
                p->n_kv_heads);
  if (p->head_dim < 8 || p->head_dim > 256 || p->head_dim % 8 != 0)
    return fail(FEDATTN_EINVAL, "head_dim %d must be a multiple of 8 in 8..256", p->head_dim);
  if (p->dtype != FEDATTN_BF16 && p->dtype != FEDATTN_F32) return fail(FEDATTN_EINVAL, "unknown dtype %d", p->dtype);
  if (!(p->softmax_scale >= 0.f) || !isfinite(p->softmax_scale))
    return fail(FEDATTN_EINVAL, "softmax_scale must be finite and >= 0");
  if (p->causal != 0 && p->causal != 1) return fail(FEDATTN_EINVAL, "causal must be 0 or 1");
  return FEDATTN_OK;
}

float resolve_scale(const fedattn_params* p) {
  return p->softmax_scale > 0.f ? p->softmax_scale : 1.0f / sqrtf((float)p->head_dim);
}

fedattn_status check_offsets(const fedattn_params* p, const int32_t* seg) {
  if (!seg) return fail(FEDATTN_EINVAL, "seg_offsets is NULL");
  if (seg[0] != 0) return fail(FEDATTN_EINVAL, "seg_offsets[0] must be 0");
  for (int n = 0; n < p->n_participants; ++n)
    if (seg[n + 1] < seg[n]) return fail(FEDATTN_EINVAL, "seg_offsets decreases at participant %d", n);
  return FEDATTN_OK;
}

bool use_mfma_prefill(const fedattn_params* p) {
  return p->dtype == FEDATTN_BF16 && (p->head_dim == 64 || p->head_dim == 128);
}

// Whether two address ranges have a byte in common.
bool ranges_meet(uintptr_t a, size_t a_bytes, uintptr_t b, size_t b_bytes) { return a < b + b_bytes && b < a + a_bytes; }

int elem_bytes(const fedattn_params* p) { return p->dtype == FEDATTN_BF16 ? 2 : 4; }

// keep chunks that are not whole 64-row tiles: the tile kernels pack the kept rows first
bool needs_row_packing(int chunk_tokens) { return chunk_tokens > 0 && chunk_tokens % kKvTile != 0; }

// Decode splits every participant's cache segment into chunks of `rows` cache rows (a
// multiple of the 64-row tile), one workgroup per (chunk, KV head).  The split aims at
// one workgroup per CU of the current device: about n_cus / Hkv chunks over all segments.
// The CU count is looked up once per device.
int device_cus() {
  constexpr int kMaxDevices = 64;
  static std::atomic<int> cus[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  const bool cached = dev >= 0 && dev < kMaxDevices;
  if (cached) {
    const int c = cus[dev].load(std::memory_order_relaxed);
    if (c > 0) return c;
  }
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
  if (cached) cus[dev].store(n, std::memory_order_relaxed);
  return n;
}

int decode_target_chunks(int Hkv) {
  const int t = device_cus() / Hkv;
  return t < 1 ? 1 : t;
}

int decode_chunk_rows(int64_t total_rows, int Hkv) {
  const int64_t target = decode_target_chunks(Hkv);
  int64_t rows = (total_rows + target - 1) / target;
  rows = (rows + kKvTile - 1) / kKvTile * kKvTile;
  return (int)(rows < kKvTile ? kKvTile : rows);
}

constexpr int64_t kMaxMergeTrips = 4;

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// prefill workspace: [kept_cum: (kMaxP+1) int32, padded][kept_tiles: int2 per 64-row tile]
// and, for keep chunks finer than a tile where a tile kernel runs: [packed K][packed V]
constexpr size_t kKeptCumBytes = 1024;
struct PrefillWs {
  size_t tiles_off, list_end, k_off, v_off, total;
};
PrefillWs prefill_ws_layout(const fedattn_params* p, int32_t tokens, int32_t chunk_tokens) {
  PrefillWs w;
  const size_t max_tiles = (size_t)tokens / kKvTile + (size_t)p->n_participants + 1;
  w.tiles_off = kKeptCumBytes;
  w.list_end = w.tiles_off + align_up(max_tiles * sizeof(int2), 256);
  w.k_off = w.v_off = w.total = w.list_end;
  if (needs_row_packing(chunk_tokens)) {
    const size_t kv_bytes = (size_t)tokens * (size_t)p->n_kv_heads * (size_t)p->head_dim * (size_t)elem_bytes(p);
    w.v_off = w.k_off + align_up(kv_bytes, 256);
    w.total = w.v_off + align_up(kv_bytes, 256);
  }
  return w;
}

// chunk counters of the fused combine, one per (KV head, participant), at the end of the workspace
size_t decode_counter_bytes(const fedattn_params* p) {
  return align_up((size_t)p->n_kv_heads * (size_t)p->n_participants * sizeof(uint64_t), 256);
}

// The partials of fp32 blocks and of bf16 blocks with head dimensions other than 64 and 128 never take more
// than the built-in array holds: larger blocks are worked off in pieces (below).  So these shapes ask for
// little memory however many participants there are, and a call with a workspace takes the route of
// fedattn_decode_static.  It costs a launch pair per piece: fp32 sync blocks, 32 x 300..900 rows, 32/8 heads of 128
// 209 us (188 with the 34 MB of the whole block's partials), 128 x 64..200 rows 1276 us (813 with 341 MB); one
// wavefront per participant and head takes 14.8 and 23.9 ms.
constexpr size_t kMostPieceBytes = FEDATTN_STATIC_SCRATCH_BYTES;

size_t decode_ws_bytes(const fedattn_params* p, int32_t capacity) {
  const size_t G = (size_t)(p->n_q_heads / p->n_kv_heads);
  const size_t N = (size_t)p->n_participants;
  // chunks <= sum_n (rows_n / chunk_rows + 1) <= target + N
  (void)capacity;
  const size_t chunks = (size_t)decode_target_chunks(p->n_kv_heads) + N;
  const size_t rows = (size_t)p->n_kv_heads * chunks * G * N;  // sync blocks: N*G query columns per chunk
  // Room for the counters: these bytes and the unused partials (there are at most target + N - 1 chunks).
  const size_t counters = align_up((size_t)p->n_kv_heads * N * sizeof(uint32_t), 256);
  const size_t whole = align_up(rows * (size_t)p->head_dim * 4, 256) + align_up(rows * 8, 256) + counters;
  return use_mfma_prefill(p) || whole < kMostPieceBytes ? whole : kMostPieceBytes;
}

// A number that no other decode call of this process gets: it tells the counters that a call's
// workgroups have set up from whatever the workspace held before.  48 bits from a start that
// differs from process to process, so that values left in memory do not meet it by design.
uint64_t next_ticket() {
  static std::atomic<uint64_t> next{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9E3779B97F4A7C15ull};
  uint64_t t;
  do t = next.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed) >> 16;
  while (t == 0);
  return t;
}

// fedattn_prefill_sync_local_kv, participants' K/V not back to back: room for one aggregated copy each
size_t local_kv_copy_bytes(const fedattn_params* p, int32_t tokens) {
  return align_up((size_t)tokens * (size_t)p->n_kv_heads * (size_t)p->head_dim * (p->dtype == FEDATTN_BF16 ? 2 : 4), 256);
}

// Sync block on matrices that lie apart: where they are (entries as in PrefillArgs::own), and room for the kept rows of a sparse exchange.
struct ApartKv {
  const void* own[2 * kMaxApart];
  unsigned char *k_packed, *v_packed;
};

fedattn_status run_prefill(const fedattn_params* p, int32_t block_idx0, int32_t n_blocks, const void* q,
                           const void* k, const void* v, void* out, int64_t q_stride, int64_t kv_stride,
                           const int32_t* seg, const uint8_t* keep_chunks, int32_t chunk_tokens,
                           int32_t sync_override, void* workspace, size_t workspace_bytes, void* stream,
                           const ApartKv* apart = nullptr) {
  fedattn_status st = check_params(p);
  if (st != FEDATTN_OK) return st;
  st = check_offsets(p, seg);
  if (st != FEDATTN_OK) return st;
  if (block_idx0 < 0 || n_blocks < 0) return fail(FEDATTN_EINVAL, "negative block index or count");
  if (sync_override < -1 || sync_override > 1) return fail(FEDATTN_EINVAL, "sync_override must be -1, 0 or 1");
  const int N = p->n_participants;
  const int32_t total = seg[N];
  if (total == 0 || n_blocks == 0) return FEDATTN_OK;
  if (!q || !k || !v || !out) return fail(FEDATTN_EINVAL, "q, k, v and out must not be NULL");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out))
    return fail(FEDATTN_EINVAL, "q, k, v and out must be 16-byte aligned");
  if (n_blocks > 1 && (q_stride % 8 != 0 || kv_stride % 8 != 0 || q_stride < 0 || kv_stride < 0))
    return fail(FEDATTN_EINVAL, "block strides must be non-negative multiples of 8 elements");
  if (n_blocks > 65535) return fail(FEDATTN_EINVAL, "at most 65535 blocks per launch");
  const bool has_keep = keep_chunks != nullptr;
  if (has_keep && chunk_tokens <= 0) return fail(FEDATTN_EINVAL, "chunk_tokens must be positive with a keep-list");

  PrefillArgs a;
  memset(&a, 0, offsetof(PrefillArgs, own));   // what lies behind is written where it is read: entries past the participants' and tiles' count are not
  a.q = q; a.k = k; a.v = v; a.out = out;
  a.q_block_stride = q_stride;
  a.kv_block_stride = kv_stride;
  a.keep_chunks = keep_chunks;
  a.chunk_tokens = has_keep ? chunk_tokens : 1;
  a.total = total;
  a.Hq = p->n_q_heads; a.Hkv = p->n_kv_heads; a.D = p->head_dim;
  a.block_idx0 = block_idx0;
  a.sync_interval = p->sync_interval;
  a.sync_override = sync_override;
  a.causal = p->causal;
  a.scale = resolve_scale(p);
  a.seg.n = N;

  if (apart) {
    a.apart = 1;
    memcpy(a.own, apart->own, sizeof(a.own));
  }
  const bool mfma = use_mfma_prefill(p);
  a.k_list = k;
  a.v_list = v;
  const int G = a.Hq / a.Hkv;
  a.heads_per_wg = heads_in_common(a.Hq / a.Hkv);
  int64_t chunks = 0;
  for (int n = 0; n <= N; ++n) {
    a.seg.seg_off[n] = seg[n];
    a.seg.chunk_cum[n] = (int32_t)chunks;
    if (n < N && has_keep) chunks += ((int64_t)seg[n + 1] - seg[n] + chunk_tokens - 1) / chunk_tokens;
  }
  lay_out_query_tiles(a, kWaveRows * (4 / a.heads_per_wg));
  a.n_cus = device_cus();
  if ((int64_t)a.n_q_tiles * a.Hkv * (G / a.heads_per_wg) > 0x7fffffffLL) return fail(FEDATTN_EUNSUPPORTED, "too many query tiles");

  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  // a block reads the keep-list only if it is a sync block
  bool any_sync = sync_override == 1;
  if (sync_override == -1)
    for (int b = 0; b < n_blocks && !any_sync; ++b) any_sync = sync_block_rule(p->sync_interval, block_idx0 + b);
  if (!has_keep || !any_sync) a.keep_chunks = nullptr;

  // fp32 and bf16 with other head dimensions: the tile kernels too, but a keep-list call that comes
  // without a workspace runs on the general kernel, which reads the flags as they are
  bool tiled = true;
  if (a.keep_chunks) {
    if (n_blocks != 1) return fail(FEDATTN_EUNSUPPORTED, "a keep-list applies to one block per call");
    const PrefillWs w = prefill_ws_layout(p, total, chunk_tokens);
    const bool have_ws = workspace && workspace_bytes >= w.total;
    if (mfma && !have_ws)
      return fail(FEDATTN_EWORKSPACE, "prefill with a keep-list needs %zu workspace bytes, got %zu", w.total,
                  workspace_bytes);
    if (mfma && !aligned16(workspace)) return fail(FEDATTN_EINVAL, "workspace must be 16-byte aligned");
    tiled = have_ws && aligned16(workspace);
    if (tiled) {
      unsigned char* ws = reinterpret_cast<unsigned char*>(workspace);
      int32_t* kept_cum = reinterpret_cast<int32_t*>(ws);
      int2* kept_tiles = reinterpret_cast<int2*>(ws + w.tiles_off);
      a.kept_cum = kept_cum;
      a.kept_tiles = kept_tiles;
      hipError_t e;
      if (apart || needs_row_packing(chunk_tokens)) {
        PackArgs pack;
        unsigned char *k_packed = apart ? apart->k_packed : ws + w.k_off, *v_packed = apart ? apart->v_packed : ws + w.v_off;
        a.k_list = k_packed;
        a.v_list = v_packed;
        pack.keep_chunks = keep_chunks;
        pack.chunk_tokens = chunk_tokens;
        pack.n = N;
        pack.row_vecs = a.Hkv * a.D * elem_bytes(p) / 16;
        pack.k_packed = reinterpret_cast<uint4*>(k_packed);
        pack.v_packed = reinterpret_cast<uint4*>(v_packed);
        pack.kept_tiles = kept_tiles;
        pack.kept_cum = kept_cum;
        pack.k = k;
        pack.v = v;
        pack.apart = a.apart;
        if (apart) memcpy(pack.own, apart->own, sizeof(pack.own));
        memcpy(pack.seg_off, a.seg.seg_off, sizeof(pack.seg_off));
        memcpy(pack.chunk_cum, a.seg.chunk_cum, sizeof(pack.chunk_cum));
        e = launch_pack_kept_rows(pack, s);
      } else {
        e = launch_build_kept_tiles(a, kept_tiles, kept_cum, s);
      }
      if (e != hipSuccess) return fail(FEDATTN_ELAUNCH, "keep-list compaction: %s", hipGetErrorString(e));
    }
  }
  hipError_t e;
  if (!tiled)
    e = launch_prefill_generic(a, n_blocks, p->dtype, s);
  else
    e = p->dtype == FEDATTN_BF16 ? launch_prefill_mfma(a, n_blocks, s) : launch_prefill_f32(a, n_blocks, s);
  if (e != hipSuccess) return fail(FEDATTN_ELAUNCH, "prefill: %s", hipGetErrorString(e));
  return FEDATTN_OK;
}

}  // namespace

extern "C" {

int fedattn_is_sync_block(int32_t sync_interval, int32_t block_idx) {
  return sync_block_rule(sync_interval, block_idx) ? 1 : 0;
}

size_t fedattn_workspace_bytes(const fedattn_params* params, int32_t op, int32_t tokens, int32_t chunk_tokens) {
  if (check_params(params) != FEDATTN_OK || tokens < 0) return 0;
  if (op == FEDATTN_OP_PREFILL) return chunk_tokens > 0 ? prefill_ws_layout(params, tokens, chunk_tokens).total : 0;
  if (op == FEDATTN_OP_DECODE) return decode_ws_bytes(params, tokens);
  if (op == FEDATTN_OP_PREFILL_SYNC_LOCAL_KV)
    return 2 * local_kv_copy_bytes(params, tokens) + (chunk_tokens > 0 ? prefill_ws_layout(params, tokens, chunk_tokens).total : 0);
  fail(FEDATTN_EINVAL, "unknown op %d", op);
  return 0;
}

fedattn_status fedattn_prefill(const fedattn_params* params, int32_t block_idx, const void* q, const void* k,
                               const void* v, void* out, const int32_t* seg_offsets, const uint8_t* keep_chunks,
                               int32_t chunk_tokens, int32_t sync_override, void* workspace,
                               size_t workspace_bytes, void* stream) {
  return run_prefill(params, block_idx, 1, q, k, v, out, 0, 0, seg_offsets, keep_chunks, chunk_tokens,
                     sync_override, workspace, workspace_bytes, stream);
}

fedattn_status fedattn_prefill_sync_local_kv(const fedattn_params* params, const void* q, const void* const* k_local,
                                             const void* const* v_local, void* out, const int32_t* seg_offsets,
                                             const uint8_t* keep_chunks, int32_t chunk_tokens, void* workspace,
                                             size_t workspace_bytes, void* stream) {
  fedattn_status st = check_params(params);
  if (st != FEDATTN_OK) return st;
  st = check_offsets(params, seg_offsets);
  if (st != FEDATTN_OK) return st;
  if (!k_local || !v_local) return fail(FEDATTN_EINVAL, "k_local and v_local must not be NULL");
  const int N = params->n_participants;
  const int32_t total = seg_offsets[N];
  if (total == 0) return FEDATTN_OK;
  const int64_t row_bytes = (int64_t)params->n_kv_heads * params->head_dim * (params->dtype == FEDATTN_BF16 ? 2 : 4);
  // Sum_n Pi_n [k_n v_n] puts row r of participant n at global row seg_offsets[n] + r.  If every
  // participant's matrices already start that many rows behind one common base address, the
  // aggregated matrices exist as they are and the attention reads them in place.
  const unsigned char* k_base = nullptr;
  const unsigned char* v_base = nullptr;
  bool in_place = true, under_out = false;   // under_out: the output lies over a matrix
  const size_t out_bytes = (size_t)total * (size_t)params->n_q_heads * (size_t)params->head_dim * (size_t)elem_bytes(params);
  for (int n = 0; n < N; ++n) {
    if (seg_offsets[n + 1] == seg_offsets[n]) continue;
    if (!k_local[n] || !v_local[n]) return fail(FEDATTN_EINVAL, "local K/V of participant %d is NULL", n);
    if (!aligned16(k_local[n]) || !aligned16(v_local[n]))
      return fail(FEDATTN_EINVAL, "local K/V of participant %d is not 16-byte aligned", n);
    const unsigned char* kb = reinterpret_cast<const unsigned char*>(k_local[n]) - (int64_t)seg_offsets[n] * row_bytes;
    const unsigned char* vb = reinterpret_cast<const unsigned char*>(v_local[n]) - (int64_t)seg_offsets[n] * row_bytes;
    if (!k_base) {
      k_base = kb;
      v_base = vb;
    } else if (kb != k_base || vb != v_base) {
      in_place = false;
    }
    const size_t bytes = (size_t)(seg_offsets[n + 1] - seg_offsets[n]) * (size_t)row_bytes;
    for (const void* m : {k_local[n], v_local[n]})
      under_out = under_out || ranges_meet(reinterpret_cast<uintptr_t>(m), bytes, reinterpret_cast<uintptr_t>(out), out_bytes);
  }
  unsigned char* ws = reinterpret_cast<unsigned char*>(workspace);
  size_t ws_left = workspace ? workspace_bytes : 0;
  if (!in_place) {
    const size_t copy = local_kv_copy_bytes(params, total);
    if (!workspace || workspace_bytes < 2 * copy)
      return fail(FEDATTN_EWORKSPACE,
                  "the participants' K/V do not lie back to back: aggregating them needs %zu workspace bytes, got %zu",
                  2 * copy, workspace_bytes);
    if (!aligned16(workspace)) return fail(FEDATTN_EINVAL, "workspace must be 16-byte aligned");
    if (keep_chunks && chunk_tokens > 0) {
      // fp32 and other head dimensions: with less than the whole the general kernel runs, as in fedattn_prefill;
      // room for the list is asked for all the same, as it was before these shapes packed rows
      const PrefillWs w = prefill_ws_layout(params, total, chunk_tokens);
      const size_t need = 2 * copy + (use_mfma_prefill(params) ? w.total : w.list_end);
      if (workspace_bytes < need)
        return fail(FEDATTN_EWORKSPACE, "workspace too small for the aggregated copy and the keep-list (%zu bytes needed)", need);
    }
    k_base = ws;
    v_base = ws + copy;
    ws += 2 * copy;
    ws_left -= 2 * copy;
  }
  // q, out and the keep-list arguments are validated by the prefill path; when they pass,
  // nothing there can fail short of a launch error, so the copy is enqueued only for valid calls
  if (!q || !out || !aligned16(q) || !aligned16(out)) return fail(FEDATTN_EINVAL, "q and out must be non-NULL and 16-byte aligned");
  if (keep_chunks && chunk_tokens <= 0) return fail(FEDATTN_EINVAL, "chunk_tokens must be positive with a keep-list");
  const auto dense_apart = [&] {   // scales that are folded only: the kernels that read dense tiles apart are of that kind
    const int heads = heads_in_common(params->n_q_heads / params->n_kv_heads);
    return folds_scale(resolve_scale(params), params->head_dim) &&
           read_apart(PrefillShape{seg_offsets, N, params->n_q_heads, params->n_kv_heads, params->head_dim, params->causal != 0, false, heads,
                                   kWaveRows * (4 / heads), device_cus()});
  };
  if (!in_place && !under_out && N <= kMaxApart && use_mfma_prefill(params) && (keep_chunks || dense_apart())) {
    // Every participant's rows are read where they are, or, the kept ones of a sparse exchange, packed from there; these
    // take the place of the aggregated copy, whose address stands for the matrices in the checks.  Not where the output
    // lies over a matrix: workgroups write rows of it while others still read.
    ApartKv apart;
    apart.k_packed = const_cast<unsigned char*>(k_base);
    apart.v_packed = const_cast<unsigned char*>(v_base);
    for (int n = 0; n < kMaxApart; ++n)
      for (int kv = 0; kv < 2; ++kv) {
        const bool has_rows = n < N && seg_offsets[n + 1] > seg_offsets[n];
        apart.own[2 * n + kv] = has_rows ? reinterpret_cast<const unsigned char*>((kv ? v_local : k_local)[n]) - (int64_t)seg_offsets[n] * row_bytes : nullptr;
      }
    return run_prefill(params, 0, 1, q, k_base, v_base, out, 0, 0, seg_offsets, keep_chunks, chunk_tokens, 1, ws, ws_left, stream, &apart);
  }
  if (!in_place) {
    st = fedattn_aggregate_kv(params, k_local, v_local, seg_offsets, const_cast<unsigned char*>(k_base),
                              const_cast<unsigned char*>(v_base), stream);
    if (st != FEDATTN_OK) return st;
  }
  return run_prefill(params, 0, 1, q, k_base, v_base, out, 0, 0, seg_offsets, keep_chunks, chunk_tokens, 1,
                     ws_left ? ws : nullptr, ws_left, stream);
}

fedattn_status fedattn_prefill_blocks(const fedattn_params* params, int32_t block_idx0, int32_t n_blocks,
                                      const void* q, const void* k, const void* v, void* out,
                                      int64_t q_block_stride, int64_t kv_block_stride,
                                      const int32_t* seg_offsets, void* stream) {
  return run_prefill(params, block_idx0, n_blocks, q, k, v, out, q_block_stride, kv_block_stride, seg_offsets,
                     nullptr, 0, -1, nullptr, 0, stream);
}

// Everything about a decode call that can be checked without the workspace or the device.
static fedattn_status check_decode_args(const fedattn_params* params, int32_t block_idx0, int32_t n_blocks, const void* q,
                                        const void* k_cache, const void* v_cache, void* out, int64_t q_block_stride,
                                        int64_t cache_block_stride, const int32_t* seg_offsets, const int32_t* seg_lens,
                                        const int32_t* remote_lens, int32_t sync_override) {
  fedattn_status st = check_params(params);
  if (st != FEDATTN_OK) return st;
  st = check_offsets(params, seg_offsets);
  if (st != FEDATTN_OK) return st;
  if (!seg_lens) return fail(FEDATTN_EINVAL, "seg_lens is NULL");
  if (block_idx0 < 0 || n_blocks < 0) return fail(FEDATTN_EINVAL, "negative block index or count");
  if (sync_override < -1 || sync_override > 1) return fail(FEDATTN_EINVAL, "sync_override must be -1, 0 or 1");
  const int N = params->n_participants;
  for (int n = 0; n < N; ++n) {
    const int cap = seg_offsets[n + 1] - seg_offsets[n];
    if (seg_lens[n] < 0 || seg_lens[n] > cap)
      return fail(FEDATTN_EINVAL, "seg_lens[%d] = %d outside 0..capacity %d", n, seg_lens[n], cap);
    if (remote_lens && (remote_lens[n] < 0 || remote_lens[n] > cap))
      return fail(FEDATTN_EINVAL, "remote_lens[%d] = %d outside 0..capacity %d", n, remote_lens[n], cap);
  }
  if (n_blocks == 0) return FEDATTN_OK;
  if (!q || !out) return fail(FEDATTN_EINVAL, "q and out must not be NULL");
  const int32_t capacity = seg_offsets[N];
  if (capacity > 0 && (!k_cache || !v_cache)) return fail(FEDATTN_EINVAL, "k_cache and v_cache must not be NULL");
  if (!aligned16(q) || !aligned16(out) || !aligned16(k_cache) || !aligned16(v_cache))
    return fail(FEDATTN_EINVAL, "q, out, k_cache and v_cache must be 16-byte aligned");
  if (n_blocks > 1 && (q_block_stride % 8 != 0 || cache_block_stride % 8 != 0 || q_block_stride < 0 ||
                       cache_block_stride < 0))
    return fail(FEDATTN_EINVAL, "block strides must be non-negative multiples of 8 elements");

  return FEDATTN_OK;
}

// Whether n_blocks blocks can run in any order, or at the same time: no block writes what it or another one reads or writes.
static bool blocks_apart(const fedattn_params* p, int32_t n_blocks, const void* q, const void* k_cache, const void* v_cache,
                         const void* out, int64_t q_block_stride, int64_t cache_block_stride, int32_t capacity) {
  const int64_t q_elems = (int64_t)p->n_participants * p->n_q_heads * p->head_dim;
  const int64_t kv_elems = (int64_t)capacity * p->n_kv_heads * p->head_dim;
  const int64_t esize = elem_bytes(p);
  if (q_block_stride < q_elems) return false;   // output blocks overlap one another
  const auto end = [&](const void* base, int64_t stride, int64_t elems) {
    return reinterpret_cast<uintptr_t>(base) + ((uintptr_t)(n_blocks - 1) * (uintptr_t)stride + (uintptr_t)elems) * (uintptr_t)esize;
  };
  const uintptr_t out_lo = reinterpret_cast<uintptr_t>(out), out_hi = end(out, q_block_stride, q_elems);
  const auto hits = [&](const void* base, int64_t stride, int64_t elems) {
    return reinterpret_cast<uintptr_t>(base) < out_hi && out_lo < end(base, stride, elems);
  };
  return !hits(q, q_block_stride, q_elems) && !hits(k_cache, cache_block_stride, kv_elems) && !hits(v_cache, cache_block_stride, kv_elems);
}

// Blocks of one kind (local / sync) share launches, as many per launch as the workspace has room for, when the caller
// says that they may (`fused`) or their memory shows it; otherwise one launch (pair) per block in block order.
// A launch of one block leaves the chip idle at its start and end, about half its time at 16 x 1152 rows.  Calls one
// launch per block and shared, us: 6 local and 2 sync blocks of 16 x 1152 rows, 32/8 heads of 128 152 -> 130 (4.65 TB/s);
// 8 sync blocks of 1 x 312..1041 rows, 8/1 heads of 64 44 -> 12; 2 of 3 x 76, 32/4 heads of 64 17.3 -> 9.0; none slower.
static fedattn_status run_decode(bool fused, const fedattn_params* params, int32_t block_idx0, int32_t n_blocks,
                                 const void* q, const void* k_cache, const void* v_cache, void* out,
                                 int64_t q_block_stride, int64_t cache_block_stride,
                                 const int32_t* seg_offsets, const int32_t* seg_lens,
                                 const int32_t* remote_lens, int32_t sync_override, void* workspace,
                                 size_t workspace_bytes, void* stream) {
  fedattn_status st = check_decode_args(params, block_idx0, n_blocks, q, k_cache, v_cache, out, q_block_stride,
                                        cache_block_stride, seg_offsets, seg_lens, remote_lens, sync_override);
  if (st != FEDATTN_OK) return st;
  if (n_blocks == 0) return FEDATTN_OK;
  const int N = params->n_participants;
  const int32_t capacity = seg_offsets[N];

  // fp32 and bf16 with other head dimensions: split too, but a call that comes without the workspace
  // runs one wavefront per (participant, head)
  const bool must_split = use_mfma_prefill(params);
  bool split = true;
  const size_t esize = (size_t)elem_bytes(params);
  DecodeArgs args[2];  // [0] local block, [1] sync block: the split differs, the layout does not
  bool built[2] = {false, false};
  uint64_t* counters = nullptr;
  const uint64_t ticket = next_ticket();
  bool counters_ready[2] = {false, false};   // a launch of this call and kind has set its counters up, and every launch leaves them at zero
  const size_t need = decode_ws_bytes(params, capacity);
  if (!workspace || workspace_bytes < need) {
    if (must_split) return fail(FEDATTN_EWORKSPACE, "decode needs %zu workspace bytes, got %zu", need, workspace_bytes);
    split = false;
  } else if (!aligned16(workspace)) {
    if (must_split) return fail(FEDATTN_EINVAL, "workspace must be 16-byte aligned");
    split = false;
  }
  // tens of thousands of KV heads: the counters alone take the piece's room
  if (split && !must_split && need == kMostPieceBytes) {
    const size_t chunks = (size_t)decode_target_chunks(params->n_kv_heads) + (size_t)N;
    if (decode_counter_bytes(params) + 512 + chunks * 16 * ((size_t)params->head_dim * 4 + 8) > need) split = false;
  }
  if (fused && split && n_blocks > 65535) return fail(FEDATTN_EINVAL, "at most 65535 blocks per fused call");
  const bool shared = split && n_blocks > 1 && n_blocks <= 65535 &&
                      (fused || blocks_apart(params, n_blocks, q, k_cache, v_cache, out, q_block_stride, cache_block_stride, capacity));
  int slices[2] = {1, 1};   // blocks of a kind in flight at once, each with partials and counters of its own in the workspace
  // blocks one after the other count their chunks in at the end of the workspace
  if (split) counters = reinterpret_cast<uint64_t*>(reinterpret_cast<unsigned char*>(workspace) + need - decode_counter_bytes(params));
  const auto block_is_sync = [&](int b) {
    return sync_override >= 0 ? sync_override != 0 : sync_block_rule(params->sync_interval, block_idx0 + b);
  };
  const auto prepare = [&](bool sync) -> fedattn_status {
    DecodeArgs& a = args[sync ? 1 : 0];
    if (!built[sync ? 1 : 0]) {
      memset(&a, 0, sizeof(a));
      a.N = N; a.Hq = params->n_q_heads; a.Hkv = params->n_kv_heads; a.D = params->head_dim;
      a.n_cus = device_cus();
      a.is_sync = sync ? 1 : 0;
      a.has_remote = (sync && remote_lens) ? 1 : 0;
      a.scale = resolve_scale(params);
      const int G = a.Hq / a.Hkv;
      a.cols = sync ? N * G : G;
      int64_t total_rows = 0;
      int32_t rows_of[kMaxP];   // cache rows that some query sees
      for (int n = 0; n < N; ++n) {
        const int rem = a.has_remote ? remote_lens[n] : seg_lens[n];
        rows_of[n] = sync && rem > seg_lens[n] ? rem : seg_lens[n];
        total_rows += rows_of[n];
      }
      a.chunk_rows = decode_chunk_rows(total_rows, a.Hkv);
      if (split && a.cols > 16 && params->dtype == FEDATTN_BF16)
        a.chunk_rows = wide_chunk_rows(rows_of, N, a.chunk_rows, a.Hkv, a.D, a.cols, a.n_cus);
      int64_t chunks = 0;
      for (int n = 0; n <= N; ++n) {
        a.seg_off[n] = seg_offsets[n];
        a.chunk_cum[n] = (int32_t)chunks;
        if (n < N) {
          a.seg_lens[n] = seg_lens[n];
          a.remote_lens[n] = remote_lens ? remote_lens[n] : seg_lens[n];
          chunks += ((int64_t)rows_of[n] + a.chunk_rows - 1) / a.chunk_rows;
        }
      }
      a.n_chunks = (int32_t)chunks;
      if (split) {
        const size_t room = need - decode_counter_bytes(params);
        const auto o_bytes_of = [&](int n_g, int n_cols) {
          return align_up((size_t)n_g * (size_t)a.n_chunks * (size_t)n_cols * (size_t)a.D * 4, 256);
        };
        const auto bytes_of = [&](int n_g, int n_cols) {
          return o_bytes_of(n_g, n_cols) + (size_t)n_g * (size_t)a.n_chunks * (size_t)n_cols * 8;
        };
        a.n_g = a.Hkv;
        a.n_cols = a.cols;
        const bool whole = bytes_of(a.Hkv, a.cols) <= room;
        if (!whole) {
          if (must_split)
            return fail(FEDATTN_EWORKSPACE, "decode partials (%zu bytes) exceed the workspace", bytes_of(a.Hkv, a.cols));
          // as many KV heads as fit, or one head's columns in whole workgroups' (64) or wavefronts' (16) shares
          const size_t fit = (room - 256) / ((size_t)a.n_chunks * ((size_t)a.D * 4 + 8));   // (KV head, column) pairs
          a.n_g = fit >= (size_t)a.cols ? (int)(fit / (size_t)a.cols) : 1;
          if (a.n_g == 1 && fit < (size_t)a.cols) a.n_cols = (int)(fit >= 64 ? fit / 64 * 64 : fit / 16 * 16);
          if (a.n_cols == 0)
            return fail(FEDATTN_EWORKSPACE, "decode partials of 16 query columns (%zu bytes) exceed the workspace", bytes_of(1, 16));
        }
        const size_t o_bytes = o_bytes_of(a.n_g, a.n_cols);
        a.part_o = reinterpret_cast<float*>(workspace);
        a.part_ml = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(workspace) + o_bytes);
        a.counters = counters;
        if (shared) {
          const size_t slice = whole ? align_up(bytes_of(a.Hkv, a.cols), 256) + decode_counter_bytes(params) : align_up(need, 256);
          if (whole) a.counters = reinterpret_cast<uint64_t*>(reinterpret_cast<unsigned char*>(workspace) + slice - decode_counter_bytes(params));
          const size_t fit = 1 + (workspace_bytes - (whole ? slice : need)) / slice;
          slices[sync ? 1 : 0] = (int)(fit < (size_t)kMaxFusedBlocks ? fit : (size_t)kMaxFusedBlocks);
          a.slice_bytes = (int64_t)slice;
        }
        // Merge inside the split kernel, by the workgroup that finishes last: up to 16 query columns
        // share a workgroup per chunk, and every output row needs a chunk to come from (an empty
        // segment's zero rows come from the separate combine kernel).  It makes a round trip to memory
        // per kMergeBatch chunks and 256 x 4 elements, about 0.9 us, where the combine kernel costs
        // 3.5 us for its launch (bf16 calls of one block, combined apart and inside: 1 x 2048 rows, 8/2 heads
        // of 128, 4 trips 10.8 and 9.3 us; 1 x 4096 rows, 8 trips 11.1 and 13.7; sync blocks of 1 x 64 rows
        // 12.0 and 8.3, of 3 x 64..400 rows 11.0 and 9.9, of 4 x 1000 rows, 16 trips 11.5 and 22.3).
        bool all_have_rows = true;
        int64_t most = 0;   // chunks merged into one row
        for (int n = 0; n < N; ++n) {
          all_have_rows = all_have_rows && seg_lens[n] > 0;
          const int64_t c = ((int64_t)seg_lens[n] + a.chunk_rows - 1) / a.chunk_rows;
          most = c > most ? c : most;
        }
        if (sync) {
          all_have_rows = chunks > 0;
          most = chunks;
        }
        const int64_t trips = ((int64_t)a.cols * (a.D / 4) + 255) / 256 * ((most + kMergeBatch - 1) / kMergeBatch);
        a.merge_in_kernel = whole && all_have_rows && a.cols <= 16 && (most == 1 || trips <= kMaxMergeTrips) ? 1 : 0;
      }
      a.q_block_bytes = q_block_stride * (int64_t)esize;
      a.cache_block_bytes = cache_block_stride * (int64_t)esize;
      built[sync ? 1 : 0] = true;
    }
    return FEDATTN_OK;
  };
  // n_z blocks of one kind: one launch (and its combine), or one per piece in stream order, all pieces through the same partials
  const auto launch = [&](const DecodeArgs& kind, int n_z) -> hipError_t {
    if (!split || (kind.n_g == kind.Hkv && kind.n_cols == kind.cols))
      return launch_decode(kind, params->dtype, split, n_z, reinterpret_cast<hipStream_t>(stream));
    DecodeArgs a = kind;
    for (a.g0 = 0; a.g0 < a.Hkv; a.g0 += kind.n_g) {
      a.n_g = kind.n_g < a.Hkv - a.g0 ? kind.n_g : a.Hkv - a.g0;
      for (a.col0 = 0; a.col0 < a.cols; a.col0 += kind.n_cols) {
        a.n_cols = kind.n_cols < a.cols - a.col0 ? kind.n_cols : a.cols - a.col0;
        const hipError_t e = launch_decode(a, params->dtype, split, n_z, reinterpret_cast<hipStream_t>(stream));
        if (e != hipSuccess) return e;
      }
    }
    return hipSuccess;
  };
  // everything that can fail validation is decided before the first launch
  for (int b = 0; b < n_blocks && !(built[0] && built[1]); ++b) {
    st = prepare(block_is_sync(b));
    if (st != FEDATTN_OK) return st;
  }
  if (shared) {
    for (int kind = 0; kind < 2; ++kind) {
      // launches of about one size: 24 blocks with room for 23 as 12 and 12
      int of_kind = 0;
      for (int b = 0; b < n_blocks; ++b) of_kind += (block_is_sync(b) ? 1 : 0) == kind ? 1 : 0;
      if (of_kind == 0) continue;
      const int launches = (of_kind + slices[kind] - 1) / slices[kind], at_once = (of_kind + launches - 1) / launches;
      int first = 0;
      while (first < n_blocks) {
        int cnt = 0;
        DecodeArgs& a = args[kind];
        int b = first;
        for (; b < n_blocks && cnt < at_once; ++b) {
          if ((block_is_sync(b) ? 1 : 0) != kind) continue;
          a.block_list[cnt++] = (uint16_t)b;
        }
        first = b;
        if (cnt == 0) continue;
        a.q = q; a.out = out; a.k_cache = k_cache; a.v_cache = v_cache;
        a.ticket = counters_ready[kind] ? 0 : ticket;   // no later launch of this kind has more blocks than the first
        counters_ready[kind] = true;
        hipError_t e = launch(a, cnt);
        if (e != hipSuccess) return fail(FEDATTN_ELAUNCH, "decode (%d blocks at once): %s", cnt, hipGetErrorString(e));
      }
    }
    return FEDATTN_OK;
  }
  for (int b = 0; b < n_blocks; ++b) {
    const bool sync = block_is_sync(b);
    st = prepare(sync);
    if (st != FEDATTN_OK) return st;
    DecodeArgs& a = args[sync ? 1 : 0];
    a.q = reinterpret_cast<const unsigned char*>(q) + (size_t)b * (size_t)q_block_stride * esize;
    a.out = reinterpret_cast<unsigned char*>(out) + (size_t)b * (size_t)q_block_stride * esize;
    a.k_cache = reinterpret_cast<const unsigned char*>(k_cache) + (size_t)b * (size_t)cache_block_stride * esize;
    a.v_cache = reinterpret_cast<const unsigned char*>(v_cache) + (size_t)b * (size_t)cache_block_stride * esize;
    a.ticket = counters_ready[sync ? 1 : 0] ? 0 : ticket;
    counters_ready[sync ? 1 : 0] = true;
    hipError_t e = launch(a, 1);
    if (e != hipSuccess) return fail(FEDATTN_ELAUNCH, "decode (block %d): %s", block_idx0 + b, hipGetErrorString(e));
  }
  return FEDATTN_OK;
}

fedattn_status fedattn_decode_blocks(const fedattn_params* params, int32_t block_idx0, int32_t n_blocks,
                                     const void* q, const void* k_cache, const void* v_cache, void* out,
                                     int64_t q_block_stride, int64_t cache_block_stride,
                                     const int32_t* seg_offsets, const int32_t* seg_lens,
                                     const int32_t* remote_lens, int32_t sync_override, void* workspace,
                                     size_t workspace_bytes, void* stream) {
  return run_decode(false, params, block_idx0, n_blocks, q, k_cache, v_cache, out, q_block_stride, cache_block_stride,
                    seg_offsets, seg_lens, remote_lens, sync_override, workspace, workspace_bytes, stream);
}

fedattn_status fedattn_decode_blocks_fused(const fedattn_params* params, int32_t block_idx0, int32_t n_blocks,
                                           const void* q, const void* k_cache, const void* v_cache, void* out,
                                           int64_t q_block_stride, int64_t cache_block_stride,
                                           const int32_t* seg_offsets, const int32_t* seg_lens,
                                           const int32_t* remote_lens, int32_t sync_override, void* workspace,
                                           size_t workspace_bytes, void* stream) {
  return run_decode(true, params, block_idx0, n_blocks, q, k_cache, v_cache, out, q_block_stride, cache_block_stride,
                    seg_offsets, seg_lens, remote_lens, sync_override, workspace, workspace_bytes, stream);
}

fedattn_status fedattn_decode(const fedattn_params* params, int32_t block_idx, const void* q, const void* k_cache,
                              const void* v_cache, void* out, const int32_t* seg_offsets, const int32_t* seg_lens,
                              const int32_t* remote_lens, int32_t sync_override, void* workspace,
                              size_t workspace_bytes, void* stream) {
  return fedattn_decode_blocks(params, block_idx, 1, q, k_cache, v_cache, out, 0, 0, seg_offsets, seg_lens,
                               remote_lens, sync_override, workspace, workspace_bytes, stream);
}

// ---- decode for callers that cannot allocate ---------------------------------------------
// The split-KV partials and chunk counters of fedattn_decode live in this array instead of a
// caller's workspace.  Every device the library runs on holds its own copy at its own address;
// in host code the array's name is only a handle for hipGetSymbolAddress, never an address.
static __device__ __align__(256) unsigned char scratch[FEDATTN_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxScratchDevices];  // device address of `scratch`, per device; NULL until looked up

// Device address of the current device's copy of `scratch` (looked up once per device).
fedattn_status static_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(FEDATTN_ELAUNCH, "hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxScratchDevices)
    return fail(FEDATTN_EUNSUPPORTED, "device %d outside 0..%d", dev, kMaxScratchDevices - 1);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(FEDATTN_ELAUNCH, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return FEDATTN_OK;
}
}  // namespace

fedattn_status fedattn_decode_static(const fedattn_params* params, int32_t block_idx, const void* q,
                                     const void* k_cache, const void* v_cache, void* out,
                                     const int32_t* seg_offsets, const int32_t* seg_lens,
                                     const int32_t* remote_lens, int32_t sync_override, void* stream) {
  fedattn_status st = check_decode_args(params, block_idx, 1, q, k_cache, v_cache, out, 0, 0, seg_offsets, seg_lens,
                                        remote_lens, sync_override);
  if (st != FEDATTN_OK) return st;
  const size_t need = decode_ws_bytes(params, seg_offsets[params->n_participants]);
  if (need > (size_t)FEDATTN_STATIC_SCRATCH_BYTES)
    return fail(FEDATTN_EWORKSPACE,
                "fedattn_decode_static: this problem needs %zu bytes of scratch, the built-in array holds %zu; "
                "use fedattn_decode with a workspace",
                need, (size_t)FEDATTN_STATIC_SCRATCH_BYTES);
  void* ptr = nullptr;
  st = static_scratch(&ptr);
  if (st != FEDATTN_OK) return st;
  return run_decode(false, params, block_idx, 1, q, k_cache, v_cache, out, 0, 0, seg_offsets, seg_lens, remote_lens,
                    sync_override, ptr, (size_t)FEDATTN_STATIC_SCRATCH_BYTES, stream);
}

fedattn_status fedattn_aggregate_kv(const fedattn_params* params, const void* const* k_local,
                                    const void* const* v_local, const int32_t* seg_offsets, void* k_global,
                                    void* v_global, void* stream) {
  fedattn_status st = check_params(params);
  if (st != FEDATTN_OK) return st;
  st = check_offsets(params, seg_offsets);
  if (st != FEDATTN_OK) return st;
  if (!k_local || !v_local) return fail(FEDATTN_EINVAL, "k_local and v_local must not be NULL");
  const int N = params->n_participants;
  if (seg_offsets[N] == 0) return FEDATTN_OK;
  if (!k_global || !v_global || !aligned16(k_global) || !aligned16(v_global))
    return fail(FEDATTN_EINVAL, "k_global and v_global must be non-NULL and 16-byte aligned");
  AggregateArgs a;
  memset(&a, 0, sizeof(a));
  a.n = N;
  a.row_bytes = params->n_kv_heads * params->head_dim * (params->dtype == FEDATTN_BF16 ? 2 : 4);
  a.k_global = k_global;
  a.v_global = v_global;
  for (int n = 0; n <= N; ++n) a.seg_off[n] = seg_offsets[n];
  for (int n = 0; n < N; ++n) {
    a.k_local[n] = k_local[n];
    a.v_local[n] = v_local[n];
    if (seg_offsets[n + 1] > seg_offsets[n]) {
      if (!k_local[n] || !v_local[n]) return fail(FEDATTN_EINVAL, "local K/V of participant %d is NULL", n);
      if (!aligned16(k_local[n]) || !aligned16(v_local[n]))
        return fail(FEDATTN_EINVAL, "local K/V of participant %d is not 16-byte aligned", n);
    }
  }
  hipError_t e = launch_aggregate(a, reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) return fail(FEDATTN_ELAUNCH, "aggregate: %s", hipGetErrorString(e));
  return FEDATTN_OK;
}

// ---- element-wise pieces of the decoder block around the attention ----------------------
namespace {
constexpr int64_t kMaxGrid = 0x7fffffffLL;
}

fedattn_status fedattn_rmsnorm(const float* x, void* out, int64_t rows, int32_t d_model, float eps, void* stream) {
  if (rows < 0 || d_model <= 0 || d_model % 4 != 0) return fail(FEDATTN_EINVAL, "rmsnorm: rows >= 0, d_model a positive multiple of 4");
  if (!(eps >= 0.f)) return fail(FEDATTN_EINVAL, "rmsnorm: eps must be non-negative");
  if (rows == 0) return FEDATTN_OK;
  if (!x || !out || !aligned16(x) || !aligned16(out)) return fail(FEDATTN_EINVAL, "rmsnorm: x and out must be non-NULL and 16-byte aligned");
  if ((rows + 3) / 4 > kMaxGrid) return fail(FEDATTN_EUNSUPPORTED, "rmsnorm: too many rows");
  hipError_t e = launch_rmsnorm(x, out, rows, d_model, eps, reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) return fail(FEDATTN_ELAUNCH, "rmsnorm: %s", hipGetErrorString(e));
  return FEDATTN_OK;
}

fedattn_status fedattn_residual_add_rmsnorm(float* x, const void* y, void* out, int64_t rows, int32_t d_model, float eps,
                                            void* stream) {
  if (rows < 0 || d_model <= 0 || d_model % 4 != 0)
    return fail(FEDATTN_EINVAL, "residual_add_rmsnorm: rows >= 0, d_model a positive multiple of 4");
  if (!(eps >= 0.f)) return fail(FEDATTN_EINVAL, "residual_add_rmsnorm: eps must be non-negative");
  if (rows == 0) return FEDATTN_OK;
  if (!x || !y || !out || !aligned16(x) || !aligned16(y) || !aligned16(out))
    return fail(FEDATTN_EINVAL, "residual_add_rmsnorm: x, y and out must be non-NULL and 16-byte aligned");
  if ((rows + 3) / 4 > kMaxGrid) return fail(FEDATTN_EUNSUPPORTED, "residual_add_rmsnorm: too many rows");
  hipError_t e = launch_residual_add_rmsnorm(x, y, out, rows, d_model, eps, reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) return fail(FEDATTN_ELAUNCH, "residual_add_rmsnorm: %s", hipGetErrorString(e));
  return FEDATTN_OK;
}

fedattn_status fedattn_rope_split_qkv(const void* qkv, const int32_t* pos, void* q, void* k, void* v, int64_t tokens,
                                      int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, float theta,
                                      void* stream) {
  if (tokens < 0 || n_q_heads <= 0 || n_kv_heads <= 0 || head_dim <= 0 || head_dim % 8 != 0)
    return fail(FEDATTN_EINVAL, "rope: tokens >= 0, positive head counts, head_dim a positive multiple of 8");
  if (!(theta > 1.f)) return fail(FEDATTN_EINVAL, "rope: theta must exceed 1");
  if (tokens == 0) return FEDATTN_OK;
  if (!qkv || !q || !k || !v || !aligned16(qkv) || !aligned16(q) || !aligned16(k) || !aligned16(v))
    return fail(FEDATTN_EINVAL, "rope: qkv, q, k and v must be non-NULL and 16-byte aligned");
  if (tokens * (head_dim / 8) / 256 + 1 > kMaxGrid) return fail(FEDATTN_EUNSUPPORTED, "rope: too many tokens");
  hipError_t e = launch_rope_split(qkv, pos, q, k, v, tokens, n_q_heads, n_kv_heads, head_dim, theta,
                                   reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) return fail(FEDATTN_ELAUNCH, "rope: %s", hipGetErrorString(e));
  return FEDATTN_OK;
}

fedattn_status fedattn_swiglu(const void* gate_up, void* out, int64_t rows, int32_t hidden, void* stream) {
  if (rows < 0 || hidden <= 0 || hidden % 8 != 0) return fail(FEDATTN_EINVAL, "swiglu: rows >= 0, hidden a positive multiple of 8");
  if (rows == 0) return FEDATTN_OK;
  if (!gate_up || !out || !aligned16(gate_up) || !aligned16(out)) return fail(FEDATTN_EINVAL, "swiglu: gate_up and out must be non-NULL and 16-byte aligned");
  if (rows * (hidden / 8) / 256 + 1 > kMaxGrid) return fail(FEDATTN_EUNSUPPORTED, "swiglu: too many elements");
  hipError_t e = launch_swiglu(gate_up, out, rows, hidden, reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) return fail(FEDATTN_ELAUNCH, "swiglu: %s", hipGetErrorString(e));
  return FEDATTN_OK;
}

fedattn_status fedattn_residual_add(float* x, const void* y, int64_t n, void* stream) {
  if (n < 0 || n % 4 != 0) return fail(FEDATTN_EINVAL, "residual_add: n must be a non-negative multiple of 4");
  if (n == 0) return FEDATTN_OK;
  if (!x || !y || !aligned16(x) || !aligned16(y)) return fail(FEDATTN_EINVAL, "residual_add: x and y must be non-NULL and 16-byte aligned");
  if (n / 4 / 256 + 1 > kMaxGrid) return fail(FEDATTN_EUNSUPPORTED, "residual_add: too many elements");
  hipError_t e = launch_residual_add(x, y, n, reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) return fail(FEDATTN_ELAUNCH, "residual_add: %s", hipGetErrorString(e));
  return FEDATTN_OK;
}

// ---- measurement aids ---------------------------------------------------------------------
int64_t fedattn_probe_stream(const void* src, int64_t bytes, int32_t pattern, void* sink, void* stream) {
  if (!src || !sink || !aligned16(src) || bytes <= 0 || (pattern != 0 && pattern != 1)) {
    fail(FEDATTN_EINVAL, "probe_stream: src and sink non-NULL, src 16-byte aligned, bytes > 0, pattern 0 or 1");
    return -1;
  }
  const int n_wgs = device_cus() / 8 * 8;
  const int64_t unit = pattern == 0 ? (int64_t)n_wgs * 32768 : (int64_t)n_wgs * 64 * 256 * 2;
  const int64_t moved = bytes / unit * unit;
  if (moved == 0) {
    fail(FEDATTN_EINVAL, "probe_stream: at least %lld bytes", (long long)unit);
    return -1;
  }
  hipError_t e = launch_stream_probe(src, moved, n_wgs, pattern, reinterpret_cast<float*>(sink), reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) {
    fail(FEDATTN_ELAUNCH, "probe_stream: %s", hipGetErrorString(e));
    return -1;
  }
  return moved;
}

int64_t fedattn_probe_mfma(void* sink, int32_t iters, void* stream) {
  if (!sink || iters <= 0) {
    fail(FEDATTN_EINVAL, "probe_mfma: sink non-NULL, iters > 0");
    return -1;
  }
  const int n_wgs = device_cus();
  hipError_t e = launch_mfma_probe(reinterpret_cast<float*>(sink), n_wgs, iters, reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) {
    fail(FEDATTN_ELAUNCH, "probe_mfma: %s", hipGetErrorString(e));
    return -1;
  }
  return (int64_t)n_wgs * 8 /* wavefronts */ * iters * 8 /* MFMAs */ * (2LL * 32 * 32 * 16);
}

const char* fedattn_last_error(void) { return g_err; }

const char* fedattn_version(void) { return "fedattn-gfx950 0.1"; }

}  // extern "C"
