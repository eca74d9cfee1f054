// The library's host side with its launchers replaced by ones that write down what they are asked to launch: which
// kernels a call takes and what it hands them, without a device.  Pointers stand for device memory and are never read.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "common.h"

namespace fedattn {
struct Launch {
  std::string kernel;
  PrefillArgs prefill;
  DecodeArgs decode;
  int blocks;
};
static std::vector<Launch> launched;
static hipError_t note(const char* kernel, const PrefillArgs* a = nullptr) {
  launched.emplace_back();
  launched.back().kernel = kernel;
  if (a) std::memcpy(static_cast<void*>(&launched.back().prefill), a, sizeof(*a));
  return hipSuccess;
}
hipError_t launch_prefill_generic(const PrefillArgs& a, int, int, hipStream_t) { return note("generic", &a); }
hipError_t launch_prefill_mfma(PrefillArgs& a, int, hipStream_t) { return note("mfma", &a); }
hipError_t launch_prefill_f32(PrefillArgs& a, int, hipStream_t) { return note("f32", &a); }
hipError_t launch_build_kept_tiles(const PrefillArgs& a, int2*, int32_t*, hipStream_t) { return note("list", &a); }
hipError_t launch_pack_kept_rows(PackArgs&, hipStream_t) { return note("pack"); }
hipError_t launch_decode(const DecodeArgs& a, int, bool, int n_z, hipStream_t) {
  note("decode");
  launched.back().decode = a;
  launched.back().blocks = n_z;
  return hipSuccess;
}
hipError_t launch_aggregate(const AggregateArgs&, hipStream_t) { return note("aggregate"); }
hipError_t launch_rmsnorm(const float*, void*, int64_t, int, float, hipStream_t) { return note("rmsnorm"); }
hipError_t launch_residual_add_rmsnorm(float*, const void*, void*, int64_t, int, float, hipStream_t) { return note("rmsnorm"); }
hipError_t launch_rope_split(const void*, const int32_t*, void*, void*, void*, int64_t, int, int, int, float, hipStream_t) { return note("rope"); }
hipError_t launch_swiglu(const void*, void*, int64_t, int, hipStream_t) { return note("swiglu"); }
hipError_t launch_residual_add(float*, const void*, int64_t, hipStream_t) { return note("add"); }
hipError_t launch_stream_probe(const void*, int64_t, int, int, float*, hipStream_t) { return note("probe"); }
hipError_t launch_mfma_probe(float*, int, int, hipStream_t) { return note("probe"); }
}  // namespace fedattn

using namespace fedattn;

static int failures = 0;
#define EXPECT(what)                                                                     \
  do {                                                                                   \
    if (!(what)) {                                                                       \
      std::printf("line %d: %s (%s)\n", __LINE__, #what, fedattn_last_error());          \
      ++failures;                                                                        \
    }                                                                                    \
  } while (0)

static std::string kernels() {
  std::string s;
  for (const Launch& l : launched) s += (s.empty() ? "" : " ") + l.kernel;
  return s;
}

// Sync block on matrices that lie apart, `out` over them or beside them: read where they are only if nobody can write them meanwhile.
static void output_over_matrices() {
  const fedattn_params p = {3, 8, 2, 128, 1, 1, FEDATTN_BF16, 0.f};
  const std::vector<int32_t> seg = {0, 130, 130, 300};
  const size_t row = 2 * 128 * 2, q_bytes = 300 * 8 * 128 * 2;
  char* base = reinterpret_cast<char*>(0x7000000000ull);
  const char *k[3] = {base, nullptr, base + (1 << 20)}, *v[3] = {base + (2 << 20), nullptr, base + (3 << 20)};
  const void *kp[3] = {k[0], k[1], k[2]}, *vp[3] = {v[0], v[1], v[2]};
  void* ws = base + (64 << 20);
  struct { const char* m; size_t rows; } const mats[] = {{k[0], 130}, {k[2], 170}, {v[0], 130}, {v[2], 170}};
  const uint8_t* const keeps[] = {nullptr, reinterpret_cast<const uint8_t*>(base + (8 << 20))};
  for (const uint8_t* keep : keeps) {
    const int chunk = keep ? 16 : 0;
    const size_t need = fedattn_workspace_bytes(&p, FEDATTN_OP_PREFILL_SYNC_LOCAL_KV, 300, chunk);
    const auto call = [&](const char* out) {
      launched.clear();
      EXPECT(fedattn_prefill_sync_local_kv(&p, base + (16 << 20), kp, vp, const_cast<char*>(out), seg.data(), keep, chunk, ws, need, nullptr) == FEDATTN_OK);
      return kernels();
    };
    const std::string where_they_are = keep ? "pack mfma" : "mfma", copied = keep ? "aggregate pack mfma" : "aggregate mfma";
    EXPECT(call(base + (32 << 20)) == where_they_are && launched.back().prefill.apart == 1);
    for (const auto& m : mats) {
      EXPECT(call(m.m) == copied && launched.back().prefill.apart == 0);
      EXPECT(call(m.m + m.rows * row - 16) == copied && launched.back().prefill.apart == 0);
      EXPECT(call(m.m + m.rows * row) == (m.m + m.rows * row + q_bytes <= m.m + (1 << 20) ? where_they_are : copied));
    }
    EXPECT(call(k[0] - q_bytes) == where_they_are);
    EXPECT(call(k[0] - q_bytes + 16) == copied);
  }
}

// Decoding: which blocks share a launch, and which launches set their chunk counters up (a round trip for every workgroup): the
// first one of a kind, as every launch leaves its counters at zero and no later one has more blocks.
static void decode_launches() {
  char* base = reinterpret_cast<char*>(0x7000000000ull);
  for (int rows : {1512, 100}) {   // workspace with room for one block of a kind, and for all
    const fedattn_params p = {1, 8, 8, 128, 2, 1, FEDATTN_BF16, 0.f};
    const std::vector<int32_t> seg = {0, rows}, lens = {rows};
    const int64_t q = 8 * 128, cache = (int64_t)rows * 8 * 128;
    const size_t need = fedattn_workspace_bytes(&p, FEDATTN_OP_DECODE, rows, 0);
    for (int out_at : {16, 2}) {   // output apart from the queries; over those of the next blocks
      launched.clear();
      EXPECT(fedattn_decode_blocks(&p, 0, 6, base, base + (32 << 20), base + (96 << 20), base + (out_at == 16 ? 16 << 20 : q * 2), q, cache, seg.data(),
                                   lens.data(), nullptr, -1, base + (200 << 20), need, nullptr) == FEDATTN_OK);
      bool seen[2] = {false, false};
      int blocks[2] = {0, 0};
      for (const Launch& l : launched) {
        EXPECT((l.decode.ticket != 0) == !seen[l.decode.is_sync]);
        EXPECT(l.blocks >= 1 && (out_at == 16 || l.blocks == 1));
        seen[l.decode.is_sync] = true;
        blocks[l.decode.is_sync] += l.blocks;
      }
      EXPECT(blocks[0] == 3 && blocks[1] == 3);
      EXPECT(launched.size() == (out_at == 16 && rows == 100 ? 2u : 6u));
    }
  }
}

// Random decode calls: every launch's partials and chunk counters lie inside the workspace, and those of the blocks that share it apart.
static void decode_workspaces() {
  std::srand(7);
  char* base = reinterpret_cast<char*>(0x7000000000ull);
  char* ws = base + (1ull << 40);
  for (int t = 0; t < 4000; ++t) {
    static const int kv[] = {1, 2, 3, 8, 16}, groups[] = {1, 2, 3, 4, 8}, dims[] = {8, 64, 72, 96, 128, 200, 256};
    const int N = 1 + std::rand() % (std::rand() % 2 ? 8 : 128), Hkv = kv[std::rand() % 5], Hq = Hkv * groups[std::rand() % 5], D = dims[std::rand() % 7];
    const int most = 1 << (std::rand() % 13), M = 1 + std::rand() % 40;
    const fedattn_params p = {N, Hq, Hkv, D, 1 + std::rand() % 4, 1, std::rand() % 2 ? FEDATTN_BF16 : FEDATTN_F32, 0.f};
    std::vector<int32_t> seg = {0}, lens, remote;
    for (int n = 0; n < N; ++n) {
      lens.push_back(std::rand() % (most + 1));
      remote.push_back(std::rand() % (lens[n] + 3));
      seg.push_back(seg[n] + lens[n] + 2);
    }
    const size_t need = fedattn_workspace_bytes(&p, FEDATTN_OP_DECODE, seg[N], 0), extra = std::rand() % 3 ? 0 : (size_t)(std::rand() % 5) * need + std::rand() % 4096;
    const size_t bytes = need + extra / 16 * 16;
    const int64_t q = (int64_t)N * Hq * D, cache = (int64_t)seg[N] * Hkv * D;
    launched.clear();
    const auto call = std::rand() % 2 ? fedattn_decode_blocks : fedattn_decode_blocks_fused;
    EXPECT(call(&p, 0, M, base, base + (1ull << 36), base + (2ull << 36), base + (3ull << 36), q, cache, seg.data(), lens.data(),
                std::rand() % 2 ? remote.data() : nullptr, -1, ws, bytes, nullptr) == FEDATTN_OK);
    for (const Launch& l : launched) {
      const DecodeArgs& a = l.decode;
      if (a.part_o == nullptr) continue;   // one wavefront per participant and head: no partials
      const size_t rows = (size_t)a.n_g * a.n_chunks * a.n_cols;
      const size_t o = (size_t)(reinterpret_cast<char*>(a.part_o) - ws), ml = (size_t)(reinterpret_cast<char*>(a.part_ml) - ws);
      const size_t cnt = (size_t)(reinterpret_cast<char*>(a.counters) - ws), last = (size_t)(l.blocks - 1) * (size_t)a.slice_bytes;
      const size_t end = cnt + (size_t)Hkv * N * sizeof(uint64_t);
      EXPECT(o + rows * D * 4 <= ml && ml + rows * 8 <= cnt);
      EXPECT(l.blocks >= 1 && l.blocks <= kMaxFusedBlocks && last + end <= bytes);
      EXPECT(l.blocks == 1 || end <= (size_t)a.slice_bytes);
      EXPECT(ml % 8 == 0 && cnt % 8 == 0 && (l.blocks == 1 || a.slice_bytes % 16 == 0));
    }
    if (failures) return;
  }
}

// The list of query tiles names, for every workgroup, the tile that the search of the segment tables finds.
static void listed_tiles() {
  std::srand(8);
  for (int t = 0; t < 4000; ++t) {
    PrefillArgs a;
    std::memset(static_cast<void*>(&a), 0, sizeof(a));
    const int N = a.seg.n = 1 + std::rand() % (std::rand() % 2 ? 6 : kMaxP), most = 1 << (std::rand() % 14), rows = 16 << (std::rand() % 4);
    const bool sync = std::rand() % 2 != 0;
    a.short_half_ascending = std::rand() % 2;
    for (int n = 0; n < N; ++n) a.seg.seg_off[n + 1] = a.seg.seg_off[n] + (std::rand() % 5 == 0 ? 0 : std::rand() % (most + 1));
    lay_out_query_tiles(a, rows);
    order_segments_by_length(a);   // pair_cum: tiles in that order
    list_heavy_first(a, sync);
    const int T = a.n_q_tiles, half = (T + 1) / 2;
    EXPECT(a.n_listed == (T <= kMaxListedTiles ? T : 0));
    for (int p = 0; p < a.n_listed; ++p) {
      const int rank = a.short_half_ascending && p >= half ? T - 1 - (p - half) : p;
      int n = 0, tile = T - 1 - rank;
      if (!sync) {
        int s = 0;
        while (rank >= a.seg.pair_cum[s + 1]) ++s;
        tile = a.seg.tile_cum[a.seg_order[s] + 1] - 1 - (rank - a.seg.pair_cum[s]);
      }
      while (tile >= a.seg.tile_cum[n + 1]) ++n;
      const uint32_t e = a.tile_list[p >> 1] >> (16 * (p & 1)) & 0xffffu;
      EXPECT((int)(e & 127) == n && (int)(e >> 7) == tile - a.seg.tile_cum[n]);
    }
    if (failures) return;
  }
}

int main() {
  listed_tiles();
  decode_launches();
  decode_workspaces();
  output_over_matrices();
  std::puts(failures ? "wrong" : "clean");
  return failures != 0;
}
