// Which piece of which cache segment a decode workgroup streams: shared by the split-KV kernels.
#pragma once

#include "common.h"

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

}  // namespace fedattn
