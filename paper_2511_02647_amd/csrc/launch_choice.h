// The rules by which a launcher chooses among its kernels and splits, in plain C++ without device code, so that a host
// program can say which launch a shape takes (the GPU tests name their layouts by it).
#pragma once

#include <math.h>
#include <stdint.h>

namespace fedattn {

constexpr int kKvTile = 64;            // KV rows per tile; also the keep-list tile
constexpr int kWaveRows = 32;          // query rows per wavefront in the bf16 prefill kernels
constexpr int kMaxListedTiles = 512;   // query tiles of a launch whose workgroups find theirs in a list
constexpr int kCombineAtOnce = 64;     // chunks up to which the decode combine kernel makes one round trip
constexpr int kMaxSegments = 128;      // participants at most

// ---- which of the launches a block takes ------------------------------------------------------
// kFour: 4-wavefront workgroups, one query tile each, several per CU; kFourOrdered: the same, causal and
// all resident at once, in an order that the host lays out.  kEight: 8-wavefront workgroups whose two
// groups share out the KV tiles of one query tile; kEightPairs: of a heavy tile and then its light mirror
// image.  kSplit: one head's 32 rows per workgroup, keys shared out among its 8 wavefronts (prefill_split.hip).  From left to right a launch has more and shorter walks for the same work and pays
// more for each: the right one depends on how far the block fills the chip, so their times are estimated.
enum PrefillLaunch { kFour, kFourOrdered, kEight, kEightPairs, kSplit };

// Measured on one MI355X, microseconds: an iteration of one workgroup alone on its CU and as its share
// of a full CU, start and end of a walk when the launch waits for it and when the CU's next workgroup
// does; workgroups resident per CU.  An iteration is 64 keys (kFour), 128 (kEight) or 256 (kSplit).
// (Bidirectional blocks of 1024, 2048 and 4096 tokens with 1 to 8 heads.)
struct Pace { float alone, full, ends, turn; int resident; };
struct Paces { Pace four, eight, split; };
inline const Paces& paces(int D) {
  static const Paces d64 = {{.87f, .53f, 3.2f, 2.0f, 3}, {1.11f, 1.26f, 3.3f, 3.3f, 1}, {.70f, .74f, 2.5f, 4.5f, 2}};
  static const Paces d128 = {{1.15f, .89f, 3.2f, 2.2f, 2}, {1.73f, 2.04f, 3.5f, 3.5f, 1}, {1.19f, 1.50f, 2.7f, 4.3f, 1}};
  // weights at full precision (other head dimensions), by padded size
  static const Paces e64 = {{1.20f, .98f, 3.2f, 1.8f, 3}, {1.95f, 2.30f, 3.3f, 3.3f, 1}, {1.05f, 1.00f, 2.5f, 4.5f, 2}};
  static const Paces e96 = {{1.53f, 1.36f, 3.2f, 2.0f, 2}, {2.41f, 3.00f, 3.5f, 3.5f, 1}, {1.38f, 1.80f, 2.7f, 3.0f, 1}};
  static const Paces e128 = {{1.89f, 1.75f, 3.2f, 2.0f, 2}, {2.82f, 3.64f, 3.5f, 3.5f, 1}, {1.64f, 2.35f, 2.8f, 3.5f, 1}};
  return D == 64 ? d64 : D == 128 ? d128 : D <= 64 ? e64 : D <= 96 ? e96 : e128;
}

struct PrefillShape {
  const int32_t* seg_off;   // [n + 1]
  int n;
  int Hq, Hkv, D;
  bool causal, keep;        // keep: a keep-list
  int heads_per_wg, q_tile_rows;
  int n_cus;
};

// Query tiles of `rows` rows (none crosses a segment's end), and pairs of them inside each segment.
struct QueryTiles { int64_t tiles, pairs; };
inline QueryTiles count_query_tiles(const int32_t* seg_off, int n_seg, int rows) {
  QueryTiles q = {0, 0};
  for (int n = 0; n < n_seg; ++n) {
    const int64_t t = ((int64_t)seg_off[n + 1] - seg_off[n] + rows - 1) / rows;
    q.tiles += t;
    q.pairs += (t + 1) / 2;
  }
  return q;
}

// Workgroups of a launch, iterations of its longest walk and of all walks together.
struct Walks { double wgs, longest, total; };
inline Walks count_walks(const PrefillShape& a, bool is_sync, int rows, int keys, int wgs_per_tile) {
  Walks w = {0, 0, 0};
  const double total = a.seg_off[a.n];
  for (int n = 0; n < a.n; ++n) {
    const double off = a.seg_off[n], len = a.seg_off[n + 1] - off;
    if (len == 0) continue;
    const double tiles = ceil(len / rows);
    double most, mean;   // keys that the segment's last rows and its rows on average see
    if (a.causal) {
      // Remote rows under a keep-list: their number is known to the device only, half are taken to be kept.
      // Every launch forced on 8 layouts (4 to 16 participants of 100..2000 tokens, 2 to 32 heads of 64, 96 and 128)
      // at shares of 0.1, 0.25, 0.5 and 1: kFour, kEight and kSplit were taken where they are the fastest, or within
      // 4 % of it at a quarter and a half, 11 % at 0.1, 13 % at 1.
      const double before = is_sync ? (a.keep ? off / 2 : off) : 0;
      most = before + len;
      mean = before + (len + fmin(rows, len)) / 2;
    } else {
      most = mean = is_sync ? (a.keep ? (total + len) / 2 : total) : len;
    }
    w.wgs += tiles;
    w.longest = fmax(w.longest, ceil(most / keys));
    w.total += tiles * (a.causal ? fmax(1.0, mean / keys + 0.5) : ceil(mean / keys));
  }
  w.wgs *= wgs_per_tile;
  w.total *= wgs_per_tile;
  return w;
}

// Whether the softmax scale is folded into the Q operand of the bf16 kernels: up to the usual 1/sqrt(D), as its rounding error grows with it.
inline bool folds_scale(float scale, int D) { return (double)scale * (double)scale * D <= 1.0 + 1e-6; }

// Microseconds of the launch without what every launch costs: the longer of its longest walk, which
// shares its CU with average ones, and the work of a CU (bidirectional blocks have walks of one length
// that fill no gaps: whole workgroups count).
inline double estimate(const Pace& p, const Walks& w, bool causal, int cus) {
  const double on_cu = ceil(w.wgs / cus);   // workgroups that the fullest CU gets
  const double together = fmin(on_cu, p.resident);
  const double mean = w.total / w.wgs;
  // with some, not all places of a CU taken, a workgroup's share is a little worse than full
  const double shared = together > 1 ? fmax(p.alone, together * p.full * (together < p.resident ? 1.15 : 1.0))
                                     : w.wgs > 0.45 * cus ? fmax(p.alone, p.full) : p.alone;
  const double path = p.ends + (w.longest - mean) * p.alone + mean * shared;
  const double work = causal ? p.turn * w.wgs / (p.resident * cus) + w.total * p.full / cus
                             : on_cu * (p.turn / p.resident + mean * p.full);
  return fmax(path, work);
}

inline PrefillLaunch choose_prefill_launch(const PrefillShape& a, bool is_sync, bool with_pairs = true) {
  const bool causal = a.causal;
  const int per_tile = a.Hkv * (a.Hq / a.Hkv / a.heads_per_wg);
  const QueryTiles q = count_query_tiles(a.seg_off, a.n, a.q_tile_rows);
  const PrefillLaunch four = causal && q.tiles <= kMaxListedTiles && q.tiles * per_tile <= 2 * (int64_t)a.n_cus ? kFourOrdered : kFour;
  if (a.D > 128) return four;   // the others' tiles do not fit LDS
  const Paces& p = paces(a.D);
  const Walks four_walks = count_walks(a, is_sync, a.q_tile_rows, kKvTile, per_tile);
  Walks eight = count_walks(a, is_sync, a.q_tile_rows, 2 * kKvTile, per_tile);
  const Walks split = count_walks(a, is_sync, kWaveRows, 256, a.Hq);
  PrefillLaunch best = four;
  double t = estimate(p.four, four_walks, causal, a.n_cus);
  const auto consider = [&](PrefillLaunch plan, double x) {
    if (x < t) {
      t = x;
      best = plan;
    }
  };
  consider(kEight, estimate(p.eight, eight, causal, a.n_cus));
  const double pairs = (double)(q.pairs * per_tile);
  if (causal && with_pairs) {   // half as many workgroups, each with a heavy and a light walk
    eight.longest = is_sync ? 2 * eight.total / eight.wgs : eight.longest + 1;
    eight.wgs = pairs;
    Pace pp = p.eight;
    pp.ends *= 1.95f;
    consider(kEightPairs, estimate(pp, eight, true, a.n_cus));
  }
  consider(kSplit, estimate(p.split, split, causal, a.n_cus));
  return best;
}

// The launch that is taken: the estimate's choice, but pairs in one round of workgroups only.  Pairs are of about one size and alone on
// their CUs, so a second round takes as long as the first, be it for 16 of 272 workgroups, where the estimate spreads its work over the chip.
// Pairs and the next best launch, us: sync blocks of 4 x 516 tokens, 32/8 heads of 128 (272 pairs) 78.4 and 50.3, 5 x 516 (344)
// 94.2 and 61.8, 8 x 454..823, 16/4 heads of 128 (320) 158 and 117, 3 x 3233, 12/4 heads of 64 (306) 195 and 169, half kept, 8 x
// 454..823, 16/8 heads of 64 (320) 84 and 63; local blocks of 2 x 2239, 16/2 heads of 128 (280) 84 and 55, 4 x 774..1290, 24/8
// heads of 64 (432) 36 and 26, 2 x 1004..3348, 16/2 heads of 96 (304) 120 and 103; the one of 11 where pairs were faster: 6 x 2373..3956,
// 6/2 heads of 64 (444) 76.3 and 79.2.  In one round: 4 x 500, 32/8 heads of 128, a tenth kept 26.2 and 29.1.
inline PrefillLaunch launch_to_take(const PrefillShape& a, bool is_sync) {
  const PrefillLaunch plan = choose_prefill_launch(a, is_sync);
  if (plan != kEightPairs) return plan;
  const QueryTiles q = count_query_tiles(a.seg_off, a.n, a.q_tile_rows);
  const int64_t wgs = (is_sync ? (q.tiles + 1) / 2 : q.pairs) * a.Hkv * (a.Hq / a.Hkv / a.heads_per_wg);
  return wgs <= a.n_cus ? plan : choose_prefill_launch(a, is_sync, false);
}

// Dense sync blocks whose participants' matrices lie apart: whether they are read where they are or aggregated first, which costs a
// launch and a copy.  Read where they are, a tile that crosses a segment's end is loaded by a longer way (every lane picks its row's
// matrix), and the 4- and 8-wavefront kernels take 1 to 4 % longer even without.  Aggregated and read apart, us:
//  - split launch, unless a CU's workgroups load many such tiles (one 32-row tile in total / (32 n) is) or, at head dimension 128, several ends
//    lie in a tile: 20 x 1..28 tokens, 8/2 heads of 64 14.7 and 12.3, 2 x 109, 1/1 heads of 64 8.6 and 5.7, 13 x 83..277, 9/3 heads
//    of 128 36.9 and 32.6, bidirectional 6 x 1..900, 16/16 heads of 64 (3.6 such tiles a CU) 74 and 67; 18 x 1..46, 16/4 heads of 128 15.6 and 17.1;
//  - others, unless segments are short or the launch is long or loads many such tiles (of 64 rows): bidirectional 6 x 300..900, 16/16 heads of 128
//    (10.8 a CU) 119 and 113; 25 x 209, 3/1 heads of 128 (14.7) 81.7 and 88.0, 16 x 20..60, 32/8 heads of 128 20.3 and 23.9, 8 x
//    500..1500, 32/8 heads of 128 431 and 436, 31 x 200..600, 16/4 580 and 605.
// Both limits of tiles that cross an end are on the safe side.  Each form forced on 192 layouts around them (2 to 25 participants, 4 to 32
// heads): split launch, from 0.6 to 1 times the limit read apart is 1.00 to 1.29 times faster in 23 of 24 (0.99), from there to 2.5 times it 0.97 to
// 1.32 (median 1.05; 19 x 431..458, 4/4 heads of 64, 5.2: 65.9 and 57.7); others, below the limit 0.97 to 1.17, beyond it 0.93 to 1.15 (median 1.02).
inline bool read_apart(const PrefillShape& a) {
  const double total = a.seg_off[a.n];
  if (a.D != 64 && total < 32.0 * a.n) return false;   // whichever launch it is; such calls are bound by the host (27 x 1..19 tokens: 18.9 and 18.6 us)
  if (launch_to_take(a, true) == kSplit)
    return count_walks(a, true, kWaveRows, 256, a.Hq).total * kWaveRows * a.n <= 4.5 * a.n_cus * total;
  const double tiles = count_walks(a, true, a.q_tile_rows, kKvTile, a.Hkv * (a.Hq / a.Hkv / a.heads_per_wg)).total / a.n_cus;
  return total >= 128.0 * a.n && tiles <= 150 && tiles * kKvTile * a.n <= 12 * total;
}

// ---- fp32 prefill ----------------------------------------------------------------------------
// Query heads of a KV group that a workgroup of 4 wavefronts takes.
inline int heads_in_common(int group) { return group % 4 == 0 ? 4 : (group % 2 == 0 ? 2 : 1); }
// Whether the wavefronts of a workgroup take different heads, each K and V tile staged once for all of them, rather than the keys of
// one head's 16 query rows: from 6 workgroups per CU on.  Keys shared out and heads shared, us, 32/8 heads of 128: 8 x 1000 tokens (8 per CU)
// sync 4257 and 3891 (137 TFLOP/s), local 664 and 661; 6 x 1000 (6) 2416 and 2281, local 497 and 502; of 64: 1199 and 1180, local 232 and 275.
// With fewer it depends on how evenly the workgroups fill the rounds: 4 x 1000 (4), heads of 64 543 and 572, bidirectional 1065
// and 1027; 4 x 700 (2.8), of 128 557 and 548, local 176 and 180; 6 x 1000, 8/2 heads of 128 (1.5) 621 and 882; 1000 tokens, 8/2 heads 27 and 133.
inline bool f32_heads_shared(const int32_t* seg_off, int n_seg, int Hq, int Hkv, int D, int n_blocks, int n_cus) {
  const int nq = D > 128 ? 1 : 2;   // 16-row sub-tiles per wavefront
  const int group = Hq / Hkv, common = heads_in_common(group);
  return count_query_tiles(seg_off, n_seg, 16 * nq * (4 / common)).tiles * Hkv * (group / common) * n_blocks >= 6 * (int64_t)n_cus;
}

// ---- decode ----------------------------------------------------------------------------------
// Sync blocks of more than 16 query columns (bf16): a chunk costs a workgroup per KV head and 64 columns,
// and partials of all columns that are written and read back, so the split that gives every CU one
// workgroup per KV head is too fine when the columns or the segments are many.  Microseconds, measured on
// one MI355X (8 to 32 participants with 64 to 4000 rows each, 24 to 256 columns): a workgroup's start and
// end 5, a 64-row tile 0.9 (head dimension 128), 0.5 (64), 1.05 (weights at full precision); workgroups
// beyond one per CU wait; the caches stream at 6.5 MB/us, partials pass at 2.5; the combine kernel takes 2
// more beyond its one-round-trip case.  Sync block before and after, us:
//   32 x 2000 rows, 8/1 heads 47.6 -> 26.0       32 x 300..800 rows, 16/4 heads 34.4 -> 21.7
//   24 x 1000..2000 rows, 32/4 heads 62.5 -> 52     16 x 200..500 rows, 32/8 heads 21.6 -> 17.1
//   20 x 500..1500 rows, 8/2 heads of 64 17.1 -> 14.1   8 x 300..1000 rows, 16/2 heads 14.9 -> 13.0
// The estimate itself takes 0.3 us at 16 participants and 1.6 at 128 (0.8 and 4.7 when every step was evaluated in full).
inline int wide_chunk_rows(const int32_t* rows, int N, int finest, int Hkv, int D, int cols, int cus) {
  const double tile_us = D == 128 ? 0.9 : D == 64 ? 0.5 : 1.05;
  const int64_t wgs_per_chunk = (int64_t)Hkv * ((cols + 63) / 64);
  int64_t total = 0;
  int longest = 1;
  double rows_d[kMaxSegments];
  for (int n = 0; n < N; ++n) {
    total += rows[n];
    longest = rows[n] > longest ? rows[n] : longest;
    rows_d[n] = rows[n];
  }
  const double stream_us = (double)total * Hkv * D * 4 / 6.5e6;
  const double partials_us = (double)Hkv * cols * (4 * D + 8) / 2.5e6;   // per chunk
  int best = finest;
  double best_us = 1e30;
  int64_t last = 0;
  // from the finest split to one chunk per segment in 24 steps, and the longest segment in up to 8 equal parts
  for (int i = 0; i < 33; ++i) {
    int64_t cr = i < 25 ? finest + (int64_t)(longest - finest) * i / 24 : ((int64_t)longest + (i - 25)) / (i - 24);
    cr = (cr + kKvTile - 1) / kKvTile * kKvTile;
    if (cr < finest || cr == last) continue;
    last = cr;
    const double per = 1.0 / (double)cr;
    const int64_t tiles = ((cr < longest ? cr : longest) + kKvTile - 1) / kKvTile;
    const auto us_of = [&](int64_t chunks) {
      const int64_t rounds = (chunks * wgs_per_chunk + cus - 1) / cus;
      const double walk_us = (double)rounds * (5 + (double)tiles * tile_us);
      return (walk_us > 5 + stream_us ? walk_us : 5 + stream_us) + (double)chunks * partials_us + (chunks > kCombineAtOnce ? 2 : 0);
    };
    if (us_of((int64_t)((double)total * per)) >= best_us) continue;   // with no segment rounded up
    int chunks = 0;   // an estimate's worth: rounding may be off by one where rows divide evenly
    for (int n = 0; n < N; ++n) chunks += (int)((rows_d[n] + (double)(cr - 1)) * per);
    const double us = us_of(chunks);
    if (us < best_us) {
      best_us = us;
      best = (int)cr;
    }
  }
  return best;
}

}  // namespace fedattn
