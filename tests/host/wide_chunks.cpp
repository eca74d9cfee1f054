// The chunk length of a wide sync block against the plain form of the same search, which evaluates every step in full.
#include <cstdio>
#include <cstdlib>

#include "launch_choice.h"

static int plain(const int32_t* rows, int N, int finest, int Hkv, int D, int cols, int cus) {
  const double tile_us = D == 128 ? 0.9 : D == 64 ? 0.5 : 1.05;
  const double wgs = (double)Hkv * ((cols + 63) / 64);
  double total = 0, best_us = 1e30;
  int longest = 1, best = finest;
  for (int n = 0; n < N; ++n) {
    total += rows[n];
    longest = rows[n] > longest ? rows[n] : longest;
  }
  for (int i = 0; i < 33; ++i) {
    long cr = i < 25 ? finest + (long)(longest - finest) * i / 24 : ((long)longest + (i - 25)) / (i - 24);
    cr = (cr + 63) / 64 * 64;
    if (cr < finest) continue;
    long chunks = 0;
    for (int n = 0; n < N; ++n) chunks += (long)((double)(rows[n] + (cr - 1)) * (1.0 / (double)cr));
    const double tiles = (double)(((cr < longest ? cr : longest) + 63) / 64);
    const double walk = (double)(((long)((double)chunks * wgs) + cus - 1) / cus) * (5 + tiles * tile_us);
    const double stream = 5 + total * Hkv * D * 4 / 6.5e6;
    const double us = (walk > stream ? walk : stream) + (double)chunks * ((double)Hkv * cols * (4 * D + 8) / 2.5e6) + (chunks > 64 ? 2 : 0);
    if (us < best_us) {
      best_us = us;
      best = (int)cr;
    }
  }
  return best;
}

int main() {
  std::srand(1);
  int bad = 0;
  for (int t = 0; t < 20000; ++t) {
    static const int heads[] = {1, 2, 3, 4, 8, 16}, dims[] = {64, 96, 128, 256};
    const int N = 1 + std::rand() % 128, most = 1 << (4 + std::rand() % 12), cus = std::rand() % 2 ? 256 : 304;
    const int Hkv = heads[std::rand() % 6], D = dims[std::rand() % 4], cols = 17 + std::rand() % 512;
    int32_t rows[128];
    long total = 0;
    for (int n = 0; n < N; ++n) total += rows[n] = std::rand() % 4 == 0 ? 0 : std::rand() % most;
    const int target = cus / Hkv;
    int finest = (int)((total + target - 1) / target + 63) / 64 * 64;
    if (finest < 64) finest = 64;
    const int got = fedattn::wide_chunk_rows(rows, N, finest, Hkv, D, cols, cus);
    if (got != plain(rows, N, finest, Hkv, D, cols, cus) || got % 64 != 0 || got < finest) {
      std::printf("case %d: %d rows, plain search %d, finest %d\n", t, got, plain(rows, N, finest, Hkv, D, cols, cus), finest);
      ++bad;
    }
  }
  std::puts(bad ? "wrong" : "clean");
  return bad != 0;
}
