// Bounds of the halves of a listed tile: every loaded row is one of the tile's, and the valid rows of
// the two halves are the tile's rows, each once.
#include <cstdio>
#include <initializer_list>

#include "half_tile.h"

int main() {
  int bad = 0;
  for (int row0 : {0, 1, 64, 1000003})
    for (int rows = 1; rows <= 64; ++rows) {
      int next = row0;   // first valid row that no half has covered yet
      for (int half = 0; half < 2; ++half) {
        const fedattn::HalfTile h = fedattn::half_of_tile(row0, rows, half);
        const bool loads = h.load_len >= 1 && h.load_len <= fedattn::kSplitRows && h.load0 >= row0 && h.load0 + h.load_len <= row0 + rows;
        const bool covers = h.len <= 0 || (h.kv0 == next && h.load0 == h.kv0 && h.load_len == h.len);
        if (!loads || !covers) {
          std::printf("tile [%d, +%d) half %d: rows [%d, +%d), loads [%d, +%d)\n", row0, rows, half, h.kv0, h.len, h.load0, h.load_len);
          ++bad;
        }
        if (h.len > 0) next = h.kv0 + h.len;
      }
      if (next != row0 + rows) {
        std::printf("tile [%d, +%d): covered up to %d\n", row0, rows, next);
        ++bad;
      }
    }
  std::puts(bad ? "wrong" : "clean");
  return bad != 0;
}
