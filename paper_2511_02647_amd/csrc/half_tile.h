// The two 32-row halves in which a wavefront of prefill_split.hip walks a listed (kept) 64-row tile.
// Plain arithmetic without device code, so that a host program can check its bounds.
#pragma once

namespace fedattn {

constexpr int kSplitRows = 32;   // keys of a wavefront's tile

struct HalfTile {
  int kv0;        // first row that the half stands for
  int len;        // its valid rows; 0 or less: none
  int load0;      // first row to load
  int load_len;   // rows that may be loaded from there, at least one
};

// Half 0 or 1 of the tile of rows [row0, row0 + rows), 1 <= rows <= 64.  A tile is a piece of one
// participant's K and V (or of its packed rows): what follows its last row belongs to somebody else, was never
// written or lies past the end, so a half without rows loads the tile's first row and is masked out.
constexpr HalfTile half_of_tile(int row0, int rows, int half) {
  const int at = half * kSplitRows;
  const int left = rows - at;
  const int len = left < kSplitRows ? left : kSplitRows;
  return len > 0 ? HalfTile{row0 + at, len, row0 + at, len} : HalfTile{row0 + at, len, row0, 1};
}

}  // namespace fedattn
