// Which workgroup does what: integer arithmetic that launches and kernels share, without anything of a GPU in it, so that a plain
// C++ program can enumerate it (tests/test_launch_plan.py).
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace moe {

// A launch has at most 2^32 - 1 threads.
constexpr bool fits_one_launch(size_t blocks, int threads) { return blocks <= 0xFFFFFFFFu / static_cast<unsigned>(threads); }

constexpr int kXcds = 8;                               // workgroup b runs on XCD b % 8

// workgroup id -> virtual tile id such that consecutive virtual ids share an XCD; -1: none
constexpr int xcd_remap(int b, int total) {
  const int per = (total + kXcds - 1) / kXcds;
  const int v = (b % kXcds) * per + b / kXcds;
  return (b / kXcds < per && v < total) ? v : -1;
}

// The row-grouped products' list of row tiles: the experts in order, the rows of each cut into tiles of bm rows (`scan`: inclusive scan of
// the experts' numbers of tiles).  Virtual tile v of a product with n_tiles_n column tiles is found through entry v / n_tiles_n.
//
// An expert of up to kGroup row tiles has its tiles in the order that keeps those of the same columns together: they share a weight
// panel, which comes from memory, and a stretch of the list that runs at one time ends between two panels, not between two row
// tiles that share them all.  Beyond, the columns of a row tile come first.  Read from memory at T = 8192, E = 128, k = 8, d = 2048, f = 768
// (512 rows per expert), columns first -> as it is: gate/up 2040 -> 1809 MB, down 718 -> 564, dX 1791 -> 1631, 8-bit gate/up 1034 -> 848.
// The time hardly follows.  Both sides of the line, whole steps in turn (two runs of one build differ by up to 0.4 %, with E = 16 by 1.6 %):
//   no groups -> 4:  E = 8, d = 4096, f = 3072, 900 rows per expert 1619 -> 1550 us; the layer above 2104 -> 2091, and at 900 to 1800 rows per
//                    expert equal; E = 16, d = 1024, f = 2048, 512 to 1800 rows 0.993-1.005; 8-bit forward at 900 rows 0.996
//   4 -> 8 and more: the layer above at 512 and 900 rows equal, at 1150, 1400 and 1800 (5 to 8 row tiles) 4142 -> 4090, 4954 -> 4913 and
//                    6254 -> 6228; E = 16 at 1400 rows 971 -> 964, else as far apart as its runs; 8-bit equal
// So the line is not too high; up to 8 row tiles it could be higher.
constexpr int kGroup = 4;
struct TileEntry {                                     // of a row tile: one scalar load finds everything
  int32_t expert, first, n;                            // its group: the list's row tiles first .. first + n - 1
  int32_t row0, row_end;                               // first row of the group; one past the expert's last
  int32_t unused[3];
};
// the expert of row tile t: the first whose inclusive scan exceeds t (the last one if none does)
constexpr int expert_of_row_tile(const int32_t* scan, int E, int t) {
  int lo = 0, hi = E - 1;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (scan[mid] > t) hi = mid; else lo = mid + 1;
  }
  return lo;
}
// its entry in a list that is cut off at `total` row tiles
constexpr TileEntry row_tile_entry(const int32_t* scan, int expert, int t, int total, int first_row, int row_end, int bm) {
  const int before = expert > 0 ? scan[expert - 1] : 0, tiles = (scan[expert] < total ? scan[expert] : total) - before;
  const bool grouped = tiles <= kGroup;
  return TileEntry{expert, grouped ? before : t, grouped ? tiles : 1, first_row + (grouped ? 0 : t - before) * bm, row_end, {0, 0, 0}};
}
struct TileAt { int e, row0, rows, n; };               // expert, first row, rows, column tile
template <class Scalar> constexpr TileAt tile_of_entry(const TileEntry& w, int v, int n_tiles_n, int bm, Scalar scalar) {
  const int l = v - w.first * n_tiles_n, n = scalar(l / w.n), row0 = w.row0 + (l - n * w.n) * bm, left = w.row_end - row0;
  return TileAt{w.expert, row0, scalar(bm < left ? bm : left), n};
}

// The weight gradients' tiles.  Work items come sorted by length, so consecutive stretches of the list differ in work: they are
// dealt to the XCDs in turn, in units of 1/g of an item's tiles -- whole items while there are at least 8 per XCD, otherwise g runs
// of the slow tile index, so that under skewed routing every XCD still gets several units of the few long items.  A unit's
// workgroups are consecutive on their XCD (shared panels).
// A workgroup takes every `grid`-th position of that order.  The last round goes the other way round: where it is not full, the
// tiles left over go to the workgroups whose tiles were the shortest (4096 skewed rows on 16 experts: 51 -> 48 and 64 -> 61 us;
// 16384 rows: dW_down 70 -> 66 us; full rounds: equal).
struct WgradWalk {
  int units, g, per_u;                                 // units in all; units and their tiles of an item
  int total, grid, last;                               // positions, workgroups (a multiple of 8), first position of the last round
};
struct WgradTile { int item, tile; bool exists; };     // tile: position among the item's tiles

// scalar: the kernel's way of saying that a value is the same in every lane
template <class Scalar> constexpr WgradWalk wgrad_walk(int n_items, int slow, int tiles, int grid, Scalar scalar) {
  int g = 1;
  while (g < slow && (n_items * g < 8 * kXcds || slow % g != 0)) ++g;
  g = scalar(g);
  const int per_u = scalar(tiles / g);                 // g divides slow, so it divides tiles
  const int total = scalar(((n_items * g + kXcds - 1) / kXcds) * per_u * kXcds);
  const int last = scalar(total > grid ? (total - 1) / grid * grid : total);
  return WgradWalk{n_items * g, g, per_u, total, grid, last};
}
// the tile at position `block` (any number >= 0: a workgroup's id plus multiples of the grid)
template <class Scalar> constexpr WgradTile wgrad_tile(const WgradWalk& w, int block, Scalar scalar) {
  const int turned = block < w.last ? block : 2 * w.last + w.grid - kXcds - block + 2 * (block % kXcds);
  const int at = block < w.last + w.grid ? turned : w.total;   // (there is no tile at `total` and beyond)
  const int q = at / kXcds, u = scalar(q / w.per_u);
  const int unit = u * kXcds + at % kXcds;
  if (unit >= w.units) return WgradTile{0, 0, false};
  const int item = scalar(unit / w.g);
  return WgradTile{item, (unit - item * w.g) * w.per_u + (q - u * w.per_u), true};
}

}  // namespace moe
