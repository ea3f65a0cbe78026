"""The integer arithmetic that says which workgroup does what (csrc/launch_plan.h), compiled by the host compiler and enumerated."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_02317_amd", "csrc")


def _run(tmp_path, body):
    """Compiles a program around the header and returns what it prints; it must end with status 0."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = str(tmp_path / "plan.cpp"), str(tmp_path / "plan")
    open(src, "w").write('#include <algorithm>\n#include <cstdio>\n#include <random>\n#include <vector>\n#include "launch_plan.h"\n'
                         "using namespace moe;\n" + body)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, src, "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stdout[-2000:]
    return res.stdout


def test_a_launch_has_fewer_than_2_to_the_32_threads(tmp_path):
    """The fp32 data and weight gradients share a launch: the workgroups of 480 million rows and of their combine weights, 32 and 256
    rows each, fit one by one but not together."""
    _run(tmp_path, """int main() {
      const size_t rows = 480000000, dx = rows / 32 + 1024, wgrad = 3 * 1024 + rows / 256;
      const bool ok = fits_one_launch(dx, 256) && fits_one_launch(wgrad, 256) && !fits_one_launch(dx + wgrad, 256) &&
                      fits_one_launch(16777215, 256) && !fits_one_launch(16777216, 256) && fits_one_launch(4194303, 1024) && !fits_one_launch(4194304, 1024);
      return ok ? 0 : 1;
    }""")


def test_every_tile_of_the_weight_gradients_is_taken_once(tmp_path):
    """Workgroups walk the tiles of sorted work items in rounds, the last one from its other end: over lists of any length, tiles per
    item and grids (fewer workgroups than positions, as many, and more), every (item, tile) comes up exactly once, in range, and a
    workgroup past its last tile finds none however far it goes on."""
    out = _run(tmp_path, """int main() {
      std::mt19937 r(1);
      auto same = [](int v) { return v; };
      long cases = 0;
      for (int n = 0; n < 6000; ++n) {
        const int few[] = {0, 1, 2, 3, 7, 8, 9, 16, 17, 33, 64, 65, 130, 1024}, grids[] = {8, 16, 64, 128, 256};
        const int items = few[r() % 14], slow = 1 + r() % (items > 100 ? 4 : 20), fast = 1 + r() % (items > 100 ? 3 : 12), tiles = slow * fast, grid = grids[r() % 5];
        const WgradWalk w = wgrad_walk(items, slow, tiles, grid, same);
        if (slow % w.g || w.per_u * w.g != tiles || w.total % kXcds) { printf("walk %d %d %d\\n", items, slow, fast); return 1; }
        std::vector<char> seen(static_cast<size_t>(items) * tiles, 0);
        size_t taken = 0;
        for (int b = 0; b < grid; ++b) {
          int block = b, past = 0;
          for (; past < 4; block += grid) {
            const WgradTile t = wgrad_tile(w, block, same);
            if (!t.exists) { ++past; continue; }
            // a workgroup ends at the first position without a tile, so no tile may follow one
            if (past || t.item < 0 || t.item >= items || t.tile < 0 || t.tile >= tiles || seen[static_cast<size_t>(t.item) * tiles + t.tile]++) {
              printf("items %d slow %d fast %d grid %d block %d\\n", items, slow, fast, grid, block);
              return 1;
            }
            ++taken;
          }
        }
        if (taken != seen.size()) { printf("missing: items %d slow %d fast %d grid %d\\n", items, slow, fast, grid); return 1; }
        ++cases;
      }
      printf("%ld\\n", cases);
      return 0;
    }""")
    assert out.strip() == "6000"


def test_every_tile_of_the_row_products_is_taken_once(tmp_path):
    """The same for the row products, whose consecutive tiles share an XCD."""
    _run(tmp_path, """int main() {
      for (int total = 0; total < 1200; ++total)
        for (int grid : {8, 64, 256, 512}) {
          std::vector<int> seen(total, 0);
          for (int b = 0; b < grid; ++b) {
            bool past = false;
            for (int block = b; block < total + 4 * grid; block += grid) {
              const int v = xcd_remap(block, total);
              if (v < 0) { past = true; continue; }
              if (past || v >= total || seen[v]++) { printf("total %d grid %d block %d\\n", total, grid, block); return 1; }
            }
          }
          if (std::count(seen.begin(), seen.end(), 1) != total) { printf("missing: total %d grid %d\\n", total, grid); return 1; }
        }
      return 0;
    }""")


def test_every_row_tile_of_the_list_is_found_with_every_column_once(tmp_path):
    """The list of row tiles and the tile at a position of it: over experts of any number of rows (none, one, a row to either side of
    one to six tiles, thousands), both heights of a tile, any number of column tiles and lists that are cut off, every (row tile, column
    tile) comes up exactly once with its expert and rows; experts of up to four row tiles have those of a column next to each
    other, larger ones the columns of a row tile."""
    out = _run(tmp_path, """int main() {
      std::mt19937 r(2);
      auto same = [](int v) { return v; };
      long grouped = 0, single = 0;
      for (int c = 0; c < 4000; ++c) {
        const int E = 1 + r() % 24, bm = r() % 2 ? 128 : 256, cols = 1 + r() % 13;
        std::vector<int> scan(E), first(E), end(E), expert, row0, rows;   // the list as it should be: expert and rows of every row tile
        int at = 0, tiles = 0;
        for (int e = 0; e < E; ++e) {
          const int kind = r() % 8;
          const int n = kind < 2 ? 0 : kind == 2 ? 1 : kind < 6 ? static_cast<int>(1 + r() % 6) * bm + static_cast<int>(r() % 3) - 1 : static_cast<int>(r() % 5000);
          first[e] = at; at += n; end[e] = at;
          for (int q = first[e]; q < end[e]; q += bm) { expert.push_back(e); row0.push_back(q); rows.push_back(std::min(bm, end[e] - q)); }
          scan[e] = tiles += (n + bm - 1) / bm;
        }
        const int total = r() % 4 ? tiles : static_cast<int>(r() % (tiles + 1));
        std::vector<TileEntry> list(total);
        for (int t = 0; t < total; ++t) {
          const int e = expert_of_row_tile(scan.data(), E, t);
          if (e != expert[t]) { printf("case %d: tile %d is expert %d's, not %d's\\n", c, t, expert[t], e); return 1; }
          list[t] = row_tile_entry(scan.data(), e, t, total, first[e], end[e], bm);
        }
        std::vector<int> seen(static_cast<size_t>(total) * cols, 0);
        int last_t = -1, last_n = -1;
        for (int v = 0; v < total * cols; ++v) {
          const TileAt a = tile_of_entry(list[v / cols], v, cols, bm, same);
          int t = 0;
          while (t < total && row0[t] != a.row0) ++t;
          if (t == total || a.e != expert[t] || a.rows != rows[t] || a.n < 0 || a.n >= cols || seen[static_cast<size_t>(t) * cols + a.n]++) {
            printf("case %d: position %d gives expert %d, rows %d + %d, column %d\\n", c, v, a.e, a.row0, a.rows, a.n);
            return 1;
          }
          const int before = a.e ? scan[a.e - 1] : 0, of_expert = std::min(scan[a.e], total) - before;
          if (last_t >= 0 && expert[last_t] == a.e) {     // the next tile of the same expert
            const bool together = of_expert <= 4;
            const int in_row = last_t + 1 - before, next_t = together ? before + in_row % of_expert : last_t + (last_n + 1 == cols),
                      next_n = together ? last_n + in_row / of_expert : (last_n + 1) % cols;
            if (t != next_t || a.n != next_n) { printf("case %d: order at %d\\n", c, v); return 1; }
            ++(together ? grouped : single);
          }
          last_t = t; last_n = a.n;
        }
        if (std::count(seen.begin(), seen.end(), 1) != static_cast<long>(seen.size())) { printf("case %d: missing\\n", c); return 1; }
      }
      return grouped > 100000 && single > 100000 ? 0 : 2;
    }""")
    assert out == ""
