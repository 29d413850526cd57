// Host check of how blocks are dealt to the XCDs (tests/test_xcd_map.py compiles and runs it; no GPU).
#include <cstdio>
#include <vector>

#include "spa2_device.h"

using namespace spa2;

static int deal(bool rows) {
  const int short_head = rows ? SHORT_ROWS : SHORT_COLUMNS;
  int bad = 0;
  for (int heads : {1, 2, 5, 9, 40}) {
    for (int blocks = 1; blocks <= 300; ++blocks) {
      const int chunk = (blocks + 7) / 8, wgs = xcd_map_wgs(heads, blocks, chunk, short_head);
      std::vector<int> seen((size_t)heads * blocks, 0);
      int dealt = 0, dead = 0, least = 1 << 30, most = 0;
      for (int xcd = 0; xcd < 8; ++xcd) {          // as a queue walks them: number s of an XCD
        int live = 0;
        for (int s = 0; s < xcd_map_share(wgs, xcd); ++s, ++dealt) {
          const HeadBlock hb = rows ? xcd_map_rows(8 * s + xcd, blocks, chunk) : xcd_map(8 * s + xcd, blocks, chunk, short_head);
          if (!hb.valid) { ++dead; continue; }
          ++live;
          if (hb.bh < 0 || hb.bh >= heads || hb.blk < 0 || hb.blk >= blocks) { ++bad; continue; }
          ++seen[(size_t)hb.bh * blocks + hb.blk];
        }
        least = live < least ? live : least;
        most = live > most ? live : most;
      }
      bool once = dealt == wgs;
      for (int n : seen) once = once && n == 1;
      // short heads: no number without a block, every XCD as many blocks as the others
      const bool even = blocks > short_head || (dead == 0 && most - least <= 1);
      if (!once || !even || dead > 7 * heads) {
        std::printf("%s: %d heads of %d blocks: once %d, dead %d, %d to %d an XCD\n", rows ? "rows" : "columns", heads, blocks, once, dead, least, most);
        ++bad;
      }
    }
  }
  return bad;
}

// Rows in stretches (stretch_row), columns in stretches, an XCD its own or all in turn: every one once, each XCD an eighth of them,
// rows one head after the other but for the rotation inside groups of four.
static int stretches() {
  int bad = 0;
  for (int heads : {1, 2, 5, 9, 40}) {
    for (int blocks = 1; blocks <= 300; ++blocks) {
      const int units = heads * blocks, wgs = stretch_wgs(units);
      std::vector<int> row((size_t)units, 0), own((size_t)units, 0), turn((size_t)units, 0);
      int live[8] = {0}, in_turn[8] = {0}, off = 0;
      for (int wg = 0; wg < wgs; ++wg) {
        const int x = wg & 7, s = wg >> 3;
        const HeadBlock hb = stretch_row(wg, heads, blocks);
        if (hb.valid) {
          const int u = hb.bh * blocks + hb.blk, at = u - stretch_first(units, x);
          if (hb.bh < 0 || hb.bh >= heads || hb.blk < 0 || hb.blk >= blocks) { ++bad; continue; }
          ++row[u]; ++live[x];
          off += at / 4 != s / 4;
        }
        if (stretch_first(units, x) + s < stretch_first(units, x + 1)) ++own[stretch_first(units, x) + s];
        const int y = stretch_in_turn(wg);
        if (y < 0 || y > 7) { ++bad; continue; }
        if (stretch_first(units, y) + s < stretch_first(units, y + 1)) { ++turn[stretch_first(units, y) + s]; ++in_turn[x]; }
      }
      bool once = stretch_first(units, 0) == 0 && stretch_first(units, 8) == units && wgs >= units && wgs % 8 == 0;
      for (int u = 0; u < units; ++u) once = once && row[u] == 1 && own[u] == 1 && turn[u] == 1;
      for (int x = 0; x < 8; ++x)
        once = once && live[x] >= units / 8 && live[x] <= (units + 7) / 8 && in_turn[x] >= units / 8 && in_turn[x] <= (units + 7) / 8;
      if (!once || off) {
        std::printf("stretches: %d heads of %d blocks: once %d, out of order %d\n", heads, blocks, once, off);
        ++bad;
      }
    }
  }
  return bad;
}

int main() {
  int bad = deal(true) + deal(false) + stretches();
  // 32 rows: four neighbours to every XCD (one below that, and 32 columns, are dealt in turn)
  for (int wg = 0; wg < 2 * 32; ++wg) {
    const HeadBlock hb = xcd_map_rows(wg, 32, 4);
    if (hb.blk / 4 != ((wg & 7) + 3 * hb.bh) % 8) ++bad;
    if (xcd_map(wg, 32, 4, SHORT_COLUMNS).blk != (wg % 32 + 3 * (wg / 32)) % 32) ++bad;
  }
  std::printf(bad ? "FAILED %d\n" : "every block once\n", bad);
  return bad ? 1 : 0;
}
