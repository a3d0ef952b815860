// How workgroups share small tiles: plain C++, so that it can be run on the host as well.
#pragma once
#include <stdint.h>

#include "host_device.h"

namespace mp {

// Rows of each m-tile that a group of n rows is cut into (the last one takes what is left); the number of tiles is
// that of tiles of `most` rows.  `even`: about equal lengths, in steps of the 64 rows that the two-kernel FFN's time
// goes in.  Its tiles share their sub-expert's weights through L2 only while they run in step: cut into 256 + 96 rows,
// 256 sub-experts of 352 x 2048 with some 350 rows each fetched every weight twice (gate-up 1.81 GB), cut into
// 192 + 160 once (1.27 GB; FFN 506 -> 485 us; 4500 tokens of 20 picks out of 256 x 256 364 -> 342, 2200 of 5 out of
// 32 x 3584 1072 -> 1006, nothing slower).  The fused kernel's time goes in steps of 128 rows and keeps full tiles.
MP_HD int mtile_rows(int n, int most, bool even) {
  const int nt = (n + most - 1) / most;
  return even && nt > 1 ? ((n + nt - 1) / nt + 63) / 64 * 64 : most;
}

// How the groups are cut into m-tiles: into tiles of at most 1 << log2 rows, `even` as above.
struct TileCut {
  int log2;
  bool even;
  int sorted = 0;  // not even: tables of up to so many tiles have the long ones first (LastTiles)
  MP_HD int tiles(int n) const { return (n + (1 << log2) - 1) >> log2; }
  MP_HD int rows(int n) const { return mtile_rows(n, 1 << log2, even); }
};

// Item of a list of (m-tile, n-tile) pairs in which a group's m-tiles of the same n-tile are neighbours: they run at the
// same time on one XCD, and its L2 serves their weights to all but the first.  first, count: the m-tiles of the
// group that m-tile item / n_tiles_n belongs to.
MP_HD void shared_item(int item, int n_tiles_n, int first, int count, int& m_tile, int& n_tile) {
  const int i = item - first * n_tiles_n;
  m_tile = first + i % count;
  n_tile = i / count;
}

// The fused kernel's table with the long tiles first: the full tiles that are not their group's last in the order of the
// groups, then the groups' last tiles in classes of 32 rows, longest first, in the order of the groups inside a class.
// Groups per class, in 16 bits each (at most 4096 groups), so that four words are added up for all eight.
struct LastTiles {
  uint32_t n[4];
  MP_HD static int cls(int rows) { return (rows - 1) % 256 >> 5; }  // of the last tile of a group of rows > 0
  MP_HD void add(int k) {
    for (int i = 0; i < 4; ++i) n[i] += k >> 1 == i ? 1u << 16 * (k & 1) : 0u;
  }
  MP_HD int from(int k) const {  // of class k and longer ones
    int s = 0;
    for (int j = 0; j < 8; ++j) s += j >= k ? (int)(n[j >> 1] >> 16 * (j & 1) & 0xffffu) : 0;
    return s;
  }
};

// Whose m-tiles are whose in the fused kernel.  An XCD's workgroups draw from a list of their own: turns of `run`
// consecutive tiles, which mostly belong to one or a few groups and so meet in one L2 with their weights and, with the other
// sub-experts of their expert, with their slot rows.  What is left after the last whole turn is dealt out evenly, in
// consecutive tiles too: fewer tiles than workgroups give every XCD its share.
struct TileLists {
  static constexpr int XCDS = 8;
  int run, turns, rest;  // whole turns, and the tiles behind them
  MP_HD TileLists(int n_tiles, int run_) : run(run_), turns(n_tiles / (run_ * XCDS)), rest(n_tiles % (run_ * XCDS)) {}
  MP_HD int count(int xcd) const { return turns * run + rest / XCDS + (xcd < rest % XCDS ? 1 : 0); }
  MP_HD int tile(int xcd, int i) const {  // i < count(xcd)
    const int turn = i / run;
    if (turn < turns) return (turn * XCDS + xcd) * run + i % run;
    const int extra = rest % XCDS;
    return turns * run * XCDS + xcd * (rest / XCDS) + (xcd < extra ? xcd : extra) + i - turns * run;
  }
};

// An m-tile of `rows` slot rows is cut into row blocks of ROWS, and each of those into n_tiles_n n-tiles.
// f(m-tile, row block, n-tile) for the share of workgroup b out of `grid` (a multiple of n_xcd; b serves XCD
// b % n_xcd, and an XCD a contiguous part of the list, in which a sub-expert's weights meet).

// For m-tiles of at most `blocks` row blocks (longer ones take longer): the list holds the first row block of every
// (m-tile, n-tile) pair, all of which exist, then the second ones, of which few do or all.  A list of every possible
// row block is mostly empty there, and brings those that exist to the same few workgroups whenever the stride
// grid / n_xcd has a factor in common with row blocks x n-tiles: one row in each of 32 groups, 4 n-tiles, 8 row
// blocks, 512 workgroups: 128 tiles on 64 of them; 20 groups, 32 n-tiles: 640 tiles on 256.
// mask(pred): bit l is pred(l), l = 0 .. 63 (a ballot), so that 64 pairs without a second row block cost one look at
// their headers (768 sub-experts of 96 with a row each, both GEMMs 200 us, with a look at every pair 225).
template <int ROWS, class Tile, class Mask, class F>
MP_HD void short_row_blocks(int b, int grid, int n_xcd, int n_mtiles, int n_tiles_n, int blocks, Tile&& tile,
                            Mask&& mask, F&& f) {
  const int xcd = b % n_xcd, total = n_mtiles * n_tiles_n, chunk = (total + n_xcd - 1) / n_xcd;
  const int begin = xcd * chunk, n = (total < begin + chunk ? total : begin + chunk) - begin;  // the XCD's pairs
  const int slot = b / n_xcd, step = grid / n_xcd;
  for (int i = slot; i < n; i += step) {
    const auto t = tile((begin + i) / n_tiles_n);
    for (int blk = 0; blk * ROWS < (blocks > 1 ? 1 : t.rows); ++blk) f(t, blk, (begin + i) % n_tiles_n);
  }
  for (int first = 1; first < blocks; ++first)  // the list goes on: start where the workgroups before this one stopped
    for (int i0 = ((slot - first * n) % step + step) % step; i0 < n; i0 += 64 * step) {
      uint64_t on = mask([&](int l) {
        const int i = i0 + l * step;
        return i < n && tile((begin + i) / n_tiles_n).rows > first * ROWS;
      });
      for (; on != 0; on &= on - 1) {
        const int i = i0 + __builtin_ctzll(on) * step;
        const auto t = tile((begin + i) / n_tiles_n);
        for (int blk = first; blk * ROWS < (first < blocks - 1 ? first * ROWS + 1 : t.rows); ++blk)
          f(t, blk, (begin + i) % n_tiles_n);
      }
    }
}

// For m-tiles of any length: the list (m-tile, row block of BLOCKS, n-tile).  What runs at the same time shares weights.
template <int ROWS, int BLOCKS, class Tile, class F>
MP_HD void all_row_blocks(int b, int grid, int n_xcd, int n_mtiles, int n_tiles_n, Tile&& tile, F&& f) {
  const int xcd = b % n_xcd, total = n_mtiles * BLOCKS * n_tiles_n, chunk = (total + n_xcd - 1) / n_xcd;
  const int end = total < (xcd + 1) * chunk ? total : (xcd + 1) * chunk;
  for (int item = xcd * chunk + b / n_xcd; item < end; item += grid / n_xcd) {
    const auto t = tile(item / (BLOCKS * n_tiles_n));
    const int blk = item / n_tiles_n % BLOCKS;
    if (blk * ROWS < t.rows) f(t, blk, item % n_tiles_n);
  }
}

}  // namespace mp
