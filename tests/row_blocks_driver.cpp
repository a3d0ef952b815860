// The deal of small tiles on the host: every tile that exists once, none that does not, and no workgroup
// with much more than its share.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../paper_2510_19366_amd/csrc/row_blocks.h"

struct Tile {
  int rows, m;
};

auto mask = [](auto&& pred) {
  uint64_t m = 0;
  for (int l = 0; l < 64; ++l) m |= (uint64_t)(pred(l) ? 1 : 0) << l;
  return m;
};

template <class Deal>
int check(Deal&& deal, int grid, int n_tiles_n, const std::vector<Tile>& tiles, bool even,
          int blocks = 1) {
  const int n = (int)tiles.size();
  std::vector<int> seen((size_t)n * 8 * n_tiles_n, 0);
  int exist = 0, most = 0;
  for (const Tile& t : tiles) exist += (t.rows + 31) / 32 * n_tiles_n;
  for (int b = 0; b < grid; ++b) {
    int mine = 0;
    deal(b, [&](int m) { return tiles.at(m); }, [&](const Tile& t, int blk, int nt) {
      if (blk * 32 >= t.rows || nt < 0 || nt >= n_tiles_n) exit(2);
      ++seen.at(((size_t)t.m * 8 + blk) * n_tiles_n + nt);
      ++mine;
    });
    most = std::max(most, mine);
  }
  int done = 0;
  for (int c : seen) {
    if (c > 1) return 3;
    done += c;
  }
  if (done != exist) return 4;
  // an even share of what an XCD gets, which is an eighth of the pairs
  const int share = (exist / blocks + 7) / 8 * blocks, per = grid / 8;
  return even && most > (share + per - 1) / per ? 5 : 0;
}

// the m-tiles of a group: as few as possible, none empty or too long, none left over; even ones differ by less
// than a step of 64 rows per tile before the last
static int check_rows(int n, int most) {
  const int nt = (n + most - 1) / most;
  for (bool even : {false, true}) {
    const int per = mp::mtile_rows(n, most, even);
    if (per > most || (nt > 1 && (per % 64 != 0 || (nt - 1) * per >= n)) || (long)nt * per < n) return 1;
    if (even && nt > 1 && per - (n + nt - 1) / nt >= 64) return 2;
    if (!even && per != most) return 3;
  }
  return 0;
}

// Groups cut into m-tiles of at most 1 << log2 rows: every row in one of them, and every (m-tile, n-tile) pair one item, the
// m-tiles of a group with the same n-tile being neighbours, so that workgroups that run side by side share their weights.
static int check_shared(const std::vector<int>& groups, int log2, int n_tiles_n) {
  struct M {
    int g, rows, first, count;
  };
  std::vector<M> tiles;
  const mp::TileCut cut{log2, false};
  for (int g = 0; g < (int)groups.size(); ++g) {
    const int nt = cut.tiles(groups[g]), first = (int)tiles.size();
    int rows = 0;
    for (int i = 0; i < nt; ++i) {
      tiles.push_back({g, std::min(cut.rows(groups[g]), groups[g] - rows), first, nt});
      rows += tiles.back().rows;
      if (tiles.back().rows < 1 || tiles.back().rows > 1 << log2) return 1;
    }
    if (rows != groups[g]) return 2;
  }
  const int total = (int)tiles.size() * n_tiles_n;
  std::vector<int> seen(total, 0);
  int last_g = -1, last_n = -1, changes = 0, exist = 0;
  for (const int n : groups) exist += n > 0 ? n_tiles_n : 0;
  for (int i = 0; i < total; ++i) {
    const M& t0 = tiles[i / n_tiles_n];
    int m, n;
    mp::shared_item(i, n_tiles_n, t0.first, t0.count, m, n);
    if (m < t0.first || m >= t0.first + t0.count || n < 0 || n >= n_tiles_n) return 3;
    if (seen[m * n_tiles_n + n]++) return 4;
    changes += tiles[m].g != last_g || n != last_n;
    last_g = tiles[m].g;
    last_n = n;
  }
  return changes != exist ? 5 : 0;  // each weight tile is one run of items
}

// The fused kernel's lists: every tile in one of them, lists of equal length but for one, turns in runs, and behind the last
// whole turn consecutive tiles as well.
static int check_lists(int n, int run) {
  const mp::TileLists lists(n, run);
  std::vector<int> seen(n, 0);
  for (int x = 0; x < 8; ++x) {
    const int c = lists.count(x);
    if (c > lists.count(0) || c < lists.count(0) - 1) return 1;
    for (int i = 0; i < c; ++i) {
      const int t = lists.tile(x, i);
      if (t < 0 || t >= n || seen[t]++) return 2;
      if (i % run != 0 && t != lists.tile(x, i - 1) + 1) return 3;
    }
  }
  for (int c : seen)
    if (c != 1) return 4;
  return 0;
}

// The groups' last tiles, longest class first: every place behind the other tiles taken once, by classes in falling order
// and by groups inside a class.  The sums over the groups before one are built as a scan would.
static int check_last(const std::vector<int>& groups) {
  mp::LastTiles total{}, run{};
  std::vector<int> at(groups.size(), -1), by(groups.size(), -1);
  int n = 0;
  for (int rows : groups)
    if (rows > 0) {
      total.add(mp::LastTiles::cls(rows));
      ++n;
    }
  if (total.from(0) != n || total.from(8) != 0) return 1;
  for (int g = 0; g < (int)groups.size(); ++g) {
    if (groups[g] == 0) continue;
    const int k = mp::LastTiles::cls(groups[g]), p = total.from(k + 1) + run.from(k) - run.from(k + 1);
    if (k != ((groups[g] + 255) % 256) / 32 || p < 0 || p >= n || by[p] >= 0) return 2;
    by[p] = g;
    run.add(k);
  }
  for (int p = 1; p < n; ++p) {
    const int a = mp::LastTiles::cls(groups[by[p - 1]]), b = mp::LastTiles::cls(groups[by[p]]);
    if (a < b || (a == b && by[p - 1] >= by[p])) return 3;
  }
  return 0;
}

int main() {
  std::mt19937 gen(3);
  for (int most : {1, 32, 33, 256, 257, 900})
    for (int n_groups : {1, 7, 512, 4096}) {
      std::vector<int> groups(n_groups);
      for (int& n : groups) n = gen() % 4 == 0 ? 0 : 1 + (int)(gen() % most);
      if (const int e = check_last(groups)) {
        printf("last tiles of %d groups of up to %d rows: %d\n", n_groups, most, e);
        return e;
      }
    }
  for (int n = 0; n < 1100; ++n)
    for (int run : {1, 32, 64})
      if (const int e = check_lists(n, run)) {
        printf("lists of %d tiles in runs of %d: %d\n", n, run, e);
        return e;
      }
  for (int log2 : {4, 5, 6})
    for (int n_tiles_n : {1, 2, 6, 11, 56})
      for (int most : {1, 15, 16, 17, 64, 65, 300, 2000}) {
        std::vector<int> groups(40);
        for (int& n : groups) n = gen() % 3 == 0 ? 0 : 1 + (int)(gen() % most);
        if (const int e = check_shared(groups, log2, n_tiles_n)) {
          printf("groups of up to %d rows in tiles of %d, n-tiles %d: %d\n", most, 1 << log2, n_tiles_n, e);
          return e;
        }
      }
  for (int n = 0; n < 5000; ++n)
    if (const int e = check_rows(n, 256)) {
      printf("m-tiles of %d rows: %d\n", n, e);
      return e;
    }
  for (int grid : {8, 64, 512})
    for (int n_tiles_n : {1, 2, 4, 6, 11, 22, 32})
      for (int n : {0, 1, 5, 20, 32, 250, 500})
        for (int kind = 0; kind < 5; ++kind) {  // one row block, all full, any length, two row blocks, one or two
          std::vector<Tile> tiles(n);
          const int blocks = kind < 3 ? 1 : 2;
          for (int m = 0; m < n; ++m) tiles[m] = {kind == 0 ? 1 + (int)(gen() % 32) : kind == 1 ? 256 : kind == 2 ? 1 + (int)(gen() % 256) : kind == 3 ? 33 + (int)(gen() % 32) : 1 + (int)(gen() % 64), m};
          int e = check([&](int b, auto tile, auto f) { mp::short_row_blocks<32>(b, grid, 8, n, n_tiles_n, blocks, tile, mask, f); }, grid,
                        n_tiles_n, tiles, kind == 0 || kind == 3, blocks);
          if (!e && kind == 2)
            e = check([&](int b, auto tile, auto f) { mp::short_row_blocks<32>(b, grid, 8, n, n_tiles_n, 2, tile, mask, f); }, grid,
                      n_tiles_n, tiles, false);
          if (!e)
            e = check([&](int b, auto tile, auto f) { mp::all_row_blocks<32, 8>(b, grid, 8, n, n_tiles_n, tile, f); }, grid,
                      n_tiles_n, tiles, kind == 1);
          if (e) {
            printf("grid %d n-tiles %d m-tiles %d kind %d: %d\n", grid, n_tiles_n, n, kind, e);
            return e;
          }
        }
  return 0;
}
