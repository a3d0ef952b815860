// The pieces of the dispatch stage (see dispatch.hip) that are also used where one workgroup does
// all of it: for a small batch, at the end of the top-k kernel.
#pragma once
#include "kernels.h"

namespace mp {

typedef unsigned long long u64;
// Of the count and place kernels: a chunk of 64 tokens has some 1300 picks, whose masks and places are chains of LDS latencies.
// Place kernel between HIP events, 256 threads | 512 | 1024, us: 300 tokens of 32 picks out of 512 11.0 | 9.8 | 10.2, 3000 11.1 | 9.3 | 9.6, 6007 of 24
// out of 256 9.9 | 8.8 | 9.3, 400 of 32 out of 256 10.4 | 9.4 | 9.7, 8192 of 12 out of 128 9.7 | 9.3 | 10.2, 1000 of 8 out of 32 7.5 | 7.5 | 8.6.
constexpr int DISPATCH_THREADS = 512;

// The picks of a run of tokens, PICKS per thread at a time, so that a memory latency is paid once per batch and not
// once per pick; the last batch loaded stays in registers.
// AGENT: the picks were stored at agent scope by other workgroups of this launch and are loaded likewise, past this CU's
// and XCD's caches; else they are an earlier launch's.
constexpr int PICKS = 8;
template <bool AGENT, int N_THREADS = DISPATCH_THREADS>
struct Picks {
  static constexpr int THREADS = N_THREADS;
  const int32_t* ids;
  int n, k_max;
  uint32_t inv;  // i / k_max = umulhi(i, inv): i k_max < 2^32 (at most 65536 or 256 k_max picks of k_max <= 1024)
  int at = -1, g[PICKS] = {};
  __device__ __forceinline__ Picks(const int32_t* ids_, int ntok, int k) : ids(ids_), n(ntok * k), k_max(k), inv(0xffffffffu / (uint32_t)k + 1u) {}
  __device__ __forceinline__ int token(int i) const { return k_max == 1 ? i : (int)__umulhi((uint32_t)i, inv); }
  __device__ __forceinline__ void load(int first) {
    if (at == first) return;
    at = first;
#pragma unroll
    for (int u = 0; u < PICKS; ++u) {
      const int i = first + u * THREADS + (int)threadIdx.x;
      if (first + u * THREADS >= n) break;  // the same for all threads
      g[u] = i >= n ? -1 : AGENT ? __hip_atomic_load(ids + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ids[i];
    }
  }
  // f(index, sub-expert) for every pick of this thread; last to first if `back`, so that a batch is used twice
  template <class F>
  __device__ __forceinline__ void each(bool back, F&& f) {
    constexpr int STEP = PICKS * THREADS;
    const int batches = (n + STEP - 1) / STEP;
    for (int b = 0; b < batches; ++b) {
      const int first = (back ? batches - 1 - b : b) * STEP;
      load(first);
#pragma unroll
      for (int u = 0; u < PICKS; ++u) {
        const int i = first + u * THREADS + (int)threadIdx.x;
        if (first + u * THREADS >= n) break;
        if (i < n) f(i, g[u]);
      }
    }
  }
};

// masks[g * W + w]: which of the run's tokens 64 w .. 64 w + 63 picked g
template <class Picks>
__device__ __forceinline__ void build_masks(Picks& picks, u64* masks, int E, int W) {
  picks.load(0);
  for (int i = threadIdx.x; i < E * W; i += Picks::THREADS) masks[i] = 0ull;
  __syncthreads();
  picks.each(false, [&](int i, int g) {
    if (g >= 0 && g < E) {
      const int tl = picks.token(i);
      atomicOr(&masks[g * W + (tl >> 6)], 1ull << (tl & 63));
    }
  });
  __syncthreads();
}

// inclusive sum over the lanes of a wave: four steps inside the rows of 16 lanes, two across them
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15, into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31, into rows 2 and 3
  return v;
}

// Exclusive prefixes over the groups by one workgroup, into LDS: off_lds[0..E]
// of the row counts cnt(g) (off_lds[E] = P) and first_lds[0..E] of the m-tile counts; in a table with the long tiles first
// (cut.sorted) without the groups' last tiles, which are written to `last` (a table of max_tiles; null: by another
// workgroup).  Returns the number of m-tiles.  A thread sums a run of consecutive groups, the partial sums are scanned, the run is walked again.
// SORTED: cut.sorted is not 0.  (Last tiles that are counted whatever it is cost every call half a microsecond, stage calls of 4 picks,
// counted | not: 1000 tokens, 32 sub-experts 6.1 | 5.8 us, 512 6.9 | 6.3; 12 000, 128 11.9 | 11.5.)
struct GroupScan {
  int32_t rows, tiles;
  LastTiles last;
};
template <bool SORTED, class Cnt>
__device__ __forceinline__ int group_offsets(Cnt cnt, int32_t* off_lds, int32_t* first_lds, GroupScan* wave_tot,
                                             const TileCut& cut, int E, MTile* last, int max_tiles) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int per = (E + DISPATCH_THREADS - 1) / DISPATCH_THREADS, lo = min(tid * per, E), hi = min(lo + per, E);
  GroupScan mine{0, 0, {}};
  for (int g = lo; g < hi; ++g) {
    const int n = cnt(g);
    mine.rows += n;
    mine.tiles += cut.tiles(n);
    if (SORTED && n > 0) mine.last.add(LastTiles::cls(n));
  }
  GroupScan run{wave_scan(mine.rows), wave_scan(mine.tiles), {}}, total{0, 0, {}};
  if constexpr (SORTED) {
#pragma unroll
    for (int i = 0; i < 4; ++i) run.last.n[i] = (uint32_t)wave_scan((int)mine.last.n[i]);
    if (lane == 63) wave_tot[wv].last = run.last;
#pragma unroll
    for (int i = 0; i < 4; ++i) run.last.n[i] -= mine.last.n[i];
  }
  if (lane == 63) {
    wave_tot[wv].rows = run.rows;
    wave_tot[wv].tiles = run.tiles;
  }
  run.rows -= mine.rows;
  run.tiles -= mine.tiles;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < DISPATCH_THREADS / 64; ++w) {
    const int rows = wave_tot[w].rows, tiles = wave_tot[w].tiles;
    const bool before = w < wv;
    run.rows += before ? rows : 0;
    run.tiles += before ? tiles : 0;
    total.tiles += tiles;
    if constexpr (SORTED) {
      const LastTiles t = wave_tot[w].last;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        run.last.n[i] += before ? t.n[i] : 0u;
        total.last.n[i] += t.n[i];
      }
    }
  }
  const bool sorted = SORTED && total.tiles <= cut.sorted;
  int first = run.tiles - (sorted ? run.last.from(0) : 0);
  for (int g = lo; g < hi; ++g) {
    const int n = cnt(g), nt = cut.tiles(n);
    off_lds[g] = run.rows;
    first_lds[g] = first;
    first += nt;
    if (sorted && n > 0) {
      const int k = LastTiles::cls(n), row = (nt - 1) << cut.log2;
      const int at = total.tiles - total.last.from(0) + total.last.from(k + 1) + run.last.from(k) - run.last.from(k + 1);
      if (last != nullptr && at < max_tiles) put_tile(last, cut, at, g, run.rows + row, n - row, at, 1);
      run.last.add(k);
      --first;
    }
    run.rows += n;
  }
  if (tid == DISPATCH_THREADS - 1) {  // lo == hi == E for the threads past the last group
    off_lds[E] = run.rows;
    first_lds[E] = first;
  }
  __syncthreads();
  return total.tiles;
}

// the header words that go with the offsets (one thread)
__device__ __forceinline__ void write_counts(int32_t* __restrict__ hdr, int P, int n_tiles, bool with_tiles, int max_tiles) {
  hdr[HDR_PAIRS] = P;
  if (with_tiles) {
    hdr[HDR_MTILES] = min(n_tiles, max_tiles);
    hdr[HDR_DYN_GATE_UP] = 0;
    hdr[HDR_DYN_DOWN] = 0;
    for (int i = 0; i < 8; ++i) hdr[HDR_DYN_FUSED + i] = 0;
    if (n_tiles > max_tiles) atomicOr(&hdr[HDR_FLAGS], 2);  // cannot happen: P <= T * k_max
  }
}
// off[0..E] and the header words that go with them (one workgroup)
__device__ __forceinline__ void write_offsets(const int32_t* off_lds, int n_tiles,
                                              int32_t* __restrict__ off, int32_t* __restrict__ hdr,
                                              bool with_tiles, int max_tiles, int E) {
  for (int g = threadIdx.x; g <= E; g += blockDim.x) off[g] = off_lds[g];
  if (threadIdx.x == 0) write_counts(hdr, off_lds[E], n_tiles, with_tiles, max_tiles);
}

// The m-tiles of all groups (a group's tiles are contiguous) that first_lds counts.  Tile i belongs to the last group
// whose first tile is <= i: every thread finds its own by bisection, so a table of hundreds of
// one-tile groups costs one round and not one per group (512 groups and one workgroup: 43-67 -> 7 us
// for the whole kernel).
__device__ __forceinline__ void write_tiles(const int32_t* off_lds, const int32_t* first_lds,
                                            MTile* __restrict__ tiles, int max_tiles, const TileCut& cut, int E,
                                            int start, int step) {
  const int n_tiles = min(first_lds[E], max_tiles);
  for (int i = start; i < n_tiles; i += step) {
    int lo = 0, hi = E;  // first_lds[lo] <= i < first_lds[hi]
    while (hi - lo > 1) {
      const int m = (lo + hi) >> 1;
      if (first_lds[m] <= i) lo = m; else hi = m;
    }
    const int n = off_lds[lo + 1] - off_lds[lo], per = cut.rows(n);
    const int first = first_lds[lo], row = (i - first) * per;
    put_tile(tiles, cut, i, lo, off_lds[lo] + row, min(per, n - row), first, min(first_lds[lo + 1] - first, max_tiles - first));
  }
}

// slots of a run's pairs, the first of which is pair0; base(g): the group's first slot plus its rows from earlier tokens
template <class Picks, class Base>
__device__ __forceinline__ void place_pairs(Picks& picks, const u64* masks, Base base, int32_t* __restrict__ sorted_pair,
                                            int32_t* __restrict__ slot_of_pair, size_t pair0, int P, int E, int W) {
  picks.each(true, [&](int i, int g) {
    int slot = -1;
    if (g >= 0 && g < E) {
      const int tl = picks.token(i), wq = tl >> 6;
      int rank = __popcll(masks[g * W + wq] & ((1ull << (tl & 63)) - 1ull));
      for (int w = 0; w < wq; ++w) rank += __popcll(masks[g * W + w]);
      slot = base(g) + rank;
      sorted_pair[slot] = (int32_t)(pair0 + i);
    }
    slot_of_pair[pair0 + i] = slot;
    if ((long)(pair0 + i) >= (long)P) sorted_pair[pair0 + i] = -1;  // tail beyond the P valid slots
  });
}

// ---------------------------------------------------------------- a small batch in one workgroup
// Up to 64 tokens, or more with few pairs, whose masks and offsets fit the default 64 KiB of LDS: the two or three launches
// of the general path cost more than their work there.  What bounds it is a chain of latencies (picks, masks, scan,
// offsets, slots); one workgroup places the pairs of all tokens by itself, and from a second 64-token word of mask on
// the general path has a workgroup for each: what counts is the pairs beyond those of 64 tokens.  The lines lie where the two met with
// workgroups of 256 threads for both, and stayed: stage calls from a captured graph, one workgroup | count and place kernels with the
// present ones, 512 sub-experts: 64 tokens of 32 picks 3.8 | 7.2 us, of 160 8.6 | 17.3, 100 of 24 4.2 | 7.1, 128 of 32 5.1 | 7.8, 160 of 12 4.1 | 6.5, 255 of
// 8 4.3 | 6.2; beyond the lines 100 of 100 8.7 | 12.8, 128 of 64 7.2 | 10.1, 80 of 256 15.3 | 25.4, 160 of 24 5.1 | 7.3, 255 of 12 4.9 | 6.6, of 24 7.0 | 7.3, of 32 8.0 |
// 7.9, of 64 13.3 | 10.3.  So they meet at about 6000 pairs beyond those of 64 tokens, and up to 128 tokens nowhere; 32, 128 and 1024
// sub-experts alike.  (Layer calls, whose workgroup is the top-k kernel's: topk_dispatches.)
struct SmallDispatch {
  int32_t *cnt, *off, *sorted_pair, *slot_of_pair;
  MTile* tiles;  // nullptr: no m-tile table
  int max_tiles;
  TileCut cut;
};
// where a kernel that picks for itself finds the logits, and what it leaves in place of the top-k kernel
struct PickArgs {
  const float* logits;
  const int32_t* k_tok;
  int32_t* ids;
  float* w;
  int32_t* hdr;
  int E, renorm;
  float scale;
  SmallDispatch small;
};
__host__ __device__ inline size_t small_dispatch_lds(int T, int E) { return (size_t)E * ((T + 63) / 64) * 8 + (size_t)E * 4; }
inline bool small_dispatch(int T, int E, int k_max) {
  return T > 0 && (T <= 64 || (T <= 128 ? (T - 64) * k_max <= 2560 : T < 256 && T * k_max <= 2048)) && small_dispatch_lds(T, E) <= 60 * 1024;
}

// Offsets, counts and m-tiles of all groups from the masks, by one workgroup of `threads` threads; returns P.  A group
// has fewer than 256 rows here: one m-tile, or a few short ones, which the thread that places the group writes.  Ends in
// front of a barrier that off_lds needs.
__device__ __forceinline__ int small_groups(const SmallDispatch& a, int32_t* __restrict__ hdr, const u64* masks,
                                            int32_t* off_lds, int32_t* wave_tot, int W, int E, int threads) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  auto count = [&](int g) {
    int n = 0;
    for (int w = 0; w < W; ++w) n += __popcll(masks[g * W + w]);
    return n;
  };
  // rows (at most 66 x 1024) in the low 18 bits of a word, m-tiles (at most 4096 and one per 16 rows of 16 x 1024, or per 32 of
  // 66 x 1024) above them: one scan for both
  constexpr int TILE = 1 << 18;
  const int per = (E + threads - 1) / threads, lo = min(tid * per, E), hi = min(lo + per, E);
  int mine = 0;
  for (int g = lo; g < hi; ++g) {
    const int n = count(g);
    mine += n + a.cut.tiles(n) * TILE;
  }
  const int incl = wave_scan(mine);
  if (lane == 63) wave_tot[wv] = incl;
  __syncthreads();
  int run = incl - mine, total = 0;
  for (int i = 0; i < threads / 64; ++i) {
    const int t = wave_tot[i];
    run += i < wv ? t : 0;
    total += t;
  }
  const int P = total & (TILE - 1);
  for (int g = lo; g < hi; ++g) {
    const int n = count(g), row0 = run & (TILE - 1), tile = run / TILE, nt = a.cut.tiles(n);
    off_lds[g] = row0;
    a.off[g] = row0;
    a.cnt[g] = n;
    if (a.tiles != nullptr) {
      const int rows = 1 << a.cut.log2, end = min(nt, a.max_tiles - tile);
      if (end > 0) put_tile(a.tiles, a.cut, tile, g, row0, min(n, rows), tile, end);  // mostly the only one
      for (int i = 1; i < end; ++i) put_tile(a.tiles, a.cut, tile + i, g, row0 + i * rows, min(n - i * rows, rows), tile, end);
    }
    run += n + nt * TILE;
  }
  if (tid == 0) {
    a.off[E] = P;
    write_counts(hdr, P, total / TILE, a.tiles != nullptr, a.max_tiles);
  }
  return P;
}

template <bool AGENT, int THREADS = DISPATCH_THREADS>
__device__ __forceinline__ void dispatch_one_workgroup(const int32_t* __restrict__ ids, const SmallDispatch& a,
                                                       int32_t* __restrict__ hdr, u64* lds,
                                                       int32_t* wave_tot, int T, int E, int k_max) {
  const int W = (T + 63) / 64;
  u64* masks = lds;
  int32_t* off_lds = reinterpret_cast<int32_t*>(masks + (size_t)E * W);
  Picks<AGENT, THREADS> picks(ids, T, k_max);
  build_masks(picks, masks, E, W);
  const int P = small_groups(a, hdr, masks, off_lds, wave_tot, W, E, THREADS);
  __syncthreads();
  place_pairs(picks, masks, [&](int g) { return off_lds[g]; }, a.sorted_pair, a.slot_of_pair, 0, P, E, W);
}

}  // namespace mp
