// The pieces of the dispatch stage (see dispatch.hip) that are also used where one workgroup does
// all of it: for a small batch, at the end of the top-k kernel.  Workgroups of 256 threads.
#pragma once
#include "kernels.h"

namespace mp {

typedef unsigned long long u64;
constexpr int DISPATCH_THREADS = 256;

// masks[g * W + w]: which of tokens 64 w .. 64 w + 63 behind t0 picked g
__device__ __forceinline__ void build_masks(const int32_t* __restrict__ ids, u64* masks, int t0,
                                            int ntok, int E, int W, int k_max) {
  for (int i = threadIdx.x; i < E * W; i += blockDim.x) masks[i] = 0ull;
  __syncthreads();
  const int n = ntok * k_max;
  const int32_t* base = ids + (size_t)t0 * k_max;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    int g = base[i];
    if (g >= 0 && g < E) {
      int tl = i / k_max;
      atomicOr(&masks[g * W + (tl >> 6)], 1ull << (tl & 63));
    }
  }
  __syncthreads();
}

// Exclusive prefixes over the groups by one workgroup of 256 threads, into LDS: off_lds[0..E]
// of the row counts cnt(g) (off_lds[E] = P) and first_lds[0..E] of the m-tile counts
// ceil(cnt(g) / FFN_BM) (first_lds[E] = number of m-tiles).  A thread sums a run of consecutive
// groups, the 256 partial sums are scanned with shuffles, the run is walked again.
template <class Cnt>
__device__ __forceinline__ void group_offsets(Cnt cnt, int32_t* off_lds, int32_t* first_lds,
                                              int32_t (*wave_tot)[2], int E) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int per = (E + 255) / 256, lo = min(tid * per, E), hi = min(lo + per, E);
  int mine = 0, mine_t = 0;
  for (int g = lo; g < hi; ++g) {
    const int n = cnt(g);
    mine += n;
    mine_t += (n + FFN_BM - 1) / FFN_BM;
  }
  int incl = mine, incl_t = mine_t;
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    const int o = __shfl_up(incl, m, 64), ot = __shfl_up(incl_t, m, 64);
    if (lane >= m) {
      incl += o;
      incl_t += ot;
    }
  }
  if (lane == 63) {
    wave_tot[wv][0] = incl;
    wave_tot[wv][1] = incl_t;
  }
  __syncthreads();
  int run = incl - mine, run_t = incl_t - mine_t;
  for (int i = 0; i < wv; ++i) {
    run += wave_tot[i][0];
    run_t += wave_tot[i][1];
  }
  for (int g = lo; g < hi; ++g) {
    const int n = cnt(g);
    off_lds[g] = run;
    first_lds[g] = run_t;
    run += n;
    run_t += (n + FFN_BM - 1) / FFN_BM;
  }
  if (tid == 255) {  // lo == hi == E for the threads past the last group
    off_lds[E] = run;
    first_lds[E] = run_t;
  }
  __syncthreads();
}

// off[0..E] and the header words that go with them (one workgroup)
__device__ __forceinline__ void write_offsets(const int32_t* off_lds, const int32_t* first_lds,
                                              int32_t* __restrict__ off, int32_t* __restrict__ hdr,
                                              bool with_tiles, int max_tiles, int E) {
  for (int g = threadIdx.x; g <= E; g += blockDim.x) off[g] = off_lds[g];
  if (threadIdx.x == 0) {
    hdr[HDR_PAIRS] = off_lds[E];
    if (with_tiles) {
      hdr[HDR_MTILES] = min(first_lds[E], max_tiles);
      hdr[HDR_DYN_GATE_UP] = 0;
      hdr[HDR_DYN_DOWN] = 0;
      for (int i = 0; i < 8; ++i) hdr[HDR_DYN_FUSED + i] = 0;
      if (first_lds[E] > max_tiles) atomicOr(&hdr[HDR_FLAGS], 2);  // cannot happen: P <= T * k_max
    }
  }
}

// The m-tiles of all groups (a group's tiles are contiguous).  Tile i belongs to the last group
// whose first tile is <= i: every thread finds its own by bisection, so a table of hundreds of
// one-tile groups costs one round and not one per group (512 groups and one workgroup: 43-67 -> 7 us
// for the whole kernel).
__device__ __forceinline__ void write_tiles(const int32_t* off_lds, const int32_t* first_lds,
                                            MTile* __restrict__ tiles, int max_tiles, bool even, int E,
                                            int start, int step) {
  const int n_tiles = min(first_lds[E], max_tiles);
  for (int i = start; i < n_tiles; i += step) {
    int lo = 0, hi = E;  // first_lds[lo] <= i < first_lds[hi]
    while (hi - lo > 1) {
      const int m = (lo + hi) >> 1;
      if (first_lds[m] <= i) lo = m; else hi = m;
    }
    const int n = off_lds[lo + 1] - off_lds[lo], per = mtile_rows(n, FFN_BM, even);
    const int first = first_lds[lo], row = (i - first) * per;
    MTile t;
    t.g = lo;
    t.row0 = off_lds[lo] + row;
    t.rows = min(per, n - row);
    t.first = first;
    t.count = min(first_lds[lo + 1] - first, max_tiles - first);
    t.pad[0] = t.pad[1] = t.pad[2] = 0;
    tiles[i] = t;
  }
}

// slots of the pairs of ntok tokens behind t0; base(g): the group's first slot plus its rows from earlier tokens
template <class Base>
__device__ __forceinline__ void place_pairs(const int32_t* __restrict__ ids, const u64* masks, Base base,
                                            int32_t* __restrict__ sorted_pair,
                                            int32_t* __restrict__ slot_of_pair, int t0, int ntok, int P,
                                            int E, int W, int k_max) {
  const int n = ntok * k_max;
  const size_t pair0 = (size_t)t0 * k_max;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    int g = ids[pair0 + i];
    int slot = -1;
    if (g >= 0 && g < E) {
      int tl = i / k_max, wq = tl >> 6;
      int rank = __popcll(masks[g * W + wq] & ((1ull << (tl & 63)) - 1ull));
      for (int w = 0; w < wq; ++w) rank += __popcll(masks[g * W + w]);
      slot = base(g) + rank;
      sorted_pair[slot] = (int32_t)(pair0 + i);
    }
    slot_of_pair[pair0 + i] = slot;
    if ((long)(pair0 + i) >= (long)P) sorted_pair[pair0 + i] = -1;  // tail beyond the P valid slots
  }
}

// ---------------------------------------------------------------- a small batch in one workgroup
// Up to 64 tokens, or more with few pairs, whose masks and prefixes fit the default 64 KiB of LDS: the three launches
// of the general path cost more than their work there.  One workgroup places the pairs of all tokens by itself, and
// from a second 64-token word of mask on the general path has a workgroup for each.  Calls of d = 64, Is = 32, 512
// sub-experts from a captured graph, one workgroup | three launches: 40 tokens of 8 picks 26.2 | 30.3 us, 64 of 64
// 50.8 | 59.2; 100 of 8 34.4 | 35.3, of 24 42.3 | 42.5, of 64 62.3 | 61.1; 160 of 4 32.7 | 31.6, of 32 54.4 | 46.1;
// 255 of 32 67.1 | 47.8 (32 to 1024 sub-experts alike).  Budgets below k_max leave fewer pairs than T k_max: 79
// tokens of up to 20, half of them on average, 36.5 | 39.2; 155 of up to 1, 39.5 | 40.7.
struct SmallDispatch {
  int32_t *cnt, *off, *sorted_pair, *slot_of_pair;
  MTile* tiles;  // nullptr: no m-tile table
  int max_tiles;
};
__host__ __device__ inline size_t small_dispatch_lds(int T, int E) { return (size_t)E * ((T + 63) / 64) * 8 + 2 * ((size_t)E + 1) * 4; }
inline bool small_dispatch(int T, int E, int k_max) {
  return T > 0 && (T <= 64 || (T < 256 && T * k_max <= (T <= 128 ? 4096 : 320))) && small_dispatch_lds(T, E) <= 60 * 1024;
}

__device__ __forceinline__ void dispatch_one_workgroup(const int32_t* __restrict__ ids, const SmallDispatch& a,
                                                       int32_t* __restrict__ hdr, u64* lds,
                                                       int32_t (*wave_tot)[2], int T, int E, int k_max) {
  const int W = (T + 63) / 64;
  u64* masks = lds;
  int32_t* off_lds = reinterpret_cast<int32_t*>(masks + (size_t)E * W);
  int32_t* first_lds = off_lds + E + 1;
  build_masks(ids, masks, 0, T, E, W, k_max);
  auto count = [&](int g) {
    int n = 0;
    for (int w = 0; w < W; ++w) n += __popcll(masks[g * W + w]);
    return n;
  };
  group_offsets(count, off_lds, first_lds, wave_tot, E);
  for (int g = threadIdx.x; g < E; g += blockDim.x) a.cnt[g] = off_lds[g + 1] - off_lds[g];
  write_offsets(off_lds, first_lds, a.off, hdr, a.tiles != nullptr, a.max_tiles, E);
  if (a.tiles != nullptr) write_tiles(off_lds, first_lds, a.tiles, a.max_tiles, false, E, threadIdx.x, blockDim.x);
  place_pairs(ids, masks, [&](int g) { return off_lds[g]; }, a.sorted_pair, a.slot_of_pair, 0, T, off_lds[E], E,
              W, k_max);
}

}  // namespace mp
