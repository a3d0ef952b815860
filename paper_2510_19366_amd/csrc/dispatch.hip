// Dispatch stage: group the token-sub-expert pairs (Sec. 2.1) by sub-expert
// with a stable counting sort that needs no global sort and no order-dependent
// atomics.
//
// Tokens are cut into chunks of 64*W tokens.  Inside a chunk, for every
// sub-expert g a bit mask over the chunk's tokens records who picked g (LDS
// atomic OR: commutative, so the result does not depend on timing).  The
// chunk's count for g is the mask's popcount, and the rank of token t among the
// chunk's pickers of g is the popcount of the mask bits below t.  A second
// kernel turns the per-chunk counts into per-chunk bases and the groups' totals (few of them
// the placing kernel itself), and the placing kernel derives the group offsets from the totals.
// A batch of fewer than 256 tokens is dispatched by one workgroup instead (dispatch_common.h).
// Because a token picks a sub-expert at most once, "token ascending" fixes the
// order inside a group completely.
#include "dispatch_common.h"

namespace mp {

int dispatch_chunk_words(int E, int T) {
  int cap = 8192 / (E > 0 ? E : 1);  // E * W * 8 bytes of LDS <= 64 KiB
  if (cap > 4) cap = 4;
  if (cap < 1) cap = 1;
  int w = T / (64 * 256);  // aim at >= 256 chunks (one per CU) before growing the chunks
  if (w > cap) w = cap;
  if (w < 1) w = 1;
  return w;
}

__global__ __launch_bounds__(DISPATCH_THREADS) void dispatch_count_kernel(const int32_t* __restrict__ ids,
                                                             int32_t* __restrict__ chunk_cnt, int T,
                                                             int E, int W, int k_max) {
  extern __shared__ u64 masks[];
  const int c = blockIdx.x, t0 = c * 64 * W;
  const int ntok = min(64 * W, T - t0);
  Picks<false> picks(ids + (size_t)t0 * k_max, ntok, k_max);
  build_masks(picks, masks, E, W);
  for (int g = threadIdx.x; g < E; g += blockDim.x) {
    int n = 0;
    for (int w = 0; w < W; ++w) n += __popcll(masks[g * W + w]);
    chunk_cnt[(size_t)c * E + g] = n;
  }
}

// chunk_cnt[c,g] -> exclusive prefix over chunks (in place) and cnt[g].  The chain over chunks
// is independent per group and moves n_chunks * E * 8 bytes, too much for one CU: a workgroup
// takes SCAN_GROUPS consecutive groups and cuts the chunk range into SCAN_PARTS pieces that run
// side by side (a thread sums its piece, the pieces' sums meet in LDS, a second walk over the
// piece writes the running prefixes).  The prefix over groups (off[]) is left to the place
// kernel, where every workgroup recomputes it in LDS from cnt[].
constexpr int SCAN_GROUPS = 16, SCAN_PARTS = 16, SCAN_THREADS = SCAN_GROUPS * SCAN_PARTS;
__global__ __launch_bounds__(SCAN_THREADS) void dispatch_scan_kernel(int32_t* __restrict__ chunk_cnt,
                                                                     int32_t* __restrict__ cnt,
                                                                     int n_chunks, int E) {
  __shared__ int32_t part_tot[SCAN_PARTS][SCAN_GROUPS];
  const int gq = threadIdx.x % SCAN_GROUPS, part = threadIdx.x / SCAN_GROUPS;
  const int g = blockIdx.x * SCAN_GROUPS + gq;
  const bool in = g < E;
  const int cp = (n_chunks + SCAN_PARTS - 1) / SCAN_PARTS;
  const int c_lo = min(part * cp, n_chunks), c_hi = min(c_lo + cp, n_chunks);
  int sum = 0;
  if (in) {
    constexpr int U = 16;
    int c = c_lo;
    for (; c + U <= c_hi; c += U) {
      int v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = chunk_cnt[(size_t)(c + u) * E + g];
#pragma unroll
      for (int u = 0; u < U; ++u) sum += v[u];
    }
    for (; c < c_hi; ++c) sum += chunk_cnt[(size_t)c * E + g];
  }
  part_tot[part][gq] = sum;
  __syncthreads();
  int run = 0, total = 0;
#pragma unroll
  for (int p = 0; p < SCAN_PARTS; ++p) {
    const int s = part_tot[p][gq];
    run += p < part ? s : 0;
    total += s;
  }
  if (!in) return;
  if (part == 0) cnt[g] = total;
  constexpr int U = 8;
  int c = c_lo;
  for (; c + U <= c_hi; c += U) {
    int v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = chunk_cnt[(size_t)(c + u) * E + g];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      chunk_cnt[(size_t)(c + u) * E + g] = run;
      run += v[u];
    }
  }
  for (; c < c_hi; ++c) {
    const int v = chunk_cnt[(size_t)c * E + g];
    chunk_cnt[(size_t)c * E + g] = run;
    run += v;
  }
}

// Where the counts of all chunks are few, the place kernel adds them up itself, every workgroup for its own chunk: totals
// and the counts of the chunks before it, four groups per load.  A launch and its latency less, for chunks x E counts read from
// L2 in each workgroup.  Layer calls, with the scan kernel | without: 500 tokens of 512 sub-experts (4096 counts) 253.5 |
// 250.4 us, 2000 of 128 (4096) 318.7 | 315.8, 8192 of 128 (16 384) 702 | 699, 2000 of 512 (16 384) 378.8 | 376.5; 6007 of 256
// (24 064) 644.1 | 644.5, 4000 of 512 (32 256) 538.3 | 539.5.  Stage calls from a captured graph: 2048 of 4 7.3 | 6.6, 16 384 of 4
// 7.9 | 7.6, of 64 9.2 | 7.8, 8192 of 128 10.7 | 7.9, 1024 of 1024 9.6 | 8.8; chunks of two and four words of tokens, 32 768 of 64
// 10.9 | 9.5, 65 536 of 64 14.2 | 12.6, of 4 8.9 | 8.6.
constexpr long SUM_COUNTS = 16384;
bool dispatch_sums(int T, int E) {
  const int nch = cdiv(T, 64 * dispatch_chunk_words(E, T));
  return T > 0 && E % 4 == 0 && E <= 1024 && nch <= 256 && (long)nch * E <= SUM_COUNTS;
}
// tot[g], before[g] (LDS): rows of group g in all chunks and in those before c.  No more threads than have U loads each: every one
// adds to the same LDS words in the end, which with all threads on four groups takes longer than the loads.  Layer calls of 4 picks,
// d = 64, Is = 32, all threads | so: 4 groups, 300 tokens 28.5 | 25.9 us, 2000 30.1 | 27.6, 16 384 46.0 | 43.6; 8, 300 27.2 | 26.0; 32, 2000
// 27.8 | 27.7.
__device__ __forceinline__ void sum_counts(const int32_t* __restrict__ chunk_cnt, int32_t* tot, int32_t* before, int c,
                                           int n_chunks, int E) {
  for (int g = threadIdx.x; g < 2 * E; g += DISPATCH_THREADS) tot[g] = 0;  // before[] lies behind tot[]
  __syncthreads();
  constexpr int U = 8;
  const int quads = E / 4, part = threadIdx.x / quads, q = threadIdx.x % quads;
  const int parts = min(DISPATCH_THREADS / quads, (n_chunks + U - 1) / U);
  if (part < parts) {
    const int4* rows = reinterpret_cast<const int4*>(chunk_cnt) + q;
    int4 t = make_int4(0, 0, 0, 0), b = t;
    for (int i = part; i < n_chunks; i += U * parts) {
      int4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = i + u * parts;
        v[u] = rows[(size_t)min(j, n_chunks - 1) * quads];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = i + u * parts;
        if (j < n_chunks) t.x += v[u].x, t.y += v[u].y, t.z += v[u].z, t.w += v[u].w;
        if (j < c) b.x += v[u].x, b.y += v[u].y, b.z += v[u].z, b.w += v[u].w;
      }
    }
    const int ts[4] = {t.x, t.y, t.z, t.w}, bs[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      atomicAdd(&tot[4 * q + e], ts[e]);
      atomicAdd(&before[4 * q + e], bs[e]);
    }
  }
  __syncthreads();
}

// Workgroup c places the pairs of chunk c.  Every workgroup derives the group offsets from
// cnt[] (E additions); workgroup 0 also writes them out: off[0..E] and the pair count.
// With tiles != nullptr the kernel also builds the grouped FFN's m-tile table (the table
// ffn_tiles_kernel builds from off[]).
// SUM: chunk_base and cnt are the chunks' counts, not yet added up, and where the groups' go (see dispatch_sums).
template <bool SUM>
__global__ __launch_bounds__(DISPATCH_THREADS) void dispatch_place_kernel(
    const int32_t* __restrict__ ids, const int32_t* __restrict__ chunk_base,
    int32_t* __restrict__ cnt, int32_t* __restrict__ off, int32_t* __restrict__ hdr,
    int32_t* __restrict__ sorted_pair, int32_t* __restrict__ slot_of_pair,
    MTile* __restrict__ tiles, int max_tiles, TileCut cut, int T, int E, int W, int k_max) {
  extern __shared__ u64 masks[];  // E * W masks, then E + 1 offsets, then E + 1 first-tile indices; SUM: then 2 E sums
  __shared__ GroupScan wave_tot[DISPATCH_THREADS / 64];
  int32_t* off_lds = reinterpret_cast<int32_t*>(masks + (size_t)E * W);
  int32_t* first_lds = off_lds + E + 1;
  const int c = blockIdx.x, t0 = c * 64 * W;
  const int ntok = max(min(64 * W, T - t0), 0);
  Picks<false> picks(ids + (size_t)t0 * k_max, ntok, k_max);
  picks.load(0);  // on their way while the offsets are derived
  int32_t *tot_lds = first_lds + E + 1, *before_lds = tot_lds + E;
  if constexpr (SUM) {
    sum_counts(chunk_base, tot_lds, before_lds, c, gridDim.x, E);
    if (c == 0)
      for (int g = threadIdx.x; g < E; g += DISPATCH_THREADS) cnt[g] = tot_lds[g];
  }
  auto count = [&](int g) { return SUM ? tot_lds[g] : cnt[g]; };
  MTile* last = c == 0 ? tiles : nullptr;
  const int n_tiles = cut.sorted != 0 ? group_offsets<true>(count, off_lds, first_lds, wave_tot, cut, E, last, max_tiles)
                                      : group_offsets<false>(count, off_lds, first_lds, wave_tot, cut, E, last, max_tiles);
  if (c == 0) write_offsets(off_lds, n_tiles, off, hdr, tiles != nullptr, max_tiles, E);
  if (tiles != nullptr)
    write_tiles(off_lds, first_lds, tiles, max_tiles, cut, E, c * DISPATCH_THREADS + threadIdx.x,
                gridDim.x * DISPATCH_THREADS);
  build_masks(picks, masks, E, W);
  place_pairs(picks, masks, [&](int g) { return off_lds[g] + (SUM ? before_lds[g] : chunk_base[(size_t)c * E + g]); }, sorted_pair,
              slot_of_pair, (size_t)t0 * k_max, off_lds[E], E, W);
}

// A thread per pick, and per two groups, as long as 256 threads are enough, else 1024, which more picks keep busy.  Stage calls from a captured graph, us, 256
// threads | 512 | 1024, 32 sub-experts unless said: 1 token of 8 picks 2.3 | 2.6 | 2.8, 64 of 4 2.4 | 2.6 | 2.8, 64 of 8 2.8 | 2.7 | 2.9, of 12 3.2 | 3.1 |
// 3.0, of 16 3.6 | 3.1 | 3.1, of 32 5.3 | 4.0 | 3.6, 200 of 8 5.6 | 4.4 | 3.9; 512 sub-experts: 4 of 32 2.8 | 2.8 | 3.0, 32 of 16 3.3 | 2.9 | 3.1, 64 of 32
// 5.7 | 4.2 | 3.8; 1024: 4 of 8 3.4 | | 3.2.  Between HIP events: 64 of 64 12.9 | 8.9 | 8.4, 100 of 71 19.6 | 12.4 | 10.3, 128 of 40 15.4 | 10.6 | 9.0, 65 of 200 30.7 | 18.8 | 14.9;
// the gate-less layer of 100 tokens, whose picks it dispatches, 251 | | 246.6.
template <int SMALL_THREADS>
__global__ __launch_bounds__(SMALL_THREADS) void dispatch_small_kernel(const int32_t* __restrict__ ids, SmallDispatch a,
                                                                       int32_t* __restrict__ hdr, int T, int E, int k_max) {
  extern __shared__ u64 masks[];
  __shared__ int32_t wave_tot[SMALL_THREADS / 64];
  dispatch_one_workgroup<false, SMALL_THREADS>(ids, a, hdr, masks, wave_tot, T, E, k_max);
}

hipError_t launch_dispatch_small(const int32_t* ids, int32_t* cnt, int32_t* off, int32_t* hdr,
                                 int32_t* sorted_pair, int32_t* slot_of_pair, MTile* tiles,
                                 int max_tiles, TileCut cut, int T, int E, int k_max, hipStream_t s) {
  const bool few = T * k_max <= 256 && E <= 512;
  (few ? dispatch_small_kernel<256> : dispatch_small_kernel<1024>)<<<1, few ? 256 : 1024, small_dispatch_lds(T, E), s>>>(
      ids, SmallDispatch{cnt, off, sorted_pair, slot_of_pair, tiles, max_tiles, cut}, hdr, T, E, k_max);
  return hipGetLastError();
}

bool dispatch_is_small(int T, int E, int k_max) { return small_dispatch(T, E, k_max); }

hipError_t launch_dispatch_count(const int32_t* ids, int32_t* chunk_cnt, int T, int E, int k_max,
                                 hipStream_t s) {
  if (T == 0) return hipSuccess;
  int W = dispatch_chunk_words(E, T);
  int nch = cdiv(T, 64 * W);
  dispatch_count_kernel<<<nch, DISPATCH_THREADS, (size_t)E * W * 8, s>>>(ids, chunk_cnt, T, E, W, k_max);
  return hipGetLastError();
}

hipError_t launch_dispatch_scan(int32_t* chunk_cnt, int32_t* cnt, int T, int E, hipStream_t s) {
  int W = dispatch_chunk_words(E, T);
  int nch = cdiv(T, 64 * W);
  dispatch_scan_kernel<<<cdiv(E, SCAN_GROUPS), SCAN_THREADS, 0, s>>>(chunk_cnt, cnt, nch, E);
  return hipGetLastError();
}

hipError_t launch_dispatch_place(const int32_t* ids, const int32_t* chunk_base, int32_t* cnt,
                                 int32_t* off, int32_t* hdr, int32_t* sorted_pair,
                                 int32_t* slot_of_pair, MTile* tiles, int max_tiles, TileCut cut, int T,
                                 int E, int k_max, bool sum, hipStream_t s) {
  int W = dispatch_chunk_words(E, T);
  int nch = cdiv(T, 64 * W);
  if (nch < 1) nch = 1;  // T == 0: one workgroup still writes the (all-zero) offsets
  const size_t lds = (size_t)E * W * 8 + 2 * ((size_t)E + 1) * 4;
  if (sum) {  // E <= 1024 where W is 1, E <= 64 where it is more: 24 KiB and 8 bytes at most
    dispatch_place_kernel<true><<<nch, DISPATCH_THREADS, lds + (size_t)E * 8, s>>>(
        ids, chunk_base, cnt, off, hdr, sorted_pair, slot_of_pair, tiles, max_tiles, cut, T, E, W, k_max);
    return hipGetLastError();
  }
  // up to 96 KiB + 8 bytes (E = 4096, W = 2): beyond the default limit for dynamic LDS
  hipError_t e = raise_lds_limit<dispatch_place_kernel<false>>(100 * 1024);
  if (e != hipSuccess) return e;
  dispatch_place_kernel<false><<<nch, DISPATCH_THREADS, lds, s>>>(
      ids, chunk_base, cnt, off, hdr, sorted_pair, slot_of_pair, tiles, max_tiles, cut, T, E, W, k_max);
  return hipGetLastError();
}

}  // namespace mp
