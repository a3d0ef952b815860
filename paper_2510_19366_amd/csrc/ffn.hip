// Grouped SwiGLU FFN over ragged per-sub-expert groups (Sec. 3.2.1, Eq. 1-3).
//
// The slot list is cut into m-tiles of up to FFN_BM rows that never straddle a
// group (ffn_tiles_kernel, on the device, from group_offset), and persistent
// workgroups walk (m-tile, n-tile) work items round-robin.  Two GEMMs:
//   gate-up : h[p, c] = SiLU(x[t_p,:] . Wg[g,c,:]) * (x[t_p,:] . Wu[g,c,:])
//   down    : y[p, q] = sum_c h[p,c] * Wd[g,q,c]
// This file: the m-tile table and the fp32 path.  The bf16 kernels are in ffn_bf16.hip and
// ffn_fused_bf16.hip.
#include "chain_tile.h"
#include "dispatch_common.h"
#include "ffn_common.h"
#include "topk_wave.h"

namespace mp {

// ---------------------------------------------------------------- m-tile table
constexpr int TILES_THREADS = 1024;

// block-wide exclusive scan of one int per thread; returns the thread's prefix, *total the sum
__device__ __forceinline__ int block_scan(int v, int32_t* wave_tot, int* total) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int incl = v;
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    int o = __shfl_up(incl, m, 64);
    if (lane >= m) incl += o;
  }
  __syncthreads();  // wave_tot may still be read from the previous call
  if (lane == 63) wave_tot[wv] = incl;
  __syncthreads();
  int wbase = 0, tot = 0;
  for (int i = 0; i < TILES_THREADS / 64; ++i) {
    if (i < wv) wbase += wave_tot[i];
    tot += wave_tot[i];
  }
  *total = tot;
  return wbase + incl - v;
}

// tiles[]: the m-tiles in group order (a group's tiles are contiguous)
__global__ __launch_bounds__(TILES_THREADS) void ffn_tiles_kernel(const int32_t* __restrict__ off,
                                                                  MTile* __restrict__ tiles,
                                                                  int32_t* __restrict__ hdr, int E,
                                                                  int max_tiles, TileCut cut, int n_rows) {
  __shared__ int32_t wave_tot[TILES_THREADS / 64];
  const int tid = threadIdx.x;
  int carry = 0;  // tiles of the groups before this round (the same in every thread)
  for (int g0 = 0; g0 < E; g0 += TILES_THREADS) {
    int g = g0 + tid;
    int lo = 0, n = 0;
    if (g < E) {  // offsets that do not describe a slot list of n_rows rows yield no tiles
      lo = off[g];
      n = off[g + 1] - lo;
      if (lo < 0 || n < 0 || lo > n_rows || n > n_rows - lo) n = 0;
    }
    const int nt = cut.tiles(n);
    int round_total = 0;
    const int first = carry + block_scan(nt, wave_tot, &round_total);
    const int per = cut.rows(n), count = min(nt, max_tiles - first);  // never points past the table
#pragma unroll 4
    for (int i = 0; i < count; ++i) put_tile(tiles, cut, first + i, g, lo + i * per, min(per, n - i * per), first, count);
    carry += round_total;
  }
  const int n_tiles = min(carry, max_tiles);
  if (tid == 0) {
    hdr[HDR_MTILES] = n_tiles;
    hdr[HDR_DYN_GATE_UP] = 0;
    hdr[HDR_DYN_DOWN] = 0;
    for (int i = 0; i < N_XCD; ++i) hdr[HDR_DYN_FUSED + i] = 0;
    // more tiles than the table holds: only possible when a caller hands offsets that do not
    // belong to this shape's pair capacity; never silent
    if (carry > max_tiles) atomicOr(&hdr[HDR_FLAGS], 2);
  }
}

hipError_t launch_ffn_tiles(const int32_t* off, MTile* tiles, int32_t* hdr, int E, int max_tiles,
                            TileCut cut, int n_rows, hipStream_t s) {
  ffn_tiles_kernel<<<1, TILES_THREADS, 0, s>>>(off, tiles, hdr, E, max_tiles, cut, n_rows);
  return hipGetLastError();
}

// ---------------------------------------------------------------- fp32
// Both GEMMs as fp32 chains on the matrix cores (chain_tile.h).  fp32 layers are small (reference
// runs of a few dozen to a few thousand tokens), so the tile is small too: 32 slot rows x 64 weight
// rows, 4 waves of 16 x 32, K in slabs of 32.  An m-tile of the table (FFN_BM = 256 rows) is up to
// eight such row blocks.  Between HIP events, against 128 x 128 tiles of v_fma_f32 (whose
// workgroups left the chip idle): 64 tokens, d = 256, 32 sub-experts of 128, gate-up 66.3 -> 8.9 us, down 35.6 -> 6.4;
// 4096 tokens, d = 1024, 32 of 256, 8 picks: both 1274 -> 576.
constexpr int F32_ROWS = 32, F32_BLOCKS = FFN_BM / F32_ROWS;
template <int NT>
using F32Tile = ChainTile<float, 2, 2, 1, NT, NT == 2 ? 5 : 4>;
// Workgroups per CU: all resident, so that a batch of no more tiles than these is one round.
template <int NT>
constexpr int F32_PER_CU = NT == 1 ? 4 : 2;
constexpr int F32_UPS_BYTES = 2 * 64 * sizeof(f32x4_t);  // the up rows' sums of NT = 1
static_assert(F32_PER_CU<1> * (F32Tile<1>::LDS_BYTES + F32_UPS_BYTES) <= 160 * 1024 && F32_PER_CU<2> * F32Tile<2>::LDS_BYTES <= 160 * 1024);

// Copies of one tile: row `row` of the stage starts at byte offset off(row) behind the base of its
// operand (slot rows first).  WIDE: an operand of 4 GiB or more, offsets of 64 bits.
template <bool WIDE, int NT, class Rows>
__device__ __forceinline__ void f32_tile(const float* a_base, const float* b_base, int K, Rows&& off,
                                         unsigned char* smem, f32x4_t (&acc)[1][NT]) {
  typedef F32Tile<NT> Tile;
  constexpr int CP = Tile::CP;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned char* base[CP];
  uint32_t voff[CP];
  uint64_t addr[CP];
#pragma unroll
  for (int j = 0; j < CP; ++j) {
    const int r0 = (wv * CP + j) * 8, row = r0 + (lane >> 3);
    base[j] = reinterpret_cast<const unsigned char*>(r0 < F32_ROWS ? a_base : b_base);
    const size_t o = off(row) * (size_t)K * 4 + (size_t)(chain_chunk(row) * 16);
    voff[j] = (uint32_t)o;
    addr[j] = reinterpret_cast<uint64_t>(base[j]) + o;
  }
  chain_tile<Tile>(smem, K / Tile::KB, [&](int j, int stage, uint32_t lds) {
    if constexpr (WIDE)
      copy_to_lds16_addr(addr[j] + (uint64_t)stage * 128, lds);
    else
      copy_to_lds16(base[j] + (size_t)stage * 128, voff[j], lds);
  }, acc);
}

// SHORT: see row_blocks.h.  tile: m-tile number m of n
template <bool SHORT, class Tile, class Body>
__device__ __forceinline__ void f32_items(Tile&& tile, int n, int block, int grid, int n_tiles_n, int T, Body&& body) {
  auto each = [&](const MTile& t, int blk, int nt) {
    body(t.g, t.row0 + blk * F32_ROWS, min(F32_ROWS, t.rows - blk * F32_ROWS), nt);
    __syncthreads();  // every wave has read the last stage before the ring is filled again
  };
  if constexpr (SHORT)
    short_row_blocks<F32_ROWS>(block, grid, N_XCD, n, n_tiles_n,
                               min((T + F32_ROWS - 1) / F32_ROWS, F32_BLOCKS), tile, [](auto&& pred) { return lane_mask(pred); },
                               each);
  else
    all_row_blocks<F32_ROWS, F32_BLOCKS>(block, grid, N_XCD, n, n_tiles_n, tile, each);
}

// PICK (gate-up of up to 64 tokens, E <= 32, k_max picks): the route's picks and their dispatch belong to this launch.  Every
// workgroup finds the picks of all tokens: a lane has a token, a wave eight sub-experts, and a sub-expert is picked if fewer
// logits than the budget are larger, or equal with a lower id.  The first workgroups, a wave per token, only write what the
// route and the dispatch leave in memory.  What it saves is the launch of the top-k kernel, which is longer than the 2 us of a
// latency and 31 comparisons for each of eight sub-experts.  Layer calls of d = 256, 32 of 128, from a captured graph, top-k kernel |
// this: 16 tokens 20.1 | 19.0 us, 32 21.9 | 19.7, 64 22.2 | 20.4; back to back, d = 1024, 32 of 256, 30 tokens 43.9 | 41.9, 60 43.9 | 42.4;
// d = 2048, 32 of 704, 60 tokens 140.9 | 134.8.
// (A lane has a token and its logits in registers, so 64 tokens, and 32 sub-experts, whose comparisons go with the square.)
constexpr int PICK_T = 64, PICK_E = 32;
struct F32Picks {
  u64 masks[PICK_E];  // tokens that picked a sub-expert
  int32_t row0[PICK_E];
  MTile tiles[PICK_E];
  uint8_t tokens[PICK_T * PICK_E];  // of the slot rows
};
// keys: PICK_T x (PICK_E + 1) words.  Returns the number of m-tiles; *rows: of slot rows.
__device__ __forceinline__ int f32_find_picks(const PickArgs& a, F32Picks& s, int* keys, int T, int k_max, int* rows) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int EACH = PICK_E / 4, LD = PICK_T / 8;  // sub-experts of a wave; logits of a thread
  const int asked = a.k_tok[min(lane, T - 1)];
  auto token = [&](int q) { return wv * (PICK_T / 4) + q * 2 + (lane >> 5); };
  float v[LD];
#pragma unroll
  for (int q = 0; q < LD; ++q) v[q] = a.logits[min(token(q), T - 1) * a.E + min(lane & 31, a.E - 1)];
#pragma unroll
  for (int q = 0; q < LD; ++q)  // absent ones are behind all others
    keys[token(q) * (PICK_E + 1) + (lane & 31)] = (lane & 31) < a.E ? topk_key(v[q]) : INT32_MIN;
  __syncthreads();
  const int kt = lane < T ? min(max(asked, 0), k_max) : 0;
  int key[PICK_E];  // of this lane's token, this wave's sub-experts first
#pragma unroll
  for (int j = 0; j < PICK_E; ++j) key[j] = keys[lane * (PICK_E + 1) + ((wv * EACH + j) & (PICK_E - 1))];
#pragma unroll
  for (int q = 0; q < EACH; ++q) {
    int larger = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int least = key[q] - (b > 0 && wv + b >= 4 ? 1 : 0);  // the ids of the blocks that wrap around are lower
#pragma unroll
      for (int j = b * EACH; j < (b + 1) * EACH; ++j) larger += b == 0 && j < q ? key[j] >= key[q] : key[j] > least;
    }
    const u64 m = __ballot(wv * EACH + q < a.E && larger < kt);
    if (lane == 0) s.masks[wv * EACH + q] = m;
  }
  __syncthreads();
  const int n = lane < PICK_E ? (int)__popcll(s.masks[lane]) : 0, incl = wave_scan(n), row0 = incl - n;
  const u64 some = __ballot(n > 0);
  if (wv == 0 && lane < PICK_E) s.row0[lane] = row0;
  if (wv == 1 && n > 0) {
    const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0));
    s.tiles[at] = MTile{lane, row0, n, at, 1, {0, 0, 0}};
  }
#pragma unroll
  for (int q = 0; q < EACH; ++q) {
    const int e = wv * EACH + q;
    const u64 m = s.masks[e];
    const int at = __builtin_amdgcn_readlane(row0, e) +
                   __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
    if (m >> lane & 1) s.tokens[at] = (uint8_t)lane;
  }
  __syncthreads();
  *rows = __builtin_amdgcn_readlane(incl, 63);
  return __popcll(some);
}
// workgroups that write: four tokens each, a whole number for each XCD
__host__ __device__ constexpr int pick_writers(int T) { return ((T + 3) / 4 + N_XCD - 1) / N_XCD * N_XCD; }
// what the top-k kernel leaves in memory: of token t, by a wave; the tables by the first workgroup
__device__ __forceinline__ void f32_write_picks(const PickArgs& a, const F32Picks& s, int* scratch, int T, int k_max, int rows, int n_tiles) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, t = blockIdx.x * 4 + wv;
  if (blockIdx.x == 0) {
    if ((int)threadIdx.x < a.E) {
      a.small.off[threadIdx.x] = s.row0[threadIdx.x];
      a.small.cnt[threadIdx.x] = __popcll(s.masks[threadIdx.x]);
    }
    if ((int)threadIdx.x < n_tiles) a.small.tiles[threadIdx.x] = s.tiles[threadIdx.x];
    if (threadIdx.x == 0) {
      a.small.off[a.E] = rows;
      write_counts(a.hdr, rows, n_tiles, true, a.small.max_tiles);
    }
  }
  if (t >= T) return;
  const int kp = topk_pad(k_max);
  int* uk = scratch + wv * 4 * kp;  // as in the top-k kernel
  float* se = reinterpret_cast<float*>(uk + 2 * kp);
  int* sid = uk + 3 * kp;
  const TopkPicks p = topk_token<1>(a.logits + (size_t)t * a.E, a.k_tok[t], a.E, k_max, a.renorm, &a.hdr[HDR_FLAGS], uk, uk + kp, se, sid);
  for (int j = lane; j < k_max; j += 64) {
    const int i = t * k_max + j;
    const bool on = j < p.kt;
    const int g = on ? sid[j] : -1;
    int slot = -1;
    if (on) {
      slot = s.row0[g] + __popcll(s.masks[g] & ((1ull << t) - 1ull));
      a.small.sorted_pair[slot] = i;
    }
    if (i >= rows) a.small.sorted_pair[i] = -1;  // tail beyond the valid slots
    a.small.slot_of_pair[i] = slot;
    a.ids[i] = g;
    a.w[i] = on ? a.scale * expf(se[j] - p.most) / p.denom : 0.0f;
  }
}

// NT = 2: a wave has 16 neurons' gate rows and the same neurons' up rows.  NT = 1: half of the chain per wave; the second
// wave of a row has the up rows, and hands its sums over through LDS.
template <bool WIDE, bool SHORT, int NT, class... Pick>
__global__ __launch_bounds__(256) void ffn_gate_up_f32_kernel(
    const float* __restrict__ x, const float* __restrict__ w_gu,
    const int32_t* __restrict__ sorted_pair, const MTile* __restrict__ tiles,
    const int32_t* __restrict__ hdr, float* __restrict__ h, int d, int Is, int k_max, int T, Pick... pick) {
  constexpr bool PICK = sizeof...(Pick) > 0;
  static_assert(!PICK || (SHORT && !WIDE));
  extern __shared__ __align__(16) unsigned char f_smem[];
  __shared__ std::conditional_t<PICK, F32Picks, int> picks;
  __shared__ f32x4_t ups[NT == 1 ? F32_UPS_BYTES / sizeof(f32x4_t) : 1];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, wm = wv >> 1, wn = wv & 1;
  int n_m_tiles, first = 0;  // the first workgroup with items
  if constexpr (PICK) {
    const PickArgs& a = (pick, ...);
    int n_rows;
    n_m_tiles = f32_find_picks(a, picks, reinterpret_cast<int*>(f_smem), T, k_max, &n_rows);
    first = pick_writers(T);
    if ((int)blockIdx.x < first) {
      f32_write_picks(a, picks, reinterpret_cast<int*>(f_smem), T, k_max, n_rows, n_m_tiles);
      return;
    }
  } else {
    n_m_tiles = hdr[HDR_MTILES];
  }
  auto tile = [&](int m) {
    if constexpr (PICK) return picks.tiles[m];
    else return tiles[m];
  };
  f32_items<SHORT>(tile, n_m_tiles, blockIdx.x - first, gridDim.x - first, Is / (16 * NT), T, [&](int g, int row0, int rows, int nt) {  // Is % 32 == 0
    f32x4_t acc[1][NT];
    f32_tile<WIDE, NT>(x, w_gu + (size_t)g * 2 * Is * d, d, [&](int row) -> size_t {
      if constexpr (PICK) {
        if (row < F32_ROWS) return picks.tokens[row0 + min(row, rows - 1)];
      } else {
        if (row < F32_ROWS) return min(max(sorted_pair[row0 + min(row, rows - 1)] / k_max, 0), T - 1);
      }
      const int b = row - F32_ROWS;
      return ((b >> 4) & 1 ? Is : 0) + nt * (16 * NT) + (b >> 5) * 16 + (b & 15);
    }, f_smem, acc);
    f32x4_t up = acc[0][NT - 1];
    if constexpr (NT == 1) {
      if (wn == 1) ups[wm * 64 + lane] = acc[0][0];
      __syncthreads();
      if (wn == 1) return;
      up = ups[wm * 64 + lane];
    }
    const int col = nt * (16 * NT) + (NT == 2 ? wn * 16 : 0) + (lane & 15);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = wm * 16 + 4 * (lane >> 4) + v;
      const float a = acc[0][0][v], u = up[v];
      if (row < rows) h[(size_t)(row0 + row) * Is + col] = a / (1.0f + expf(-a)) * u;
    }
  });
}

template <bool WIDE, bool SHORT>
__global__ __launch_bounds__(256) void ffn_down_f32_kernel(const float* __restrict__ h,
                                                           const float* __restrict__ w_dn,
                                                           const MTile* __restrict__ tiles,
                                                           const int32_t* __restrict__ hdr,
                                                           float* __restrict__ y, int T, int d, int Is) {
  extern __shared__ __align__(16) unsigned char f_smem[];
  constexpr int NT = 2, COLS = F32Tile<NT>::BE;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, wm = wv >> 1, wn = wv & 1;
  auto tile = [&](int m) { return tiles[m]; };
  f32_items<SHORT>(tile, hdr[HDR_MTILES], blockIdx.x, gridDim.x, d / COLS, T, [&](int g, int row0, int rows, int nt) {  // d % 64 == 0
    f32x4_t acc[1][NT];
    f32_tile<WIDE, NT>(h + (size_t)row0 * Is, w_dn + (size_t)g * d * Is, Is, [&](int row) -> size_t {
      return row < F32_ROWS ? min(row, rows - 1) : nt * COLS + row - F32_ROWS;
    }, f_smem, acc);
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = wm * 16 + 4 * (lane >> 4) + v, col = nt * COLS + (wn * NT + j) * 16 + (lane & 15);
        if (row < rows) y[(size_t)(row0 + row) * d + col] = acc[0][j][v];
      }
  });
}

// ---------------------------------------------------------------- launchers
// Which list of row blocks (row_blocks.h) and tile the fp32 kernels take: 0 the list of all row blocks, else the list of
// first blocks, then second, with gate-up tiles of 1 or 2 column blocks per wave.
// The list of all eight possible blocks of an m-tile is mostly empty where groups are short, and brings those that exist
// to few workgroups, the more so the fewer n-tiles a GEMM has; but what runs at the same time shares weights.  Both GEMMs
// between HIP events, us, all | first, second: 64 tokens of 8 picks on 32 sub-experts of 128 x 256 15.5 | 15.3, 100 28 | 16, 300
// 29 | 18, 1024 32 | 31; 32 of 256 x 1024: 100 79 | 32, 300 79 | 49, 1000 129 | 113.  Layer calls back to back, 4 picks, weights
// beyond the memory-side cache of 256 MB, by possible rows, even load, then skewed (router bias N(0, 1) per expert):
//   128 of 256 x 1024: 20 314 | 124, 207 | 179; 50 315 | 181, 268 | 277; 62 315 | 196, 267 | 287;  256 of them: 50 623 | 331, 405 |
//     367; 62 623 | 386, 443 | 449;  32 of 256 x 4096: 62 291 | 206, 342 | 302;  128 of 704 x 512: 62 316 | 245, 247 | 254;
//   64 of 512 x 1024: 40 202 | 139, 261 | 255; 62 203 | 187, 280 | 285;  128 of 704 x 1024: 40 386 | 295, 251 | 262; 50 428 | 397; 62 444 | 446,
//     632 | 657;  32 of 1024 x 1024: 40 148 | 140, 191 | 201; 50 165 | 167; 62 172 | 182, 279 | 291;  32 of 704 x 2048: 37 189 | 174,
//     222 | 236; 62 229 | 243, 554 | 567.
// So up to 64 possible rows, 56 where the gate-up has more than 16 n-tiles and the down GEMM 16, 256 where the weights fit that cache (32 of 256 x
// 1024, 8 picks: 250 rows 151 | 136, 182 | 183).
// The list of all blocks wants full m-tiles: 2000 tokens on the last shape (two m-tiles a group) 228, with tiles of even
// length 258; 4000 on 32 of 704 x 2048 975, 1005.  The other list is a little better off with even ones where the
// load is skewed (256 of 256 x 1024, 50 and 62 rows 367 and 449, full 389 and 464; 32 of 256 x 4096 the other way round, 302
// and 287).
// One column block halves a wave's chain where there are CUs to spare: 64 tokens, 32 of 128 x 256, gate-up 8.1 | 9.4, 100
// tokens on 32 of 256 x 1024 17.4 | 19.4; 300 tokens there (768 tiles) 29.9 | 28.3, 16 on 128 of them (640) 29.3 | 27.0.  Four
// workgroups fit a CU, so two tiles of two column blocks per CU are one round.  Both GEMMs, 64 tokens on 32 of d = 256 | 1024 |
// 2048, one column block, two: 320 tiles 18.6, 19.5 | 32.5, 38.2 | 54.9, 64.5; 512 23.3, 24.1 | 41.3, 43.1 | 96.9, 92.5, skewed
// load 25.2, 26.8 | 56.0, 61.8 | 103, 109.  (With a ring of six stages three fit: 512 tiles 26.5 | 46.2 | 99.9.)
int ffn_f32_list(int T, int k_max, int E, int d, int Is) {
  const long pairs = (long)T * k_max, groups = pairs < E ? pairs : E;
  const bool cached = 12.0 * E * d * Is <= 256e6, many_tiles = Is > 16 * 32 && d >= 16 * 64;
  if (T > 2 * F32_ROWS && pairs > (cached ? 256L : many_tiles ? 56L : 64L) * E) return 0;
  return groups * (Is / 32) * cdiv(cdiv(pairs, E), F32_ROWS) <= 2L * num_cus() ? 1 : 2;
}

static bool f32_wide(int T, int d, int Is) { return (long)T * d >= (1L << 30) || (long)Is * d >= (1L << 29); }

hipError_t launch_ffn_gate_up(int dtype, const void* x, const void* w_gu, const int32_t* sorted_pair,
                              const MTile* tiles, int32_t* hdr, void* h, int T, int d, int Is,
                              int k_max, int few, int max_mtiles, hipStream_t s) {
  if (max_mtiles <= 0) return hipSuccess;
  if (dtype != 0)
    return launch_gate_up_bf16((const uint16_t*)x, (const uint16_t*)w_gu, sorted_pair, tiles, hdr,
                               (uint16_t*)h, T, d, Is, k_max, few, max_mtiles, s);
  const bool wide = f32_wide(T, d, Is);
  auto run = [&](auto* kern, int nt) {
    const int grid = persistent_grid((long)max_mtiles * F32_BLOCKS * (Is / (16 * nt)), nt == 1 ? F32_PER_CU<1> : F32_PER_CU<2>);
    const int lds = nt == 1 ? F32Tile<1>::LDS_BYTES : F32Tile<2>::LDS_BYTES;
    kern<<<grid, 256, lds, s>>>((const float*)x, (const float*)w_gu, sorted_pair, tiles, hdr, (float*)h, d, Is, k_max, T);
  };
  if (few == 1) {
    if (wide) run(ffn_gate_up_f32_kernel<true, true, 1>, 1);
    else run(ffn_gate_up_f32_kernel<false, true, 1>, 1);
  } else if (few == 2) {
    if (wide) run(ffn_gate_up_f32_kernel<true, true, 2>, 2);
    else run(ffn_gate_up_f32_kernel<false, true, 2>, 2);
  } else {
    if (wide) run(ffn_gate_up_f32_kernel<true, false, 2>, 2);
    else run(ffn_gate_up_f32_kernel<false, false, 2>, 2);
  }
  return hipGetLastError();
}

hipError_t launch_ffn_down(int dtype, const void* h, const void* w_dn, const MTile* tiles,
                           int32_t* hdr, void* y, int T, int d, int Is, int few, int max_mtiles,
                           hipStream_t s) {
  if (max_mtiles <= 0) return hipSuccess;
  if (dtype != 0)
    return launch_down_bf16((const uint16_t*)h, (const uint16_t*)w_dn, tiles, hdr, (uint16_t*)y, T, d,
                            Is, few, max_mtiles, s);
  const int grid = persistent_grid((long)max_mtiles * F32_BLOCKS * (d / F32Tile<2>::BE), F32_PER_CU<2>);
  const bool wide = (long)Is * d >= (1L << 30);
  auto* kern = few != 0 ? (wide ? ffn_down_f32_kernel<true, true> : ffn_down_f32_kernel<false, true>)
                            : (wide ? ffn_down_f32_kernel<true, false> : ffn_down_f32_kernel<false, false>);
  kern<<<grid, 256, F32Tile<2>::LDS_BYTES, s>>>((const float*)h, (const float*)w_dn, tiles, hdr, (float*)y, T, d, Is);
  return hipGetLastError();
}

// The gate-up's tiles of 16 nt columns: an XCD's share of them (groups x n-tiles) rounded up, as short_row_blocks deals them, for one row block
struct F32PickGrid {
  int nt, cap;  // cap: resident workgroups
  long tiles;
  F32PickGrid(int few, int T, int k_max, int E, int Is) : nt(few == 1 ? 1 : 2), cap(num_cus() * (nt == 1 ? F32_PER_CU<1> : F32_PER_CU<2>)) {
    const long groups = (long)T * k_max < E ? (long)T * k_max : E;
    tiles = (groups * (Is / (16 * nt)) + N_XCD - 1) / N_XCD * N_XCD;
  }
};
// Not where the workgroups that write would push tiles into one more round: layer calls, us, top-k kernel | picking for itself, 8 sub-experts of 1024 x
// 64, 64 tokens of 6 picks 31.9 | 35.5, 16 of them, 40 of 2 28.7 | 31.2.
bool ffn_picks(int dtype, int few, int T, int k_max, int E, int d, int Is) {
  if (dtype != 0) return picks_bf16(few, T, k_max, E);
  if (few == 0 || T < 1 || T > PICK_T || E > PICK_E || f32_wide(T, d, Is)) return false;
  const F32PickGrid g(few, T, k_max, E, Is);
  const long items = g.tiles * cdiv(cdiv((long)T * k_max, E), F32_ROWS);  // of groups of the same length
  return cdiv(items + pick_writers(T), g.cap) == cdiv(items, g.cap);
}

hipError_t launch_ffn_pick_gate_up(int dtype, const PickArgs& p, const void* x, const void* w_gu, void* h, int T, int d, int Is,
                                   int k_max, int few, hipStream_t s) {
  if (dtype != 0)
    return launch_pick_gate_up_bf16(p, (const uint16_t*)x, (const uint16_t*)w_gu, (uint16_t*)h, T, d, Is, k_max, s);
  const F32PickGrid g(few, T, k_max, p.E, Is);
  auto run = [&](auto* kern, int nt) {
    const long all = g.tiles * cdiv(T, F32_ROWS), room = (g.cap - pick_writers(T)) / N_XCD * N_XCD;  // beside those that write
    const int grid = (int)(all < room ? all : room);
    const int lds = nt == 1 ? F32Tile<1>::LDS_BYTES : F32Tile<2>::LDS_BYTES;
    kern<<<grid + pick_writers(T), 256, lds, s>>>((const float*)x, (const float*)w_gu, nullptr, nullptr, nullptr, (float*)h, d, Is, k_max, T, p);
  };
  if (few == 1) run(ffn_gate_up_f32_kernel<false, true, 1, PickArgs>, 1);
  else run(ffn_gate_up_f32_kernel<false, true, 2, PickArgs>, 2);
  return hipGetLastError();
}

}  // namespace mp
