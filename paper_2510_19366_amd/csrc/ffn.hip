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
#include "ffn_common.h"

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
                                                                  int max_tiles, int even, int n_rows) {
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
    const int nt = (n + FFN_BM - 1) / FFN_BM;
    int round_total = 0;
    const int first = carry + block_scan(nt, wave_tot, &round_total);
    const int per = mtile_rows(n, FFN_BM, even != 0);
    for (int i = 0; i < nt; ++i) {
      MTile t;
      t.g = g;
      t.row0 = lo + i * per;
      t.rows = min(per, n - i * per);
      t.first = first;
      t.count = min(nt, max_tiles - first);  // never points past the table
      t.pad[0] = t.pad[1] = t.pad[2] = 0;
      if (first + i < max_tiles) tiles[first + i] = t;
    }
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
                            bool even_tiles, int n_rows, hipStream_t s) {
  ffn_tiles_kernel<<<1, TILES_THREADS, 0, s>>>(off, tiles, hdr, E, max_tiles, even_tiles, n_rows);
  return hipGetLastError();
}

// ---------------------------------------------------------------- fp32
// Both GEMMs as fp32 chains on the matrix cores (chain_tile.h).  fp32 layers are small (reference
// runs of a few dozen to a few thousand tokens), so the tile is small too: 32 slot rows x 64 weight
// rows, 4 waves of 16 x 32, K in slabs of 32.  An m-tile of the table (FFN_BM = 256 rows) is up to
// eight such row blocks.  Between HIP events, against 128 x 128 tiles of v_fma_f32 (whose
// workgroups left the chip idle): 64 tokens, d = 256, 32 sub-experts of 128, gate-up 66.3 -> 8.9 us, down 35.6 -> 6.4;
// 4096 tokens, d = 1024, 32 of 256, 8 picks: both 1274 -> 576.
constexpr int F32_ROWS = 32, F32_COLS = 64, F32_BLOCKS = FFN_BM / F32_ROWS;
typedef ChainTile<float, 2, 2, 1, 2, 5> F32Tile;

// Copies of one tile: row `row` of the stage starts at byte offset off(row) behind the base of its
// operand (slot rows first).  WIDE: an operand of 4 GiB or more, offsets of 64 bits.
template <bool WIDE, class Rows>
__device__ __forceinline__ void f32_tile(const float* a_base, const float* b_base, int K, Rows&& off,
                                         unsigned char* smem, f32x4_t (&acc)[1][2]) {
  constexpr int CP = F32Tile::CP;
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
  chain_tile<F32Tile>(smem, K / F32Tile::KB, [&](int j, int stage, uint32_t lds) {
    if constexpr (WIDE)
      copy_to_lds16_addr(addr[j] + (uint64_t)stage * 128, lds);
    else
      copy_to_lds16(base[j] + (size_t)stage * 128, voff[j], lds);
  }, acc);
}

// SHORT: see row_blocks.h
template <bool SHORT, class Body>
__device__ __forceinline__ void f32_items(const MTile* __restrict__ tiles, const int32_t* __restrict__ hdr,
                                          int n_tiles_n, int T, Body&& body) {
  auto tile = [&](int m) { return tiles[m]; };
  auto each = [&](const MTile& t, int blk, int nt) {
    body(t.g, t.row0 + blk * F32_ROWS, min(F32_ROWS, t.rows - blk * F32_ROWS), nt);
    __syncthreads();  // every wave has read the last stage before the ring is filled again
  };
  if constexpr (SHORT)
    short_row_blocks<F32_ROWS>(blockIdx.x, gridDim.x, N_XCD, hdr[HDR_MTILES], n_tiles_n,
                               (T + F32_ROWS - 1) / F32_ROWS, tile, [](auto&& pred) { return lane_mask(pred); },
                               each);
  else
    all_row_blocks<F32_ROWS, F32_BLOCKS>(blockIdx.x, gridDim.x, N_XCD, hdr[HDR_MTILES], n_tiles_n, tile, each);
}

// Weight rows of a tile: per wave column 16 neurons' gate rows, then their up rows.
template <bool WIDE, bool SHORT>
__global__ __launch_bounds__(256) void ffn_gate_up_f32_kernel(
    const float* __restrict__ x, const float* __restrict__ w_gu,
    const int32_t* __restrict__ sorted_pair, const MTile* __restrict__ tiles,
    const int32_t* __restrict__ hdr, float* __restrict__ h, int d, int Is, int k_max, int T) {
  extern __shared__ __align__(16) unsigned char f_smem[];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, wm = wv >> 1, wn = wv & 1;
  f32_items<SHORT>(tiles, hdr, Is / 32, T, [&](int g, int row0, int rows, int nt) {  // Is % 32 == 0
    f32x4_t acc[1][2];
    f32_tile<WIDE>(x, w_gu + (size_t)g * 2 * Is * d, d, [&](int row) -> size_t {
      if (row < F32_ROWS) return min(max(sorted_pair[row0 + min(row, rows - 1)] / k_max, 0), T - 1);
      const int b = row - F32_ROWS;
      return ((b >> 4) & 1 ? Is : 0) + nt * 32 + (b >> 5) * 16 + (b & 15);
    }, f_smem, acc);
    const int col = nt * 32 + wn * 16 + (lane & 15);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = wm * 16 + 4 * (lane >> 4) + v;
      const float a = acc[0][0][v], u = acc[0][1][v];
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
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, wm = wv >> 1, wn = wv & 1;
  f32_items<SHORT>(tiles, hdr, d / F32_COLS, T, [&](int g, int row0, int rows, int nt) {  // d % 64 == 0
    f32x4_t acc[1][2];
    f32_tile<WIDE>(h + (size_t)row0 * Is, w_dn + (size_t)g * d * Is, Is, [&](int row) -> size_t {
      return row < F32_ROWS ? min(row, rows - 1) : nt * F32_COLS + row - F32_ROWS;
    }, f_smem, acc);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = wm * 16 + 4 * (lane >> 4) + v, col = nt * F32_COLS + (wn * 2 + j) * 16 + (lane & 15);
        if (row < rows) y[(size_t)(row0 + row) * d + col] = acc[0][j][v];
      }
  });
}

// ---------------------------------------------------------------- launchers
// A token picks a sub-expert at most once, so a group of a dispatched batch has at most T rows: two row blocks (a
// caller's own tables may hold more, which then take longer).  Both GEMMs between HIP events, 16 | 64 tokens, 32
// sub-experts of 256, 8 picks, d = 1024: 30.5 | 30.6 us, with the list of all row blocks 77 | 77; 64 tokens of the
// tiny layer 15.5 | 27.8.
static bool f32_short(int T) { return T <= 2 * F32_ROWS; }

hipError_t launch_ffn_gate_up(int dtype, const void* x, const void* w_gu, const int32_t* sorted_pair,
                              const MTile* tiles, int32_t* hdr, void* h, int T, int d, int Is,
                              int k_max, int few, int max_mtiles, hipStream_t s) {
  if (max_mtiles <= 0) return hipSuccess;
  if (dtype != 0)
    return launch_gate_up_bf16((const uint16_t*)x, (const uint16_t*)w_gu, sorted_pair, tiles, hdr,
                               (uint16_t*)h, T, d, Is, k_max, few, max_mtiles, s);
  const int grid = persistent_grid((long)max_mtiles * F32_BLOCKS * (Is / 32), 2);
  const bool wide = (long)T * d >= (1L << 30) || (long)Is * d >= (1L << 29);
  auto* kern = f32_short(T) ? (wide ? ffn_gate_up_f32_kernel<true, true> : ffn_gate_up_f32_kernel<false, true>)
                            : (wide ? ffn_gate_up_f32_kernel<true, false> : ffn_gate_up_f32_kernel<false, false>);
  kern<<<grid, 256, F32Tile::LDS_BYTES, s>>>((const float*)x, (const float*)w_gu, sorted_pair, tiles, hdr, (float*)h,
                                             d, Is, k_max, T);
  return hipGetLastError();
}

hipError_t launch_ffn_down(int dtype, const void* h, const void* w_dn, const MTile* tiles,
                           int32_t* hdr, void* y, int T, int d, int Is, int few, int max_mtiles,
                           hipStream_t s) {
  if (max_mtiles <= 0) return hipSuccess;
  if (dtype != 0)
    return launch_down_bf16((const uint16_t*)h, (const uint16_t*)w_dn, tiles, hdr, (uint16_t*)y, T, d,
                            Is, few, max_mtiles, s);
  const int grid = persistent_grid((long)max_mtiles * F32_BLOCKS * (d / F32_COLS), 2);
  const bool wide = (long)Is * d >= (1L << 30);
  auto* kern = f32_short(T) ? (wide ? ffn_down_f32_kernel<true, true> : ffn_down_f32_kernel<false, true>)
                            : (wide ? ffn_down_f32_kernel<true, false> : ffn_down_f32_kernel<false, false>);
  kern<<<grid, 256, F32Tile::LDS_BYTES, s>>>((const float*)h, (const float*)w_dn, tiles, hdr, (float*)y, T, d, Is);
  return hipGetLastError();
}

}  // namespace mp
