// Internal launcher interface between the C ABI (api.hip) and the kernel files.
// gfx950 only.  Every launcher enqueues on `s` and returns hipGetLastError().
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "row_blocks.h"

namespace mp {

// Workspace header: int32 words at the start of ws.
// HDR_DYN_*: cursors of the FFN kernels' work pools (cleared with the m-tile table)
// HDR_TOPK_DONE: workgroups of the top-k kernel that have written their picks (cleared by the logits kernel)
// HDR_DYN_FUSED .. +7: the fused FFN kernel's per-XCD tile cursors
enum { HDR_FLAGS = 0, HDR_PAIRS = 1, HDR_MTILES = 2, HDR_DYN_GATE_UP = 3, HDR_DYN_DOWN = 4, HDR_TOPK_DONE = 5, HDR_DYN_FUSED = 8, HDR_WORDS = 64 };

constexpr int FFN_BM = 256;  // rows of one m-tile of the grouped GEMMs

struct MTile {  // one m-tile of a group: rows [row0, row0 + rows) of the slot list
  int32_t g, row0, rows;
  int32_t first;  // table index of the group's first m-tile
  int32_t count;  // m-tiles of the group
  int32_t pad[3];
};
// ... and one of at most 64 rows (ffn_few_kernel): half of the bytes, so that the table of tiles of 256 rows,
// rows / 256 + E entries, holds 2 E of them
struct FewTile {
  int32_t g, row0, rows_count, first;  // rows | m-tiles of the group << 8
};
static_assert(2 * sizeof(FewTile) == sizeof(MTile));
// m-tile `i` into the table: FewTiles where the cut is below FFN_BM
__device__ __forceinline__ void put_tile(MTile* tiles, const TileCut& cut, int i, int g, int row0, int rows, int first, int count) {
  if ((1 << cut.log2) < FFN_BM) reinterpret_cast<FewTile*>(tiles)[i] = FewTile{g, row0, rows | count << 8, first};
  else tiles[i] = MTile{g, row0, rows, first, count, {0, 0, 0}};
}

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

hipError_t launch_expand_k(int R, int T, const int32_t* req_k, const int32_t* req_off,
                           int32_t* k_tok, hipStream_t s);

// S: sub-experts of an expert, whose rows of w may be equal; differ: scratch of E / S words (not used with S = 1)
hipError_t launch_logits(int dtype, const void* x, const void* w, const float* bias, float* logits,
                         int32_t* hdr, int T, int d, int E, int S, int32_t* differ, hipStream_t s);
// with `small` (only where topk_dispatches): the kernel also dispatches its picks
bool topk_dispatches(int T, int E, int k_max);
struct MTile;
struct SmallDispatch;
hipError_t launch_topk(const float* logits, const int32_t* k_tok, int32_t* ids, float* w,
                       int32_t* hdr, int T, int E, int k_max, int renorm, float scale,
                       const SmallDispatch* small, hipStream_t s);

// dispatch: chunk_cnt is [n_chunks, E] scratch
int dispatch_chunk_words(int E, int T);          // 64-token words per chunk
hipError_t launch_dispatch_count(const int32_t* ids, int32_t* chunk_cnt, int T, int E, int k_max,
                                 hipStream_t s);
// proxy gate (Sec. 3.2.2): per-expert top-kappa on the gate-neuron activations
constexpr int PROXY_MAX_SUB = 16;
hipError_t launch_proxy_select(int dtype, const void* act, int act_ld, const int32_t* ids0,
                               const float* w0, const int32_t* slot0, const int32_t* k_tok,
                               const int32_t* kappa, int32_t* ids, float* w, int32_t* hdr, int T,
                               int S, int r, int m, int k_max, hipStream_t s);
// few counts: no scan, the place kernel adds them up (its `sum`)
bool dispatch_sums(int T, int E);
hipError_t launch_dispatch_scan(int32_t* chunk_cnt, int32_t* cnt, int T, int E, hipStream_t s);
bool dispatch_is_small(int T, int E, int k_max);  // the whole stage in one workgroup (launch_dispatch_small)
hipError_t launch_dispatch_small(const int32_t* ids, int32_t* cnt, int32_t* off, int32_t* hdr,
                                 int32_t* sorted_pair, int32_t* slot_of_pair, MTile* tiles,
                                 int max_tiles, TileCut cut, int T, int E, int k_max, hipStream_t s);
// also writes off[0..E] and hdr[HDR_PAIRS] (from cnt[]) and, with tiles != nullptr, the grouped
// FFN's m-tile table and its header words (what launch_ffn_tiles builds from off[])
hipError_t launch_dispatch_place(const int32_t* ids, const int32_t* chunk_base, int32_t* cnt,
                                 int32_t* off, int32_t* hdr, int32_t* sorted_pair,
                                 int32_t* slot_of_pair, MTile* tiles, int max_tiles, TileCut cut, int T,
                                 int E, int k_max, bool sum, hipStream_t s);

// grouped FFN
hipError_t launch_ffn_tiles(const int32_t* off, MTile* tiles, int32_t* hdr, int E, int max_tiles,
                            TileCut cut, int n_rows, hipStream_t s);
hipError_t launch_ffn_gate_up(int dtype, const void* x, const void* w_gu, const int32_t* sorted_pair,
                              const MTile* tiles, int32_t* hdr, void* h, int T, int d, int Is,
                              int k_max, int few, int max_mtiles, hipStream_t s);
hipError_t launch_ffn_down(int dtype, const void* h, const void* w_dn, const MTile* tiles,
                           int32_t* hdr, void* y, int T, int d, int Is, int few, int max_mtiles,
                           hipStream_t s);
// bf16: so few rows per sub-expert that the tiles of ffn_few_kernel are the faster ones: their blocks of 16 slot rows, or
// 0.  fused: the fused kernel would run instead
int ffn_few_blocks(int T, int k_max, int E, int d, int Is, bool fused);
// the gate-up of a few tokens that picks and dispatches for itself, in place of the top-k kernel (layer calls; few: of ffn_few_blocks
// or ffn_f32_list)
struct PickArgs;
bool ffn_picks(int dtype, int few, int T, int k_max, int E, int d, int Is);
hipError_t launch_ffn_pick_gate_up(int dtype, const PickArgs& p, const void* x, const void* w_gu, void* h, int T, int d, int Is,
                                   int k_max, int few, hipStream_t s);
// the down projection of the few-rows tiles and the combine in one kernel (layer calls; few: of ffn_few_blocks)
bool ffn_down_combines(int few, int T, int k_max, int E, int d, int Is);
hipError_t launch_ffn_down_combine(const uint16_t* h, const uint16_t* w_dn, const MTile* tiles, const int32_t* hdr,
                                   int max_tiles, const int32_t* slot_of_pair, const float* w, const int32_t* k_tok,
                                   uint16_t* y, uint16_t* out, int T, int d, int Is, int k_max, hipStream_t s);
// fp32: the list of row blocks and the tile (`few` of the launchers)
int ffn_f32_list(int T, int k_max, int E, int d, int Is);

// fused gate-up -> SwiGLU -> down for narrow sub-experts (bf16); see ffn_fused_bf16.hip
bool ffn_fused_supported(int T, int d, int Is);
// sorted: tables of up to so many tiles have the long ones first (TileCut)
hipError_t launch_ffn_fused_bf16(const uint16_t* x, const uint16_t* w_gu, const uint16_t* w_dn,
                                 const int32_t* sorted_pair, const MTile* tiles, int32_t* hdr,
                                 uint16_t* y, int T, int d, int Is, int k_max, int max_mtiles,
                                 int sorted, hipStream_t s);
// the same kernel without the matrix products (measurement: its memory traffic alone)
hipError_t launch_ffn_fused_traffic_bf16(const uint16_t* x, const uint16_t* w_gu,
                                         const uint16_t* w_dn, const int32_t* sorted_pair,
                                         const MTile* tiles, int32_t* hdr, uint16_t* y, int T,
                                         int d, int Is, int k_max, int max_mtiles, hipStream_t s);

hipError_t launch_combine(int dtype, const void* y, const int32_t* slot_of_pair, const float* w,
                          const int32_t* k_tok, void* out, int T, int d, int k_max, hipStream_t s);

int num_cus();  // compute units of the current device (cached)

// Kernels that need more than the default 64 KiB of dynamic LDS (the CU has 160 KiB): the
// attribute is set once per kernel and device, so the launch path makes no other runtime call
// (which also keeps it usable while the caller's stream is being captured into a graph, after one
// eager call).
template <auto Kern>
inline hipError_t raise_lds_limit(size_t bytes) {
  static bool done[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = -1;
  if (dev >= 0 && done[dev]) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(Kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess && dev >= 0) done[dev] = true;
  return e;
}

// bf16 helpers (bit patterns in uint16_t)
__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(((uint32_t)b) << 16);
}
// two fp32 -> two bf16 (round to nearest even) in one word, a in the low half: v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f32x2_t;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
  const f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

}  // namespace mp
