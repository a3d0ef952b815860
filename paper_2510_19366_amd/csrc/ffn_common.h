// Shared by the grouped-FFN kernel files: persistent work distribution.
#pragma once
#include "kernels.h"

namespace mp {

// Persistent work distribution that keeps neighbouring work items on one XCD.
// Workgroups are handed to the 8 XCDs round-robin by workgroup id, and each XCD
// has its own L2.  Workgroup b therefore serves XCD b % 8 and walks a contiguous
// eighth of the item list together with the other workgroups of that XCD, so
// the tiles that share an activation tile or a sub-expert's weights meet in one L2.
constexpr int N_XCD = 8;
struct ItemRange {
  int begin, end, step;
};
__device__ __forceinline__ ItemRange xcd_items(int total, int block, int grid) {
  const int xcd = block % N_XCD, slot = block / N_XCD;
  const int per = grid / N_XCD;  // the grid is a multiple of N_XCD
  const int chunk = (total + N_XCD - 1) / N_XCD;
  ItemRange r;
  r.begin = min(total, xcd * chunk) + slot;
  r.end = min(total, (xcd + 1) * chunk);
  r.step = per;
  return r;
}
__device__ __forceinline__ ItemRange xcd_items(int total) { return xcd_items(total, blockIdx.x, gridDim.x); }

// SiLU(a) * u = a / (1 + e^-a) * u.  v_rcp_f32 and one correction of the quotient by its remainder,
// in a third of the instructions of the IEEE division the compiler emits (which also scales its operands for
// quotients this one cannot have).  With the reciprocal off by an ulp either way, 40 million quotients over
// a in [-20, 20] are all the division's; below 2e-36, a < -87.3, a quotient may come out as zero.  Where a or the denominator is infinite the remainder
// is not a number and the uncorrected quotient is the result.
__device__ __forceinline__ float silu_mul(float a, float u) {
  const float den = 1.0f + __expf(-a), r = __builtin_amdgcn_rcpf(den);
  const float q = a * r, c = fmaf(fmaf(-den, q, a), r, q);
  return (c == c ? c : q) * u;
}

// bit l: pred(l), in every lane
template <class P>
__device__ __forceinline__ uint64_t lane_mask(P&& pred) {
  return __ballot(pred((int)(threadIdx.x & 63)));
}

inline int persistent_grid(long max_items, int per_cu) {  // a multiple of N_XCD
  long g = (long)num_cus() * per_cu;
  if (g > max_items) g = max_items;
  if (g < 1) g = 1;
  return (int)((g + N_XCD - 1) / N_XCD * N_XCD);
}

// bf16 kernels (ffn_bf16.hip); few: see ffn_few_blocks
hipError_t launch_gate_up_bf16(const uint16_t* x, const uint16_t* w_gu, const int32_t* sorted_pair,
                               const MTile* tiles, int32_t* hdr, uint16_t* h, int T, int d,
                               int Is, int k_max, int few, int max_mtiles, hipStream_t s);
hipError_t launch_down_bf16(const uint16_t* h, const uint16_t* w_dn, const MTile* tiles,
                            int32_t* hdr, uint16_t* y, int T, int d, int Is, int few, int max_mtiles,
                            hipStream_t s);

bool picks_bf16(int few, int T, int k_max, int E);
hipError_t launch_pick_gate_up_bf16(const PickArgs& p, const uint16_t* x, const uint16_t* w_gu, uint16_t* h, int T, int d, int Is, int k_max,
                                    hipStream_t s);

}  // namespace mp
