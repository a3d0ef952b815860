// The picks of one token by one wave, shared by the top-k kernel and the gate-up that picks for itself.
#pragma once
#include "kernels.h"
#include "topk_search.h"

namespace mp {

typedef unsigned long long u64;

// Wave-wide reductions that leave the result in every lane: four DPP steps inside each row
// of 16 lanes (lane ^ 1, lane ^ 2, mirror inside 8, mirror inside 16), then the four row
// results are read with v_readlane and combined.  No LDS traffic, unlike shuffles.
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_XOR3 = 0x1B, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140,
              DPP_ROR8 = 0x128;

__device__ __forceinline__ float wave_max_f(float v) {
  v = fmaxf(v, __int_as_float(dpp_i<DPP_XOR1>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_i<DPP_XOR2>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_i<DPP_HALF_MIRROR>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_i<DPP_MIRROR>(__float_as_int(v))));
  const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
  const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
  const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
  const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
  return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}
__device__ __forceinline__ int wave_min_i(int v) {
  v = min(v, dpp_i<DPP_XOR1>(v));
  v = min(v, dpp_i<DPP_XOR2>(v));
  v = min(v, dpp_i<DPP_HALF_MIRROR>(v));
  v = min(v, dpp_i<DPP_MIRROR>(v));
  const int r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
  const int r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
  return min(min(r0, r1), min(r2, r3));
}
// the butterfly over lane ^ 32, 16, 8, 4, 2, 1 (every lane ends with the same sum)
__device__ __forceinline__ float wave_sum(float x) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const auto add = [](u32x2 v) { return __uint_as_float(v.x) + __uint_as_float(v.y); };
  const auto bits = [](float f) { return __float_as_uint(f); };
  x = add(__builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(bits(x), bits(x), false, false)));
  x = add(__builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(bits(x), bits(x), false, false)));
  x += __int_as_float(dpp_i<DPP_ROR8>(__float_as_int(x)));
  x += __int_as_float(dpp_i<DPP_HALF_MIRROR>(dpp_i<DPP_XOR3>(__float_as_int(x))));  // 7 - l, then ^ 3
  x += __int_as_float(dpp_i<DPP_XOR2>(__float_as_int(x)));
  x += __int_as_float(dpp_i<DPP_XOR1>(__float_as_int(x)));
  return x;
}

// Budgets up to this take a maximum per pick, larger ones the search, whose time is mostly the
// compaction and ranking behind it.  16 384 x 512 between HIP events, picks | search: 2 picks 14.7 | 18.2 us,
// 6 picks 20.5 | 20.4, 8 picks 23.7 | 21.3; 16 384 x 2048: 30.5 | 41.6, 44.6 | 47.2, 52.8 | 47.4.  With one element
// per lane a maximum is cheaper: 4096 x 64, 8 picks 7.9 | 8.6, 12 picks 9.1 | 8.6 (16 384 x 64: 15.6 | 14.9).
constexpr int topk_few(int elems) { return elems == 1 ? 8 : 6; }
__host__ __device__ inline int topk_pad(int k_max) { return (k_max + 7) / 8 * 8; }
// a wave's own LDS writes are readable by all its lanes
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

__device__ __forceinline__ int wave_max_i(int v) {
  v = max(v, dpp_i<DPP_XOR1>(v));
  v = max(v, dpp_i<DPP_XOR2>(v));
  v = max(v, dpp_i<DPP_HALF_MIRROR>(v));
  v = max(v, dpp_i<DPP_MIRROR>(v));
  const int r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
  const int r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
  return max(max(r0, r1), max(r2, r3));
}

struct TopkPicks {
  int kt;            // picks: the budget, inside 0 .. k_max
  float most, denom;  // the weight of a pick is scale expf(logit - most) / denom
};
// Lane l holds logits g = 64 i + l of `row`.  Leaves logits and ids of the picks in pick order in se and sid; uk and uid are scratch,
// all of topk_pad(k_max) words.  flags: of the header, or null where another wave reports this token's budget.
// SET: only which they are, bit l of set[i] for g = 64 i + l (set[] is zero before).
template <int ELEMS, bool SET = false>
__device__ __forceinline__ TopkPicks topk_token(const float* __restrict__ row, int asked, int E, int k_max, int renorm,
                                                int32_t* __restrict__ flags, int* uk, int* uid, float* se, int* sid, u64* set = nullptr) {
  const int lane = threadIdx.x & 63, kp = topk_pad(k_max);
  const float NEG_INF = -__builtin_inff();
  constexpr int GONE = (int)0x80000000;  // key of an element beyond E
  float v[ELEMS];
#pragma unroll
  for (int i = 0; i < ELEMS; ++i) {
    int g = i * 64 + lane;
    v[i] = g < E ? row[g] : NEG_INF;
  }
  // (behind the loads of the logits, so that one memory latency covers both)
  int kt = __builtin_amdgcn_readfirstlane(asked);
  if (kt < 0 || kt > k_max) {
    if (lane == 0 && flags != nullptr) atomicOr(flags, 1);
    kt = kt < 0 ? 0 : k_max;
  }
  // full-softmax denominator (only needed when weights are not renormalised)
  float lmax = NEG_INF;
#pragma unroll
  for (int i = 0; i < ELEMS; ++i) lmax = fmaxf(lmax, v[i]);
  const float mx = wave_max_f(lmax);
  float denom = 0.0f;
  if (!SET && !renorm) {
#pragma unroll
    for (int i = 0; i < ELEMS; ++i)
      if (i * 64 + lane < E) denom += expf(v[i] - mx);
    denom = wave_sum(denom);
  }

  int key[ELEMS];
  int best = GONE;
#pragma unroll
  for (int i = 0; i < ELEMS; ++i) {
    const int k = topk_key(v[i]);  // outside the choice, or it becomes a branch per element
    key[i] = i * 64 + lane < E ? k : GONE;
    best = max(best, key[i]);
  }
  if (kt > 0 && kt <= topk_few(ELEMS)) {
    // One wave-wide maximum per pick: g = 64 i + lane, so inside a lane the lower element index is
    // the lower id, and the winner's lane is g & 63.  Only that lane retires its element.
    constexpr int NONE = 0x7fffffff;
    for (int j = 0; j < kt; ++j) {
      const int top = wave_max_i(best);
      int mine = NONE;  // this lane's first element with that key
      if (best == top) {
#pragma unroll
        for (int i = ELEMS - 1; i >= 0; --i) mine = key[i] == top ? i * 64 + lane : mine;
      }
      const int g = wave_min_i(mine);
      if (lane == 0) {
        if (SET) {
          set[g >> 6] |= 1ull << (g & 63);
        } else {
          se[j] = topk_unkey(top);
          sid[j] = g;
        }
      }
      if (g == mine) {
        best = GONE;
#pragma unroll
        for (int i = 0; i < ELEMS; ++i) {
          key[i] = i * 64 + lane == g ? GONE : key[i];
          best = max(best, key[i]);
        }
      }
    }
    wave_lds_fence();
  } else if (kt > 0) {
    // Lower bound of the border: the best keys of 64 lanes are 64 elements, so for k_t <= 64 the k_t-th
    // largest is at least their minimum.  Fewer picks need fewer such sets of elements: with the best
    // of 2, 4, 8 or 16 neighbouring lanes the bound is tighter (at 2 picks 2.6 steps instead of 4.5).
    // Twice as many sets as picks are kept: where the bound is the border itself the search is long.
    int low = best;
    if (kt <= 16) low = max(low, dpp_i<DPP_XOR1>(low));
    if (kt <= 8) low = max(low, dpp_i<DPP_XOR2>(low));
    if (kt <= 4) low = max(low, dpp_i<DPP_HALF_MIRROR>(low));
    if (kt <= 2) low = max(low, dpp_i<DPP_MIRROR>(low));
    auto uniform = [](int m) { return __builtin_amdgcn_readfirstlane(m); };
    auto at_least = [&](int m) {
      // eight ballots at a time into registers of their own: a bit count right behind its comparison waits for it
      constexpr int G = ELEMS < 8 ? ELEMS : 8;
      int c = 0;
#pragma unroll
      for (int i0 = 0; i0 < ELEMS; i0 += G) {
        u64 b[G];
#pragma unroll
        for (int i = 0; i < G; ++i) b[i] = __ballot(key[i0 + i] >= m);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < G; ++i) c += __popcll(b[i]);
      }
      return c;
    };
    const TopkCut cut = topk_cut(kt <= 64 ? wave_min_i(low) : GONE, wave_max_i(best) + 1, kt, uniform, at_least);
    const int thr = cut.thr;
    // compact in id order (g = 64 i + lane: element by element, lanes ascending)
    int base = 0, rem = cut.rem;
#pragma unroll
    for (int i = 0; i < ELEMS; ++i) {
      u64 take = __ballot(key[i] > thr);
      if (rem > 0) {
        const u64 eq = __ballot(key[i] == thr);
        const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(eq >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eq, 0));
        take |= __ballot(key[i] == thr && before < rem);
        rem -= min(rem, (int)__popcll(eq));
      }
      if (SET) {
        if (lane == 0) set[i] = take;
      } else if ((take >> lane) & 1) {
        const int pos = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(take >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)take, 0));
        uk[pos] = key[i];
        uid[pos] = i * 64 + lane;
      }
      base += __popcll(take);
    }
    if (SET) return {kt, mx, denom};
    if (lane < 8 && kt + lane < kp) uk[kt + lane] = GONE;  // the ranking reads eight at a time
    wave_lds_fence();
    // rank = number of larger keys plus equal keys of smaller ids (= earlier positions)
    for (int j = lane; j < kt; j += 64) {
      const int mine = uk[j];
      int rank = 0;
      for (int q = 0; q < kt; q += 8) {
        const int4 o = *reinterpret_cast<const int4*>(uk + q), p = *reinterpret_cast<const int4*>(uk + q + 4);
        rank += o.x > mine - (q < j ? 1 : 0);
        rank += o.y > mine - (q + 1 < j ? 1 : 0);
        rank += o.z > mine - (q + 2 < j ? 1 : 0);
        rank += o.w > mine - (q + 3 < j ? 1 : 0);
        rank += p.x > mine - (q + 4 < j ? 1 : 0);
        rank += p.y > mine - (q + 5 < j ? 1 : 0);
        rank += p.z > mine - (q + 6 < j ? 1 : 0);
        rank += p.w > mine - (q + 7 < j ? 1 : 0);
      }
      se[rank] = topk_unkey(mine);
      sid[rank] = uid[j];
    }
    wave_lds_fence();
  }
  if (SET) return {kt, mx, denom};
  float dsel = 0.0f;
  for (int j = lane; j < kt; j += 64) dsel += expf(se[j] - mx);
  if (renorm) denom = wave_sum(dsel);
  return {kt, mx, denom};
}

}  // namespace mp
