// Route stage (Sec. 3.2.2, expanded linear gate): router logits with a fixed
// summation order, then per-token top-k_t and softmax weights.
#include "chain_tile.h"
#include "dispatch_common.h"
#include "topk_wave.h"

namespace mp {

// ---------------------------------------------------------------- expand_k
// Sec. 3.3.1: a token inherits its request's budget.
__global__ void expand_k_kernel(int R, const int32_t* __restrict__ req_k,
                                const int32_t* __restrict__ req_off, int32_t* __restrict__ k_tok) {
  int r = blockIdx.x;
  if (r >= R) return;
  int lo = req_off[r], hi = req_off[r + 1], k = req_k[r];
  for (int t = lo + threadIdx.x; t < hi; t += blockDim.x) k_tok[t] = k;
}

hipError_t launch_expand_k(int R, int T, const int32_t* req_k, const int32_t* req_off,
                           int32_t* k_tok, hipStream_t s) {
  (void)T;
  if (R > 0) expand_k_kernel<<<R, 256, 0, s>>>(R, req_k, req_off, k_tok);
  return hipGetLastError();
}

// ---------------------------------------------------------------- equal router rows
// An expanded gate that has not been trained yet repeats an expert's router row for each of its sub-experts (Sec. 3.2.2), and
// equal rows have equal chains.  differ[e]: the rows of expert e's sub-experts are not all the same, bit for bit.
__global__ __launch_bounds__(256) void rows_differ_kernel(const uint32_t* __restrict__ w, int32_t* __restrict__ differ,
                                                          int words, int S) {
  const uint32_t* row = w + (size_t)blockIdx.x * S * words;
  int any = 0;
  for (int i0 = 0; i0 < words && any == 0; i0 += 4 * 256) {
    const int i = i0 + 4 * (int)threadIdx.x;
    uint32_t diff = 0;
    if (i < words) {  // words % 32 == 0
      uint32_t first[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) first[q] = row[i + q];
      for (int s0 = 1; s0 < S; s0 += 3)
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
          for (int q = 0; q < 4; ++q) diff |= first[q] ^ row[(size_t)min(s0 + u, S - 1) * words + i + q];
    }
    any = __syncthreads_or(diff != 0);
  }
  if (threadIdx.x == 0) differ[blockIdx.x] = any;
}

// ---------------------------------------------------------------- logits on the matrix cores
// Every logit is ONE chain of d binary32 fused multiply-adds over the hidden index in
// ascending order, then the fp32 bias add: the fixed summation order is what makes the
// routing reproducible bit for bit.  The chains run on the matrix cores, see chain_tile.h.
// SHARE: the rows were compared.  (An instance of its own: with the branch and its epilogue in one kernel the 64 x 64 tile took 53 registers
// instead of 37, and its stores waited for one bias after the other; route calls, one kernel | two, d = 384: 14 000 x 512 63.5 | 58.9 us, 20 200 x 512 83.2 | 80.7.)
struct SharedRows {
  const int32_t* differ;  // of the experts (rows_differ_kernel)
  int S;
};
template <typename InT, int WM, int WN, int MT, int NT, int NS, bool APART, bool SHARE>
__global__ __launch_bounds__(64 * WM * WN * (APART ? 2 : 1)) void logits_kernel(
    const InT* __restrict__ x, const InT* __restrict__ w, const float* __restrict__ bias,
    float* __restrict__ logits, int32_t* __restrict__ hdr, int T, int d, int E, SharedRows shared) {
  using C = ChainTile<InT, WM, WN, MT, NT, NS>;
  constexpr int CP = C::CP;
  extern __shared__ __align__(16) unsigned char lg_smem[];
  const int lane = threadIdx.x & 63, w0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wv = APART ? w0 % C::NW : w0;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    hdr[HDR_FLAGS] = 0;
    hdr[HDR_TOPK_DONE] = 0;
  }
  int bx = blockIdx.x, by = blockIdx.y, cols = E, step = 1;  // columns of C are every step-th row of w
  if constexpr (SHARE) {
    bool same = true;
    for (int e = lane; e < E / shared.S; e += 64) same = same && shared.differ[e] == 0;
    if (__all(same)) {
      step = shared.S;
      cols = E / step;
      const int nx = (cols + C::BE - 1) / C::BE, id = by * gridDim.x + bx;  // the first workgroups have all there is to do
      by = id / nx;
      bx = id % nx;
      if (by * C::BT >= T) return;
    }
  }
  const int m0 = by * C::BT, n0 = bx * C::BE;
  const unsigned char* base[CP];
  uint32_t voff[CP];
#pragma unroll
  for (int j = 0; j < CP; ++j) {
    const int r0 = (wv * CP + j) * 8, row = r0 + (lane >> 3);
    const bool tok = r0 < C::BT;  // the same for the whole copy
    base[j] = reinterpret_cast<const unsigned char*>(tok ? x + (size_t)m0 * d : w + (size_t)n0 * step * d);
    const int rr = tok ? min(row, T - 1 - m0) : min(row - C::BT, cols - 1 - n0) * step;
    voff[j] = (uint32_t)rr * (uint32_t)(d * (int)sizeof(InT)) + (uint32_t)(chain_chunk(row) * 16);
  }
  f32x4_t acc[MT][NT];
  chain_tile<C, APART>(lg_smem, d / C::KB, [&](int j, int stage, uint32_t lds) {  // d % 64 == 0
    copy_to_lds16(base[j] + (size_t)stage * 128, voff[j], lds);
  }, acc);
  if (APART && w0 >= C::NW) return;

  const int wm = wv / WN, wn = wv % WN, r = lane & 15, g = lane >> 4;
  if (SHARE && step > 1) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int col = n0 + (wn * NT + j) * 16 + r;
      for (int c = col * step; c < (col + 1) * step && col < cols; c += step % 4 == 0 ? 4 : 1) {
        float bv[4] = {};
        if (bias != nullptr)
#pragma unroll
          for (int u = 0; u < 4; ++u) bv[u] = u == 0 || step % 4 == 0 ? bias[c + u] : 0.0f;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int row = m0 + (wm * MT + i) * 16 + 4 * g + v;
            const float a = acc[i][j][v];
            float o[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) o[u] = bias != nullptr ? a + bv[u] : a;
            if (row >= T) continue;
            if (step % 4 == 0) __builtin_memcpy(logits + (size_t)row * E + c, o, 16);
            else logits[(size_t)row * E + c] = o[0];
          }
      }
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int col = n0 + (wn * NT + j) * 16 + r;
    const float bv = bias != nullptr && col < E ? bias[col] : 0.0f;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = m0 + (wm * MT + i) * 16 + 4 * g + v;
        if (row < T && col < E) {
          const float s = acc[i][j][v];
          logits[(size_t)row * E + col] = bias != nullptr ? s + bv : s;
        }
      }
  }
}

__global__ void clear_flags_kernel(int32_t* hdr) { hdr[HDR_FLAGS] = 0; }

template <typename InT, bool SHARE, int MT, int NT, int NS, bool APART>
static void launch_logits_cfg(const InT* x, const InT* w, const float* bias, float* logits,
                              int32_t* hdr, int T, int d, int E, SharedRows shared, hipStream_t s) {
  using C = ChainTile<InT, 2, 2, MT, NT, NS>;
  constexpr int MOST = 65535 * C::BT;  // tokens that the second dimension of a grid holds: 2.1 or 4.2 million
  for (long t0 = 0; t0 < T; t0 += MOST) {
    const int n = (int)(T - t0 < MOST ? T - t0 : MOST);
    logits_kernel<InT, 2, 2, MT, NT, NS, APART, SHARE><<<dim3(cdiv(E, C::BE), cdiv(n, C::BT)), 64 * C::NW * (APART ? 2 : 1), C::LDS_BYTES, s>>>(
        x + t0 * d, w, bias, logits + t0 * E, hdr, n, d, E, shared);
  }
}

// Workgroups of 2 x 2 waves on tiles of 32 x 32, 32 x 64 or 64 x 64 logits: 1, 2 or 4 sub-tiles
// per SIMD.  The time is the number of sub-tiles the busiest SIMD works through (workgroups per
// CU, rounded up, times sub-tiles), so the tile with the smallest such number is taken; among
// equals, and up to 5 % more, the widest, which re-reads less, but where one or two sub-tiles are all there
// is its single workgroup per CU has nothing to overlap its start with (4096 x 128: 20.7 us on 32 x 32, 21.5 on
// 32 x 64).  The narrow tiles have their copies done by waves of their own (APART); not 32 x 32 for short rows on CUs with many
// tiles, where other workgroups' products hide the copies and what is left is twice the waves at a barrier.  Route calls, copies by the
// same waves | apart: 41 000 x 256, d = 256 73.0 | 78.3, d = 384 89.6 | 93.9; 17 293 x 256, d = 256 37.5 | 38.9; but d = 512 54.2 | 53.5, d = 1024 90.9 | 87.8; and
// with few tiles, 1024 x 512, d = 256 9.5 | 9.4.  The 64 x 64 tile does not: three of its
// workgroups share a CU, and six waves per SIMD measured 152 us where three took 137 (8192 x 512).  A workgroup of it that is
// left alone, the last of 4, 7, 10 .., takes a quarter longer, which narrow tiles are worth where rows are long, or with 4 and as many
// in 32 x 64.  Route calls, 64 x 64 | narrow: 8192 x 512, d = 128 25.4 | 26.4, d = 256 35.8 | 34.2, d = 1024 86.1 | 73.1; 25 200 x 512, d = 256 78.8 | 88.8, d = 512 122.1 |
// 128.7, 1024 212.7 | 212.6; 27 340 x 256, d = 512 72.6 | 75.0, d = 2048 219.5 | 211.5; fp32, 27 340 x 256, d = 512 75.6 | 80.8, 2048 231 | 261, 8192 x 512, d = 256 35.6 | 34.1, d =
// 1024 78.6 | 80.7.  Between HIP events, d = 2048, all in 32 x 64 | 64 x 64: 8192 x 512
// 126.5 | 134.5, 16 384 x 256 126 | 140, 10 000 x 512 156.0 | 154.0, 12 000 185.6 | 182.3, 16 384 245 | 241, 65 536 955 | 947.
// Copies by the same waves | apart: 1 x 512 13.6 | 11.8, 1024 22.1 | 20.6, 3000 56.4 | 50.2, 5000 89.5 | 79.6, 2741 x 128 21.9 |
// 20.0, 8192 39.5 | 35.6, 6007 x 256 56.6 | 50.1; 100 x 32, d = 4096 23.1 | 19.4; fp32, 1024 x 32, d = 256 6.4 | 6.4.
template <typename InT, bool SHARE = false>
static void launch_logits_t(const InT* x, const InT* w, const float* bias, float* logits,
                            int32_t* hdr, int T, int d, int E, SharedRows shared, hipStream_t s) {
  auto cost = [&](int bt, int be, int sub) { return (long)cdiv((long)cdiv(T, bt) * cdiv(E, be), num_cus()) * sub; };
  const long c1 = cost(32, 32, 1), c2 = cost(32, 64, 2), c4 = cost(64, 64, 4);  // c1 <= c2 <= c4
  const bool alone = sizeof(InT) == 2 && c4 / 4 % 3 == 1 && (d >= 2048 || (d >= 256 && c4 == 16 && c2 == 16));
  if (c4 > 4 && c4 * 20 + (alone ? 22 : 0) <= c1 * 21)
    launch_logits_cfg<InT, SHARE, 2, 2, 3, false>(x, w, bias, logits, hdr, T, d, E, shared, s);
  else if (c2 == c1 && c1 > 2)
    launch_logits_cfg<InT, SHARE, 1, 2, 5, true>(x, w, bias, logits, hdr, T, d, E, shared, s);
  else if (SHARE || d * sizeof(InT) >= 1024 || c1 <= 8)
    launch_logits_cfg<InT, SHARE, 1, 1, 6, true>(x, w, bias, logits, hdr, T, d, E, shared, s);
  else
    launch_logits_cfg<InT, SHARE, 1, 1, 6, false>(x, w, bias, logits, hdr, T, d, E, shared, s);
}

// Rows are compared beyond 2^34 multiply-adds, where a gate whose rows differ loses less than 2 % of its route call by it: a launch, and
// in every workgroup the latency of its result.  Route calls from a captured graph, rows not compared | compared, rows that differ, equal rows, 512
// sub-experts, 4 to an expert, d = 2048: 2^31 40.7 | 43.6, 27.4; 2^32 73.5 | 77.5, 46.7; 2^33 130 | 142, 49.5; 2^33.5 190 | 194.5, 79; 2^34 (16 384 tokens) 250.6 |
// 254.6, 82; 2^35 492 | 497, 162; 2^36 976 | 981, 286.  256 of d = 4096, 128 of 2 to an expert, 1024 of 8 and d = 1024: 6 to 10 % at 2^31, 3 to 9 at 2^32, 2.5 to 7 at 2^33, 1.5 to
// 2.9 at 2^33.5, 1.6 to 1.8 at 2^34, up to 1.8 and falling beyond (between HIP events, 2^34 272 | 280).  Below the line equal rows are left alone: trained
// gates, which are the more frequent, would pay for them.
static bool compare_rows(int dtype, int T, int d, int E, int S) {
  return S > 1 && (double)T * E * d > 17179869184.0 && (long)E * d * (dtype == 0 ? 4 : 2) < (1L << 31);
}
hipError_t launch_logits(int dtype, const void* x, const void* w, const float* bias, float* logits,
                         int32_t* hdr, int T, int d, int E, int S, int32_t* differ, hipStream_t s) {
  if (T == 0) {
    clear_flags_kernel<<<1, 1, 0, s>>>(hdr);
    return hipGetLastError();
  }
  const SharedRows shared{differ, S};
  if (compare_rows(dtype, T, d, E, S)) {
    rows_differ_kernel<<<E / S, 256, 0, s>>>((const uint32_t*)w, differ, dtype == 0 ? d : d / 2, S);
    if (dtype == 0)
      launch_logits_t<float, true>((const float*)x, (const float*)w, bias, logits, hdr, T, d, E, shared, s);
    else
      launch_logits_t<uint16_t, true>((const uint16_t*)x, (const uint16_t*)w, bias, logits, hdr, T, d, E, shared, s);
  } else if (dtype == 0) {
    launch_logits_t((const float*)x, (const float*)w, bias, logits, hdr, T, d, E, shared, s);
  } else {
    launch_logits_t((const uint16_t*)x, (const uint16_t*)w, bias, logits, hdr, T, d, E, shared, s);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------- top-k_t + weights
// One wavefront per token, lane l holds logits g = i*64 + l in registers.  The k_t picks are the
// keys above a threshold that topk_search.h finds (a ballot and a scalar bit count per element and
// step), compacted in id order and ranked by counting; no sort and no global traffic besides the
// logits row and the outputs.
constexpr int TOPK_WAVES = 4;
// What follows the picks of a small batch in the same launch.
//   LAST: the last workgroup to finish dispatches the picks of all T tokens, which it reads back.
//   SOLO: one workgroup of up to WAVES waves has all tokens, and dispatches their picks from LDS.
enum { TOPK_ONLY, TOPK_LAST, TOPK_SOLO };
constexpr int SOLO_WAVES = 16;
template <int ELEMS, int MODE, int WAVES = TOPK_WAVES>
__global__ __launch_bounds__(64 * WAVES) void topk_kernel(
    const float* __restrict__ logits, const int32_t* __restrict__ k_tok, int32_t* __restrict__ ids,
    float* __restrict__ wout, int32_t* __restrict__ hdr, int T, int E, int k_max, int renorm,
    float scale, SmallDispatch small) {
  extern __shared__ __align__(16) unsigned char topk_smem[];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int t = MODE == TOPK_SOLO ? wv : blockIdx.x * WAVES + wv;
  // per wave: keys and ids of the picks in id order, then logits and ids in pick order
  const int kp = topk_pad(k_max);
  int* uk = reinterpret_cast<int*>(topk_smem) + (size_t)wv * 4 * kp;
  int* uid = uk + kp;
  float* se = reinterpret_cast<float*>(uid + kp);
  int* sid = reinterpret_cast<int*>(se + kp);
  u64* solo_masks = reinterpret_cast<u64*>(topk_smem + (size_t)(blockDim.x / 64) * 16 * kp);  // behind all waves' picks
  if constexpr (MODE == TOPK_SOLO) {
    for (int g = threadIdx.x; g < E; g += blockDim.x) solo_masks[g] = 0ull;
    __syncthreads();
  }
  int picked = 0;
  if (t < T) {
    const int asked = k_tok != nullptr ? k_tok[t] : k_max;  // null: every token takes k_max
    const TopkPicks p = topk_token<ELEMS>(logits + (size_t)t * E, asked, E, k_max, renorm, &hdr[HDR_FLAGS], uk, uid, se, sid);
    const int kt = picked = p.kt;
    for (int j = lane; j < k_max; j += 64) {
      bool on = j < kt;
      const int32_t id = on ? sid[j] : -1;
      if constexpr (MODE == TOPK_LAST)
        __hip_atomic_store(&ids[(size_t)t * k_max + j], id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else
        ids[(size_t)t * k_max + j] = id;
      if (MODE == TOPK_SOLO && on) atomicOr(&solo_masks[sid[j]], 1ull << t);
      wout[(size_t)t * k_max + j] = on ? scale * expf(se[j] - p.most) / p.denom : 0.0f;
    }
  }
  if constexpr (MODE == TOPK_SOLO) {
    int32_t* off_lds = reinterpret_cast<int32_t*>(solo_masks + E);
    __syncthreads();
    const int P = small_groups(small, hdr, solo_masks, off_lds, off_lds + E, 1, E, blockDim.x);
    __syncthreads();
    if (t >= T) return;
    for (int j = lane; j < k_max; j += 64) {
      const int i = t * k_max + j;
      int slot = -1;
      if (j < picked) {
        const int g = sid[j];
        slot = off_lds[g] + __popcll(solo_masks[g] & ((1ull << t) - 1ull));
        small.sorted_pair[slot] = i;
      }
      small.slot_of_pair[i] = slot;
      if (i >= P) small.sorted_pair[i] = -1;  // tail beyond the P valid slots
    }
  }
  if constexpr (MODE == TOPK_LAST) {
    // behind the dispatch's tables in the same dynamic LDS: the picks of the largest budget take all of
    // the default 64 KiB, so there is no room for static LDS beside them
    int32_t* is_last = reinterpret_cast<int32_t*>(topk_smem + small_dispatch_lds(T, E));
    int32_t* wave_tot = is_last + 1;
    // The picks were stored at agent scope, i.e. through this XCD's L2, so once they are acknowledged every CU can read
    // them: no release fence, which would have each workgroup write back all of its L2 (64 fp32 tokens of 8 x 4
    // sub-experts, layer calls: 24.5 -> 23.6 us)
    wait_vmem<0>();
    __syncthreads();
    if (threadIdx.x == 0) *is_last = atomicAdd(&hdr[HDR_TOPK_DONE], 1) == (int)gridDim.x - 1;
    __syncthreads();
    if (!*is_last) return;
    dispatch_one_workgroup<true, 64 * WAVES>(ids, small, hdr, reinterpret_cast<u64*>(topk_smem), wave_tot, T, E, k_max);
  }
}

// TOPK_LAST has eight waves where their picks fit the default 64 KiB of LDS: four, which the general top-k has, take twice as long
// to dispatch (masks, groups and places of 3200 pairs 7.7 of the kernel's 13.4 us), and sixteen get in each other's way at the
// picks.  Layer calls back to back, us, four waves | eight | sixteen: 512 sub-experts of 32 picks, 37 tokens 105.3 | 104.5 | 106.1, 64 122.6 |
// 121.7 | 123.1, 100 143.1 | 140.3 | 141.3; 256 of 24, 100 tokens 226.4 | 224.7 | 224.9; fp32, 32 of 8, 250 29.6 | 27.9 | 28.2; 2048 of 8, d = 256, 120
// 37.6 | 34.5 | 34.5.
constexpr int LAST_WAVES = 8;
static bool wide_last(int k_max) { return (size_t)LAST_WAVES * 4 * topk_pad(k_max) * sizeof(float) <= 60 * 1024; }
// So with eight waves the last workgroup is ahead of count and place kernels for more pairs than one of four (small_dispatch, which the
// stage call goes by).  The line lies where they met while those had 256 threads.  Layer calls from a captured graph, d = 64, Is = 32, one workgroup |
// count and place kernels of 512, 512 sub-experts, by the pairs beyond those of 64 tokens: 128 tokens of 24 picks (1536) 25.4 | 28.1, 255 of 12 (2292) 24.7 | 26.2, 128 of
// 48 (3072) 31.8 | 32.9, 160 of 32 (3072) 29.7 | 30.2, 200 of 24 (3264) 28.4 | 28.2, 128 of 64 (4096) 35.2 | 35.3, 200 of 32 (4352) 31.2 | 29.7, 255 of 24 (4584)
// 30.2 | 28.7, 160 of 48 (4608) 33.5 | 32.4, beyond it 128 of 100 (6400) 50.9 | 48.8, 255 of 32 (6112) 33.1 | 30.0; 32, 128 and 1024 alike.  So they meet at 4100 up to 128
// tokens, at 3100 beyond.
bool topk_dispatches(int T, int E, int k_max) {
  return small_dispatch(T, E, k_max) ||
         (T > 0 && T < 256 && (T - 64) * k_max <= 4608 && wide_last(k_max) && small_dispatch_lds(T, E) <= 60 * 1024);
}

hipError_t launch_topk(const float* logits, const int32_t* k_tok, int32_t* ids, float* w,
                       int32_t* hdr, int T, int E, int k_max, int renorm, float scale,
                       const SmallDispatch* small, hipStream_t s) {
  if (T == 0) return hipSuccess;
  const size_t sh_wave = (size_t)4 * topk_pad(k_max) * sizeof(float);
  const int elems = cdiv(E, 64);
  // One workgroup saves the count and the reading back of the picks, but its waves are in each other's way.  Layer calls from a
  // captured graph, us, one workgroup | the last of several of eight waves, d = 128, Is = 64: 9 tokens of 2 picks out of 32 sub-experts 15.7 |
  // 16.7, of 32 out of 32 19.6 | 20.4, out of 512 21.5 | 22.0, out of 1024 24.6 | 25.7; 12 tokens of 2 out of 16 15.9 | 16.7, of 24 out of 512
  // 21.4 | 21.7, of 32 21.6 | 21.9, out of 1024 24.0 | 23.4; 16 tokens of 2 out of 16 16.7 | 17.7, of 12 out of 128 0.3 less, of 20 20.4 |
  // 20.4, equal logits among them (long searches) 2 more; of 2 out of 256 17.1 | 17.5, of 8 19.2 | 19.0, of 32 22.2 | 21.8; of 12 out of 512 20.5 | 20.0, out
  // of 1024 23.1 | 22.0.  Equal logits cost one workgroup of 12 tokens 1, too.
  const int solo_waves = T < TOPK_WAVES ? TOPK_WAVES : T;
  const size_t sh_solo = solo_waves * sh_wave + (size_t)E * 12 + SOLO_WAVES * sizeof(int32_t);
  const bool solo = small != nullptr && ((T <= 12 && T * E <= 10 * 1024) || (T <= SOLO_WAVES && E <= 128 && k_max <= 12)) && elems <= 16 && sh_solo <= 60 * 1024;
  const int waves = !small || solo || !wide_last(k_max) ? TOPK_WAVES : LAST_WAVES;
  const size_t sh_small = small_dispatch_lds(T, E) + (1 + waves) * sizeof(int32_t);  // the last flag and wave_tot
  dim3 grid(cdiv(T, waves)), block(64 * waves);
  size_t sh = waves * sh_wave;
  if (solo) {
    sh = sh_solo;
    grid = dim3(1);
    block = dim3(64 * solo_waves);
  } else if (small != nullptr && sh_small > sh) {
    sh = sh_small;
  }
  const SmallDispatch sd = small != nullptr ? *small : SmallDispatch{};
#define MP_TOPK_MODE(N, ...) \
  topk_kernel<N, __VA_ARGS__><<<grid, block, sh, s>>>(logits, k_tok, ids, w, hdr, T, E, k_max, renorm, scale, sd)
#define MP_TOPK(N)                                                           \
  do {                                                                       \
    if (small == nullptr) MP_TOPK_MODE(N, TOPK_ONLY);                        \
    else if (solo && T <= 8) MP_TOPK_MODE((N <= 16 ? N : 16), TOPK_SOLO, 8); \
    else if (solo) MP_TOPK_MODE((N <= 16 ? N : 16), TOPK_SOLO, SOLO_WAVES);  \
    else if (waves == LAST_WAVES) MP_TOPK_MODE(N, TOPK_LAST, LAST_WAVES);    \
    else MP_TOPK_MODE(N, TOPK_LAST);                                         \
  } while (0)
  if (elems <= 1) MP_TOPK(1);
  else if (elems <= 2) MP_TOPK(2);
  else if (elems <= 4) MP_TOPK(4);
  else if (elems <= 8) MP_TOPK(8);
  else if (elems <= 16) MP_TOPK(16);
  else if (elems <= 32) MP_TOPK(32);
  else MP_TOPK(64);
#undef MP_TOPK
#undef MP_TOPK_MODE
  return hipGetLastError();
}

// ---------------------------------------------------------------- proxy gate: per-expert top-kappa
// Sec. 3.2.2, training-free proxy gating.  One thread per (token, expert rank j).  For the expert
// the original router ranked j, the S sub-experts are scored by the mean absolute activation of
// their r gate neurons (act: row slot(t, j) of the proxy activations, sub-expert n at columns
// n r .. n r + r - 1, summed in ascending column order in fp32), and the best kappa[k_t][j] are
// taken, score descending, equal scores to the smaller index.  Selected sub-experts are
// appended in rank order with the expert's weight: rank j writes at the sum of the ranks'
// allocations before it, the last rank also pads the tail.
// A chain of latencies: budget, allocations, slot, activations.  What a step needs is requested at once: the allocations of
// eight ranks, and of every sub-expert the next activation, or four where r % 4 == 0 (rows of act are whole multiples
// of 32 elements, so that four are aligned).  MOST: 4 or 16, the largest S.  Between HIP events, one activation after the other
// | this: 300 tokens of 8 experts, S = r = 4, 15.9 | 7.6 us, 4096 15.3 | 8.1, 16384 23.4 | 12.0.
template <int N>
__device__ __forceinline__ void act_abs(const float* p, float (&v)[N]) {
  float f[N];
  __builtin_memcpy(f, __builtin_assume_aligned(p, 4 * N), sizeof(f));
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = fabsf(f[i]);
}
template <int N>
__device__ __forceinline__ void act_abs(const uint16_t* p, float (&v)[N]) {
  uint16_t f[N];
  __builtin_memcpy(f, __builtin_assume_aligned(p, 2 * N), sizeof(f));
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = fabsf(bf16_to_f32(f[i]));
}
// sums of |a[n r + c]| over ascending c
template <int N, int MOST, typename ActT>
__device__ __forceinline__ void proxy_sums(const ActT* a, int S, int r, float (&sum)[MOST]) {
#pragma unroll
  for (int n = 0; n < MOST; ++n) sum[n] = 0.0f;
  for (int c = 0; c < r; c += N) {
    float v[MOST][N];
#pragma unroll
    for (int n = 0; n < MOST; ++n) act_abs(a + min(n, S - 1) * r + c, v[n]);
#pragma unroll
    for (int n = 0; n < MOST; ++n)
#pragma unroll
      for (int i = 0; i < N; ++i) sum[n] += v[n][i];
  }
}

template <typename ActT, int MOST>
__global__ __launch_bounds__(256) void proxy_select_kernel(
    const ActT* __restrict__ act, int act_ld, const int32_t* __restrict__ ids0,
    const float* __restrict__ w0, const int32_t* __restrict__ slot0,
    const int32_t* __restrict__ k_tok, const int32_t* __restrict__ kappa, int32_t* __restrict__ ids,
    float* __restrict__ w, int32_t* __restrict__ hdr, int T, int S, int r, int m, int k_max) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= T * m) return;
  const int t = idx / m, j = idx % m;
  const int k_cap = min(k_max, m * S);
  int kt = k_tok[t];
  if (kt < 0 || kt > k_cap) {
    if (j == 0) atomicOr(&hdr[HDR_FLAGS], 1);
    kt = kt < 0 ? 0 : k_cap;
  }
  const int32_t* kap_row = kappa + (size_t)kt * m;
  auto alloc = [&](int jj) {
    const int e = ids0[(size_t)t * m + jj], slot = slot0[(size_t)t * m + jj];
    int kap = kap_row[jj];
    kap = kap < 0 ? 0 : (kap > S ? S : kap);
    return (e < 0 || slot < 0) ? 0 : kap;
  };
  int pos = 0;
  for (int j0 = 0; j0 < j; j0 += 8) {
    int al[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) al[u] = alloc(min(j0 + u, j));
#pragma unroll
    for (int u = 0; u < 8; ++u) pos += j0 + u < j ? al[u] : 0;
  }
  const int kap = alloc(j);
  int32_t* o = ids + (size_t)t * k_max;
  float* ow = w + (size_t)t * k_max;
  if (kap > 0) {
    const int e = ids0[idx];
    const ActT* a = act + (size_t)slot0[idx] * act_ld;
    const float inv_r = 1.0f / (float)r;
    float sc[MOST];
    if (r % 4 == 0) proxy_sums<4>(a, S, r, sc);
    else proxy_sums<1>(a, S, r, sc);
#pragma unroll
    for (int n = 0; n < MOST; ++n) sc[n] = n < S ? sc[n] * inv_r : -1.0f;  // scores are >= 0: -1 marks taken or absent
    const float wj = w0[idx];
    for (int i = 0; i < kap && pos < k_max; ++i) {
      int best = 0;
      float most = sc[0];
#pragma unroll
      for (int n = 1; n < MOST; ++n)
        if (sc[n] > most) {
          most = sc[n];
          best = n;
        }
#pragma unroll
      for (int n = 0; n < MOST; ++n)
        if (n == best) sc[n] = -1.0f;
      o[pos] = e * S + best;
      ow[pos] = wj;
      ++pos;
    }
  }
  if (j == m - 1)
    for (; pos < k_max; ++pos) {
      o[pos] = -1;
      ow[pos] = 0.0f;
    }
}

hipError_t launch_proxy_select(int dtype, const void* act, int act_ld, const int32_t* ids0,
                               const float* w0, const int32_t* slot0, const int32_t* k_tok,
                               const int32_t* kappa, int32_t* ids, float* w, int32_t* hdr, int T,
                               int S, int r, int m, int k_max, hipStream_t s) {
  if (T == 0) return hipSuccess;
  auto run = [&](auto* kern, auto* a) {
    kern<<<cdiv(T * m, 256), 256, 0, s>>>(a, act_ld, ids0, w0, slot0, k_tok, kappa, ids, w, hdr, T, S, r, m, k_max);
  };
  if (dtype == 0) {
    const float* a = (const float*)act;
    if (S <= 4) run(proxy_select_kernel<float, 4>, a);
    else run(proxy_select_kernel<float, PROXY_MAX_SUB>, a);
  } else {
    const uint16_t* a = (const uint16_t*)act;
    if (S <= 4) run(proxy_select_kernel<uint16_t, 4>, a);
    else run(proxy_select_kernel<uint16_t, PROXY_MAX_SUB>, a);
  }
  return hipGetLastError();
}

}  // namespace mp
