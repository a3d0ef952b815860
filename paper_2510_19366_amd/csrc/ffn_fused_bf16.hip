// bf16 grouped SwiGLU FFN (Sec. 3.2.1, Eq. 1-3) for narrow sub-experts, fused: gate-up,
// SwiGLU and the down projection of an m-tile run in one workgroup and the activations
// h never leave the registers.
//
//   y[p, :] = ( SiLU(x[t_p,:] Wg[g]^T) * (x[t_p,:] Wu[g]^T) ) Wd[g]^T        p in group g
//
// Split: a persistent workgroup (8 wavefronts, one per CU) owns an m-tile of 256 slot rows of
// one group; wave w owns rows 32w .. 32w+31 and ALL 2*Is gate/up rows and all d output
// columns.  With v_mfma_f32_32x32x16_bf16 and the weight rows as first operand, a lane ends
// phase 1 with gate and up of 8 consecutive neurons of one slot row (the weight rows of a
// 32-row block are fed in a permuted order: 16 neurons' gate rows and the same neurons' up
// rows).  After SiLU(g)*u those 8 values, packed to bf16, are exactly the second-operand
// fragment of one K step of the down GEMM for the same 32 slot rows: phase 2 takes h from
// registers, no LDS round trip, no barrier between the phases, and neither h nor a second
// pass over the tile table touches HBM.
//
// Operands travel global -> LDS directly (global_load_lds_dwordx4), in whole 128-byte lines.
// Weights: a ring of 4 slots of Is*128 bytes shared by the waves (phase 1: Is rows, half of gate and
// up, x 64 K-elements; phase 2: 64 output columns x Is K-elements; both fill a slot exactly),
// published by one s_barrier per stage; two stages are in flight while one is multiplied.  Slot
// rows of x: one slot of 4 KiB PRIVATE to each wave (a wave copies the rows it multiplies itself,
// so x needs no barrier), refilled as soon as its fragments are in registers.  vmcnt retires in
// issue order, so a wait is for the number of operations issued behind the ones needed.
#include <type_traits>

#include "dma.h"
#include "ffn_common.h"

namespace mp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

namespace fused {

constexpr int NT = 512;   // threads: 8 waves
constexpr int BM = FFN_BM;
constexpr int NSW = 4;    // weight ring slots
constexpr int X_WAVE = 32 * 128;       // bytes of one wave's x slot: 32 rows x 64 K-elements
constexpr int EPI_WAVE = 16 * 128;     // bytes of a wave's output staging: 16 rows x 64 columns
// Consecutive tiles of a list's turn; 1 where the long tiles come first, so that every list has its share of them (skewed, 700 |
// 1024 tokens in runs of 32: 212 | 232 us, so 210 | 227).  With 32, one tile for each of an XCD's workgroups, | 64, 512
// sub-experts of 192 x 2048, fused kernel between HIP events, three layers in turn: proxy gate, 2000 tokens 318 | 306 us, 4096
// 368 | 355, 6000 434 | 436, 12000 666 | 667; skewed, 3000 tokens 313 | 304, 8000 497 | 501, 16384 885 | 890; 12000 of 32 picks 986 | 987.
constexpr int RUN = 64;
constexpr int PD = 4;     // fragment reads in flight ahead of the MFMAs

template <int IS>
struct Cfg {
  static_assert(IS % 64 == 0 && IS >= 64 && IS <= 192, "fused path: Is in {64, 128, 192}");
  static constexpr int NBLK = IS / 16;     // 32-row weight blocks of phase 1 = K steps of phase 2
  static constexpr int HB = NBLK / 2;      // blocks of a phase-1 stage
  static constexpr int WPW = IS / 64;      // copy instructions per wave and weight stage
  static constexpr int W_SLOT = IS * 128;  // bytes
  static constexpr int CPR = IS / 8;       // 16-byte chunks per weight row in phase 2
  static constexpr int ROW2 = IS * 2;      // bytes per weight row in phase 2
  static constexpr int OFF_X = NSW * W_SLOT;
  static constexpr int OFF_PAIR = OFF_X + 8 * X_WAVE;
  static constexpr int OFF_EPI = OFF_PAIR + 2 * BM * 4;   // output transposition
  static constexpr int OFF_DYN = OFF_EPI + 8 * EPI_WAVE;  // the tile number drawn by wave 0, and the number of tiles
  static constexpr int LDS_BYTES = OFF_DYN + 16;
  // steps of a stage (one MFMA each) behind which things happen
  static constexpr int STEPS = 2 * NBLK;
  static constexpr int BAR = 1;                        // the stage's wait and barrier
  static constexpr int W0 = 2, W_END = W0 + WPW;       // copies of weights, one per step
  static constexpr int PREP = STEPS - 1;               // the next stage's weight copies are prepared
  // copy j of the four of x; in phase 1 behind the step that waits for the last read of the slot
  static constexpr int X0 = W_END > PD ? W_END : PD;
  static constexpr int x_copy(int j) { return X0 + (STEPS > 8 ? j : j / 2); }
  static constexpr int XW = STEPS - 5;                 // phase 1: x of the next stage pair has to be there
  // phase 2, output of the previous stage: half h goes into the staging buffer, quarter k (8 rows)
  // is read back and stored
  static constexpr int out_write(int h) { return STEPS > 8 ? W0 + 1 + h * (STEPS * 5 / 12) : 2 + 2 * h; }
  static constexpr int out_read(int k) {
    return out_write(k / 2) + (STEPS > 16 ? 3 + k % 2 * 2 : STEPS > 8 ? 2 + k % 2 : 1);
  }
  static constexpr int out_store(int k) { return out_read(k) + (STEPS > 16 ? 3 : STEPS > 8 ? 2 : 1); }
  static_assert(STEPS % PD == 0 && 3 * HB >= PD && XW + PD < STEPS && XW + 2 >= 3 * HB - 1, "fragment registers");
  static_assert(out_write(0) < out_read(0) && out_read(1) <= out_write(1) && out_store(0) >= W_END &&
                    out_store(3) < STEPS && XW >= W_END && x_copy(3) < STEPS,
                "order inside a stage");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS per CU");
};

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// wave-wide copy of 4 bytes per lane (see copy_to_lds16)
__device__ __forceinline__ void dma4(const void* base, uint32_t voff, uint32_t lds) {
  uint32_t keep;
  asm volatile(
      "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\t"
      "global_load_lds_dword %1, %2\n\ts_mov_b32 m0, %0"
      : "=&s"(keep)
      : "v"(voff), "s"(base), "s"(lds)
      : "memory");
}
// 16-byte store at base + voff, counted by hand like the copies (the compiler neither
// merges nor splits it).  A store of more than 8 bytes reads its data registers for a few
// cycles after issue and the compiler's hazard handling does not look inside an asm block:
// the s_nop keeps the next VALU write away from them.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store16(void* base, uint32_t voff, u32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, %2\n\ts_nop 1" ::"v"(voff), "v"(v), "s"(base) : "memory");
}
// until at most n of this wave's vector memory operations are pending, for n one of the given
// counts, largest first (another n: the next smaller one).  The steady state falls through; a branch per
// count would cost more than the waits.
template <int A, int B, int C, int D>
__device__ __forceinline__ void wait_one_of4(int n) {
  asm volatile(
      "s_waitcnt vmcnt(%1)\n\ts_cmp_ge_i32 %0, %1\n\ts_cbranch_scc1 1f\n\t"
      "s_waitcnt vmcnt(%2)\n\ts_cmp_ge_i32 %0, %2\n\ts_cbranch_scc1 1f\n\t"
      "s_waitcnt vmcnt(%3)\n\ts_cmp_ge_i32 %0, %3\n\ts_cbranch_scc1 1f\n\t"
      "s_waitcnt vmcnt(%4)\n1:" ::"s"(n),
      "n"(A), "n"(B), "n"(C), "n"(D)
      : "memory", "scc");
}
template <int A, int B, int... MORE>
__device__ __forceinline__ void wait_one_of(int n) {
  if constexpr (sizeof...(MORE) == 0)
    asm volatile("s_waitcnt vmcnt(%1)\n\ts_cmp_ge_i32 %0, %1\n\ts_cbranch_scc1 1f\n\ts_waitcnt vmcnt(%2)\n1:" ::"s"(n),
                 "n"(A), "n"(B)
                 : "memory", "scc");
  else
    wait_one_of4<A, B, MORE...>(n);
}
// weight-row permutations (MFMA row i = 8a + 4hi + b of a 32-row block):
// phase 1: block row 16*(a>>1) + 8hi + 4(a&1) + b, block rows 0..15 = gate rows of 16 neurons,
// 16..31 = their up rows: accumulators 0..7 of a lane = gate of neurons 8hi..8hi+7, 8..15 = up
__device__ __forceinline__ int wrow_gu(int i) {
  const int a = i >> 3, hi = (i >> 2) & 1, b = i & 3;
  return 16 * (a >> 1) + 8 * hi + 4 * (a & 1) + b;
}
// phase 2: block row 16hi + 4a + b: a lane's 16 accumulators = output columns 16hi .. 16hi+15
__device__ __forceinline__ int wrow_dn(int i) {
  const int a = i >> 3, hi = (i >> 2) & 1, b = i & 3;
  return 16 * hi + 4 * a + b;
}
// LDS swizzles (16-byte chunk c of row r sits at chunk position c ^ f(r)); 16 lanes read 16
// rows at one chunk index, f spreads them over all banks.
// 128-byte rows (phase 1, both operands, and the output staging), 16 consecutive rows: rows of
// equal parity share banks
__device__ __forceinline__ int f1(int r) { return (r >> 1) & 7; }
// Is*2-byte rows (phase 2): 384- and 128-byte rows alternate between two bank halves (8 rows of
// equal parity must differ), 256-byte rows all start in bank 0 (16 rows must differ); the 16
// rows read together are {0..7, 16..23} + const
template <int IS>
__device__ __forceinline__ int f2(int r) {
  return IS == 128 ? ((r & 7) | (((r >> 4) & 1) << 3)) : (((r >> 1) & 3) | (((r >> 4) & 1) << 2));
}

struct TileHdr {  // wave-uniform
  int g, row0, rows;
};

// One matrix-core step.  MATH = false is the traffic probe: the same operand reads, copies,
// barriers, waits and stores, without the multiply (the fragments count as used, the results mean
// nothing).
template <bool MATH>
__device__ __forceinline__ f32x16 mma(bf16x8 a, bf16x8 b, f32x16 c) {
  if constexpr (MATH) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  } else {
    asm volatile("" ::"v"(a), "v"(b));
    return c;
  }
}

template <int IS, bool MATH>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void ffn_fused_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ w_gu,
    const uint16_t* __restrict__ w_dn, const int32_t* __restrict__ sorted_pair,
    const MTile* __restrict__ tiles, int32_t* __restrict__ hdr, uint16_t* __restrict__ y, int T,
    int d, int k_max, int sorted, int help) {
  using C = Cfg<IS>;
  constexpr int NBLK = C::NBLK, WPW = C::WPW;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, wv = uni(threadIdx.x >> 6);
  const int S1 = d / 32, S2 = d / 64, ST = S1 + S2;

  // Tiles are drawn at run time, in the order of TileLists (long tables with the long tiles first measured slower): the first one
  // of a workgroup is given, the next one is drawn at the end of phase 1 of the one before, from the list of its XCD
  // (workgroup b runs on XCD b % 8) and, once that is empty, from the longest of the others.
  // A list is always drained by its own workgroups, whatever the others take of it.  What this is about is the end of the
  // kernel: a workgroup has a few tiles of 70 to 150 us.  With two tiles drawn ahead, lists that did not help each other and
  // runs of 32 to the last tile | so, between HIP events, three layers in turn, 128 x 4 sub-experts of 192 x 2048, budgets 8 to
  // 32, router bias N(0, 1) per expert: 3000 tokens 336 | 317 us, 8000 533 | 513, 16384 906 | 864; 12000 of 32 picks 980 | 950,
  // 65536 5365 | 5300.
  // A draw is a latency that wave 0 stands still for, with its copies, and its line is one that all workgroups wait for: the
  // number of tiles is kept in LDS, or short tiles take up to 40 % longer (see fused_help for the helping, which is one more).  Fused
  // kernel, number of tiles read with each draw | kept: 512 sub-experts of 32 picks, 192 x 2048, 1500 tokens 279 | 273, 64 x 2048, 5000 217 |
  // 195; 1024 of 16 picks, 64 x 512, 6772 116 | 95; 768 of 16 picks, 192 x 512, 1682 119 | 107; 64 of 64 picks, 128 x 256, 6535 95 | 82.
  const int xcd = blockIdx.x % N_XCD, slot = blockIdx.x / N_XCD;
  int32_t* dyn_lds = reinterpret_cast<int32_t*>(smem + C::OFF_DYN);
  auto lists_of = [&](int n) { return TileLists(n, n <= sorted ? 1 : RUN); };
  auto ask = [&](int list) { return lane == 0 ? atomicAdd(&hdr[HDR_DYN_FUSED + list], 1) : 0; };
  auto draw = [&](int asked) {  // wave 0, what ask(xcd) returned; -1: none is left
    const TileLists lists = lists_of(uni(dyn_lds[1]));  // (from the header it is a line that all workgroups' draws are waiting for)
    const int slots = gridDim.x / N_XCD;
    int from = xcd, i = slots + uni(asked);
    if (i >= lists.count(xcd) && !help) return -1;
#pragma nounroll
    for (int tries = 0; i >= lists.count(from); ++tries) {
      // lane l looks at list l
      const int l = lane % N_XCD;
      const int left = lists.count(l) - slots - __hip_atomic_load(&hdr[HDR_DYN_FUSED + l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      int most = left * N_XCD + l;
      most = max(most, __builtin_amdgcn_mov_dpp(most, 0xB1, 0xf, 0xf, true));   // lane ^ 1
      most = max(most, __builtin_amdgcn_mov_dpp(most, 0x4E, 0xf, 0xf, true));   // lane ^ 2
      most = uni(max(most, __builtin_amdgcn_mov_dpp(most, 0x141, 0xf, 0xf, true)));  // 7 - lane
      if (most < N_XCD || tries == N_XCD) return -1;
      from = most % N_XCD;
      i = slots + uni(ask(from));
    }
    return lists.tile(from, i);
  };
  const int n_tiles = hdr[HDR_MTILES];
  if (threadIdx.x == 0) dyn_lds[1] = n_tiles;  // (read behind the barriers of the first tile's start)
  const TileLists lists = lists_of(n_tiles);
  if (slot >= lists.count(xcd)) return;  // uniform over the workgroup

  const uint32_t lds0 = lds_offset(smem);
  const int32_t* pair_lds = reinterpret_cast<const int32_t*>(smem + C::OFF_PAIR);

  auto load_hdr = [&](int k, TileHdr& t) {
    const MTile m = tiles[k];
    t.g = uni(m.g);
    t.row0 = uni(m.row0);
    t.rows = uni(m.rows);
  };

  // A copy of the lane id that the optimiser cannot see through: per-lane constants of one
  // phase are derived from it at the start of that phase, so they do not occupy registers
  // during the other (phase 1 runs at the register limit).
  auto opaque_lane = [&]() {
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  };
  // (by hand: the compiler would take a 64-bit multiply-add and keep a pair of registers)
  const uint32_t d2 = (uint32_t)d * 2u;
  auto row_bytes = [&](int row) {
    uint32_t v;
    asm("v_mul_lo_u32 %0, %1, %2" : "=v"(v) : "v"(row), "s"(d2));
    return v;
  };
  // Offsets of the weight copies.  Phase 1: piece pc = 8 ring rows of 64 K-elements; ring row lr
  // holds block row lr & 31 of block lr >> 5 of the stage's half of the blocks: the piece starts at
  // a weight row that is the same for all lanes (piece_row, of the first half), and odd pieces have
  // the other swizzle (f1).  Phase 2: a wave copies ring rows 8 wv .. 8 wv + 7, piece j = 64
  // consecutive 16-byte positions of them.
  const uint32_t voff_w1 = row_bytes(lane >> 3) + (uint32_t)(((lane & 7) ^ (lane >> 4)) * 16);
  auto piece_row = [&](int pc) { return (pc >> 2) * 16 + (pc & 1) * 8 + ((pc & 2) ? IS : 0); };
  auto voff_w2 = [&](int j) {
    const uint32_t p = j * 64 + opaque_lane(), r2 = p / C::CPR;
    return (p ^ (uint32_t)f2<IS>(r2) ^ (uint32_t)f2<IS>(wv * 8)) * 16u;
  };
  // x offsets of the rows this lane copies (4 pieces of 8 rows) from a tile's slot list in LDS
  uint32_t xoff[4];
  auto x_offsets = [&](int parity) {
    const int l = opaque_lane();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int lr = j * 8 + (l >> 3), pos = l & 7;
      int tok = pair_lds[parity * BM + wv * 32 + lr] / k_max;
      tok = min(max(tok, 0), T - 1);
      xoff[j] = row_bytes(tok) + (uint32_t)((pos ^ f1(lr)) * 16);
    }
  };
  auto fetch_pairs = [&](const TileHdr& t, int parity) {  // waves 0..3, 64 rows each
    if (wv >= 4) return;
    const int r = max(min(wv * 64 + opaque_lane(), t.rows - 1), 0);
    dma4(sorted_pair + t.row0, (uint32_t)r * 4u, lds0 + C::OFF_PAIR + (uint32_t)(parity * BM + wv * 64) * 4u);
  };

  // ---- prologue: tile 0's slot list
  TileHdr cur, nxt;
  load_hdr(lists.tile(xcd, slot), cur);
  nxt = cur;
  bool has_next = false;  // known from stage next_at + 2 of a tile on
  int par = 0;            // which half of the slot-list buffer holds the current tile's entries
  fetch_pairs(cur, 0);
  wait_vmem<0>();
  raw_barrier();

  // ---- producer of weights, stage q + 3.  It keeps a running global pointer and LDS address and
  // counts the stages left in its phase; it runs ahead of the multiplying code across phase and
  // tile borders (the next tile's header `nxt` is known by then).  Behind the last tile's
  // last stage that stage is copied again (nobody reads it), so that every stage issues the same
  // number of copies.
  const int half_w = IS / 2 * d;  // elements from a gate row of the first half to that of the second
  const uint16_t* pw_ptr = w_gu + (size_t)cur.g * (2 * IS) * d + half_w - 64;
  int pw_g = cur.g, pw_phase = 0, pw_cnt = S1;
  const uint32_t pw_dst0 = lds0 + (uint32_t)(wv * WPW) * 1024u;
  uint32_t pw_dst = pw_dst0 + (NSW - 1) * C::W_SLOT;
  auto prep_w = [&]() {
    pw_dst = pw_dst == pw_dst0 + (NSW - 1) * C::W_SLOT ? pw_dst0 : pw_dst + C::W_SLOT;
    if (pw_cnt == 0) {
      if (pw_phase == 0) {  // on to the down weights of the same group
        pw_phase = 1;
        pw_cnt = S2;
        pw_ptr = w_dn + (size_t)pw_g * d * IS - 64 * IS;
      } else if (has_next) {  // on to the next tile
        pw_phase = 0;
        pw_cnt = S1;
        pw_g = nxt.g;
        pw_ptr = w_gu + (size_t)pw_g * (2 * IS) * d + half_w - 64;
      } else {
        return;
      }
    }
    pw_ptr += pw_phase ? 64 * IS : (pw_cnt & 1) ? half_w : 64 - half_w;  // S1 is even
    --pw_cnt;
  };
  auto copy_w1 = [&](int j) {
    const int pc = wv * WPW + j;
    copy_to_lds16(pw_ptr + (size_t)(uint32_t)(piece_row(pc) * d), voff_w1 ^ (uint32_t)((pc & 1) * 64), pw_dst + j * 1024u);
  };
  // (phase 1 has no registers for the offsets of phase 2: it computes them for the few copies)
  auto copy_w = [&](int j) {
    if (pw_phase) copy_to_lds16(pw_ptr + wv * 8 * IS, voff_w2(j), pw_dst + j * 1024u);
    else copy_w1(j);
  };
  // ---- x: the rows of stage pair m + 1 are copied during the first stage of pair m, once its
  // fragments of x are in registers; the next tile's first rows during phase 2
  const uint32_t x_dst = lds0 + C::OFF_X + (uint32_t)wv * X_WAVE;
  auto copy_x = [&](const uint16_t* src, int j) { copy_to_lds16(src, xoff[j], x_dst + j * 1024u); };

  // Stage numbering: q counts the stages this workgroup walks.  Per iteration q a wave
  //   (a) multiplies stage q (W(q) was published by the barrier of iteration q - 1, x is its own),
  //   (b) waits for its part of W(q+1) and passes barrier(q): every wave has finished reading
  //       W(q-1), and W(q+1) is published,
  //   (c) issues its copies of W(q+3) (into the slot of W(q-1)), then those of x, then the stores,
  //   (d) at the end of a stage pair of phase 1 waits for the next pair's x.
  // They are dealt out behind single MFMAs of (a) (Cfg).
  // Vector memory operations retire in issue order, so a wait is for "at most n pending" with n the
  // number of operations issued behind the ones waited for.  With w = WPW copies of weights per
  // stage and s stores per stage of phase 2 (from its second on):
  //   (d) x was issued in the pair's first stage, behind its W: behind it one stage's W
  //   (b) second stage of a pair: W(q+1) was issued in iteration q - 2, behind it W(q+2), x
  //       first stage of a pair: the wait (d) of iteration q - 1 was for x issued behind W(q+1)
  //       phase 2: W(q+1) was issued in iteration q - 2, behind it s(q-2), W(q+2), s(q-1)
  prep_w();
#pragma unroll
  for (int j = 0; j < WPW; ++j) copy_w(j);  // W(0)
  x_offsets(0);
  if (cur.rows > wv * 32) {
#pragma unroll
    for (int j = 0; j < 4; ++j) copy_x(x, j);
  }
  prep_w();
#pragma unroll
  for (int j = 0; j < WPW; ++j) copy_w(j);  // W(1)
  prep_w();
#pragma unroll
  for (int j = 0; j < WPW; ++j) copy_w(j);  // W(2)
  prep_w();
  wait_vmem<WPW>();  // W(0), x, W(1) have landed
  raw_barrier();

  // The next tile: wave 0 asks for a number ahead of SwiGLU, behind which it is there (the wait for it is also one for that
  // wave's copies: near the end of phase 2, 65 536 tokens of 32 picks took 5370 us instead of 5300), every wave picks it up two
  // barriers later, then the slot list is fetched.  The offsets of the next tile's rows are computed at stage xo_at, before
  // the first copy of them at ST - 4, which is also where the copies of its weights start.  Phases 2 of few stages have
  // no time for that: the tile is drawn at the start of the one before.
  const bool early = S2 < 13;
  const int next_at = early ? 0 : S1, xo_at = early ? S1 : ST - 5;
  auto next_tile = [&](int s) {  // at the start of stage next_at + s
    if (s == 2) {
      const int k = uni(dyn_lds[0]);
      has_next = k >= 0;
      if (has_next) load_hdr(k, nxt);
    }
    if (s == 4 && has_next) fetch_pairs(nxt, par ^ 1);
  };
  auto draw_next = [&](int asked) {
    if (wv != 0) return;
    const int k = draw(asked);
    if (lane == 0) dyn_lds[0] = k;
  };
  uint32_t c_w = 0;  // byte offset of the weight slot of stage q
  auto next_w = [&](uint32_t c) { return c + C::W_SLOT == NSW * C::W_SLOT ? 0u : c + C::W_SLOT; };
  constexpr int STEPS = C::STEPS;          // MFMAs per wave and stage, both phases

  for (;;) {
    if (early) draw_next(wv == 0 ? ask(xcd) : 0);
    if (cur.rows <= wv * 32) {
      // a wave whose 32 rows lie beyond the tile's rows only takes part in the copies and barriers
#pragma nounroll
      for (int s = 0; s < ST; ++s) {
        next_tile(s - next_at);
        wait_vmem<WPW>();
        raw_barrier();
#pragma unroll
        for (int j = 0; j < WPW; ++j) copy_w(j);
        if (s == xo_at) x_offsets(par ^ 1);
        if (s == ST - 4 && has_next && nxt.rows > wv * 32) {
#pragma unroll
          for (int j = 0; j < 4; ++j) copy_x(x, j);
        }
        prep_w();
        c_w = next_w(c_w);
      }
      wait_vmem<WPW>();  // x and W(1) of the next tile
    } else {
      bf16x8 hfrag[NBLK];
      {
        // ---- phase 1: acc1[blk] += W-block(blk) x-rows^T.  A stage is 64 K-elements (4 K steps) of half
        // of the blocks, so that a copy takes whole 128-byte lines: with 32 K-elements of all blocks
        // the L2 serves every line twice, half a line at a time (between HIP events, 16384
        // tokens of 20 picks, 512 sub-experts of 192 x 2048: 1016 us, with whole lines, also in the stores of y, 947).
        // The fragment of step i + PD is read right after the MFMA of step i is issued (the
        // scheduling barriers keep that order), and the stream of reads runs on into the next
        // stage (after the last stage of the phase it reads a slot whose values are not used).
        const int l = opaque_lane(), fr = l & 31, fh = l >> 5;
        // fragment reads: row wrow_gu(fr) (+ 32 per block), chunk 2 ks + fh; the swizzled chunks
        // of the K steps differ in two address bits
        const int rw = wrow_gu(fr);
        const uint32_t rd_w1 = lds0 + (uint32_t)(rw * 128 + ((fh ^ f1(rw)) * 16));
        const uint32_t rd_x = lds0 + (uint32_t)(C::OFF_X + wv * X_WAVE + fr * 128 + ((fh ^ f1(fr)) * 16));
        // Reads go into fixed registers (tied operands) and are waited for by count: left to itself
        // the compiler rotates them through twice as many and spills what the loop needs.
        bf16x8 xa[4] = {}, wf[PD] = {};
        auto rd_w = [&](uint32_t slot, auto step_c) {  // the weight fragment of `step` of the stage in `slot`
          constexpr int step = decltype(step_c)::value;
          read_lds16<step % C::HB * 4096>(wf[step % PD], (slot + rd_w1) ^ (uint32_t)(step / C::HB * 32));
        };
        auto rd_xf = [&](int ks) { read_lds16<0>(xa[ks], rd_x ^ (uint32_t)(ks * 32)); };
        f32x16 acc1[NBLK];
#pragma unroll
        for (int b = 0; b < NBLK; ++b)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc1[b][v] = 0.0f;
        rd_xf(0), rd_xf(1), rd_xf(2);
        static_loop<0, PD>([&](auto I) { rd_w(c_w, I); });
        const uint16_t* x_src = x + 64;
        auto stage = [&](int m, auto half_c) {
          constexpr int half = decltype(half_c)::value;
          const uint32_t nw = next_w(c_w);
          const int x_go = m + 1 < S1 / 2;
          __builtin_amdgcn_sched_barrier(0);
          static_loop<0, STEPS>([&](auto I) {
            constexpr int i = decltype(I)::value;
            // all but the youngest PD - 1 reads have returned: this step's weights, and x, which is
            // read more than PD steps ahead
            wait_lds<PD - 1>(wf[i % PD], xa[i / C::HB]);
            acc1[half * C::HB + i % C::HB] = mma<MATH>(wf[i % PD], xa[i / C::HB], acc1[half * C::HB + i % C::HB]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (i + PD < STEPS) rd_w(c_w, std::integral_constant<int, i + PD>{});
            else rd_w(nw, std::integral_constant<int, i + PD - STEPS>{});
            if constexpr (half == 0 && i == 0) rd_xf(3);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (i == C::BAR) {
              if constexpr (half == 1) wait_one_of<WPW + 4, WPW>(x_go ? WPW + 4 : WPW);
              raw_barrier();
            }
            if constexpr (i >= C::W0 && i < C::W_END) copy_w(i - C::W0);
            static_loop<0, 4>([&](auto J) {
              constexpr int j = decltype(J)::value;
              if constexpr (half == 0 && i == C::x_copy(j)) {
                if (x_go) copy_x(x_src, j);
              }
            });
            if constexpr (half == 1 && i >= C::XW && i < C::XW + 3) {
              if constexpr (i == C::XW) wait_vmem<WPW>();
              rd_xf(i - C::XW);
            }
            if constexpr (i == C::PREP) prep_w();
            __builtin_amdgcn_sched_barrier(0);
          });
          c_w = nw;
        };
#pragma nounroll
        for (int m = 0; m < S1 / 2; ++m) {
          if (early) next_tile(2 * m);
          stage(m, std::integral_constant<int, 0>{});
          stage(m, std::integral_constant<int, 1>{});
          x_src += 64;
        }
        static_loop<0, PD>([&](auto I) { wait_lds<0>(wf[decltype(I)::value], xa[decltype(I)::value]); });  // unused, but on their way
        const int asked = !early && wv == 0 ? ask(xcd) : 0;  // on its way during what follows
        // ---- SwiGLU: gate/up accumulators -> the bf16 K-step fragments of phase 2, block by
        // block (16 accumulator registers become 4), before anything of phase 2 is read
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
          const f32x16 v = acc1[b];
          const uint4 pk = make_uint4(pack_bf16x2(silu_mul(v[0], v[8]), silu_mul(v[1], v[9])),
                                      pack_bf16x2(silu_mul(v[2], v[10]), silu_mul(v[3], v[11])),
                                      pack_bf16x2(silu_mul(v[4], v[12]), silu_mul(v[5], v[13])),
                                      pack_bf16x2(silu_mul(v[6], v[14]), silu_mul(v[7], v[15])));
          hfrag[b] = __builtin_bit_cast(bf16x8, pk);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (!early) draw_next(asked);
      }
      // ---- phase 2: 64 output columns per stage (2 blocks of 32), K = Is (NBLK K steps) from
      // the register-resident h fragments; step i = K step i >> 1 of block i & 1
      const int l = opaque_lane(), fr = l & 31, fh = l >> 5;
      const int r2rd = wrow_dn(fr), f2rd = f2<IS>(r2rd);
      const uint32_t rd_w2_row = (uint32_t)r2rd * C::ROW2;
      auto rd_w2f = [&](uint32_t slot, int step) {
        const uint32_t co = (uint32_t)(((2 * (step >> 1) + fh) ^ f2rd) * 16);
        return *reinterpret_cast<const bf16x8*>(smem + slot + rd_w2_row + (step & 1) * 32 * C::ROW2 + co);
      };
      // Output staging: a lane ends a stage with 2 x 16 consecutive columns of ONE slot row, and
      // neighbouring lanes hold different rows, 2*d bytes apart; stored like that every lane's 16
      // bytes are a memory access of their own (measured: 64 accesses per instruction, and the
      // stores alone keep the address unit busy for a quarter of the kernel).  So 16 rows x 64
      // columns at a time go through 2 KiB of wave-private LDS and are stored with 8 adjacent lanes
      // covering a 128-byte line of a row.
      // A stage ends by packing its 64 columns to bf16 (16 registers); they are stored during the
      // next stage.
      unsigned char* epi = smem + C::OFF_EPI + wv * EPI_WAVE;
      const int er = fr & 15;
      const uint32_t epi_wr = (uint32_t)(er * 128 + ((2 * fh) ^ f1(er)) * 16);  // chunk 2 fh; 1, 4, 5 further: xor
      const uint32_t epi_rd = (uint32_t)l * 16u;  // row l >> 3 of the 8, position l & 7
      const int srow = wv * 32 + (l >> 3);        // + 8 per quarter
      const int echunk = (l & 7) ^ (l >> 4);      // the chunk that sits there (odd quarters: ^ 4)
      uint32_t vo[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) vo[k] = row_bytes(srow + 8 * k) + (uint32_t)(echunk ^ (k & 1) * 4) * 16u;
      uint16_t* ybase = y + (size_t)cur.row0 * d - 64;  // columns of the stage before
      // (set here: as an undefined value `out` would hold its registers through phase 1 as well)
      uint4 out[4] = {}, oq[2] = {};  // packed columns 0..7, 8..15 of either block; two quarters read back
      auto out_write = [&](auto H) {  // lane (row fr, half fh): columns 32 b + 16 fh + 0..15 of slot row 32 wv + fr
        if ((fr >> 4) == decltype(H)::value) {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            *reinterpret_cast<uint4*>(epi + (epi_wr ^ (uint32_t)((c >> 1) * 64 + (c & 1) * 16))) = out[c];
        }
      };
      auto out_read = [&](auto Q) {
        constexpr int k = decltype(Q)::value;
        oq[k & 1] = *reinterpret_cast<const uint4*>(epi + epi_rd + (k & 1) * 1024);
      };
      auto out_store = [&](auto Q) {
        constexpr int k = decltype(Q)::value;
        const uint4 v = oq[k & 1];
        if (srow + 8 * k < cur.rows) store16(ybase, vo[k], u32x4{v.x, v.y, v.z, v.w});
      };
      // stores issued per stage: the quarters that have a row of the tile
      const int n_st = min((cur.rows - wv * 32 + 7) / 8, 4);
      uint32_t vo_w2[WPW];
#pragma unroll
      for (int j = 0; j < WPW; ++j) vo_w2[j] = voff_w2(j);
      bf16x8 wd[PD];
#pragma unroll
      for (int i = 0; i < PD; ++i) wd[i] = rd_w2f(c_w, i);
#pragma nounroll
      for (int s2 = 0; s2 < S2; ++s2) {
        const uint32_t nw = next_w(c_w);
        if (!early) next_tile(s2);
        if (S1 + s2 == xo_at) x_offsets(par ^ 1);  // of the next tile, if there is one
        const int x_go = s2 == S2 - 4 && has_next && nxt.rows > wv * 32;
        f32x16 acc2[2];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc2[b][v] = 0.0f;
        __builtin_amdgcn_sched_barrier(0);
        static_loop<0, STEPS>([&](auto I) {
          constexpr int i = decltype(I)::value;
          acc2[i & 1] = mma<MATH>(wd[i % PD], hfrag[i >> 1], acc2[i & 1]);
          wd[i % PD] = i + PD < STEPS ? rd_w2f(c_w, i + PD) : rd_w2f(nw, i + PD - STEPS);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (i == C::BAR) {
            wait_one_of<WPW + 8, WPW + 4, WPW + 2, WPW>(s2 >= 3 ? WPW + 2 * n_st : s2 == 2 ? WPW + n_st : WPW);
            raw_barrier();
          }
          if constexpr (i >= C::W0 && i < C::W_END) {
            constexpr int j = i - C::W0;
            if (pw_phase) copy_to_lds16(pw_ptr + wv * 8 * IS, vo_w2[j], pw_dst + j * 1024u);
            else copy_w1(j);
          }
          static_loop<0, 4>([&](auto Q) {
            constexpr int k = decltype(Q)::value;
            if constexpr (i == C::x_copy(k)) {
              if (x_go) copy_x(x, k);
            }
            if constexpr (k < 2 && i == C::out_write(k)) out_write(Q);  // s2 = 0: nothing meaningful, not stored
            if constexpr (i == C::out_read(k)) out_read(Q);
            if constexpr (i == C::out_store(k)) {
              if (s2 > 0) out_store(Q);
            }
          });
          if constexpr (i == C::PREP) prep_w();
          __builtin_amdgcn_sched_barrier(0);
        });
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const f32x16 a = acc2[b];
          out[2 * b] = make_uint4(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(a[4], a[5]),
                                  pack_bf16x2(a[6], a[7]));
          out[2 * b + 1] = make_uint4(pack_bf16x2(a[8], a[9]), pack_bf16x2(a[10], a[11]), pack_bf16x2(a[12], a[13]),
                                      pack_bf16x2(a[14], a[15]));
        }
        ybase += 64;
        c_w = nw;
      }
      // W(1) of the next tile (and x, issued before it): behind it s, W, s
      wait_one_of<WPW + 8, WPW + 4, WPW + 2, WPW>(WPW + 2 * n_st);
      static_loop<0, 2>([&](auto H) {  // the last stage's columns
        constexpr int k = 2 * decltype(H)::value;
        out_write(H);
        out_read(std::integral_constant<int, k>{});
        out_read(std::integral_constant<int, k + 1>{});
        out_store(std::integral_constant<int, k>{});
        out_store(std::integral_constant<int, k + 1>{});
      });
    }
    // ---- next tile
    if (!has_next) {
      wait_vmem<0>();  // no copy may land in LDS that is no longer this workgroup's
      break;
    }
    cur = nxt;
    par ^= 1;
    has_next = false;
  }
}

// Whether a workgroup whose list is empty draws from the others'.  It has to look at them first, and even load has the
// workgroups do so all at once: 6 to 10 us, which long tiles get back with skewed load and short ones don't.  Fused kernel, us, not |
// helping, even load (512 sub-experts, 2500 tokens of 32 picks) and skewed (256, 6000 of 16): 192 x 512 78 | 88, 78 | 79; 128 x 1024 98.5 | 107.0,
// 103 | 96; 128 x 1536 151 | 158, 149 | 149; 128 x 2048 237 | 239, 201 | 199; 64 x 4096 281 | 287, 323 | 314; 192 x 1536 215.7 | 217.6, 186 | 179;
// 128 x 2560 252 | 258, 248 | 248; 192 x 2048 317 | 317, 247 | 241; 128 x 4096 446 | 445, 393 | 380; skewed, 512 of 192 x 2048, 16 384 tokens 911 | 869.
// Layer calls, helping over not, on average over 9 calls of 256 to 560 sub-experts, even load, skewed: 128 x 1792 1.007, 0.980; 64 x 3840 1.008, 0.981;
// 192 x 1280 1.015, 0.977; 64 x 4096 1.005, 0.990; 128 x 2048 0.996, 0.992; 192 x 1536 1.012, 0.975.
static bool fused_help(int d, int Is) { return (long)d * Is >= 128L * 2048; }

template <int IS, bool MATH>
static hipError_t launch_is(const uint16_t* x, const uint16_t* w_gu, const uint16_t* w_dn,
                            const int32_t* sorted_pair, const MTile* tiles, int32_t* hdr,
                            uint16_t* y, int T, int d, int k_max, int max_mtiles, int sorted, hipStream_t s) {
  hipError_t e = raise_lds_limit<ffn_fused_kernel<IS, MATH>>(Cfg<IS>::LDS_BYTES);
  if (e != hipSuccess) return e;
  const int grid = persistent_grid(max_mtiles, 1);
  const int help = fused_help(d, IS);
  ffn_fused_kernel<IS, MATH><<<grid, NT, Cfg<IS>::LDS_BYTES, s>>>(x, w_gu, w_dn, sorted_pair, tiles, hdr, y,
                                                            T, d, k_max, sorted, help);
  return hipGetLastError();
}

}  // namespace fused

// Shapes the fused kernel takes: Is in {64, 128, 192}; d a multiple of 64 with at least 8
// phase-1 stages (the next tile's slot list is fetched while the current tile runs); 32-bit
// byte offsets inside x and inside one sub-expert's weights.
bool ffn_fused_supported(int T, int d, int Is) {
  if (Is != 64 && Is != 128 && Is != 192) return false;
  if (d % 64 != 0 || d < 256) return false;
  if ((long)T * d * 2 >= (1L << 32) || (long)2 * Is * d * 2 >= (1L << 32)) return false;
  if ((long)FFN_BM * d * 2 >= (1L << 32)) return false;
  return true;
}

template <bool MATH>
static hipError_t launch_fused(const uint16_t* x, const uint16_t* w_gu, const uint16_t* w_dn,
                               const int32_t* sorted_pair, const MTile* tiles, int32_t* hdr,
                               uint16_t* y, int T, int d, int Is, int k_max, int max_mtiles,
                               int sorted, hipStream_t s) {
  if (max_mtiles <= 0) return hipSuccess;
  switch (Is) {
    case 64: return fused::launch_is<64, MATH>(x, w_gu, w_dn, sorted_pair, tiles, hdr, y, T, d, k_max, max_mtiles, sorted, s);
    case 128: return fused::launch_is<128, MATH>(x, w_gu, w_dn, sorted_pair, tiles, hdr, y, T, d, k_max, max_mtiles, sorted, s);
    case 192: return fused::launch_is<192, MATH>(x, w_gu, w_dn, sorted_pair, tiles, hdr, y, T, d, k_max, max_mtiles, sorted, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_ffn_fused_bf16(const uint16_t* x, const uint16_t* w_gu, const uint16_t* w_dn,
                                 const int32_t* sorted_pair, const MTile* tiles, int32_t* hdr,
                                 uint16_t* y, int T, int d, int Is, int k_max, int max_mtiles,
                                 int sorted, hipStream_t s) {
  return launch_fused<true>(x, w_gu, w_dn, sorted_pair, tiles, hdr, y, T, d, Is, k_max, max_mtiles, sorted, s);
}

// The kernel's memory operations alone (see mma<false>): what y holds afterwards means nothing.
hipError_t launch_ffn_fused_traffic_bf16(const uint16_t* x, const uint16_t* w_gu,
                                         const uint16_t* w_dn, const int32_t* sorted_pair,
                                         const MTile* tiles, int32_t* hdr, uint16_t* y, int T,
                                         int d, int Is, int k_max, int max_mtiles, hipStream_t s) {
  return launch_fused<false>(x, w_gu, w_dn, sorted_pair, tiles, hdr, y, T, d, Is, k_max, max_mtiles, 0, s);
}

}  // namespace mp
