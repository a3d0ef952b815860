// A tile of C = A B^T in which every element is ONE chain of binary32 fused multiply-adds in
// ascending k, on the matrix cores: v_mfma_f32_16x16x4_f32 adds its four k terms as four fused
// multiply-adds in ascending k with one rounding each (checked on the device against fmaf
// chains, subnormal sums included: bit-identical), so issuing it for k = 0, 4, 8, ... computes
// exactly that chain.  No split-K, no reordering.  Used for the router logits (fp32 or bf16
// operands) and for the fp32 FFN.
//
// What bounds it: the matrix pipe.  One instruction takes 32 cycles whether or not it depends on
// the previous one, so one chain per wave and one wave per SIMD already run at the full rate, and
// K = 2048 is 6.8 us for every 16 x 16 sub-tile a SIMD works through.  The fp32 matrix instructions
// do NOT overlap with vector ALU work (measured: an ALU instruction between two of them costs its
// 4 cycles plus about 16 for the change-over, LDS reads and scalar work nothing), so the loop
// contains no vector ALU instruction at all:
//   * bf16 operands are widened by the LDS read: ds_read_u16_d16_hi writes the upper half of a
//     register whose lower half stays zero;
//   * the eight LDS addresses of a lane never change: ring slot, sub-tile and k step are immediate
//     offsets (the stage loop is unrolled over the ring);
//   * the copies global -> LDS advance scalar bases.
//
// Operands: slabs of 128 bytes per row (64 bf16 or 32 fp32 of K) go global -> LDS directly into
// a ring of NS stages, NS - 2 of them in flight while one is multiplied and the next one is
// already published (its first fragments are read early).  Lane l feeds row l & 15 and k = l >> 4
// of a step.  Chunk c (16 bytes) of row r sits at position c ^ ((r >> 1) & 7): conflict-free reads.
#pragma once
#include "dma.h"

namespace mp {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

template <typename InT, int WM, int WN, int MT, int NT, int NS>
struct ChainTile {  // WM x WN waves, MT x NT sub-tiles of 16 x 16 per wave
  typedef InT In;
  static constexpr int M = MT, N = NT, WAVES_N = WN, STAGES = NS;
  static constexpr int NW = WM * WN, BT = WM * MT * 16, BE = WN * NT * 16, ROWS = BT + BE;
  static constexpr int CP = ROWS / 8 / NW;  // copy instructions (8 rows) per wave and stage
  static constexpr int STAGE = ROWS * 128;
  static constexpr int LDS_BYTES = NS * STAGE;
  static constexpr int KB = 128 / (int)sizeof(InT);
  static constexpr int STEPS = KB / 4;      // matrix steps (4 k) per stage
  static constexpr int NF = MT + NT;        // fragments per step
  // fragment sets and how many steps ahead they are read: lgkmcnt counts up to 15 reads
  static constexpr int R = NF <= 2 ? 8 : 4, PD = NF <= 2 ? 7 : NF <= 5 ? 3 : NF <= 7 ? 2 : 1;
  static_assert(CP * NW * 8 == ROWS && BT % 8 == 0, "whole copies");
  static_assert(NS >= 3 && (NS - 1) * CP < 63 && PD * NF <= 15 && STEPS % R == 0, "counters");
  static_assert(LDS_BYTES <= 65536, "immediate offsets of 16 bits");
};

// value of this lane's element: bf16 into the upper half (the lower half stays as it is: zero), fp32 whole
template <typename InT, int OFF>
__device__ __forceinline__ void read_elem(uint32_t& v, uint32_t addr) {
  if constexpr (sizeof(InT) == 2)
    asm volatile("ds_read_u16_d16_hi %0, %1 offset:%2" : "+v"(v) : "v"(addr), "n"(OFF));
  else
    asm volatile("ds_read_b32 %0, %1 offset:%2" : "+v"(v) : "v"(addr), "n"(OFF));
}

// Copy j of this wave (CP of them per stage) fetches rows 8 (wave CP + j) .. + 7 of the stage, A rows
// first: lane i fetches 16-byte chunk chain_chunk(row) of row 8 (wave CP + j) + i / 8.
__device__ __forceinline__ int chain_chunk(int row) { return (threadIdx.x & 7) ^ ((row >> 1) & 7); }

// acc[i][j] of wave (wm, wn), sub-tile rows (wm MT + i) 16 .., columns (wn NT + j) 16 ..: accumulator v
// of lane l is row 4 (l >> 4) + v, column l & 15.  copy(j, stage, lds) issues copy j of `stage`.
// All LDS reads of the tile have returned when it ends, but other waves may still be reading.
// COPIES_APART: waves NW .. 2 NW - 1 of the workgroup copy, wave NW + w what else were the copies of wave w; their acc is not
// set.  For short rows of sub-tiles on a SIMD: an LDS read behind a copy of the same wave waits until the copy's addresses are
// out, some 45 cycles, and the multiply with it.  The tile alone, one token, 512 rows, K = 256 | 2048 | 4096: 2.0 | 9.8 | 18.8 us,
// 10.5 cycles per k; apart 2.1 | 8.2 | 15.3, 8.3 per k.
template <class C, bool COPIES_APART = false, class Copy>
__device__ __forceinline__ void chain_tile(unsigned char* smem, int ns, Copy&& copy, f32x4_t (&acc)[C::M][C::N]) {
  typedef typename C::In InT;
  constexpr int CP = C::CP, PD = C::PD, R = C::R, NF = C::NF, NS = C::STAGES, MT = C::M, NT = C::N;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wv = COPIES_APART ? w % C::NW : w, wm = wv / C::WAVES_N, wn = wv % C::WAVES_N;
  const uint32_t lds0 = lds_offset(smem);
  const uint32_t dst0 = lds0 + (uint32_t)(wv * CP) * 1024u;
  auto produce = [&](int stage, int slot) {
    if (stage < ns) {
#pragma unroll
      for (int j = 0; j < CP; ++j) copy(j, stage, dst0 + (uint32_t)(slot * C::STAGE + j * 1024));
    }
  };
  auto landed_first = [&] {  // this wave's copies of stage 0
    if (ns >= NS - 1)
      wait_vmem<(NS - 2) * CP>();
    else
      wait_vmem<0>();
  };
  auto landed_after = [&](int q) {  // of stage q + 1
    if (q + NS - 2 < ns)
      wait_vmem<(NS - 3) * CP>();
    else
      wait_vmem<0>();
  };
  if (!COPIES_APART || w >= C::NW) {
#pragma unroll
    for (int i = 0; i < NS - 1; ++i) produce(i, i);
  }
  if (COPIES_APART && w >= C::NW) {
    landed_first();
    raw_barrier();
    int slot = NS - 1;
    for (int q = 0; q < ns; ++q) {
      landed_after(q);
      raw_barrier();
      produce(q + NS - 1, slot);
      slot = slot == NS - 1 ? 0 : slot + 1;
    }
    return;
  }

  // consumer: addresses of this lane's element of chunk c, in token rows and in sub-expert rows
  const int r = lane & 15, g = lane >> 4;
  uint32_t at[8], bt[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const uint32_t o = lds0 + (uint32_t)(r * 128 + ((c ^ ((r >> 1) & 7)) * 16) + g * (int)sizeof(InT));
    at[c] = o + (uint32_t)(wm * MT) * 2048u;
    bt[c] = o + (uint32_t)(C::BT + wn * NT * 16) * 128u;
  }
  uint32_t fa[R][MT], fb[R][NT];
#pragma unroll
  for (int s = 0; s < R; ++s) {
#pragma unroll
    for (int i = 0; i < MT; ++i) fa[s][i] = 0;
#pragma unroll
    for (int i = 0; i < NT; ++i) fb[s][i] = 0;
  }
  auto read = [&](auto slot_c, auto step_c) {  // the fragments of step (0 .. STEPS - 1) of ring slot
    constexpr int SLOT = decltype(slot_c)::value, STEP = decltype(step_c)::value;
    constexpr int CH = STEP * 4 * (int)sizeof(InT) / 16;
    constexpr int OFF = SLOT * C::STAGE + (STEP * 4 * (int)sizeof(InT)) % 16;
    static_loop<0, MT>([&](auto i) { read_elem<InT, OFF + decltype(i)::value * 2048>(fa[STEP % R][i], at[CH]); });
    static_loop<0, NT>([&](auto i) { read_elem<InT, OFF + decltype(i)::value * 2048>(fb[STEP % R][i], bt[CH]); });
  };
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

  if (!COPIES_APART) landed_first();
  raw_barrier();
  static_loop<0, PD>([&](auto s) { read(std::integral_constant<int, 0>{}, s); });
  // Stage q: its successor's copies have landed for this wave (wait) and, behind the barrier,
  // for all.  The barrier also frees the slot of stage q - 1 (every wave had its last fragments in
  // registers before its last multiply), which takes stage q + NS - 1.
  for (int q0 = 0; q0 < ns; q0 += NS) {
    static_loop<0, NS>([&](auto slot_c) {
      constexpr int SLOT = decltype(slot_c)::value, NSLOT = (SLOT + 1) % NS;
      const int q = q0 + SLOT;
      if (q >= ns) return;
      if (!COPIES_APART) landed_after(q);
      raw_barrier();
      if (!COPIES_APART) produce(q + NS - 1, (SLOT + NS - 1) % NS);
      __builtin_amdgcn_sched_barrier(0);
      static_loop<0, C::STEPS>([&](auto step_c) {
        constexpr int S = decltype(step_c)::value, A = S + PD;
        if constexpr (A < C::STEPS)
          read(slot_c, std::integral_constant<int, A>{});
        else  // after the last stage: an old slot, not used
          read(std::integral_constant<int, NSLOT>{}, std::integral_constant<int, A - C::STEPS>{});
        // the reads of this step have returned (the tie brings a wait state in front of the multiply: 2741 x 128
        // logits 22.0 -> 22.3 us, 16 384 x 512 240 either way)
        uint32_t(&ua)[MT] = fa[S % R], (&ub)[NT] = fb[S % R];
        if constexpr (MT == 2)
          wait_lds<PD * NF>(ua[0], ua[1], ub[0], ub[1]);
        else if constexpr (NT == 2)
          wait_lds<PD * NF>(ua[0], ub[0], ub[1]);
        else
          wait_lds<PD * NF>(ua[0], ub[0]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j)  // ascending k
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(ua[i]), __uint_as_float(ub[j]),
                                                            acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  }
  // fragments read ahead: not used, but on their way into registers
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int s = 0; s < R; ++s) {
#pragma unroll
    for (int i = 0; i < MT; ++i) asm volatile("" ::"v"(fa[s][i]));
#pragma unroll
    for (int i = 0; i < NT; ++i) asm volatile("" ::"v"(fb[s][i]));
  }
}

}  // namespace mp
