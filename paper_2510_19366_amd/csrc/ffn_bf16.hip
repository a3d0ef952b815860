// bf16 grouped SwiGLU FFN on MFMA (Sec. 3.2.1, Eq. 1-3): the two grouped GEMMs
//   gate-up : h[p, c] = SiLU(x[t_p,:] . Wg[g,c,:]) * (x[t_p,:] . Wu[g,c,:])
//   down    : y[p, q] = sum_c h[p,c] * Wd[g,q,c]
// over ragged groups, as persistent workgroups that walk (m-tile, n-tile) items.
//
// Tile: 256 slot rows x 256 weight rows, 8 wavefronts (4 along the slot rows x 2 along the weight
// rows), one workgroup per CU, v_mfma_f32_32x32x16_bf16.  Drivers:
//   run_items_ring (K > 192): operands go global -> LDS directly through a ring of two stages of
//     64 K-elements that is refilled piece by piece;
//   run_items (shorter K, and tiles whose outputs are 4 GiB and more): 64-wide slabs through registers
//     into a double-buffered, XOR-swizzled LDS tile, one slab ahead of the MFMAs.  The weight block is the MFMA's first operand and its
//     rows are fed in a permuted order, so that a lane ends up with 8 or 16 consecutive output
//     columns of one slot row and stores them as 16-byte words (ffn_few_kernel likewise).
// Few rows per sub-expert take ffn_few_kernel (tiles of 64 or 128 weight rows, see ffn_few_blocks), and so does the
// gate-up of up to 32 neurons.
// Narrow sub-experts (Is in {64, 128, 192}) take the fused kernel in ffn_fused_bf16.hip
// instead; these two kernels serve every other shape.
#include <type_traits>

#include "dispatch_common.h"
#include "dma.h"
#include "ffn_common.h"
#include "topk_wave.h"

namespace mp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int BM = FFN_BM;   // slot rows per tile
constexpr int BN = 256;      // weight rows per tile
constexpr int BK = 64;       // bf16 elements of K per stage: 128 bytes per row
constexpr int NT_ = 512;     // threads per workgroup
constexpr int NB = 4, MB = 2;  // 32-row weight and slot blocks per wave

// Block b (0..7) of 32 rows of the tile that a wave multiplies.  Slot rows are dealt out so that
// every 64 rows of a ragged tile add one block to every SIMD (waves v and v + 4 share SIMD v mod 4,
// i.e. slot quarters wm and wm + 2): a tile takes as long as its rows, in steps of 64.  Weight
// rows: blocks 0..3 are the tile's first half (B0), 4..7 its second (B1); a wave takes two
// neighbouring blocks of either (64 consecutive output columns of the down projection).
__device__ __forceinline__ int slot_block(int wm, int mb) { return wm + 4 * mb; }
__device__ __forceinline__ int weight_block(int wn, int nb) { return (nb >> 1) * 4 + 2 * wn + (nb & 1); }

// 16-byte chunk c (0..7) of row r is stored at chunk position c ^ f(r).  A fragment
// read is served 16 lanes at a time (16 rows at one chunk index) from 64 banks: even
// rows fall into one half of the banks, odd rows into the other, so f must differ
// over the 8 rows of equal parity that one such group reads.
//   SWZ_SEQ: the group reads 16 consecutive rows            -> f = (r >> 1) & 7
//   SWZ_SPLIT: it reads rows {0..7, 16..23} or {8..15, 24..31} of a 32-row block
//                                                           -> f = ((r >> 1) & 3) | ((r >> 4) & 1) << 2
constexpr int SWZ_SEQ = 0, SWZ_SPLIT = 1;
template <int MODE>
__device__ __forceinline__ int swz_f(int r) {
  return MODE == SWZ_SEQ ? ((r >> 1) & 7) : (((r >> 1) & 3) | (((r >> 4) & 1) << 2));
}
template <int MODE>
__device__ __forceinline__ int swz(int r, int c) {  // in elements
  return r * BK + ((c ^ swz_f<MODE>(r)) << 3);
}

// 32-bit byte offsets into a tile's output rows
__host__ __device__ constexpr bool out_fits(int n_cols) { return (long)BM * n_cols * 2 < (1L << 32); }

// Tile header fields are the same for every lane: keep them in scalar registers.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ uint32_t pack2(float a, float b) { return pack_bf16x2(a, b); }

// What every lane knows about a work item: group, first slot row, valid rows, first
// output column (or neuron) of the n-tile.  Wave-uniform.
struct Sc {
  int g, row0, rows, n0;
};
// 32-row slot blocks of wave row wm that hold a valid row
__device__ __forceinline__ int blocks_on(const Sc& sc, int wm) {
  const int n = (sc.rows + 31) >> 5;
  return uni((n > slot_block(wm, 0) ? 1 : 0) + (n > slot_block(wm, 1) ? 1 : 0));
}

// ---------------------------------------------------------------- gate-up
// A tile holds BN/2 neurons.  Each 32-row weight block is 16 neurons: rows 0..15 are their
// gate rows, rows 16..31 their up rows, so a lane's accumulators v and v + 8 are the gate
// and up value of one neuron.  MFMA row i = 8a + 4hi + b reads block row 16*(a >> 1) +
// 8hi + 4(a & 1) + b, which makes accumulators 0..7 of a lane the 8 consecutive neurons
// 8hi .. 8hi + 7.
struct GateUpOp {
  static constexpr int WSWZ = SWZ_SEQ;
  static constexpr int N_PER_ROW = 2;  // weight rows per output column
  static constexpr bool GATHER = true;
  const uint16_t* x;
  const uint16_t* w_gu;
  const int32_t* sorted_pair;
  uint16_t* h;
  int T, d, Is, k_max;

  __device__ __forceinline__ int K() const { return d; }
  __device__ __forceinline__ int n_cols() const { return Is; }
  static __device__ __forceinline__ int wrow(int i) {
    const int a = i >> 3, hi = (i >> 2) & 1, b = i & 3;
    return 16 * (a >> 1) + 8 * hi + 4 * (a & 1) + b;
  }
  __device__ __forceinline__ const int32_t* idx_src(const Sc& sc, int r) const {
    return sorted_pair + sc.row0 + min(r, sc.rows - 1);
  }
  // rows are K elements each, behind a wave-uniform base
  __device__ __forceinline__ void bases(const Sc& sc, const uint16_t*& ba, const uint16_t*& bb) const {
    ba = x;
    bb = w_gu + (size_t)sc.g * 2 * Is * d;
  }
  // slot row r with slot-list entry `pair`, weight row br of the tile
  __device__ __forceinline__ int a_row(const Sc&, int, int pair) const { return min(max(pair / k_max, 0), T - 1); }
  __device__ __forceinline__ int b_row(const Sc& it, int br) const {
    const int blk = br >> 5, rr = br & 31;
    const int neuron = min(it.n0 + blk * 16 + (rr & 15), Is - 1);
    return (rr >> 4) ? Is + neuron : neuron;
  }
  bool offsets_fit() const {  // 32-bit byte offsets into the operands
    return (long)T * d * 2 < (1L << 32) && 2L * Is * d * 2 < (1L << 32);
  }
  // ---- ring driver (weight rows as second operand: lane n of a block holds ITS row's products with 16
  // slot rows).  The two blocks of a phase are the gate and the up rows of the same 32 neurons.
  static constexpr int CHUNK = 32;  // output columns of a wave and phase
  static constexpr int PUTS = 8;    // stores per phase and slot block
  __device__ __forceinline__ int ring_row(const Sc& it, int br) const {
    const int neuron = min(it.n0 + (br >> 7) * 64 + ((br >> 6) & 1) * 32 + (br & 31), Is - 1);
    return (br & 32) ? Is + neuron : neuron;
  }
  __device__ __forceinline__ uint16_t* out() const { return h; }
  // offset of what a lane stores: even lanes row v, odd lanes row v + 1 of two neighbouring neurons
  __device__ __forceinline__ uint32_t put_off(int lane) const {
    return ((uint32_t)(4 * (lane >> 5) + (lane & 1)) * (uint32_t)Is + (uint32_t)(lane & 30)) * 2u;
  }
  // slot rows v, v + 1 (v even) of a slot block: one store of 4 rows x 64 bytes
  template <class Store>
  __device__ __forceinline__ void put(const f32x16& a0, const f32x16& a1, int v, Store&& store) const {
    const uint32_t mine = pack2(silu_mul(a0[v], a1[v]), silu_mul(a0[v + 1], a1[v + 1]));
    const uint32_t other = __builtin_amdgcn_mov_dpp(mine, 0xB1, 0xF, 0xF, true);  // of the lane's neighbour
    // even lanes: low halves (row v), odd lanes: high halves (row v + 1)
    store(v, __builtin_amdgcn_perm(other, mine, (threadIdx.x & 1) ? 0x03020706u : 0x05040100u));
  }
  // one lane's share of a 32-row weight block: 8 neurons of one slot row
  __device__ __forceinline__ void store_block(const Sc& it, int row, int block, int hi, const f32x16& v) const {
    const int col = it.n0 + block * 16 + 8 * hi;
    if (col < Is)  // Is % 32 == 0 and col % 8 == 0: all 8 neurons are inside
      *reinterpret_cast<uint4*>(h + (size_t)(it.row0 + row) * Is + col) = make_uint4(
          pack2(silu_mul(v[0], v[8]), silu_mul(v[1], v[9])), pack2(silu_mul(v[2], v[10]), silu_mul(v[3], v[11])),
          pack2(silu_mul(v[4], v[12]), silu_mul(v[5], v[13])), pack2(silu_mul(v[6], v[14]), silu_mul(v[7], v[15])));
  }
  // ---- few rows: weight rows 0..7 of a wave are the gate rows of 8 neurons, 8..15 their up rows, so lanes 0..31 hold
  // gates and lanes 32..63 the same neurons' ups
  __device__ __forceinline__ int few_row(const Sc& it, int i) const { return it.n0 + (i & 7) + (i >> 3) * Is; }
  __device__ __forceinline__ void few_store(const Sc& it, int row, int g, const f32x4& v) const {
    float u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t b = __float_as_uint(v[i]);
      u[i] = __uint_as_float(__builtin_amdgcn_permlane32_swap(b, b, false, false)[1]);  // of lane + 32
    }
    if (g < 2 && row < it.rows)
      *reinterpret_cast<uint2*>(h + (size_t)(it.row0 + row) * Is + it.n0 + 4 * g) =
          make_uint2(pack2(silu_mul(v[0], u[0]), silu_mul(v[1], u[1])), pack2(silu_mul(v[2], u[2]), silu_mul(v[3], u[3])));
  }
  __device__ __forceinline__ void epilogue(const Sc& it, f32x16 (&acc)[NB][MB], uint16_t*) const {  // short K
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int wm = wv >> 1, wn = wv & 1;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int row = slot_block(wm, mb) * 32 + (lane & 31);
      if (row >= it.rows) continue;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) store_block(it, row, weight_block(wn, nb), lane >> 5, acc[nb][mb]);
    }
  }
};

// ---------------------------------------------------------------- down
// A 32-row weight block is 32 consecutive output columns.  MFMA row i = 8a + 4hi + b reads
// block row 16hi + 4a + b, so a lane's 16 accumulators are the consecutive columns
// 16hi .. 16hi + 15.
constexpr int EPI_WAVE_BYTES = 2048;
struct DownOp {
  static constexpr int WSWZ = SWZ_SPLIT;
  static constexpr int N_PER_ROW = 1;
  static constexpr bool GATHER = false;
  const uint16_t* h;
  const uint16_t* w_dn;
  uint16_t* y;
  int d, Is;

  __device__ __forceinline__ int K() const { return Is; }
  __device__ __forceinline__ int n_cols() const { return d; }
  static __device__ __forceinline__ int wrow(int i) {
    const int a = i >> 3, hi = (i >> 2) & 1, b = i & 3;
    return 16 * hi + 4 * a + b;
  }
  __device__ __forceinline__ const int32_t* idx_src(const Sc&, int) const { return nullptr; }
  __device__ __forceinline__ void bases(const Sc& sc, const uint16_t*& ba, const uint16_t*& bb) const {
    ba = h + (size_t)sc.row0 * Is;
    bb = w_dn + (size_t)sc.g * d * Is;
  }
  __device__ __forceinline__ int a_row(const Sc& sc, int r, int) const { return min(r, sc.rows - 1); }
  __device__ __forceinline__ int b_row(const Sc& it, int br) const { return min(it.n0 + br, d - 1); }
  bool offsets_fit() const { return (long)(d < BM ? BM : d) * Is * 2 < (1L << 32); }
  // ---- ring driver: the two blocks of a phase are the even and the odd ones of 64 columns, so that
  // a lane holds two neighbouring columns
  static constexpr int CHUNK = 64;
  static constexpr int PUTS = 16;
  __device__ __forceinline__ int ring_row(const Sc& it, int br) const {
    return min(it.n0 + (br & ~63) + (br & 31) * 2 + ((br >> 5) & 1), d - 1);
  }
  __device__ __forceinline__ uint16_t* out() const { return y; }
  __device__ __forceinline__ uint32_t put_off(int lane) const {
    return ((uint32_t)(4 * (lane >> 5)) * (uint32_t)d + (uint32_t)(lane & 31) * 2u) * 2u;
  }
  // slot rows v, v + 1: two stores of 2 rows x 128 bytes
  template <class Store>
  __device__ __forceinline__ void put(const f32x16& a0, const f32x16& a1, int v, Store&& store) const {
    store(v, pack2(a0[v], a1[v]));
    store(v + 1, pack2(a0[v + 1], a1[v + 1]));
  }
  // ---- few rows
  __device__ __forceinline__ int few_row(const Sc& it, int i) const { return it.n0 + i; }
  __device__ __forceinline__ void few_store(const Sc& it, int row, int g, const f32x4& v) const {
    if (row < it.rows)
      *reinterpret_cast<uint2*>(y + (size_t)(it.row0 + row) * d + it.n0 + 4 * g) = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
  }
  // one lane's share of a 32-row weight block: 16 columns of one slot row
  __device__ __forceinline__ void store_block(const Sc& it, int row, int block, int hi, const f32x16& v) const {
    const int col = it.n0 + block * 32 + 16 * hi;
    if (col >= d) return;  // d % 64 == 0: all 16 columns are inside
    uint4* o = reinterpret_cast<uint4*>(y + (size_t)(it.row0 + row) * d + col);
    o[0] = make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
    o[1] = make_uint4(pack2(v[8], v[9]), pack2(v[10], v[11]), pack2(v[12], v[13]), pack2(v[14], v[15]));
  }
  // (short K)  16 rows x 64 columns at a time go through wave-private LDS and are read back row-major, so
  // that every store instruction writes 8 rows x 128 contiguous bytes (whole cache lines) instead
  // of 64 scattered 16-byte pieces: y is the layer's largest HBM stream.  LDS rows are 128 bytes,
  // 16-byte chunk c of row r sits at position c ^ ((r >> 1) & 7): conflict-free both ways.
  // Rows beyond the tile are dropped by the buffer's bound, and blocks of 16 without a row skipped.
  // (Tiles of 4 GiB and more, which a buffer cannot bound, are stored as they stand.)
  __device__ __forceinline__ void epilogue(const Sc& it, f32x16 (&acc)[NB][MB], uint16_t* scratch) const {
    const int lane = threadIdx.x & 63, wv = uni(threadIdx.x >> 6);
    const int wm = wv >> 1, wn = wv & 1;
    if (!out_fits(d)) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int row = slot_block(wm, mb) * 32 + (lane & 31);
        if (row >= it.rows) continue;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) store_block(it, row, weight_block(wn, nb), lane >> 5, acc[nb][mb]);
      }
      return;
    }
    const int r = lane & 15, hi = lane >> 5, sw = (r >> 1) & 7;
    const uint32_t ld2 = (uint32_t)d * 2u;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(y + (size_t)it.row0 * d + it.n0, 0,
                                                        (int)((uint32_t)it.rows * ld2 - (uint32_t)it.n0 * 2u), 0x00020000);
    uint32_t at = (uint32_t)(lane >> 3) * ld2 + (uint32_t)(lane & 7) * 16u;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int row0 = slot_block(wm, mb) * 32;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int col0 = weight_block(wn, 2 * half) * 32;
        if (it.n0 + col0 >= d) continue;  // d % 64 == 0: a half is inside or outside as a whole
#pragma unroll
        for (int q = 0; q < 2; ++q) {  // rows 16 q .. 16 q + 15 of the block
          if (row0 + 16 * q >= it.rows) continue;
          if (((lane >> 4) & 1) == q) {
#pragma unroll
            for (int nbl = 0; nbl < 2; ++nbl) {
              const f32x16 v = acc[half * 2 + nbl][mb];
              const int c = nbl * 4 + 2 * hi;
              *reinterpret_cast<uint4*>(scratch + r * 64 + ((c ^ sw) << 3)) =
                  make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
              *reinterpret_cast<uint4*>(scratch + r * 64 + (((c + 1) ^ sw) << 3)) = make_uint4(
                  pack2(v[8], v[9]), pack2(v[10], v[11]), pack2(v[12], v[13]), pack2(v[14], v[15]));
            }
          }
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int row = j * 8 + (lane >> 3), c = lane & 7;
            const u32x4 o = *reinterpret_cast<const u32x4*>(scratch + row * 64 + ((c ^ ((row >> 1) & 7)) << 3));
            asm volatile("" : "+v"(at));  // or the offsets of all pieces are kept in registers
            __builtin_amdgcn_raw_buffer_store_b128(
                o, rsrc, (int)(at + (uint32_t)(row0 + 16 * q + 8 * j) * ld2 + (uint32_t)col0 * 2u), 0, 0);
          }
        }
      }
    }
  }
};

// ---------------------------------------------------------------- short K
// Slabs of 64 K-elements through registers into a double-buffered LDS tile, one barrier per slab.
// Items are one to three slabs here, so what bounds it is the way to an item's first slab: tile header,
// slot list, rows.  Each of the three is fetched while earlier items are multiplied: the header three
// items ahead, the slot list two, the first slab during the last slab of the item before.  Measured between
// HIP events, 256 sub-experts of 32 | 96 x 2048, 4 to 16 picks, down: 8192 tokens 94 | 169 -> 84 | 131 us, 1024 tokens
// 31 | 47 -> 24 | 38, against starting each item with its own loads (and 64-bit offsets and every block of 16 rows
// in the epilogue).  The addresses of the loads and stores are recomputed throughout: with them in
// registers the accumulators spill, and a reload waits for the loads in flight.
constexpr int LD = BM * 8 / NT_;  // 16-byte loads per thread and slab, slot rows and weight rows alike
constexpr size_t SLAB_LDS_BYTES = 2 * (size_t)(BM + BN) * BK * 2;
constexpr size_t SHORT_LDS_BYTES = SLAB_LDS_BYTES + (NT_ / 64) * EPI_WAVE_BYTES;

template <class Op>
__device__ __forceinline__ void run_items(const Op& op, const MTile* __restrict__ tiles,
                                          const int32_t* __restrict__ hdr, int n_tiles_n) {
  extern __shared__ __align__(16) uint16_t smem[];
  const int lane = threadIdx.x & 63, wv = uni(threadIdx.x >> 6), wm = wv >> 1, wn = wv & 1;
  const int wrow = Op::wrow(lane & 31);
  uint16_t* epi_lds = smem + SLAB_LDS_BYTES / 2 + (size_t)wv * (EPI_WAVE_BYTES / 2);
  const int lc = threadIdx.x & 7, lr = threadIdx.x >> 3;  // this thread copies chunk lc of rows lr + 64 i
  const int K = op.K(), nslab = (K + BK - 1) / BK;
  const int total = hdr[HDR_MTILES] * n_tiles_n;
  const ItemRange ir = xcd_items(total);
  if (ir.begin >= ir.end) return;  // the whole workgroup
  auto load_sc = [&](int item) {  // an item past the end: the first one, in bounds and not used
    if (item >= ir.end) item = ir.begin;
    const MTile t = tiles[item / n_tiles_n];
    Sc sc;
    sc.g = uni(t.g);
    sc.row0 = uni(t.row0);
    sc.rows = uni(t.rows);
    sc.n0 = uni(item % n_tiles_n) * (BN / Op::N_PER_ROW);
    return sc;
  };
  int pair[LD] = {}, row[LD] = {};  // slot-list entries of the next item, operand rows of the one being loaded
  auto load_pairs = [&](const Sc& sc) {
    if constexpr (Op::GATHER)
#pragma unroll
      for (int i = 0; i < LD; ++i) pair[i] = *op.idx_src(sc, lr + 64 * i);
  };
  auto enter = [&](const Sc& sc) {
    if constexpr (Op::GATHER)
#pragma unroll
      for (int i = 0; i < LD; ++i) row[i] = op.a_row(sc, lr + 64 * i, pair[i]);
  };
  // (everything else about the addresses is recomputed: the accumulators need the registers)
  u32x4 ra[LD], rb[LD];
  auto gload = [&](const Sc& sc, int k0) {
    const int k = min(k0 + lc * 8, K - 8);  // K % 64 == 32: chunks 4..7 do not exist (not used)
    const uint16_t *ba, *bb;
    op.bases(sc, ba, bb);
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      const int r = lr + 64 * i, ao = Op::GATHER ? row[i] : op.a_row(sc, r, 0);
      ra[i] = *reinterpret_cast<const u32x4*>(ba + (size_t)ao * K + k);
      rb[i] = *reinterpret_cast<const u32x4*>(bb + (size_t)op.b_row(sc, r) * K + k);
    }
  };
  auto sstore = [&](int buf) {
    uint16_t* sa = smem + buf * (BM + BN) * BK;
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      *reinterpret_cast<u32x4*>(sa + swz<SWZ_SEQ>(lr + 64 * i, lc)) = ra[i];
      *reinterpret_cast<u32x4*>(sa + BM * BK + swz<Op::WSWZ>(lr + 64 * i, lc)) = rb[i];
    }
  };

  Sc cur = load_sc(ir.begin), nxt = load_sc(ir.begin + ir.step), aft = load_sc(ir.begin + 2 * ir.step);
  load_pairs(cur);
  enter(cur);
  gload(cur, 0);
  load_pairs(nxt);
  int buf = 0;
  for (int item = ir.begin; item < ir.end; item += ir.step) {
    f32x16 acc[NB][MB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[nb][mb][v] = 0.0f;
    const int mb_on = blocks_on(cur, wm);
    for (int s = 0; s < nslab; ++s) {
      // the buffer was read two slabs ago, and every wave has passed the barrier of the slab between
      sstore(buf);
      __syncthreads();
      if (s + 1 < nslab) {
        gload(cur, (s + 1) * BK);
      } else if (item + ir.step < ir.end) {
        enter(nxt);
        gload(nxt, 0);
        load_pairs(aft);
      }
      const uint16_t* sa = smem + buf * (BM + BN) * BK;
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        if (ks == 2 && s * BK + 32 == K) break;  // K % 64 == 32
        const int c = ks * 2 + (lane >> 5);
        bf16x8 fw[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          fw[nb] = *reinterpret_cast<const bf16x8*>(sa + BM * BK + swz<Op::WSWZ>(weight_block(wn, nb) * 32 + wrow, c));
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          if (mb < mb_on) {
            const bf16x8 ft = *reinterpret_cast<const bf16x8*>(sa + swz<SWZ_SEQ>(slot_block(wm, mb) * 32 + (lane & 31), c));
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
              acc[nb][mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[nb], ft, acc[nb][mb], 0, 0, 0);
          }
      }
      buf ^= 1;
    }
    const Sc done = cur;
    cur = nxt;
    nxt = aft;
    aft = load_sc(item + 3 * ir.step);
    op.epilogue(done, acc, epi_lds);
  }
}

// ---------------------------------------------------------------- ring driver
// Stages of 64 K-elements: 128 bytes per row and copy, so that 8 lanes of a copy instruction fetch
// one whole cache line (the caches move whole lines; copies of half lines carry every byte twice).
// LDS holds two stages of 256 + 256 rows (128 KiB).
//
// What bounds it.  At the full matrix rate a stage takes 2048 cycles, in which a CU needs 64 KiB
// through its L1 and its LDS serves 192 KiB of fragment reads beside the 64 KiB of copies: both
// pipes are near their limits, so what counts is that copies flow all the time and have long to
// land.  A ring slot is therefore refilled in two pieces, each as soon as its rows have been read:
//   phase 0 of stage q: slot rows x first half of the weight rows (B0).  The slot-row fragments
//           stay in registers for phase 1, so A and B0 are free two K steps into it.
//     X(q): wait for this wave's copies of B1(q), barrier (A, B0 of q are read, B1(q) is complete),
//           issue the copies of A, B0 of stage q + 2 into their place
//   phase 1 of stage q: slot rows x second half (B1), free two K steps into it.
//     Y(q): wait for this wave's copies of A, B0 of q + 1, barrier, issue B1 of stage q + 2
// Every copy has one and a half stages of flight (one stage when a slot is refilled as a whole:
// 8 waves then wait for the slowest of 64 KiB of copies issued in one burst).
// Fragments are read two steps ahead of their MFMAs, across phase, stage and item borders;
// sched_barriers pin that order.
// Vector memory operations retire in issue order, so "my copies of B1(q) have landed" is s_waitcnt
// vmcnt(n) with n = (a lower bound of) what this wave issued after them.
// K % 64 == 32: the last stage has two K steps; its copies fetch the row's valid half twice.
constexpr int SLOT_BYTES = (BM + BN) * BK * 2;   // A rows, then B rows
constexpr int B_OFF = BM * BK * 2;
constexpr int FIRST = 0, MIDDLE = 1, LAST = 2;  // stages of an item
constexpr int DYN_DIV = 8;  // 1/DYN_DIV of the work items go to the shared pool
template <bool GATHER>
struct Ring {
  static constexpr int OFF_PAIR = 2 * SLOT_BYTES;
  static constexpr int OFF_DYN = OFF_PAIR + (GATHER ? 2 * BM * 4 : 0);
  static constexpr int LDS_BYTES = OFF_DYN + 16;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS per CU");
};

// wave-wide copy of 4 bytes per lane
__device__ __forceinline__ void dma4(const void* g, uint32_t lds) {
  uint32_t keep;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 1\n\tglobal_load_lds_dword %1, off\n\t"
               "s_mov_b32 m0, %0"
               : "=&s"(keep)
               : "v"(g), "s"(lds)
               : "memory");
}
// FAR: an operand of 4 GiB or more.  Byte offsets are 64 bits and added to the base by the vector ALU,
// an addition per copy.
template <class Op, bool HALF, bool FAR>
__device__ __forceinline__ void run_items_ring(const Op& op, const MTile* __restrict__ tiles,
                                               int32_t* __restrict__ hdr, int n_tiles_n, int dyn_word) {
  using RG = Ring<Op::GATHER>;
  extern __shared__ __align__(16) uint16_t smem[];
  unsigned char* sm8 = reinterpret_cast<unsigned char*>(smem);
  int32_t* pair_lds = reinterpret_cast<int32_t*>(sm8 + RG::OFF_PAIR);  // [2][BM]
  int32_t* dyn_next = reinterpret_cast<int32_t*>(sm8 + RG::OFF_DYN);
  const int lane = threadIdx.x & 63, wv = uni(threadIdx.x >> 6);
  const int wm = wv >> 1, wn = wv & 1;
  // Work split: about 1 - 1/DYN_DIV of the item list is dealt out statically (XCD-aware, see
  // xcd_items), the rest is a pool that workgroups draw from in batches once their own share is
  // done, which evens out the finishing times (m-tiles differ in their row counts).  The static
  // part is a whole number of items per workgroup: with 6.5 each, those that got 7 finished last
  // whatever the pool did (64 x 2 sub-experts of 704, 8192 tokens: 15 % of the kernel).
  const int total_items = hdr[HDR_MTILES] * n_tiles_n;
  const int grid = (int)gridDim.x;
  const int rounds = max(1, (total_items - total_items / DYN_DIV) / grid);
  const int n_static = min(total_items, rounds * grid);
  const int K = op.K(), nst = (K + BK - 1) / BK;
  // A batch from the pool: 12 stages, since a run's start costs a few, but no more than an even share (with 264 items of
  // 5 stages on 256 workgroups, one took the last three: 3000 tokens, 66 sub-experts of 256 x 320, 8 picks, both GEMMs
  // 73 us instead of 48).
  const int batch = max(1, min((12 + nst - 1) / nst, (total_items - n_static + grid - 1) / grid));
  ItemRange ir = xcd_items(n_static);
  int n_my = ir.begin < ir.end ? (ir.end - ir.begin + ir.step - 1) / ir.step : 0;
  const uint32_t smem_base = lds_offset(smem);
  const uint32_t pair_base = smem_base + RG::OFF_PAIR;
  const int sub = lane >> 3, pos = lane & 7;  // a copy covers 8 rows: row lane / 8, position lane % 8

  Sc cur, nxt;
  // Item -> (m-tile, n-tile).  A group's items are contiguous; inside a group they are walked
  // in chunks of C n-tiles x all of the group's m-tiles, so that the ~32 items an XCD works on
  // at a time form a block a x b of m-tiles x n-tiles with a + b small: each activation tile
  // is then fetched once for b n-tiles and each weight tile once for a m-tiles.
  auto load_sc = [&](int my_idx, Sc& sc) {
    const int item = ir.begin + my_idx * ir.step;
    const MTile t0 = tiles[item / n_tiles_n];
    const int first = uni(t0.first), cnt = uni(t0.count);
    const int L = item - first * n_tiles_n;
    int C = 32 / (cnt < 6 ? cnt : 6);
    C = C > n_tiles_n ? n_tiles_n : C;
    const int per = cnt * C;
    const int c = L / per, r = L % per;
    const int Cc = min(C, n_tiles_n - c * C);
    const MTile t = tiles[first + r / Cc];
    sc.g = uni(t.g);
    sc.row0 = uni(t.row0);
    sc.rows = uni(t.rows);
    sc.n0 = uni(c * C + r % Cc) * (BN / Op::N_PER_ROW);
  };
  auto fetch_pairs = [&](const Sc& sc, int parity) {
    if (Op::GATHER && wv < 4) dma4(op.idx_src(sc, wv * 64 + lane), pair_base + (uint32_t)(parity * BM + wv * 64) * 4);
  };
  // Producers of the two pieces: uniform bases that advance 64 elements per stage, byte offsets of
  // this lane's rows.  A copy covers 8 rows; chunk position pos holds chunk pos ^ f(row).
  struct Piece {
    int left, stage, par;  // stages to go in this run; stages issued of the item; slot and slot-list parity
  };
  typedef std::conditional_t<FAR, uint64_t, uint32_t> Off;
  const uint16_t *pa, *pb0, *pb1;
  Off va[4], vb0[2], vb1[2];
  Piece px, py;
  auto row_bytes = [&](int row) { return (Off)row * (Off)K * 2u; };
  auto copy = [&](const uint16_t* base, Off off, uint32_t lds) {
    if constexpr (FAR)
      copy_to_lds16_addr((uint64_t)base + off, lds);
    else
      copy_to_lds16(base, off, lds);
  };
  auto rows_x = [&](const Sc& sc, int parity) {
    op.bases(sc, pa, pb0);
    pa -= BK;  // advanced before every stage
    pb0 -= BK;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = wv * 32 + j * 8 + sub;
      va[j] = row_bytes(op.a_row(sc, r, Op::GATHER ? pair_lds[parity * BM + r] : 0)) + (uint32_t)(pos ^ swz_f<SWZ_SEQ>(r)) * 16u;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = (wv * 2 + j) * 8 + sub;
      vb0[j] = row_bytes(op.ring_row(sc, r)) + (uint32_t)(pos ^ swz_f<SWZ_SEQ>(r)) * 16u;
    }
  };
  auto rows_y = [&](const Sc& sc) {
    const uint16_t* unused;
    op.bases(sc, unused, pb1);
    pb1 -= BK;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = 128 + (wv * 2 + j) * 8 + sub;
      vb1[j] = row_bytes(op.ring_row(sc, r)) + (uint32_t)(pos ^ swz_f<SWZ_SEQ>(r)) * 16u;
    }
  };
  // K % 64 == 32, last stage: chunks 4..7 of a row do not exist, their lanes fetch chunks 0..3 (not used)
  auto tail_off = [&](int f) { return (pos ^ f) & 4 ? 64u : 0u; };
  // What the next copies of a piece need is prepared ahead of the barrier that allows them.  Behind
  // the last stage of a run the last stage is copied again (nobody reads it), so that the number of
  // operations in flight is always the same.
  uint32_t x_lds, y_lds;
  Off xa[4], xb[2], yb[2];
  auto prep_x = [&]() {  // A, B0 of the next stage
    if (px.left > 0) {
      --px.left;
      if (px.stage == nst) {  // on to the next item
        px.stage = 0;
        px.par ^= 2;
        rows_x(nxt, px.par >> 1);
      }
      ++px.stage;
      pa += BK;
      pb0 += BK;
    }
    x_lds = smem_base + (uint32_t)(px.par & 1) * SLOT_BYTES + (uint32_t)wv * 4096u;
    px.par ^= 1;
    if (HALF) {
      const bool cut = px.stage == nst;
#pragma unroll
      for (int j = 0; j < 4; ++j) xa[j] = va[j] - (cut ? tail_off(swz_f<SWZ_SEQ>(j * 8)) : 0u);
#pragma unroll
      for (int j = 0; j < 2; ++j) xb[j] = vb0[j] - (cut ? tail_off(swz_f<SWZ_SEQ>((wv * 2 + j) * 8)) : 0u);
    }
  };
  auto copy_x = [&](int j) {  // copies 0..5
    if (j < 4)
      copy(pa, HALF ? xa[j] : va[j], x_lds + j * 1024u);
    else
      copy(pb0, HALF ? xb[j - 4] : vb0[j - 4], x_lds + (B_OFF - (uint32_t)wv * 2048u) + (j - 4) * 1024u);
  };
  auto prep_y = [&]() {  // B1 of the next stage
    if (py.left > 0) {
      --py.left;
      if (py.stage == nst) {
        py.stage = 0;
        rows_y(nxt);
      }
      ++py.stage;
      pb1 += BK;
    }
    y_lds = smem_base + (uint32_t)(py.par & 1) * SLOT_BYTES + B_OFF + 128 * BK * 2 + (uint32_t)wv * 2048u;
    py.par ^= 1;
    if (HALF) {
      const bool cut = py.stage == nst;
#pragma unroll
      for (int j = 0; j < 2; ++j) yb[j] = vb1[j] - (cut ? tail_off(swz_f<SWZ_SEQ>((wv * 2 + j) * 8)) : 0u);
    }
  };
  auto copy_y = [&](int j) { copy(pb1, HALF ? yb[j] : vb1[j], y_lds + j * 1024u); };
  auto all_x = [&] {
    prep_x();
#pragma unroll
    for (int j = 0; j < 6; ++j) copy_x(j);
  };
  auto all_y = [&] {
    prep_y();
    copy_y(0);
    copy_y(1);
  };

  // fragment addresses: slot-row block mb at + 4 * 32 rows, weight block nb at + (nb & 1) * 32 and
  // (nb >> 1) * 128 rows; K step ks toggles two bits of the address
  const int fr = lane & 31, fh = lane >> 5;
  const uint32_t frag = (uint32_t)(fr * 128 + ((fh ^ swz_f<SWZ_SEQ>(fr)) * 16));
  const uint32_t ra = smem_base + (uint32_t)(wm * 32 * 128) + frag, rb = smem_base + (uint32_t)(2 * wn * 32 * 128) + frag;
  auto read_a = [&](bf16x8& v, uint32_t slot, auto ks, auto mb) {
    read_lds16<decltype(mb)::value * 128 * 128>(v, (ra + slot) ^ (uint32_t)(decltype(ks)::value * 32));
  };
  auto read_b = [&](bf16x8& v, uint32_t slot, auto ks, auto nb_c) {
    constexpr int nb = decltype(nb_c)::value;
    read_lds16<B_OFF + (nb & 1) * 32 * 128 + (nb >> 1) * 128 * 128>(v, (rb + slot) ^ (uint32_t)(decltype(ks)::value * 32));
  };

  for (;;) {
  if (n_my > 0) {
    const int total = n_my * nst;
    // ---- prologue of one pipeline run over n_my items
    load_sc(0, cur);
    nxt = cur;
    if (n_my > 1) load_sc(1, nxt);
    fetch_pairs(cur, 0);
    wait_vmem<0>();
    raw_barrier();
    px = Piece{total, 0, 0};
    py = Piece{total, 0, 0};
    rows_x(cur, 0);
    rows_y(cur);
    if (n_my > 1) fetch_pairs(nxt, 1);
    all_x();  // stages 0 and 1 (every item has at least 4)
    all_y();
    all_x();
    all_y();
    wait_vmem<10>();  // A, B0 of stage 0 (and the slot-list fetch) have landed
    raw_barrier();

    f32x16 acc[NB][MB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[nb][mb][v] = 0.0f;

    bf16x8 fa[4][MB] = {}, fb[4][2] = {};
    int mb_on = blocks_on(cur, wm);
    auto p1_of = [&](const Sc& sc) { return uni(sc.n0 + BN / 2 / Op::N_PER_ROW < op.n_cols() ? 1 : 0); };
    int p1_on = p1_of(cur);  // the second half of weight rows exists
    // ---- output.  The first half's products are complete one phase before the item's end, and the
    // second half's registers are free until the next item's phase 1: the results of phase 0 are
    // stored during phase 1 of the last stage, those of phase 1 during phase 0 of the next stage, a
    // pair of slot rows behind each MFMA.  The weight rows are the MFMA's second operand, so that
    // lanes are output columns and a store covers whole lines of a few rows as it stands.  (With the
    // columns in registers, through LDS and as a run of code behind the last stage, the down
    // projection of 6007 tokens, 64 x 4 sub-experts of 352, took 241 us instead of 223; what is left
    // of its 56 us is the stores themselves, 128 KiB per CU in one stage's time.)
    // Rows beyond the tile are dropped by the buffer's bound.
    const uint32_t ld2 = (uint32_t)op.n_cols() * 2u;
    const uint32_t put_off = op.put_off(lane) + (uint32_t)(slot_block(wm, 0) * 32) * ld2 + (uint32_t)wn * (Op::CHUNK * 2);
    uint16_t* out_ptr = nullptr;
    uint32_t out_bytes = 0;
    int out_a = 0, out_b = 0;  // slot blocks to store of phase 0 (in the last stage), of phase 1 (behind it)
    auto chunk_on = [&](int ph) { return cur.n0 + (2 * ph + wn) * Op::CHUNK < op.n_cols() ? mb_on : 0; };
    auto put = [&](auto ph_c, auto slot_c, int blocks) {  // piece 0..15 of a phase's results
      constexpr int ph = decltype(ph_c)::value, mb = decltype(slot_c)::value >> 3, v = (decltype(slot_c)::value & 7) * 2;
      if (mb < blocks) {
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(out_ptr, 0, (int)out_bytes, 0x00020000);
        uint32_t off = put_off;
        asm volatile("" : "+v"(off));  // or the offsets of all pieces are kept in registers
        op.put(acc[2 * ph][mb], acc[2 * ph + 1][mb], v, [&](int vv, uint32_t w) {
          const uint32_t row = (uint32_t)(mb * 128 + 8 * (vv >> 2) + (vv & 3));
          __builtin_amdgcn_raw_buffer_store_b32(w, rsrc, (int)(off + row * ld2 + ph * (4 * Op::CHUNK)), 0, 0);
        });
      }
    };
    // X(q) and Y(q): this wave has its fragments of the piece in registers (lgkmcnt), its copies of
    // the piece that is read next have landed, barrier.  Issued after those copies: the 8 of a stage
    // and `more` stores.
    int more_x = 0, more_y = 0;
    auto sync = [&](int more) {
      asm volatile(
          "s_waitcnt vmcnt(40) lgkmcnt(0)\n\t"
          "s_cmp_gt_u32 %0, 31\n\ts_cbranch_scc1 1f\n\t"
          "s_waitcnt vmcnt(24)\n\t"
          "s_cmp_gt_u32 %0, 15\n\ts_cbranch_scc1 1f\n\t"
          "s_waitcnt vmcnt(16)\n\t"
          "s_cmp_gt_u32 %0, 7\n\ts_cbranch_scc1 1f\n\t"
          "s_waitcnt vmcnt(8)\n1:" ::"s"(more)
          : "memory", "scc");
      raw_barrier();
    };
    // The eight steps of a stage: step t is K step t & 3 of phase t >> 2, four MFMAs.  Everything else
    // is dealt out behind single MFMAs, so that the matrix pipe never waits for a run of scalar work:
    //   fragments of step t + 2         behind MFMAs 0, 1 (steps 2, 6: behind 2, 3)
    //   X, Y                            behind MFMA 1 of steps 2, 6
    //   the copies that X, Y allow      behind MFMAs 2, 3 of steps 3, 4, 5 and of step 7
    //   preparing them                  behind MFMA 3 of steps 1 and 6
    //   a finished item's output        behind every MFMA of one phase
    // Waves with one slot block skip MFMAs 2 and 3.
    // Three copies of a stage (`kind`), run one behind the other for an item: what its first and last
    // stage have besides would be 40 branches in every one (measured: 15 % of the kernel), and three
    // alternatives in one loop spill the accumulators.
    auto step = [&](uint32_t q, auto kind_c, auto t_c) {
      constexpr int kind = decltype(kind_c)::value;
      constexpr int t = decltype(t_c)::value, ph = t >> 2, ks = t & 3, u = t + 2;
      const uint32_t slot = q * SLOT_BYTES, nslot = slot ^ SLOT_BYTES;
      const bool on = (ph == 0 || p1_on != 0) && (!HALF || ks < 2 || kind != LAST);
      auto mm = [&](int mb, int n) {
        f32x16& c = acc[2 * ph + n][mb];
        if constexpr (kind == FIRST && ks == 0)
          c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][mb], fb[t & 3][n], f32x16{}, 0, 0, 0);
        else
          c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][mb], fb[t & 3][n], c, 0, 0, 0);
      };
      auto piece = [&](auto e) {  // output behind MFMA e of the step
        constexpr std::integral_constant<int, 4 * ks + decltype(e)::value> slot_c{};
        if constexpr (kind == LAST && ph == 1) put(std::integral_constant<int, 0>{}, slot_c, out_a);
        if constexpr (kind == FIRST && ph == 0) put(std::integral_constant<int, 1>{}, slot_c, out_b);
      };
      auto rd = [&](auto e_c) {
        constexpr int e = decltype(e_c)::value;
        constexpr std::integral_constant<int, (u & 3)> k{};
        if constexpr (e < 2)
          read_b(fb[u & 3][e], u < 8 ? slot : nslot, k, std::integral_constant<int, 2 * (u >> 2 & 1) + e>{});
        else if constexpr (u < 4 || u >= 8)
          read_a(fa[u & 3][e - 2], u < 8 ? slot : nslot, k, std::integral_constant<int, e - 2>{});
      };
      constexpr bool LATE = t == 2 || t == 6;
      __builtin_amdgcn_sched_barrier(0);
      // all but the reads of the step before have returned
      wait_lds<(t >= 3 && t <= 6) ? 2 : 4>(fb[t & 3][0], fb[t & 3][1], fa[ks][0], fa[ks][1]);
      if (on) mm(0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!LATE) {
        rd(std::integral_constant<int, 0>{});
        rd(std::integral_constant<int, 2>{});
      }
      piece(std::integral_constant<int, 0>{});
      __builtin_amdgcn_sched_barrier(0);
      if (on) mm(0, 1);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!LATE) {
        rd(std::integral_constant<int, 1>{});
        rd(std::integral_constant<int, 3>{});
      }
      if constexpr (t == 2) sync(more_x);
      if constexpr (t == 6) sync(more_y);
      piece(std::integral_constant<int, 1>{});
      __builtin_amdgcn_sched_barrier(0);
      if (on && mb_on == 2) mm(1, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (LATE) {
        rd(std::integral_constant<int, 0>{});
        rd(std::integral_constant<int, 2>{});
      }
      if constexpr (t >= 3 && t <= 5) copy_x(2 * (t - 3));
      if constexpr (t == 7) copy_y(0);
      piece(std::integral_constant<int, 2>{});
      __builtin_amdgcn_sched_barrier(0);
      if (on && mb_on == 2) mm(1, 1);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (LATE) {
        rd(std::integral_constant<int, 1>{});
        rd(std::integral_constant<int, 3>{});
      }
      if constexpr (t >= 3 && t <= 5) copy_x(2 * (t - 3) + 1);
      if constexpr (t == 7) copy_y(1);
      if constexpr (t == 1) prep_x();
      if constexpr (t == 6) prep_y();
      piece(std::integral_constant<int, 3>{});
      __builtin_amdgcn_sched_barrier(0);
    };
    auto stage = [&](uint32_t q, auto kind_c) { static_loop<0, 8>([&](auto t_c) { step(q, kind_c, t_c); }); };
    auto first_frags = [&](uint32_t slot) {  // of steps 0 and 1
      static_loop<0, 2>([&](auto k) {
        static_loop<0, 2>([&](auto e) {
          read_b(fb[decltype(k)::value][decltype(e)::value], slot, k, e);
          read_a(fa[decltype(k)::value][decltype(e)::value], slot, k, e);
        });
      });
    };
    first_frags(0u);
    uint32_t q = 0;  // parity of the stage's slot
    for (int c_item = 0; c_item < n_my; ++c_item) {
      if (mb_on > 0) {
        stage(q, std::integral_constant<int, FIRST>{});
        q ^= 1;
        more_x = more_y;  // phase-1 stores of the item before
        more_y = 0;
#pragma nounroll
        for (int s = 2; s < nst; ++s) {
          stage(q, std::integral_constant<int, MIDDLE>{});
          q ^= 1;
          more_x = 0;
        }
        out_ptr = op.out() + (size_t)cur.row0 * op.n_cols() + cur.n0;
        out_bytes = (uint32_t)cur.rows * ld2 - (uint32_t)cur.n0 * 2u;
        out_a = chunk_on(0);
        out_b = chunk_on(1);
        more_y = out_a * Op::PUTS / 2;
        stage(q, std::integral_constant<int, LAST>{});
        q ^= 1;
      } else {  // no slot rows: only the copies, waits and barriers
        out_a = out_b = 0;
#pragma nounroll
        for (int s = 0; s < nst; ++s) {
          sync(0);
          all_x();
          sync(0);
          all_y();
          q ^= 1;
        }
      }
      // what the waits of the next stage may leave pending: the stores of phase 0 (X), of phase 1 (Y)
      more_x = out_a * Op::PUTS;
      more_y = out_b * Op::PUTS;
      const bool idle = mb_on == 0;
      cur = nxt;
      mb_on = blocks_on(cur, wm);
      p1_on = p1_of(cur);
      if (mb_on == 0 || c_item + 1 == n_my) {  // no stage follows that could
        static_loop<0, 16>([&](auto e) { put(std::integral_constant<int, 1>{}, e, out_b); });
        out_b = 0;
      }
      if (idle && mb_on > 0) first_frags(q * SLOT_BYTES);
      if (c_item + 2 < n_my) {
        load_sc(c_item + 2, nxt);
        fetch_pairs(nxt, c_item & 1);
      }
    }
    // fragments read ahead of a stage that does not come: not used, but on their way into registers
    static_loop<0, 4>([&](auto k) {
      constexpr int s = decltype(k)::value;
      wait_lds<0>(fb[s][0], fb[s][1], fa[s][0], fa[s][1]);
    });
  }
    // ---- next batch from the pool (every copy of this run has landed, every wave is here)
    wait_vmem<0>();
    __syncthreads();
    if (threadIdx.x == 0) *dyn_next = atomicAdd(&hdr[dyn_word], batch);
    __syncthreads();
    ir.begin = n_static + uni(*dyn_next);
    if (ir.begin >= total_items) break;
    ir.end = min(total_items, ir.begin + batch);
    ir.step = 1;
    n_my = ir.end - ir.begin;
  }
}

// HALF: K % 64 == 32, the last stage of an item has two K steps
template <class Op, bool HALF, bool FAR>
__global__ __launch_bounds__(NT_) void ffn_ring_kernel(Op op, const MTile* __restrict__ tiles,
                                                       int32_t* __restrict__ hdr, int n_tiles_n, int dyn_word) {
  run_items_ring<Op, HALF, FAR>(op, tiles, hdr, n_tiles_n, dyn_word);
}
template <class Op>
__global__ __launch_bounds__(NT_) void ffn_short_kernel(Op op, const MTile* __restrict__ tiles,
                                                        int32_t* __restrict__ hdr, int n_tiles_n) {
  run_items<Op>(op, tiles, hdr, n_tiles_n);
}

// ---------------------------------------------------------------- few rows per sub-expert
// A decode batch gives a sub-expert a row or a few, so the time is that of its weights' bytes, or with few of them that
// of a tile's chain of latencies.  A wave has 16 weight rows and up to 64 slot rows
// (v_mfma_f32_16x16x32_bf16: 16 cycles per 32 of K, and bit for bit what two v_mfma_f32_32x32x16_bf16 in a row give, so
// that which driver a batch takes does not show in its results).  Weights go through a ring of 2 KiB stages that is the
// wave's own: a stage is a wait, its LDS reads, two copies and its matrix instructions, no barrier.  Slot rows are shared
// by the waves, in chunks of 4 to 8 stages of K, two of them, and one barrier per chunk.
//   MOST = 1, 2 (blocks of 16 slot rows at a time): 4 waves, two workgroups per CU with 80 KB of weights in flight;
//   MOST = 4: 8 waves, which halves what is copied of the slot rows per weight row.
// The groups are cut into m-tiles of 16 MOST rows (FewTile), and those of a longer group with the same weight rows are
// neighbours in the list (shared_item): they run side by side on an XCD, and its L2 serves the weights to all but the first.
// Items are then of one length, whatever the load.  With m-tiles of 256 rows, which a workgroup went through 16 MOST at a
// time, it fetched its weights again each time, and the XCD that had the long group finished last.  Both GEMMs, us, so |
// now (| ring driver), router bias N(0, 1) per expert: 100 tokens on 32 of 3584 x 4096 (longest group 87) 610 | 405 | 410, 256
// on 128 of 704 (170) 250 | 164 | 184, 192 on 256 of 256 (166) 195 | 132 | 156, 384 on 512 of 192 (213) 277 | 169, fused
// kernel 247; even load: the same as before.  All tokens with the same picks, which nothing but the number of tokens bounds,
// are better off with the ring driver from some four m-tiles per group on: 256 tokens on 12 of the 128 62 | 66, 590 97 | 71.
// Two tokens of 32 sub-experts each, 192 x 2048, both GEMMs between HIP events 17.6 us, with tiles that shared a stage of
// weight and slot rows behind a barrier 24.4; 100 tokens of 4 to 12 on 128 of 704 231 -> 196 us (5.6 TB/s of weights)
// against the ring driver.  (Weights straight into the registers of the matrix instruction: its lanes are rows, so that
// every lane's 16 bytes are a cache access of their own, 330 cycles a step.)
constexpr int FP_WAVE_N = 16, NARROW_COLS = 32;
// SHORT: K of at most 3 stages (192), one chunk of slot rows; an item is then one chain of latencies, and three
// workgroups per CU have more of them side by side.  Both GEMMs, us between HIP events, with two per CU and with three:
// 1 token of the 128 x 4 layer 19.1 -> 18.1, 37 90.1 -> 88.6, 64 tokens on 256 of 64 x 1024 29.8 -> 26.0 (K = 256, 4 stages:
// 180 tokens on 256 of 256 160 -> 163).
constexpr int PICK_K = 64;  // ELEMS: the largest k_max
template <int MOST, bool SHORT, bool NARROW, int ELEMS = 0, int TOKENS = 0>
struct Few {
  static_assert((!SHORT || MOST <= 2) && (!NARROW || MOST == 4) && (ELEMS == 0 || (MOST == 1 && !SHORT)));
  static constexpr int WAVES = MOST == 4 && !NARROW ? 8 : 4, THREADS = 64 * WAVES, N = WAVES * FP_WAVE_N;
  static constexpr int NS = SHORT || NARROW ? 4 : ELEMS > 0 ? 7 : MOST == 4 ? 5 : 6, STAGE = FP_WAVE_N * BK * 2, RING = WAVES * NS * STAGE;
  static constexpr int CHUNK = WAVES * 4096;
  // ELEMS: a row of a chunk is 1 KiB, and there are no more than TOKENS; what is read of the others is not used
  static constexpr int CHUNK_STEP = ELEMS > 0 ? TOKENS * 1024 : CHUNK, GROUPS = RING + 2 * CHUNK_STEP;
  static constexpr int LDS_BYTES = ELEMS > 0 ? RING + CHUNK_STEP + CHUNK : RING + (SHORT ? 1 : 2) * CHUNK;
  static_assert(ELEMS == 0 || (GROUPS + TOKENS * PICK_K * 8 <= LDS_BYTES && 2 * LDS_BYTES <= 160 * 1024 && TOKENS <= WAVES));
  static constexpr int PER_CU = 160 * 1024 / LDS_BYTES, PARTS = NARROW ? BM / (16 * MOST) : 1;
  static constexpr int CP = 2;           // copies of a wave per stage
  static constexpr int AHEAD = NS - 1;   // stages in flight
};

// NARROW (gate-up of up to 32 neurons, any number of rows, K > 192): the ring driver's tile has 256 weight rows, of which only 64
// exist, and one workgroup per m-tile, so that CUs without one are idle.  Here four waves have the 64 weight rows, and the
// blocks of 64 slot rows of an m-tile are items of their own, PARTS of them one behind the other in the list, so that they
// meet in an L2 with their weights; two workgroups per CU.  Bound by what the copies bring from L2 (twice the slot rows' bytes).
// Gate-up between HIP events, us, ring driver | this: d = 2048, 256 sub-experts of 32, 8 picks, skewed: 2000 tokens 42.1 | 33.8,
// 4096 69.6 | 44.6, 8192 81.1 | 67.9; even load on 128 of them: 1000 36.2 | 25.9, 4096 44.2 | 35.6, 16384 123 | 93; 64 of 32 x
// 512: 1024 18.0 | 9.4, 8192 21.7 | 17.9; 128 of 32 x 4096: 4096 76.5 | 69.7.  (Blocks of 32 slot rows: 32.6, 42.2, 119 on the
// 128.)  64 neurons are two such tiles, which read the slot rows twice, and half of a ring tile: 4096 tokens 45 | 56.  Where
// few == 4 applies, it is ahead with even load (600 tokens on the 128 18.3 | 23.9).
//
// ELEMS, TOKENS (gate-up of up to TOKENS tokens, E <= 64 ELEMS): the route's picks and their dispatch belong to this launch.  Every
// workgroup picks for itself, a wave per token, and lists the groups in LDS; the first one only writes what the route and the
// dispatch leave in memory.  What it saves is the launch of the top-k kernel.  Layer calls that find their weights in HBM, us, top-k
// kernel | this: 128 x 4 sub-experts of 192 x 2048, 1 token 30.7 | 27.1, 2 36.0 | 32.8, 4 44.5 | 41.4; 64 x 4 of 256 x 2048, 1 31.5 | 27.9, 4
// 75.4 | 71.3; 64 x 2 of 704 x 2048, 1 31.1 | 27.9, 4 62.6 | 59.0; 8 x 4 of 3584 x 4096, 1 105.0 | 102.8; 512 of 128 x 256, 4 23.9 | 22.0.
// With two tokens per wave 8 tokens of the first 61.0 | 59.8, but of the last 26.6 | 33.1: the first workgroup comes last.  (Where every
// workgroup ranks its picks, which only the first one has to, one token 28.9.)
// The groups of the picks of T tokens, a bit per token and sub-expert in `takes` [token][element]: f(group, its place in the list, its
// first row, its tokens as bits); returns the rows.  ALL: also the sub-experts that nobody took.
template <int ELEMS, int TOKENS, bool ALL, class F>
__device__ __forceinline__ int pick_groups(const u64* takes, int E, int& n_groups, F&& f) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  auto below = [](u64 m) { return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0)); };
  int groups = 0, rows = 0;
#pragma unroll
  for (int i = 0; i < ELEMS; ++i) {
    u64 take[TOKENS], any = 0;
    int row0 = rows, bits = 0;
#pragma unroll
    for (int t = 0; t < TOKENS; ++t) {
      take[t] = takes[t * ELEMS + i];
      any |= take[t];
      row0 += below(take[t]);
      rows += __popcll(take[t]);
      bits |= (int)(take[t] >> lane & 1) << t;
    }
    if (i % 4 == wv && (ALL ? i * 64 + lane < E : bits != 0)) f(i * 64 + lane, groups + below(any), row0, bits);
    groups += __popcll(any);
  }
  n_groups = groups;
  return rows;
}

template <class Op, int MOST, bool SHORT, bool NARROW, int ELEMS = 0, int TOKENS = 0, class... Pick>
__global__ __launch_bounds__((Few<MOST, SHORT, NARROW, ELEMS, TOKENS>::THREADS)) void ffn_few_kernel(Op op, const MTile* __restrict__ tiles,
                                                                            const int32_t* __restrict__ hdr,
                                                                            int n_tiles_n, Pick... pick) {
  typedef Few<MOST, SHORT, NARROW, ELEMS, TOKENS> F;
  extern __shared__ __align__(16) unsigned char fp_smem[];
  constexpr int FP_NS = F::NS, FP_STAGE = F::STAGE, FP_CHUNK = F::CHUNK, STEP = F::CHUNK_STEP;
  constexpr int CP = F::CP, AHEAD = F::AHEAD, XCP = FP_CHUNK / 1024 / F::WAVES;  // XCP: copies of a wave per chunk
  const int lane = threadIdx.x & 63, wv = uni(threadIdx.x >> 6), r = lane & 15, g = lane >> 4;
  const int K = op.K(), ns = (K + BK - 1) / BK;
  const uint32_t lds0 = lds_offset(fp_smem), ring = lds0 + (uint32_t)(wv * FP_NS * FP_STAGE), xs = lds0 + F::RING;
  int2* groups = reinterpret_cast<int2*>(fp_smem + F::GROUPS);  // ELEMS: sub-expert and tokens as bits << 16, first row
  int n_m_tiles = 0, tokens = 0;  // m-tiles; ELEMS: tokens of the item's rows, as bits
  if constexpr (ELEMS > 0) {
    if (blockIdx.x > 0 && blockIdx.x < N_XCD) return;  // so that the items' workgroups keep their XCDs
    const PickArgs& p = (pick, ...);
    const int kp = topk_pad(op.k_max);
    int* uk = reinterpret_cast<int*>(fp_smem) + wv * 4 * kp;  // as in the top-k kernel
    int* uid = uk + kp;
    float* se = reinterpret_cast<float*>(uid + kp);
    int* sid = reinterpret_cast<int*>(se + kp);
    u64* takes = reinterpret_cast<u64*>(fp_smem + F::WAVES * PICK_K * 16);
    if (threadIdx.x < TOKENS * ELEMS) takes[threadIdx.x] = 0ull;
    __syncthreads();
    const bool first = blockIdx.x == 0;
    TopkPicks picks{0, 0.0f, 1.0f};
    if (wv < op.T) {
      const float* row = p.logits + (size_t)wv * p.E;
      const int asked = p.k_tok[wv];
      u64* mine = takes + wv * ELEMS;
      if (first) {
        picks = topk_token<ELEMS>(row, asked, p.E, op.k_max, p.renorm, &p.hdr[HDR_FLAGS], uk, uid, se, sid);
        for (int j = lane; j < picks.kt; j += 64) atomicOr(&mine[sid[j] >> 6], 1ull << (sid[j] & 63));
      } else {
        topk_token<ELEMS, true>(row, asked, p.E, op.k_max, p.renorm, nullptr, nullptr, nullptr, nullptr, nullptr, mine);
      }
    }
    __syncthreads();
    if (first) {
      int* first_row = reinterpret_cast<int*>(takes + TOKENS * ELEMS);  // of a sub-expert's group; its tokens as bits << 16
      const int rows = pick_groups<ELEMS, TOKENS, true>(takes, p.E, n_m_tiles, [&](int gr, int at, int row0, int bits) {
        if (bits) {
          put_tile(p.small.tiles, p.small.cut, at, gr, row0, __popc(bits), at, 1);
          first_row[gr] = row0 | bits << 16;
        }
        p.small.off[gr] = row0;
        p.small.cnt[gr] = __popc(bits);
      });
      __syncthreads();
      if (threadIdx.x == 0) {
        p.small.off[p.E] = rows;
        write_counts(p.hdr, rows, n_m_tiles, true, p.small.max_tiles);
      }
      if (wv >= op.T) return;
      for (int j = lane; j < op.k_max; j += 64) {
        const int i = wv * op.k_max + j;
        const bool on = j < picks.kt;
        const int gr = on ? sid[j] : -1;
        int slot = -1;
        if (on) {
          const int f = first_row[gr];
          slot = (f & 0xffff) + __popc((f >> 16) & ((1 << wv) - 1));
          p.small.sorted_pair[slot] = i;
        }
        if (i >= rows) p.small.sorted_pair[i] = -1;  // tail beyond the valid slots
        p.small.slot_of_pair[i] = slot;
        p.ids[i] = gr;
        p.w[i] = on ? p.scale * expf(se[j] - picks.most) / picks.denom : 0.0f;
      }
      return;
    }
    pick_groups<ELEMS, TOKENS, false>(takes, p.E, n_m_tiles, [&](int gr, int at, int row0, int bits) { groups[at] = int2{gr | bits << 16, row0}; });
    n_m_tiles = uni(n_m_tiles);
    __syncthreads();  // the ring takes the place of what was read
  }
  auto tile = [&](const Sc& sc, bool on, auto nb_c) {
    constexpr int NB = decltype(nb_c)::value;  // blocks of 16 slot rows
    constexpr int CPR = FP_CHUNK / 256 / NB, SPC = CPR / 8;  // 16-byte pieces of a row in a chunk, stages
    const uint16_t *bx, *bw;
    op.bases(sc, bx, bw);
    const uint32_t row2 = (uint32_t)K * 2u;
    uint32_t voff[CP], tail[CP], xrow[XCP], xcol[XCP];
#pragma unroll
    for (int j = 0; j < CP; ++j) {
      const int row = j * 8 + (lane >> 3), piece = (lane & 7) ^ swz_f<SWZ_SEQ>(row);
      voff[j] = (uint32_t)op.few_row(sc, row) * row2 + (uint32_t)piece * 16u;
      tail[j] = piece & 4 ? 64u : 0u;
    }
    uint32_t p_slot = ring;
    auto produce = [&](int stage) {  // one stage after the other
      if (stage >= ns) return;
      const bool cut = (stage + 1) * BK > K;  // K % 64 == 32: pieces 4..7 do not exist, fetch 0..3 (not used)
#pragma unroll
      for (int j = 0; j < CP; ++j)
        copy_to_lds16(bw + (size_t)stage * BK, cut ? voff[j] - tail[j] : voff[j], p_slot + j * 1024u);
      p_slot = p_slot == ring + (FP_NS - 1) * FP_STAGE ? ring : p_slot + FP_STAGE;
    };
    produce(0);  // on its way while the slot list is read
    // piece p of row i sits at p ^ (i & 15): rows start in the same bank
    constexpr int CROWS = CPR < 64 ? 64 / CPR : 1;  // rows of a copy
    const int x_on = min(max((sc.rows + CROWS - 1) / CROWS - wv * XCP, 0), XCP);  // copies that have a row of the tile
#pragma unroll
    for (int j = 0; j < XCP; ++j) {
      const int row = (wv * XCP + j) * CROWS + lane % 64 / CPR;
      int pair = 0;
      if constexpr (ELEMS > 0) {
        int left = min(row, sc.rows - 1);  // the token of bit number `row`
#pragma unroll
        for (int t = 0; t < TOKENS; ++t)
          if (tokens >> t & 1) pair = left-- == 0 ? t : pair;
        pair *= op.k_max;
      } else if constexpr (Op::GATHER) {
        // a copy of one row: the same for all lanes, and a scalar load does not wait for the copies
        typedef const __attribute__((address_space(4))) int32_t* Scalar;
        const int32_t* src = op.idx_src(sc, row);
        pair = CROWS == 1 ? *(Scalar)(uintptr_t)src : *src;
      }
      xrow[j] = (uint32_t)op.a_row(sc, row, pair) * row2;
      xcol[j] = (uint32_t)((lane % CPR) ^ (row & 15)) * 16u;
    }
    auto produce_x = [&](int c) {
#pragma unroll
      for (int j = 0; j < XCP; ++j) {
        if (j >= x_on) break;
        const uint32_t col = (uint32_t)(c * CPR * 16) + xcol[j];
        copy_to_lds16(bx, xrow[j] + (col < row2 ? col : 0u), xs + (uint32_t)((c & 1) * STEP + (wv * XCP + j) * 1024));
      }
    };
    produce_x(0);
#pragma nounroll
    for (int i = 1; i < AHEAD; ++i) produce(i);
    f32x4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // fragment addresses of an even and an odd stage of a chunk
    uint32_t rd_w[2], rd_x[2][2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      rd_w[ks] = ring + (uint32_t)(r * 128) + (uint32_t)((ks * 4 + g) ^ swz_f<SWZ_SEQ>(r)) * 16u;
#pragma unroll
      for (int set = 0; set < 2; ++set) rd_x[set][ks] = xs + (uint32_t)(r * CPR * 16) + (uint32_t)((set * 8 + ks * 4 + g) ^ r) * 16u;
    }
    bf16x8 fw[2][2] = {}, fx[2][2][NB] = {};
    auto multiply = [&](auto set_c, int steps) {
      constexpr int set = decltype(set_c)::value;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        if (ks < steps)
#pragma unroll
          for (int b = 0; b < NB; ++b)
            acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[set][ks], fx[set][ks][b], acc[b], 0, 0, 0);
    };
    // Copies land in the order of their issue, so a wait is a count of what may still be on its way behind what is needed:
    //   stage 0, chunk 0, stages 1 .. AHEAD - 1 (above); then chunk by chunk: chunk c + 1, and in step q of it stage q + AHEAD.
    // Stage q + AHEAD takes the slot of stage q - 1, which this wave has read; chunk c + 1 the place of chunk c - 1, which all
    // have read at the barrier.  Stages that do not exist are not issued: near the end everything is waited for.
    static_assert(FP_NS == AHEAD + 1 && (!SHORT || SPC >= 3));  // SHORT has one chunk
    const int nc = (ns + SPC - 1) / SPC;
    uint32_t w_slot = 0;  // of the stage that is read next
    for (int c = 0; c < nc; ++c) {
      // Chunk c has landed for this wave, behind the barrier for all.  Issued after it: AHEAD - 1 stages for the first one, SPC
      // for the others.
      static_assert(SPC >= AHEAD - 1);
      if (c * SPC + AHEAD - 1 < ns) wait_vmem<(AHEAD - 1) * CP>();
      else wait_vmem<0>();
      raw_barrier();
      const bool more = c + 1 < nc;
      if (more) produce_x(c + 1);
      // stage q: its copies have landed, its fragments are read while those of stage q - 1 are multiplied
      auto stage = [&](int s, auto set_c) {
        constexpr int set = decltype(set_c)::value;
        const int q = c * SPC + s;
        if (q >= ns) return;
        // issued after stage q: AHEAD - 1 stages, and chunk c + 1 where stage q was issued before this chunk
        if (q + AHEAD - 1 >= ns) wait_vmem<0>();
        else if (s < AHEAD && more && x_on == XCP) wait_vmem<(AHEAD - 1) * CP + XCP>();
        else wait_vmem<(AHEAD - 1) * CP>();
        const uint32_t x_at = (uint32_t)((c & 1) * STEP + s / 2 * 256);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          read_lds16<0>(fw[set][ks], rd_w[ks] + w_slot);
          read_lds16<0>(fx[set][ks][0], rd_x[set][ks] + x_at);
          static_loop<1, NB>([&](auto b) {
            read_lds16<decltype(b)::value * 16 * CPR * 16>(fx[set][ks][decltype(b)::value], rd_x[set][ks] + x_at);
          });
        }
        w_slot = w_slot == (FP_NS - 1) * FP_STAGE ? 0u : w_slot + FP_STAGE;
        produce(q + AHEAD);  // into the slot of stage q - 1, which has been read
        if (q > 0) multiply(std::integral_constant<int, 1 - set>{}, 2);
        wait_lds<0>(fw[set][0], fw[set][1], fx[set][0][0], fx[set][1][0]);
        static_loop<1, NB>([&](auto b) { wait_lds<0>(fx[set][0][decltype(b)::value], fx[set][1][decltype(b)::value]); });
      };
#pragma nounroll
      for (int s = 0; s < SPC; s += 2) {
        stage(s, std::integral_constant<int, 0>{});
        stage(s + 1, std::integral_constant<int, 1>{});
      }
    }
    const int steps = (K - (ns - 1) * BK) / 32;
    if (ns & 1) multiply(std::integral_constant<int, 0>{}, steps);
    else multiply(std::integral_constant<int, 1>{}, steps);
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (on) op.few_store(sc, b * 16 + r, g, acc[b]);
    raw_barrier();  // the first chunk is copied again
  };
  ItemRange ir;
  if constexpr (ELEMS > 0) ir = xcd_items(n_m_tiles * n_tiles_n, blockIdx.x - N_XCD, gridDim.x - N_XCD);
  else ir = xcd_items(hdr[HDR_MTILES] * n_tiles_n * F::PARTS);
  for (int i = ir.begin; i < ir.end; i += ir.step) {
    Sc sc;
    int nt;
    if constexpr (ELEMS > 0) {
      const int2 group = groups[i / n_tiles_n];
      nt = i % n_tiles_n;
      tokens = uni(group.x) >> 16;
      sc.g = uni(group.x) & 0xffff;
      sc.row0 = uni(group.y);
      sc.rows = __popc(tokens);
    } else if constexpr (NARROW) {
      const int item = i / F::PARTS, row = i % F::PARTS * 16 * MOST;
      const MTile t = tiles[item / n_tiles_n];
      nt = item % n_tiles_n;
      sc.g = uni(t.g);
      sc.row0 = uni(t.row0) + row;
      sc.rows = min(16 * MOST, uni(t.rows) - row);
      if (sc.rows <= 0) continue;
    } else {
      const FewTile* few = reinterpret_cast<const FewTile*>(tiles);
      FewTile t = few[i / n_tiles_n];
      nt = i % n_tiles_n;
      const int count = uni(t.rows_count) >> 8;
      if (count > 1) {
        int m;
        shared_item(i, n_tiles_n, uni(t.first), count, m, nt);
        t = few[m];
      }
      sc.g = uni(t.g);
      sc.row0 = uni(t.row0);
      sc.rows = uni(t.rows_count) & 255;
    }
    constexpr int PER_WAVE = FP_WAVE_N / Op::N_PER_ROW;
    const int n0 = (nt * F::WAVES + wv) * PER_WAVE;
    sc.n0 = min(n0, op.n_cols() - PER_WAVE);  // of eight waves the last tile's second four may have none: again the last rows
    if (MOST == 2 && sc.rows <= 16) tile(sc, n0 == sc.n0, std::integral_constant<int, 1>{});
    else tile(sc, n0 == sc.n0, std::integral_constant<int, MOST>{});
  }
}

// ---------------------------------------------------------------- down projection and combine of a few tokens
// A workgroup has 8 or 16 columns of the output and all slot rows: y of them is kept in LDS, and the picks of a token are
// added behind one barrier, in the combine's order.  The m-tiles are cut into blocks of 16 slot rows for 16 columns.  For 8
// columns they are blocks of 8 rows, and a wave multiplies two of them at a time: weight rows 0 .. 7 of the matrix instruction
// are the columns of one block's sub-expert, 8 .. 15 of the other's, and so are the slot rows; what it makes of one's weights
// and the other's rows is dropped.  Weights and slot rows share the stages of a ring that is the wave's own.
// Bound by the weights' bytes, as ffn_few_kernel is, and by one launch's latency; what it saves is the combine's launch, 3 us of
// a call, and y's way back from memory.  Layer calls that find their weights in HBM, us, two kernels | this one: 128 x 4
// sub-experts of 192 x 2048, 8 to 32 picks, skewed: 1 token 32.9 | 30.6, 4 46.7 | 44.8, 16 78.2 | 75.5, 37 100.9 | 96.9, 64 119 | 117; of 64 x
// 2048 20 tokens 82.2 | 73.6, 60 111 | 97; 64 x 4 of 256 x 2048 20 tokens 149.3 | 140.4; 64 x 2 of 704 x 2048 40 tokens 207 | 205; 8 x 4 of 3584 x 4096 1 token
// 104.8 | 99.8, 47 513 | 491; 32 x 4 of 256 x 3072 60 tokens 126.4 | 120.8.  (Pairs of m-tiles instead of blocks dealt to the waves: 37 tokens
// 2 us more, as a wave with a long group came last.)
template <int COLUMNS, int SLOTS>
struct DownCombine {
  static constexpr int COLS = COLUMNS, BLOCK = COLUMNS, PAIR = 16 / COLUMNS;  // columns, rows of a block, blocks at a time
  static constexpr int WAVES = 8, THREADS = 64 * WAVES;
  static constexpr int NS = SLOTS, AHEAD = NS - 1, STAGE = 4096, RING = WAVES * NS * STAGE, CP = 4;
  static constexpr int TOKENS = THREADS / (COLS / 2);  // at a time: a thread adds up two columns of a token
  // behind the ring, of each possible slot row: y, a block (at most one per row, and one more), a pick's weight and slot
  static constexpr int ROW = COLS * 2 + 4 + 4 + 2, LDS_BYTES = 160 * 1024 - 256, ROWS = (LDS_BYTES - RING - 16) / ROW;
  static constexpr int PER_THREAD = (ROWS + THREADS - 1) / THREADS;
  static_assert(ROWS < 1 << 12);  // dc_block
  static size_t lds_bytes(int rows) { return RING + (size_t)rows * ROW + 16; }
};
// a block: sub-expert, first slot row, rows - 1
__device__ __forceinline__ uint32_t dc_block(int g, int row0, int rows) { return (uint32_t)(g | row0 << 12 | (rows - 1) << 24); }
__device__ __forceinline__ int dc_group(uint32_t b) { return b & 4095; }
__device__ __forceinline__ int dc_row0(uint32_t b) { return b >> 12 & 4095; }
__device__ __forceinline__ int dc_rows(uint32_t b) { return (int)(b >> 24) + 1; }

template <int COLUMNS, int SLOTS, int STAGES>  // STAGES: of K, or 0: any number
__global__ __launch_bounds__((DownCombine<COLUMNS, SLOTS>::THREADS)) void ffn_down_combine_kernel(
    const uint16_t* __restrict__ h, const uint16_t* __restrict__ w_dn, const MTile* __restrict__ tiles,
    const int32_t* __restrict__ hdr, int max_tiles, const int32_t* __restrict__ slot_of_pair, const float* __restrict__ w,
    const int32_t* __restrict__ k_tok, uint16_t* __restrict__ y, uint16_t* __restrict__ out, int T, int d, int Is, int k_max) {
  typedef DownCombine<COLUMNS, SLOTS> D;
  extern __shared__ __align__(16) unsigned char dc_smem[];
  __shared__ int sums[D::WAVES];
  const int K = STAGES ? STAGES * BK : Is, ns = STAGES ? STAGES : (K + BK - 1) / BK;
  const uint32_t row2 = (uint32_t)K * 2u;
  const int lane = threadIdx.x & 63, wv = uni(threadIdx.x >> 6), r = lane & 15, g = lane >> 4;
  // neighbouring columns on one XCD: a line of the output has eight or four writers
  const int b = blockIdx.x, n0 = D::COLS * (gridDim.x % N_XCD != 0 ? b : b % N_XCD * (int)(gridDim.x / N_XCD) + b / N_XCD);
  const int n_rows = T * k_max;
  unsigned char* ys = dc_smem + D::RING;
  uint32_t* blocks = reinterpret_cast<uint32_t*>(ys + n_rows * (D::COLS * 2));
  float* pick_w = reinterpret_cast<float*>(blocks + (n_rows + 2));
  int16_t* pick_slot = reinterpret_cast<int16_t*>(pick_w + n_rows);
  // everything that is read before the ring starts, at once
  const FewTile* few = reinterpret_cast<const FewTile*>(tiles);
  FewTile tile = few[min((int)threadIdx.x, max_tiles - 1)];
  const int first = threadIdx.x / (D::COLS / 2);
  const int first_budget = k_tok[min(first, T - 1)];
  int slot[D::PER_THREAD];
  float weight[D::PER_THREAD];
#pragma unroll
  for (int i = 0; i < D::PER_THREAD; ++i) {
    const int at = min((int)threadIdx.x + i * D::THREADS, n_rows - 1);
    slot[i] = slot_of_pair[at];
    weight[i] = w[at];
  }
  const int n_tiles = uni(hdr[HDR_MTILES]), n_slots = uni(hdr[HDR_PAIRS]);
#pragma unroll
  for (int i = 0; i < D::PER_THREAD; ++i) {
    const int at = (int)threadIdx.x + i * D::THREADS;
    asm volatile("" : "+v"(slot[i]), "+v"(weight[i]));  // the loads stay where they are
    if (at < n_rows) {
      pick_slot[at] = (int16_t)(slot[i] < n_rows ? slot[i] : -1);
      pick_w[at] = weight[i];
    }
  }
  int n_blocks = 0;
  for (int base = 0; base < n_tiles; base += D::THREADS) {
    if (base > 0) tile = few[min(base + (int)threadIdx.x, max_tiles - 1)];
    const int rows = base + (int)threadIdx.x < n_tiles ? tile.rows_count & 255 : 0, n = (rows + D::BLOCK - 1) / D::BLOCK;
    int at = base + threadIdx.x, total = min(n_tiles - base, D::THREADS);
    if (T > D::BLOCK) {  // tiles of several blocks
      int sum = n;
#pragma unroll
      for (int i = 1; i < 64; i *= 2) {
        const int v = __shfl_up(sum, i);
        if (lane >= i) sum += v;
      }
      if (base > 0) __syncthreads();
      if (lane == 63) sums[wv] = sum;
      __syncthreads();
      at = n_blocks + sum - n;
      total = 0;
#pragma unroll
      for (int i = 0; i < D::WAVES; ++i) {
        if (i < wv) at += sums[i];
        total += sums[i];
      }
    }
    n_blocks += total;
    for (int i = 0; i < n; ++i) {
      const uint32_t bl = dc_block(tile.g, tile.row0 + i * D::BLOCK, min(rows - i * D::BLOCK, D::BLOCK));
      blocks[at + i] = bl;
      if (at + i == n_blocks - 1 && base + D::THREADS >= n_tiles) blocks[at + i + 1] = bl;  // of an odd number the last one twice
    }
  }
  __syncthreads();
  n_blocks = uni(n_blocks);

  const uint32_t ring = lds_offset(dc_smem) + (uint32_t)(wv * D::NS * D::STAGE);
  uint32_t piece[2], tail[2], rd[2], w_row[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = j * 8 + (lane >> 3);
    piece[j] = (uint32_t)((lane & 7) ^ swz_f<SWZ_SEQ>(row)) * 16u;
    tail[j] = piece[j] & 64u;
    w_row[j] = (uint32_t)(row % D::COLS) * row2 + piece[j];
    rd[j] = (uint32_t)(r * 128) + (uint32_t)((j * 4 + g) ^ swz_f<SWZ_SEQ>(r)) * 16u;
  }
  uint32_t p_slot = ring, c_slot = ring;
  int ahead = 0, p_at = D::PAIR * wv, p_stage = 0;  // stages on their way; what is copied next
  uint2 next = {0, 0};                              // ... and its blocks
  auto look = [&] {
    if (p_at >= n_blocks) return;
    if constexpr (D::PAIR == 2) next = *reinterpret_cast<const uint2*>(blocks + p_at);
    else next.x = next.y = blocks[p_at];
  };
  look();
  const uint16_t* wp[2];
  uint32_t h_off[2];
  auto produce = [&](uint32_t b0, uint32_t b1) {
    if (p_at >= n_blocks) return;
    if (p_stage == 0) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint32_t bl = j == 0 ? b0 : b1;
        wp[j] = w_dn + ((size_t)dc_group(bl) * d + n0) * K;
        h_off[j] = (uint32_t)(dc_row0(bl) + min((j * 8 + (lane >> 3)) % D::BLOCK, dc_rows(bl) - 1)) * row2 + piece[j];
      }
    }
    const bool cut = STAGES == 0 && (p_stage + 1) * BK > K;  // K % 64 == 32: pieces 4 .. 7 do not exist, fetch 0 .. 3 (not used)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t back = cut ? tail[j] : 0u;
      copy_to_lds16(wp[j] + p_stage * BK, w_row[j] - back, p_slot + j * 1024u);
      copy_to_lds16(h + p_stage * BK, h_off[j] - back, p_slot + 2048u + j * 1024u);
    }
    p_slot = p_slot == ring + (D::NS - 1) * D::STAGE ? ring : p_slot + D::STAGE;
    ++ahead;
    if (++p_stage == ns) {
      p_stage = 0;
      p_at += D::PAIR * D::WAVES;
      look();
    }
  };
#pragma nounroll
  for (int i = 0; i < D::AHEAD; ++i) produce(uni(next.x), uni(next.y));
  for (int c_at = D::PAIR * wv; c_at < n_blocks; c_at += D::PAIR * D::WAVES) {
    const uint32_t block = blocks[c_at + (D::PAIR == 2 ? g >> 1 : 0)];
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    auto stage = [&](int steps) {
      const uint32_t b0 = uni(next.x), b1 = uni(next.y);  // here, where no LDS read is waited for with it
      // the copies of this stage have landed; AHEAD - 1 stages were issued after it, or fewer near the end
      if (ahead == D::AHEAD) wait_vmem<(D::AHEAD - 1) * D::CP>();
      else wait_vmem<0>();
      bf16x8 fw[2] = {}, fx[2] = {};
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        read_lds16<0>(fw[ks], rd[ks] + c_slot);
        read_lds16<2048>(fx[ks], rd[ks] + c_slot);
      }
      c_slot = c_slot == ring + (D::NS - 1) * D::STAGE ? ring : c_slot + D::STAGE;
      --ahead;
      produce(b0, b1);  // into the slot of the stage before, which has been read
      wait_lds<0>(fw[0], fw[1], fx[0], fx[1]);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        if (ks < steps) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[ks], fx[ks], acc, 0, 0, 0);
    };
    if constexpr (STAGES > 0) {
      static_loop<0, STAGES>([&](auto) { stage(2); });
    } else {
      for (int s = 1; s < ns; ++s) stage(2);
      stage(K % BK != 0 ? 1 : 2);
    }
    const int row = r % D::BLOCK;
    if ((D::PAIR == 1 || r >> 3 == g >> 1) && row < dc_rows(block))
      *reinterpret_cast<uint2*>(ys + (dc_row0(block) + row) * (D::COLS * 2) + g % (D::COLS / 4) * 8) =
          make_uint2(pack2(acc[0], acc[1]), pack2(acc[2], acc[3]));
  }
  __syncthreads();
  // y is one of the layer's intermediates, so it is left in memory too.  These stores are on their way during the sums below; among
  // the copies of the loop above they make its waits stricter.  Layer calls without y | with it | from the loop, 128 x 4 of 192 x 2048,
  // 37 tokens 107.2 | 109.3 | 112.8 us, 64 tokens 121.4 | 124.3 | 129.1, 1 token 32.2 | 32.4 | 32.2.
  for (int row = threadIdx.x; row < min(n_slots, n_rows); row += D::THREADS) {
    const uint4* src = reinterpret_cast<const uint4*>(ys + row * (D::COLS * 2));
    uint4* dst = reinterpret_cast<uint4*>(y + (size_t)row * d + n0);
#pragma unroll
    for (int q = 0; q < D::COLS / 8; ++q) dst[q] = src[q];
  }
  const int c = threadIdx.x % (D::COLS / 2);
  for (int token = first; token < T; token += D::TOKENS) {
    const int kt = min(max(token == first ? first_budget : k_tok[token], 0), k_max);
    float a0 = 0.0f, a1 = 0.0f;
    for (int j0 = 0; j0 < kt; j0 += 8) {
      int at[8];
      float wt[8];
      uint32_t v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = token * k_max + min(j0 + u, k_max - 1);
        at[u] = j0 + u < kt ? pick_slot[j] : -1;
        wt[u] = pick_w[j];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const uint32_t*>(ys + max(at[u], 0) * (D::COLS * 2) + c * 4);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float wu = at[u] < 0 ? 0.0f : wt[u];  // a pick without a slot adds nothing
        const uint32_t vu = at[u] < 0 ? 0u : v[u];
        a0 = fmaf(wu, __uint_as_float(vu << 16), a0);
        a1 = fmaf(wu, __uint_as_float(vu & 0xffff0000u), a1);
      }
    }
    *reinterpret_cast<uint32_t*>(out + (size_t)token * d + n0 + 2 * c) = pack2(a0, a1);
  }
}

// ---------------------------------------------------------------- launchers
// The ring driver runs its producers two stages ahead, enters at most one new item per stage and
// needs the next item's slot list one barrier before that: at least 4 stages per item.
constexpr int RING_MIN_STAGES = 4;

template <auto Kern, class Op, class... A>
static hipError_t launch_big(size_t lds, int grid, hipStream_t s, const Op& op, A... a) {
  hipError_t e = raise_lds_limit<Kern>(lds);
  if (e != hipSuccess) return e;
  Kern<<<grid, NT_, lds, s>>>(op, a...);
  return hipGetLastError();
}

// Operands of 4 GiB and more: 1.1 million tokens of d = 2048, 8 sub-experts of 704 | 192, gate-up between HIP
// events: 5.78 | 1.79 ms; through the short-K driver, whose offsets can be of any size, 7.79 | 2.63.
template <class Op, bool HALF>
static hipError_t launch_ring(const Op& op, int ntn, int grid, int dyn_word, const MTile* tiles, int32_t* hdr,
                              hipStream_t s) {
  constexpr size_t lds = Ring<Op::GATHER>::LDS_BYTES;
  if (op.offsets_fit()) return launch_big<ffn_ring_kernel<Op, HALF, false>>(lds, grid, s, op, tiles, hdr, ntn, dyn_word);
  return launch_big<ffn_ring_kernel<Op, HALF, true>>(lds, grid, s, op, tiles, hdr, ntn, dyn_word);
}

template <class Op, int MOST, bool SHORT = false, bool NARROW = false>
static hipError_t launch_few(const Op& op, int n_cols, int max_tiles, const MTile* tiles, const int32_t* hdr, hipStream_t s) {
  typedef Few<MOST, SHORT, NARROW> F;
  hipError_t e = raise_lds_limit<ffn_few_kernel<Op, MOST, SHORT, NARROW>>(F::LDS_BYTES);
  if (e != hipSuccess) return e;
  const int ntn = cdiv(n_cols, F::N / Op::N_PER_ROW);
  const int grid = persistent_grid((long)max_tiles * ntn * F::PARTS, F::PER_CU);
  ffn_few_kernel<Op, MOST, SHORT, NARROW><<<grid, F::THREADS, F::LDS_BYTES, s>>>(op, tiles, hdr, ntn);
  return hipGetLastError();
}

template <class Op>
static hipError_t launch_op(const Op& op, int T, int K, int n_cols, int few, int dyn_word, int max_mtiles,
                            const MTile* tiles, int32_t* hdr, hipStream_t s) {
  if constexpr (!Op::GATHER) {
    if (few == 1 && K <= 3 * BK) return launch_few<Op, 1, true>(op, n_cols, 2 * max_mtiles, tiles, hdr, s);
    if (few == 2 && K <= 3 * BK) return launch_few<Op, 2, true>(op, n_cols, 2 * max_mtiles, tiles, hdr, s);
  }
  if (few == 1) return launch_few<Op, 1>(op, n_cols, 2 * max_mtiles, tiles, hdr, s);
  if (few == 2) return launch_few<Op, 2>(op, n_cols, 2 * max_mtiles, tiles, hdr, s);
  if (few == 4) return launch_few<Op, 4>(op, n_cols, 2 * max_mtiles, tiles, hdr, s);
  if constexpr (Op::GATHER) {
    if (n_cols <= NARROW_COLS && K > 3 * BK && op.offsets_fit())
      return launch_few<Op, 4, false, true>(op, n_cols, max_mtiles, tiles, hdr, s);
  }
  const int ntn = cdiv(n_cols, BN / Op::N_PER_ROW);
  const int grid = persistent_grid((long)max_mtiles * ntn, 1);
  if (cdiv(K, BK) < RING_MIN_STAGES || !out_fits(n_cols))
    return launch_big<ffn_short_kernel<Op>>(SHORT_LDS_BYTES, grid, s, op, tiles, hdr, ntn);
  if constexpr (!Op::GATHER)  // Is % 32 == 0, d % 64 == 0
    if (K % BK != 0) return launch_ring<Op, true>(op, ntn, grid, dyn_word, tiles, hdr, s);
  return launch_ring<Op, false>(op, ntn, grid, dyn_word, tiles, hdr, s);
}

// T k_max pairs are what a batch can have, its pairs are that for one budget and about 0.6 of it for mixed ones.  Stage
// calls back to back, us, two blocks, four | what else would run; mixed budgets and d = 2048 unless said; skewed: a router
// bias N(0, 1) per expert.  By possible rows per sub-expert:
//   up to 16 tokens, one block: no group has more rows;
//   two blocks up to 24, then four | ring driver: 128 of 704: 18.8 201, 209 | 239, skewed 151, 152 | 179; 37.5 217, 218 | 244,
//     skewed 190, 191 | 212; 256 of 256: 18.8 157, 176 | 191; 32 169, 179 | 196; 128 of 768, 8 picks each: 24 230, 227 | 269; 32
//     257, 230 | 272, skewed 213, 179 | 196; 32 of 3584 x 4096: 40 511, 474 | 519;
//   four up to 56 | ring driver: 128 of 704: 48 221 | 249, skewed 199 | 223; 60 228 | 251, 205 | 228; 256 of 352: 48 235 | 262, 226 |
//     244; 60 242 | 265, 210 | 206; 75 262 | 270, 242 | 216; 128 of 768, 8 picks: 50 257 | 282, 231 | 224; 56 259 | 284, 248 | 245; 62
//     278 | 287, 249 | 233; 32 of 3584 x 4096: 50 477 | 518, 502 | 491 (other tokens 506 | 514); 72 485 | 523, 526 | 499.  So with
//     skewed load they meet at 50 to 60, with even load at 75 and beyond.  With a bias N(0, 3^2) nearly all tokens have the same
//     picks, groups are as long as the batch and the ring driver is ahead where that is many tiles of 64.  Layer calls of 400 |
//     200 tokens, four | ring driver: 128 of 704 130 | 124, 89 | 91; 256 of 352 145 | 131, 96 | 103; 256 of 256 127 | 123, 89 |
//     106; the same 400 without a bias 254 | 267, 261 | 290, 215 | 237;
//   where the fused kernel is what else would run: it gives a tile a workgroup, so it wants long groups and more of them than
//     CUs.  Layer calls that find their weights in HBM, these | fused kernel, of 192 x 2048 unless said, by possible rows; even load,
//     skewed: bias N(0, 1) per sub-expert, N(0, 3^2).
//     Up to 24 rows, any number of sub-experts: 8, 300 tokens 41 | 96, 43 | 126; 128, 300 90 | 118, 77 | 139; 192 121 | 141, 103 | 144; 256 154 | 158, 125 | 155; 512, 448 of 9 rows
//     243 | 266, 126 | 167, 65 | 142, of 24 269 | 281, 190 | 236, 112 | 149; 1024, 1024 tokens of 5 454 | 486, 173 | 208, 90 | 166, of 24 525 | 573, 329 | 398, but 212 | 183;
//     64 x 2048, 256 of 24 83 | 89, 71 | 98; 192 x 1536, 512 of 24 208 | 214, 145 | 178, 87 | 121; x 1024, 20 144 | 147, 83 | 94.  They meet at 512 of 128 x 1024, 20 115 |
//     114, 70 | 77, 24 125 | 116, 89 | 85, and at 1024 of 192 x 1024, 22 267 | 280, 149 | 141.
//     Beyond, four blocks: up to 3/4 as many sub-experts as CUs, 128, 400 tokens of 40 104 | 117, 98 | 143, 600 of 56 124 | 118, 147 | 147; 192 of 40 145 | 148, 133 | 157, of
//     56 150 | 150, 154 | 158; of 128 x 1024, 40 68 | 63, 60 | 73.  Not with 224: 40 150 | 151, 136 | 161, of 128 x 1024 73 | 67, 64 | 75; 256 of 40 164 | 163, 148 | 162 (what
//     skewed load would gain, even load of short phases would lose).  With more than CUs, where the phases are long
//     and no group can be: 512, 400 tokens of 25 279 | 283, 213 | 238, 120 | 152, 640 of 40 298 | 302, 254 | 259, 161 | 164; x 4096, 40 549 | 571, 529 | 532, 325 | 316; 320 of 40
//     196 | 232, 166 | 197, 111 | 148; 512 of 128 x 2048, 448 of 28 231 | 240, 190 | 195, 98 | 122, 640 of 40 243 | 253, 205 | 205, 131 | 133; x 4096, 28 391 | 388, 350 | 380, 36 410 |
//     406, 385 | 398.  Not with longer groups, 1024, 896 of 28 551 | 538, 379 | 410, 218 | 194, 1280 of 40 560 | 580, 436 | 436, 272 | 217; nor with short phases, 512 of 192 x
//     1536, 28 219 | 216, 166 | 178; x 1024, 24.4 159 | 151, 95 | 96, 40 163 | 156, 123 | 122; 64 x 2048, 256 of them, 28 94 | 91, 80 | 108.
int ffn_few_blocks(int T, int k_max, int E, int d, int Is, bool fused) {
  const long pairs = (long)T * k_max;
  if (!GateUpOp{nullptr, nullptr, nullptr, nullptr, T, d, Is, k_max}.offsets_fit() || !DownOp{nullptr, nullptr, nullptr, d, Is}.offsets_fit()) return 0;
  if (T <= 16) return 1;
  if (fused && T > 64 && pairs > 24L * E && 4 * E > 3 * num_cus()) {
    const int longest = d < 2048 ? 0 : Is >= 192 ? 640 : Is >= 128 ? 448 : 0;  // rows of a group: at most T
    if (E <= num_cus() || T > longest || pairs > 40L * E) return 0;
  }
  if (pairs <= 24L * E) return 2;
  return T <= 64 || pairs <= 56L * E ? 4 : 0;
}

// Eight logits per lane are the most: 1024 sub-experts would gain too with sixteen, 1 token of 192 x 2048 35.9 | 31.8, of 32 x 256 17.0 | 14.2.
bool picks_bf16(int few, int T, int k_max, int E) { return few == 1 && T >= 1 && T <= 4 && k_max <= PICK_K && E <= 512; }

hipError_t launch_pick_gate_up_bf16(const PickArgs& p, const uint16_t* x, const uint16_t* w_gu, uint16_t* h, int T, int d, int Is, int k_max,
                                    hipStream_t s) {
  const GateUpOp op{x, w_gu, nullptr, h, T, d, Is, k_max};
  auto launch = [&](auto elems, auto tokens) {
    typedef Few<1, false, false, decltype(elems)::value, decltype(tokens)::value> F;
    constexpr auto Kern = ffn_few_kernel<GateUpOp, 1, false, false, decltype(elems)::value, decltype(tokens)::value, PickArgs>;
    hipError_t e = raise_lds_limit<Kern>(F::LDS_BYTES);
    if (e != hipSuccess) return e;
    const int ntn = cdiv(Is, F::N / GateUpOp::N_PER_ROW);
    const long most = (long)T * k_max < p.E ? (long)T * k_max : p.E;  // groups
    const int grid = persistent_grid(most * ntn, F::PER_CU) + N_XCD;  // the first one writes, its neighbours have nothing to do
    Kern<<<grid, F::THREADS, F::LDS_BYTES, s>>>(op, nullptr, nullptr, ntn, p);
    return hipGetLastError();
  };
  auto of = [&](auto elems) {  // one token: a quarter of the looks at the picks, 0.6 us of 27.7
    return T == 1 ? launch(elems, std::integral_constant<int, 1>{}) : launch(elems, std::integral_constant<int, 4>{});
  };
  if (p.E <= 64) return of(std::integral_constant<int, 1>{});
  if (p.E <= 128) return of(std::integral_constant<int, 2>{});
  if (p.E <= 256) return of(std::integral_constant<int, 4>{});
  return of(std::integral_constant<int, 8>{});
}

hipError_t launch_gate_up_bf16(const uint16_t* x, const uint16_t* w_gu, const int32_t* sorted_pair,
                               const MTile* tiles, int32_t* hdr, uint16_t* h, int T, int d,
                               int Is, int k_max, int few, int max_mtiles, hipStream_t s) {
  return launch_op(GateUpOp{x, w_gu, sorted_pair, h, T, d, Is, k_max}, T, d, Is, few, HDR_DYN_GATE_UP,
                   max_mtiles, tiles, hdr, s);
}

hipError_t launch_down_bf16(const uint16_t* h, const uint16_t* w_dn, const MTile* tiles,
                            int32_t* hdr, uint16_t* y, int T, int d, int Is, int few, int max_mtiles,
                            hipStream_t s) {
  return launch_op(DownOp{h, w_dn, y, d, Is}, T, Is, d, few, HDR_DYN_DOWN, max_mtiles, tiles, hdr, s);
}

// Three stages of ring leave room for twice the rows of four, and are as fast in 8 columns (37 tokens of 512 of 192 x 2048 96.9 us, four
// 97.6).  In 16 four are the faster ones where they do: 32 of 3584 x 4096, 1 token 107.0 | 104.1, 5 307 | 304.
typedef DownCombine<8, 3> Columns8;
typedef DownCombine<16, 4> Columns16;
typedef DownCombine<16, 3> Columns16Rows;
// Two kernels | one, layer calls, us:
//   As many workgroups as three quarters of the CUs, or they don't draw the weights' bytes: 512 of 192 x 1024 8 tokens 52.6 | 55.4, 30
//   99.7 | 108.5, x 512 37.8 | 42.5, 62 | 75; at d = 1536, 256 of 256, 10 tokens 63.0 | 61.0.  And no more than CUs, or some have two: in
//   8 columns, d = 4096, 32 of 3584, 1 token 110.7 | 118, 100 tokens 504 | 616.
//   A sub-expert's weights are fetched again for each block of its rows: 8 of 704 x 2048, possible rows per sub-expert 12.5 33.1 | 32.1,
//   30 38.6 | 40.3; 64 of 704 7.5 124.6 | 117.4, 12 126.5 | 125.4; 128 of 704 9.75 223 | 221; 256 of 256 9.5 180.6 | 169.5.  Where rows of
//   half a line straddle lines: 256 of 352 4.9 220 | 216, 5.6 224 | 219, 7.5 225 | 226, 9.4 236 | 238.
//   Every workgroup reads h of all slot rows, and a sub-expert's weights again for each block, 64 bytes a clock: a time that goes with
//   pairs x Is, hides behind the weights' bytes as long as it is shorter, and is longer where some CUs have no columns or the load is skewed.
//   Layer calls of 256 sub-experts unless said, bias N(0, 1) per expert, N(0, 3^2); pairs x Is in thousands.  d = 2048: 192, 20 tokens of 12 picks (46)
//   49 | 48, 38 | 37; 37 of 32 (227) 75 | 74, 51 | 52; 64 of 24 (295) 77 | 80, 53 | 55; 704, 20 of 12 (169) 106 | 103, 62 | 62, 64 of 12 (541) 165 | 167, 63 | 71, 64 of
//   24 (1081) 227 | 231, 123 | 136; 832, 64 of 24 (1278) 244 | 248, 109 | 124.  d = 1536: 128, 64 of 12 (98) 42 | 42, 34 | 35; 192, 64 of 12 (147) 47 | 49, 34 | 36; 704, 37 of 32
//   (834) 170 | 181, 102 | 118.  In 16 columns d = 3072: 448, 64 of 12 (344) 170 | 171, 86 | 92; 704, 37 of 32 376 | 384, 189 | 200; d = 4096: 704, 64 of 24 517 | 504, 244 | 243.
//   Half a stage of K at d = 1536: 352, 4 of 16 (23) 36 | 34, 40 of 12 (169) 58 | 60; 608, 4 of 16 (39) 45 | 44, 20 of 12 (146) 76 | 81; 864, 64 of 12 (664) 133 | 156; d = 2048: 480, 20 of
//   12 (115) 85 | 83; 608 (146) 108 | 111; 864, 64 of 12 203 | 218.  (Up to 352, where six possible rows per sub-expert are the line, 128 sub-experts of
//   352 x 1536, 64 tokens of 12 picks (270) 58 | 65.)
template <class D>
static bool down_combine_fits(int T, int k_max, int d) {
  return (long)T * k_max <= D::ROWS && d <= D::COLS * num_cus() && 4 * d >= 3 * D::COLS * num_cus();
}
template <class D>
static bool down_combine_pays(int T, int k_max, int d, int Is) {
  if (!down_combine_fits<D>(T, k_max, d)) return false;
  const double work = (double)T * k_max * Is, share = 4.0 * d / (D::COLS * num_cus()) - 3.0;  // 0 .. 1: of the CUs beyond three quarters
  if (Is % BK != 0) return Is <= 352 || work <= 50e3 + 70e3 * share;
  return work <= (D::COLS == 8 ? 100e3 + 460e3 * share : 300e3 + 1000e3 * share);
}
bool ffn_down_combines(int few, int T, int k_max, int E, int d, int Is) {
  if (few == 0 || T < 1 || (long)T * k_max > (Is % BK != 0 ? 6L : 12L) * E) return false;
  return down_combine_pays<Columns8>(T, k_max, d, Is) || down_combine_pays<Columns16Rows>(T, k_max, d, Is);
}

hipError_t launch_ffn_down_combine(const uint16_t* h, const uint16_t* w_dn, const MTile* tiles, const int32_t* hdr,
                                   int max_tiles, const int32_t* slot_of_pair, const float* w, const int32_t* k_tok,
                                   uint16_t* y, uint16_t* out, int T, int d, int Is, int k_max, hipStream_t s) {
  auto launch = [&](auto shape, auto stages) {
    typedef decltype(shape) D;
    constexpr auto Kern = ffn_down_combine_kernel<D::COLS, D::NS, decltype(stages)::value>;
    hipError_t e = raise_lds_limit<Kern>(D::LDS_BYTES);
    if (e != hipSuccess) return e;
    Kern<<<d / D::COLS, D::THREADS, D::lds_bytes(T * k_max), s>>>(h, w_dn, tiles, hdr, max_tiles, slot_of_pair, w, k_tok, y, out, T, d, Is,
                                                                  k_max);
    return hipGetLastError();
  };
  const std::integral_constant<int, 0> any;
  // Up to three whole stages unrolled.  Layer calls, us, any number | so, d = 2048, 256 sub-experts of 24 picks: Is = 64, 1 token 24.3 | 24.1, 16
  // 35.4 | 34.9, 64 53.6 | 51.6; 128, 1 26.1 | 25.9, 64 75.0 | 74.3; 192, 1 29.3 | 29.0, 64 82.2 | 82.1; but 256 29.8 | 29.6, 32 tokens 87.4 | 88.3.
  if (down_combine_fits<Columns8>(T, k_max, d)) {
    if (Is == BK) return launch(Columns8{}, std::integral_constant<int, 1>{});
    if (Is == 2 * BK) return launch(Columns8{}, std::integral_constant<int, 2>{});
    if (Is == 3 * BK) return launch(Columns8{}, std::integral_constant<int, 3>{});
    return launch(Columns8{}, any);
  }
  return down_combine_fits<Columns16>(T, k_max, d) ? launch(Columns16{}, any) : launch(Columns16Rows{}, any);
}

}  // namespace mp
