// bf16 backward kernels of the attention variants for gfx950: gradients of the fused forward
// pass (Eq. 3 with the score_mod of Eq. 4 and the masks of the attention listing) with respect
// to Q, K and V, from the saved log-sum-exp -- the training extension the paper's conclusion
// leaves open.  Like the forward pass, nothing of size [Sq, Sk] ever reaches device memory: each
// score tile is recomputed on the matrix cores, turned into probabilities with the saved
// row statistics and consumed at once.
//
//     P  = exp(s - lse)                 s: the transformed, masked score of the forward pass
//     dP = dO V^T
//     dS = P * (dP - delta)             delta_i = sum_c dO_ic O_ic  (= rowsum(P * dP))
//     dZ = dS * (1 - tanh^2)            soft-cap only
//     dV = P^T dO,   dK = scale * dZ^T Q,   dQ = scale * dZ K
//
// Two passes, both without atomics (bitwise reproducible results):
//   * bwd_dq_kernel (first: it also writes the row statistics that the other reads): a workgroup owns 128 query rows (one per lane, as in the forward kernel)
//     and walks the key tiles; per tile S^T = K Q^T and dP^T = V dO^T land in the 32x32
//     accumulator layout with the query in the lane, dS^T rounded to bf16 is the B operand of
//     dQ^T += K^T dS^T, whose A operand is the same K tile read through the transposing LDS load.
//   * dK / dV: a workgroup owns 128 keys (one per lane) and walks the query tiles of the query
//     heads of its group; S = Q K^T and dP = dO V^T have the key in the lane and the query row in
//     the register index, so P and dS are the B operands of dV^T += dO^T P and dK^T += Q^T dS with
//     dO^T / Q^T read transposed from LDS.  bwd_dkdv_kernel (D = 64) does all of it in every wave,
//     software-pipelined over 32-row blocks; bwd_dkdv_ws_kernel (D = 128, where one wave's
//     accumulators fill a SIMD's registers) splits it over two specialised waves per SIMD.
//     With grouped heads and few workgroups, the group's heads are cut over several workgroups
//     whose fp32 partials bwd_reduce_kv_kernel adds in a fixed order.
// The row statistics are delta and the log2-scaled lse (+inf for rows without a visible key, so that their probabilities come out
// as exactly 0).
//
// LDS tiles are row-major [rows][D] bf16 with one 16-byte-chunk swizzle that serves both access
// patterns without bank conflicts: the row read (32 consecutive rows, one chunk per lane) and
// the transposing read (4 rows x 4 chunks per 32 lanes).
#pragma once
#include "fl_kernel_bf16.hpp"

namespace fl {

struct BwdParams {
  View q, k, v, o, dout;           // inputs  [B, G, H | Hkv, S, D]; o.ptr null: delta and lse2 are given
  View dq, dk, dv;                 // outputs (ptr is written)
  const float* lse;                // [B, G, H, Sq] from the forward pass
  int64_t lse_sb, lse_sg, lse_sh;
  float* delta;                    // workspace [B, G, H, Sq]: rowsum(dO * O)
  float* lse2;                     // workspace [B, G, H, Sq]: lse * log2(e), +inf for dead rows
  const float* alibi_slopes;
  const int32_t* q_doc;            // [B, Sq]
  const int32_t* kv_doc;           // [B, Sk]
  int2* q_sum;                     // (min, max) document id per block of 32 rows / keys
  int2* kv_sum;
  int32_t B, G, H, Hkv, Sq, Sk;
  int32_t window, prefix;
  float scale, softcap;
  int32_t dq_f32, dk_f32, dv_f32;  // 1: that output is float, 0: bf16
  int32_t n_qtiles, n_ktiles;      // workgroups per (b, g, h) of the dQ kernel / per (b, g, hkv) of the dK/dV kernel
  int32_t order_q, order_k;        // 1: XCD-aware workgroup order (whole (b, g, h) problems per XCD) in that kernel
  int32_t step_q, step_k;          // > 0: the longest tiles of so many problems (all, or an XCD's) come first, 0: one problem after the other
  int32_t order_heads;             // dQ kernel, order_q 1: heads with the same keys that an XCD takes one after the other (FwdParams)
  int32_t hsplit;                  // dK/dV kernel: the query heads of a group are cut into hsplit subsets, one workgroup each
  int32_t heads_kv, heads_wg;      // query heads per kv head; of those, what a workgroup of the dK/dV kernel sums over
  // what a workgroup's index is divided by: dQ kernel, dK/dV kernel, both (set where they are launched)
  Divisor q_tiles, q_share, q_heads, q_group, k_tiles, k_split, k_heads, by_g;
  float* part_dk;                  // hsplit > 1: fp32 partial sums [hsplit][B, G, Hkv, Sk, D | DV], summed by bwd_reduce_kv_kernel
  float* part_dv;
  const float* dv_add;             // added to dV before it is written, dense fp32 [B, G, Hkv, Sk, DV]: the first softmax
                                   // stream's dV in the pass over the second stream (null: nothing to add)
  BiasView bias[2];                // the forward pass's additive biases (kernels built with NBIAS > 0), bf16
  int32_t q_off;                   // query row i sits at sequence position i + q_off (positional masks, ALiBi); >= 0
  const void* user_aux[4];         // run-time compiled variants: the caller's device arrays that the expressions read
  // Bias gradients wanted: dS of every score in bf16, as the 32 x 32 blocks in which the dQ kernel holds it,
  // [B, G, H, ceil(Sq / 32), ceil(Sk / 32)][ds_block(Sq)]; the host sums it afterwards over the axes each bias broadcasts along
  // (null: not wanted).
  uint16_t* ds_stage;
};

// One staged block: registers 0..7 of its 64 lanes, then registers 8..15 (lane L and register r are query row L % 32 and
// key 8 * (r / 4) + 4 * (L / 32) + r % 4 of the block), so that every store and load is 16 bytes per lane and 1 KiB
// contiguous per wave.  In the row-major order [Sq, Sk] a lane's four consecutive keys were an 8-byte store of their own:
// the dQ kernel of the Evoformer rows (128 x 8 heads x 384, D = 32) took 200 us that way, 143 us this way.
// A call of fewer than 32 query rows keeps only the lanes of rows that exist: a block is [2][2 halves][rows][8].
__host__ __device__ inline int ds_rows(int64_t Sq) { return Sq < 32 ? (int)Sq : 32; }
__host__ __device__ inline int ds_block(int64_t Sq) { return 32 * ds_rows(Sq); }

// Item `idx`, `tiles` of them for every problem: the tiles of one problem after the other, or tile by tile through all problems.
// Under a mask the tiles of a problem are unequal, the first ones the longest.  With few of them per compute unit the last problem's long ones, begun when
// the rest was half done, were the launch's end (us, problem by problem / tile by tile: dQ causal 16 x 8 heads x 999, D = 64 55 / 42, 8 x 16 x 2048 154 / 126, D = 128
// 8 x 16 x 1024 98 / 80, 4 x 16 x 4096 552 / 487, windows and documents 8 x 16 x 2048, D = 64 82 / 73; dK / dV there 77 / 59, 217 / 185, 123 / 108).
// step > 0: so many problems, tile by tile; 0: problem by problem.  per: divides by step, or by the tiles of a problem.
__device__ __forceinline__ void tile_of(int step, int idx, const Divisor& per, int& problem, int& tile) {
  int a, b;
  per.split(idx, a, b);
  problem = step > 0 ? b : a;
  tile = step > 0 ? a : b;
}
// Problem bh of the dK/dV kernels, (b, g, kv head, subset of the group's query heads)
struct KeyProblem {
  int split, hk, g, b, h_first;
};
__device__ __forceinline__ KeyProblem key_problem(const BwdParams& p, int bh) {
  KeyProblem r;
  int bhk, bg;
  p.k_split.split(bh, bhk, r.split);
  p.k_heads.split(bhk, bg, r.hk);
  p.by_g.split(bg, r.b, r.g);
  r.h_first = r.hk * p.heads_kv + r.split * p.heads_wg;
  return r;
}

// chunk swizzle of a tile row (see the header comment): an XOR on the 16-byte chunk index that
// depends on row % 16 only.
template <int D>
__device__ __forceinline__ int swz_u(int r) {
  if constexpr (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  else if constexpr (D == 64) return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
  else return (r >> 2) & 3;                        // 64-byte rows: four of them are one line of all banks
}

// a + b for a, b >= 0, not past the largest number (a key and a window may each have 31 bits)
__host__ __device__ __forceinline__ int capped_sum(int a, int b) {
  const uint32_t sum = (uint32_t)a + (uint32_t)b;
  return sum > 0x7fffffffu ? 0x7fffffff : (int)sum;
}

// Query rows [lo, hi) that can see any key in [j_lo, j_hi] under the positional masks.
__host__ __device__ __forceinline__ void query_range(const uint32_t MASK, int j_lo, int j_hi, int Sq, int window, int prefix,
                                                     int& lo, int& hi) {
  lo = 0;
  hi = Sq;
  if ((MASK & kMaskPrefix) != 0) {
    if (j_lo >= prefix) lo = j_lo;
  } else if ((MASK & (kMaskCausal | kMaskWindow)) != 0) {
    lo = j_lo;
  }
  if ((MASK & kMaskWindow) != 0) hi = min(Sq, capped_sum(j_hi, window + 1));
  lo = min(lo, hi);
}

// classify_block() under the positional masks for a wave whose rows, or keys, stay the same: what the other side is compared with, formed
// once.  (Two dozen scalar instructions per 32 x 32 block otherwise, in front of its first product: windows and documents 8 x 16 heads x
// 2048 rows, D = 64, 239 -> 236 us for the training step, dK / dV 109 -> 104.)
constexpr int kFarBelow = -0x7fffffff - 1, kFarAbove = 0x7fffffff;
struct KeyBounds {                                 // of rows at the positions [q_lo, q_hi]
  int end, first, whole_last, whole_first;
  __host__ __device__ __forceinline__ bool hidden(int k_lo, int k_hi) const { return k_lo >= end || k_hi < first; }
  __host__ __device__ __forceinline__ bool whole(int k_lo, int k_hi) const { return k_hi <= whole_last && k_lo >= whole_first; }
};
__host__ __device__ __forceinline__ KeyBounds key_bounds(const uint32_t MASK, int q_lo, int q_hi, int Sk, int window, int prefix) {
  KeyBounds b = {Sk, kFarBelow, Sk - 1, kFarBelow};
  if ((MASK & kMaskPrefix) != 0) {
    b.end = min(Sk, max(q_hi + 1, prefix));
    b.whole_last = min(Sk - 1, max(q_lo, prefix - 1));
  } else if ((MASK & (kMaskCausal | kMaskWindow)) != 0) {
    b.end = min(Sk, q_hi + 1);
    b.whole_last = min(Sk - 1, q_lo);
  }
  if ((MASK & kMaskWindow) != 0) {
    b.first = q_lo - window;
    b.whole_first = q_hi - window;
  }
  return b;
}
struct RowBounds {                                 // of the keys [k_lo, k_hi]; rows as positions
  int first, last, whole_first, whole_last;
  __host__ __device__ __forceinline__ bool hidden(int q_lo, int q_hi) const { return q_hi < first || q_lo > last; }
  __host__ __device__ __forceinline__ bool whole(int q_lo, int q_hi) const { return q_lo >= whole_first && q_hi <= whole_last; }
};
__host__ __device__ __forceinline__ RowBounds row_bounds(const uint32_t MASK, int k_lo, int k_hi, int Sk, int window, int prefix) {
  RowBounds b = {kFarBelow, kFarAbove, kFarBelow, kFarAbove};
  if ((MASK & kMaskPrefix) != 0) {
    if (k_lo >= prefix) b.first = k_lo;
    if (k_hi >= prefix) b.whole_first = k_hi;
  } else if ((MASK & (kMaskCausal | kMaskWindow)) != 0) {
    b.first = k_lo;
    b.whole_first = k_hi;
  }
  if ((MASK & kMaskWindow) != 0) {
    b.last = capped_sum(min(k_hi, Sk - 1), window);
    b.whole_last = capped_sum(k_lo, window);
  }
  if (k_lo >= Sk) b.last = kFarBelow;
  if (k_hi >= Sk) b.whole_first = kFarAbove;
  return b;
}

// D: channels of Q and K, DV: of V and dO.  The two contractions over D and the two (dK/dV kernel) or one (dQ kernel) over
// or into DV are tiled separately, so that D != DV and head dim 32 do no matrix work on zero padding.
template <int D_, int MOD_, uint32_t MASK_, int BN_, int WPE_, int NBIAS_ = 0, int DV_ = D_>
struct BwdCfg {
  static constexpr int D = D_, DV = DV_, MOD = MOD_, BN = BN_, WPE = WPE_, NBIAS = NBIAS_;
  static constexpr uint32_t MASK = MASK_;
  static constexpr int NW = 4, NT = NW * 64;
  static constexpr int BM = NW * 32;               // rows (dQ kernel) or keys (dK/dV kernel) per workgroup
  static constexpr int NB = BN / 32;               // 32-row blocks of a streamed tile
  static constexpr int KK = D / 16, KV = DV / 16;  // k-steps over the channels of Q / K and of V / dO
  static constexpr int DB = D / 32, DBV = DV / 32; // 32-channel blocks of them
  static constexpr int ROW = D * 2, ROWV = DV * 2; // bytes of a tile row
  static constexpr int TILE = BN * ROW, TILEV = BN * ROWV;   // bytes of one streamed tile (Q or K, V or dO)
  static constexpr int STAT = BN * 4;              // bytes of one per-row statistic of a tile (dK/dV kernel)
  static constexpr int STATS = TILE + TILEV;       // offset of the statistics in a stage
  static constexpr bool DOC = (MASK_ & kMaskDoc) != 0;   // the document ids of a tile's keys / rows are staged with the tile
  static constexpr int STAGE_DQ = TILE + TILEV + (DOC ? STAT : 0);   // K, V, key ids
  static constexpr int STAGE_KV = STATS + (DOC ? 3 : 2) * STAT;      // Q, dO, lse2, delta, row ids
  static_assert(!DOC || BN == 64, "one 4-byte load instruction fetches a tile's ids");
  static constexpr int TILE_INSTR = TILE / 1024, TILEV_INSTR = TILEV / 1024;   // 64-lane x 16-byte direct loads per tile
  static constexpr int RPI = 1024 / ROW;           // rows of a Q / K tile per load instruction
  static constexpr int GR = WPE == 1 ? 4 : 2;      // dK/dV pipeline: row fragments read ahead (a lone wave per SIMD hides LDS latency itself)
  static constexpr int GT = WPE == 1 ? 4 : 2;      // dK/dV pipeline: transposed fragments read ahead
  static_assert((D == 32 || D == 64 || D == 128) && (DV == 32 || DV == 64 || DV == 128), "head dims of the backward kernels");
  static_assert(TILE_INSTR % NW == 0 && TILEV_INSTR % NW == 0, "every wave issues the same number of loads");
  static_assert((NW * RPI) % 16 == 0 && (NW * 1024 / ROWV) % 16 == 0, "a lane's destination row keeps its residue mod 16");
};

// Fragment -> LDS offset maps of the pipelined loops.  RowPair: KK row fragments of the block at
// OFF0, then those of the block at OFF1.  TrQuad: transposed fragments of (block at OFF0, rows 0..15; DB0 of
// them), (block at OFF1, rows 0..15; DB1), (OFF0, rows 16..31), (OFF1, rows 16..31).
template <int OFF0, int OFF1, int KK>
struct RowPair {
  static constexpr int off(int f) { return f < KK ? OFF0 : OFF1; }
};
template <int OFF0, int OFF1, int DB0, int DB1, int ROW0, int ROW1>
struct TrQuad {
  static constexpr int off(int f) {
    return f % (DB0 + DB1) < DB0 ? OFF0 + (f / (DB0 + DB1)) * 16 * ROW0 : OFF1 + (f / (DB0 + DB1)) * 16 * ROW1;
  }
};

template <int OFF>
struct RowOne {                                    // KK row fragments of the block at OFF
  static constexpr int off(int) { return OFF; }
};
template <int OFF, int DB, int ROW>
struct TrOne {                                     // DB transposed fragments of rows 0..15, then DB of rows 16..31
  static constexpr int off(int f) { return OFF + (f / DB) * 16 * ROW; }
};

template <class C>
struct BwdWave {
  static constexpr int D = C::D, DV = C::DV, KK = C::KK, DB = C::DB, ROW = C::ROW;
  static constexpr uint32_t MASK = C::MASK;

  int lane, half, col;
  uint32_t ra[C::KK];              // per-lane byte offset of the row-read fragment of k-step kk (row block 0) of a Q / K tile
  uint32_t ta[C::DB][2];           // per-lane byte offsets of the transposing read of channel block d (rows +0 / +8)
  uint32_t rv[C::KV], tv[C::DBV][2];   // the same in a V / dO tile

  __device__ __forceinline__ void init(int lane_) {
    lane = lane_;
    half = lane >> 5;
    col = lane & 31;
    lane_offsets<D>(ra, ta);
    lane_offsets<DV>(rv, tv);
  }
  template <int W>
  __device__ __forceinline__ void lane_offsets(uint32_t (&r_off)[W / 16], uint32_t (&t_off)[W / 32][2]) const {
#pragma unroll
    for (int kk = 0; kk < W / 16; ++kk) r_off[kk] = col * (W * 2) + ((2 * kk + half) ^ swz_u<W>(col)) * 16;
    const int s16 = lane & 15;
    const int r0 = 4 * half + (s16 >> 2);          // row this lane addresses in the transposing read
#pragma unroll
    for (int d = 0; d < W / 32; ++d) {
      const int ch = 32 * d + 16 * ((lane >> 4) & 1) + 4 * (s16 & 3);   // first of its 4 channels
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int r = r0 + 8 * u;
        t_off[d][u] = r * (W * 2) + ((ch >> 3) ^ swz_u<W>(r)) * 16 + (ch & 7) * 2;
      }
    }
  }

  static __device__ __forceinline__ f32x16 zero16() {
    return f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  }

  // LDS reads are issued by hand with explicit lgkmcnt waits (LDS returns in order): the compiler
  // then sees no LDS read in the loop and cannot tie one to the direct global->LDS loads of the
  // next tile that are in flight.
  template <int OFF>
  static __device__ __forceinline__ void read_b128(i32x4& dst, uint32_t addr) {
    if constexpr (OFF <= 65535) {
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
    } else {
      const uint32_t a = addr + (uint32_t)OFF;
      asm volatile("ds_read_b128 %0, %1" : "=v"(dst) : "v"(a) : "memory");
    }
  }
  template <int OFF>
  static __device__ __forceinline__ void read_tr(i32x2& dst, uint32_t addr) {
    if constexpr (OFF <= 65535) {
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
    } else {
      const uint32_t a = addr + (uint32_t)OFF;
      asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(dst) : "v"(a) : "memory");
    }
  }
  template <int OFF>
  static __device__ __forceinline__ void write_b128(uint32_t addr, i32x4 v) {
    asm volatile("ds_write_b128 %0, %1 offset:%2" : : "v"(addr), "v"(v), "n"(OFF) : "memory");
  }
  // Values read by hand that only a branch uses: keeps their registers theirs until the reads have landed (called behind
  // the wait that covers them), also on the path around the branch.
  static __device__ __forceinline__ void landed(const i32x4& a, const i32x4& b) { asm volatile("" : : "v"(a), "v"(b)); }
  template <int N>
  static __device__ __forceinline__ void wait_lds() {
    static_assert(N >= 0 && N <= 15, "lgkmcnt is a 4-bit counter");
    asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(N) : "memory");
    __builtin_amdgcn_sched_barrier(0);
  }

  // The row-read fragments (A operand, 32 tile rows x 16 channels each; lane offsets off) of the 32-row block at
  // LDS byte offset OFF, read two ahead; body(kk, fragment).
  template <int OFF, int NF, class Body>
  __device__ __forceinline__ void row_stream(const uint32_t (&off)[NF], Body&& body) const {
    constexpr int G = 2, NG = NF / G;
    i32x4 fr[NF];
    static_for<0, G>([&](auto f) __attribute__((always_inline)) { read_b128<OFF>(fr[f], off[f]); });
    static_for<0, NG>([&](auto gc) __attribute__((always_inline)) {
      constexpr int g = gc;
      if constexpr (g + 1 < NG)
        static_for<(g + 1) * G, (g + 2) * G>([&](auto f) __attribute__((always_inline)) { read_b128<OFF>(fr[f], off[f]); });
      wait_lds<(g + 1 < NG) ? G : 0>();
      static_for<g * G, (g + 1) * G>([&](auto f) __attribute__((always_inline)) { body(f, __builtin_bit_cast(bf16x8, fr[f])); });
    });
  }
  // 2 * DB transposed fragments (A operand, 32 channels x 16 tile rows each) of the 32-row block
  // at OFF: fragment f = ks * DB + d covers rows 16 * ks .. + 15 and channels 32 * d .. + 31, with
  // the contraction index order of the accumulator registers (element e <-> row 8*(e/4) + 4*half + e%4).
  template <int OFF, class Body>
  __device__ __forceinline__ void tr_stream(Body&& body) const {
    constexpr int NF = 2 * DB, G = 2, NG = NF / G;
    i32x2 lo[NF], hi[NF];
    static_for<0, G>([&](auto f) __attribute__((always_inline)) {
      read_tr<OFF + (f / DB) * 16 * ROW>(lo[f], ta[f % DB][0]);
      read_tr<OFF + (f / DB) * 16 * ROW>(hi[f], ta[f % DB][1]);
    });
    static_for<0, NG>([&](auto gc) __attribute__((always_inline)) {
      constexpr int g = gc;
      if constexpr (g + 1 < NG)
        static_for<(g + 1) * G, (g + 2) * G>([&](auto f) __attribute__((always_inline)) {
          read_tr<OFF + (f / DB) * 16 * ROW>(lo[f], ta[f % DB][0]);
          read_tr<OFF + (f / DB) * 16 * ROW>(hi[f], ta[f % DB][1]);
        });
      wait_lds<(g + 1 < NG) ? 2 * G : 0>();
      static_for<g * G, (g + 1) * G>([&](auto f) __attribute__((always_inline)) {
        body(f, __builtin_bit_cast(bf16x8, (i32x4){lo[f][0], lo[f][1], hi[f][0], hi[f][1]}));
      });
    });
  }

  // Generic forms for the software-pipelined loops: O::off(f) is the LDS byte offset of fragment
  // f (a compile-time function), addr(f) the lane's part of it, fragments are read G ahead, body(f, fragment) runs in order.
  template <class O, int NF, int G, class Addr, class Body>
  __device__ __forceinline__ void row_stream_g(Addr&& addr, Body&& body) const {
    constexpr int NG = NF / G;
    static_assert(NF % G == 0 && G <= 15, "fragment groups");
    i32x4 fr[NF];
    static_for<0, G>([&](auto f) __attribute__((always_inline)) { read_b128<O::off(f)>(fr[f], addr(f)); });
    static_for<0, NG>([&](auto gc) __attribute__((always_inline)) {
      constexpr int g = gc;
      if constexpr (g + 1 < NG)
        static_for<(g + 1) * G, (g + 2) * G>([&](auto f) __attribute__((always_inline)) { read_b128<O::off(f)>(fr[f], addr(f)); });
      wait_lds<(g + 1 < NG) ? G : 0>();
      static_for<g * G, (g + 1) * G>([&](auto f) __attribute__((always_inline)) { body(f, __builtin_bit_cast(bf16x8, fr[f])); });
    });
  }
  template <class O, int NF, int G, class Addr, class Body>
  __device__ __forceinline__ void tr_stream_g(Addr&& addr, Body&& body) const {   // addr(f, 0 | 1): rows +0 / +8
    constexpr int NG = NF / G;
    static_assert(NF % G == 0 && 2 * G <= 15, "fragment groups");
    i32x2 lo[NF], hi[NF];
    static_for<0, G>([&](auto f) __attribute__((always_inline)) {
      read_tr<O::off(f)>(lo[f], addr(f, 0));
      read_tr<O::off(f)>(hi[f], addr(f, 1));
    });
    static_for<0, NG>([&](auto gc) __attribute__((always_inline)) {
      constexpr int g = gc;
      if constexpr (g + 1 < NG)
        static_for<(g + 1) * G, (g + 2) * G>([&](auto f) __attribute__((always_inline)) {
          read_tr<O::off(f)>(lo[f], addr(f, 0));
          read_tr<O::off(f)>(hi[f], addr(f, 1));
        });
      wait_lds<(g + 1 < NG) ? 2 * G : 0>();
      static_for<g * G, (g + 1) * G>([&](auto f) __attribute__((always_inline)) {
        body(f, __builtin_bit_cast(bf16x8, (i32x4){lo[f][0], lo[f][1], hi[f][0], hi[f][1]}));
      });
    });
  }
};

// One 64-lane x 16-byte direct load instruction `inst` of a [rows][W] tile whose row 0 is at
// `base` (row stride `row_bytes`); rows at or past n_valid are replaced by row n_valid - 1.
template <int W>
__device__ __forceinline__ void tile_load_instr(const unsigned char* base, int64_t row_bytes, int n_valid, int inst,
                                                int lane, unsigned char* lds_tile) {
  const int dst_row = inst * (512 / W) + lane / (W / 8);
  const int chunk = (lane % (W / 8)) ^ swz_u<W>(dst_row);
  const int row = dst_row < n_valid ? dst_row : n_valid - 1;
  lds_void* dst = (lds_void*)(lds_tile + inst * 1024);
  __builtin_amdgcn_global_load_lds((global_cvoid*)(base + (int64_t)row * row_bytes + chunk * 16), dst, 16, 0, 0);
}

// The lane's part of a tile's address in load instruction `inst` of it, in rows of `row_bytes` < 2^24 (tile_load_instr away from the
// end of the tensor)
template <int W>
__device__ __forceinline__ uint32_t tile_lane_offset(int inst, int lane, uint32_t row_bytes) {
  const int dst_row = inst * (512 / W) + lane / (W / 8);
  return dst_row * row_bytes + ((lane % (W / 8)) ^ swz_u<W>(dst_row)) * 16;
}

// The tile skipper's view of 64 consecutive tiles of a list, one per lane: the range of document ids in tile base + lane, and
// which of them hold something visible to the workgroup.  One memory round trip serves 64 tiles; finding the next visible
// tile is a bit scan and its id range a lane read.
// The ids of a tile's keys (dQ) or rows (dK / dV) arrive in LDS with the tile, and a tile in which the wave's rows and keys are
// all of one document skips the mask.  Before, every block fetched its 16 ids per lane from global memory behind the loads of
// the next tile, and so waited for that tile, and every step waited for the next tile's summary.  Windows and packed
// documents, 8 x 16 heads x 2048 rows, D = 64: dQ 110 -> 88 us, dK / dV 167 -> 154 us; 4 x 32 / 8 heads x 4096, D = 128, the
// whole training step 1193 -> 1018 us.
struct TileWindow {
  int base;
  int2 ids;
  unsigned long long vis;
  __device__ __forceinline__ int2 at(int t) const {      // base <= t < base + 64, uniform
    return make_int2(__builtin_amdgcn_readlane(ids.x, t - base), __builtin_amdgcn_readlane(ids.y, t - base));
  }
};
// Smallest and largest id of NB consecutive 32-element blocks from block s0 (n blocks in all)
template <int NB>
__device__ __forceinline__ int2 merge_summaries(const int2* sum, int s0, int n) {
  int2 r = sum[min(s0, n - 1)];
#pragma unroll
  for (int u = 1; u < NB; ++u) {
    const int2 x = sum[min(s0 + u, n - 1)];
    r.x = min(r.x, x.x);
    r.y = max(r.y, x.y);
  }
  return r;
}
// Do two id ranges hold one and the same document (nothing is masked) / none in common (everything is)?
__device__ __forceinline__ bool same_document(int2 a, int2 b) { return a.x == a.y && b.x == b.y && a.x == b.x; }
__device__ __forceinline__ bool no_common_document(int2 a, int2 b) { return a.y < b.x || b.y < a.x; }

// The score pipeline of the forward pass replayed on one raw dot product x = <q_i, k_j>:
// returns the log2-domain exponent argument a (P = exp2(a)) and the soft-cap derivative factor.
//   rel = i - j;  slope2 = slope * log2(e);  lse2 = lse * log2(e).
template <int MOD>
__device__ __forceinline__ float replay_score(float x, float c_scale, float lse2, float softcap, float slope2,
                                              float rel, float& fac) {
  fac = 1.f;
  if constexpr (MOD == kModSoftcap) {
    const float e = fast_exp2(x * (2.f * c_scale / softcap));     // exp(2 z / cap)
    const float t = fmaf(fast_rcp(e + 1.f), -2.f, 1.f);           // tanh(z / cap)
    fac = fmaf(-t, t, 1.f);
    return fmaf(t, softcap * kLog2e, -lse2);
  } else if constexpr (MOD == kModAlibi) {
    return fmaf(x, c_scale, -lse2) - slope2 * fabsf(rel);
  } else {
    return fmaf(x, c_scale, -lse2);
  }
}

// The positional masks and the ends of the tensors leave a lane one range of keys (dQ kernel: the lane is a query row) or of query
// rows (dK / dV kernel: the lane is a key): per score one subtraction and one compare, instead of every condition on (i, j).
// These kernels are bound by instruction issue where many blocks are cut by a mask: windows and packed documents, 8 x 16 heads x
// 2048 rows, D = 64: dK / dV 146 -> 127 us, dQ 92 -> 81 us; 4 x 32 / 8 heads x 4096, D = 128, the training step 952 -> 870 us.
struct Span {
  int first;
  uint32_t more;                                   // first .. first + more
  __device__ __forceinline__ bool outside(int x) const { return (uint32_t)(x - first) > more; }   // x >= 0
  __device__ __forceinline__ void set(int lo, int hi) {
    const bool none = lo > hi;
    first = none ? -1 : lo;                        // (no x >= 0 is -1)
    more = none ? 0u : (uint32_t)(hi - lo);
  }
};
// keys that query row i sees
__device__ __forceinline__ Span visible_keys(const uint32_t MASK, int i, int Sq, int Sk, int q_off, int window, int prefix) {
  const int ip = i + q_off;
  int lo = 0, hi = Sk - 1;
  if ((MASK & kMaskPrefix) != 0) hi = min(hi, max(ip, prefix - 1));
  else if ((MASK & (kMaskCausal | kMaskWindow)) != 0) hi = min(hi, ip);
  if ((MASK & kMaskWindow) != 0) lo = max(lo, ip - window);
  Span s;
  s.set(lo, i < Sq ? hi : -1);
  return s;
}
// query rows that see key j
__device__ __forceinline__ Span seeing_rows(const uint32_t MASK, int j, int Sq, int Sk, int q_off, int window, int prefix) {
  int lo = 0, hi = Sq - 1;
  if ((MASK & kMaskPrefix) != 0) lo = j < prefix ? 0 : max(j - q_off, 0);
  else if ((MASK & (kMaskCausal | kMaskWindow)) != 0) lo = max(j - q_off, 0);
  if ((MASK & kMaskWindow) != 0) hi = (int)min((int64_t)hi, (int64_t)j + window - q_off);
  Span s;
  s.set(lo, j < Sk ? hi : -1);
  return s;
}

// Run-time compiled variants (kModCustom / kMaskCustom): the caller's expressions see the sizes of the call and their
// captured arrays through the forward pass's parameter block; this is the part of it they read.
__device__ __forceinline__ FwdParams user_context(const BwdParams& p) {
  FwdParams u;
  u.B = p.B; u.G = p.G; u.H = p.H; u.Sq = p.Sq; u.Sk = p.Sk;
#pragma unroll
  for (int n = 0; n < 4; ++n) u.user_aux[n] = p.user_aux[n];
  return u;
}
// The score pipeline of a compiled score_mod replayed on the raw dot product x of (i, j) (valid indices): exponent
// argument and derivative factor, as replay_score.
template <int MOD>
__device__ __forceinline__ float replay_user(float x, const BwdParams& p, const FwdParams& u, float lse2, int b, int g, int h,
                                             int i, int j, float& fac) {
  const int ic = i < p.Sq ? i : p.Sq - 1, jc = j < p.Sk ? j : p.Sk - 1;
  const float s = x * p.scale;
  fac = fl_user_score_mod_grad(s, b, g, h, ic + p.q_off, jc, u);
  return fmaf(fl_user_score_mod(s, b, g, h, ic + p.q_off, jc, u), kLog2e, -lse2);
}
// Is the score of (i, j) hidden?  outside: by the positional masks or the ends of the tensors (then a compiled mask expression,
// which takes valid indices only, is not evaluated)
template <uint32_t MASK>
__device__ __forceinline__ bool hidden(bool outside, int i, int j, const BwdParams& p, const FwdParams& u, int b, int g, int h, int qdoc,
                                       int kdoc) {
  if (outside || ((MASK & kMaskDoc) != 0 && qdoc != kdoc)) return true;
  if constexpr ((MASK & kMaskCustom) != 0) return fl_user_mask(b, g, h, i + p.q_off, j, u);
  return false;
}

// The sum of a score's biases in log2 units, a rounding of its own: never half of an FMA (biased_exponent)
__device__ __forceinline__ float bias_log2(float sum) {
#pragma clang fp contract(off)
  return sum * kLog2e;
}
// The argument of P = exp2(score + biases - lse) from a = score - lse and the biases, in log2 units.  A row all of whose keys are hidden
// by a large finite bias has lse = bias up to its rounding, and the two have to cancel: the rounded biases against the rounded lse.
// What is left can still be a few units in the last place of numbers like 1e9, in either direction, so that the argument is
// bounded by what it is mathematically, P <= 1.  NaN stays NaN.
__device__ __forceinline__ float biased_exponent(float a, float bl) {
#pragma clang fp contract(off)
  return __builtin_elementwise_minimum(a + bl, 0.f);
}

// Offsets of the (b, g, h) slice of each bias / bias gradient (elements).
template <int NBIAS>
struct BiasHead {
  int64_t off[NBIAS > 0 ? NBIAS : 1];
  __device__ __forceinline__ void set(const BwdParams& p, int b, int g, int h) {
#pragma unroll
    for (int n = 0; n < NBIAS; ++n) off[n] = b * p.bias[n].sb + g * p.bias[n].sg + h * p.bias[n].sh;
  }
  // can four consecutive keys of a row be fetched with one 8-byte load?  (uniform)
  __device__ __forceinline__ bool rows_vec4(const BwdParams& p) const {
    bool ok = true;
#pragma unroll
    for (int n = 0; n < NBIAS; ++n) {
      const BiasView& v = p.bias[n];
      ok = ok && v.sj == 1 && ((uint64_t)v.ptr) % 8 == 0 && ((v.sb | v.sg | v.sh | v.si) & 3) == 0;
    }
    return ok;
  }
  // the four bf16 values of keys j .. j + 3 of row i of bias n, as loaded (j a multiple of 4, rows_vec4())
  __device__ __forceinline__ uint2 raw4(const BwdParams& p, int n, int i, int j) const {
    return *(const uint2*)((const uint16_t*)p.bias[n].ptr + off[n] + (int64_t)i * p.bias[n].si + j);
  }
  __device__ __forceinline__ uint16_t raw1(const BwdParams& p, int n, int i, int j) const {
    return ((const uint16_t*)p.bias[n].ptr)[off[n] + (int64_t)i * p.bias[n].si + (int64_t)j * p.bias[n].sj];
  }
  // sum of the biases of score (i, j) in log2 units; i, j are valid indices
  __device__ __forceinline__ float value(const BwdParams& p, int i, int j) const {
    float s = 0.f;
#pragma unroll
    for (int n = 0; n < NBIAS; ++n)
      s += bf16_to_f32(((const uint16_t*)p.bias[n].ptr)[off[n] + (int64_t)i * p.bias[n].si + (int64_t)j * p.bias[n].sj]);
    return bias_log2(s);
  }
};

// Four consecutive channels of a dK (V false) or dV row: to the output tensor, or (grouped-query heads cut
// over several workgroups) to this workgroup's fp32 partial.
template <bool V, int W>
__device__ __forceinline__ void store_kv_grad(const BwdParams& p, int split, int b, int g, int hk, int j, int ch, float x0,
                                              float x1, float x2, float x3) {
  const int64_t dense = (((int64_t)b * p.G + g) * p.Hkv + hk) * p.Sk + j;
  if (p.hsplit > 1) {
    const int64_t row = (int64_t)split * p.B * p.G * p.Hkv * p.Sk + dense;
    *(float4*)((V ? p.part_dv : p.part_dk) + row * W + ch) = make_float4(x0, x1, x2, x3);
  } else {
    if (V && p.dv_add != nullptr) {
      const float4 a = *(const float4*)(p.dv_add + dense * W + ch);
      x0 += a.x; x1 += a.y; x2 += a.z; x3 += a.w;
    }
    const View& out = V ? p.dv : p.dk;
    const int64_t row = b * out.sb + g * out.sg + hk * out.sh + (int64_t)j * out.ss;
    if (V ? p.dv_f32 : p.dk_f32) *(float4*)((float*)out.ptr + row + ch) = make_float4(x0, x1, x2, x3);
    else *(uint2*)((uint16_t*)out.ptr + row + ch) = make_uint2(pack_bf16(x0, x1), pack_bf16(x2, x3));
  }
}

// Sum of the hsplit partials of dK and dV, in a fixed order (reproducible), written in the output dtype.  One thread per
// four channels of a dK row or of a dV row (grid.y).
template <int D, int DV>
__global__ void __launch_bounds__(256) bwd_reduce_kv_kernel(const BwdParams p) {
  const bool is_v = blockIdx.y != 0;
  const int W = is_v ? DV : D, cpr = W / 4;        // channels and float4 chunks per row
  const int64_t rows = (int64_t)p.B * p.G * p.Hkv * p.Sk;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= rows * cpr) return;
  const int64_t row = idx / cpr;
  const int ch = (int)(idx % cpr) * 4;
  const int j = (int)(row % p.Sk);
  const int hk = (int)((row / p.Sk) % p.Hkv);
  const int g = (int)((row / ((int64_t)p.Sk * p.Hkv)) % p.G);
  const int b = (int)(row / ((int64_t)p.Sk * p.Hkv * p.G));
  const float* part = is_v ? p.part_dv : p.part_dk;
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s = 0; s < p.hsplit; ++s) {
    const float4 a = *(const float4*)(part + ((int64_t)s * rows + row) * W + ch);
    x.x += a.x; x.y += a.y; x.z += a.z; x.w += a.w;
  }
  if (is_v && p.dv_add != nullptr) {
    const float4 a = *(const float4*)(p.dv_add + row * W + ch);
    x.x += a.x; x.y += a.y; x.z += a.z; x.w += a.w;
  }
  const View& out = is_v ? p.dv : p.dk;
  const int64_t orow = b * out.sb + g * out.sg + hk * out.sh + (int64_t)j * out.ss;
  if (is_v ? p.dv_f32 : p.dk_f32) *(float4*)((float*)out.ptr + orow + ch) = x;
  else *(uint2*)((uint16_t*)out.ptr + orow + ch) = make_uint2(pack_bf16(x.x, x.y), pack_bf16(x.z, x.w));
}

// ------------------------------------------------------------------------------------------------
// dQ
// ------------------------------------------------------------------------------------------------
template <class C>
__global__ void __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::WPE, C::WPE)))
bwd_dq_kernel(const BwdParams p) {
  constexpr int BN = C::BN, NB = C::NB, KK = C::KK, KV = C::KV, DB = C::DB, ROW = C::ROW, ROWV = C::ROWV;
  constexpr uint32_t MASK = C::MASK;
  constexpr uint32_t POS = MASK & ~kMaskDoc;
  typedef BwdWave<C> W;
#ifdef FL_LDS_STATIC   // instantiated at run time: the size is part of the code object (a launch through the module API
                       // cannot ask for more than 64 KiB of dynamic LDS)
  __shared__ __attribute__((aligned(16))) unsigned char lds_raw[2 * C::STAGE_DQ];
#else
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
#endif

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  W w;
  w.init(tid & 63);
  const int lane = w.lane;

  // grid decode: longest q-tiles (under a causal mask) first, of one head after the other or of all heads
  const int nq = p.n_qtiles;
  int qt, bh;
  if (p.order_q == 1) {
    // consecutive workgroup ids go round-robin to the 8 XCDs: give each XCD whole heads, so that a
    // head's K / V tiles stay in one L2 (the host checks that the head count is a multiple of 8), with the heads that read
    // the same K / V side by side
    int n, inner, r;                               // which of the XCD's heads, or sets of heads
    tile_of(p.step_q, blockIdx.x >> 3, p.q_tiles, n, inner);
    if (p.step_q == 0) {
      p.q_share.split(inner, qt, r);
    } else {
      qt = inner;
      p.q_share.split(n, n, r);
    }
    bh = (n * 8 + (int)(blockIdx.x & 7)) * (int)p.q_share.d + r;
  } else {
    tile_of(p.step_q, blockIdx.x, p.q_tiles, bh, qt);
  }
  qt = nq - 1 - qt;
  int bg, h, b, g;
  p.q_heads.split(bh, bg, h);
  p.by_g.split(bg, b, g);
  const int hk = p.q_group.div(h);
  const FwdParams uctx = user_context(p);          // what a compiled variant's expressions read (unused otherwise)
  const int i0 = qt * C::BM, iw = i0 + 32 * wave;
  const int i = iw + w.col, ic = i < p.Sq ? i : p.Sq - 1;
  const int64_t srow = ((int64_t)(b * p.G + g) * p.H + h) * p.Sq + ic;

  // per-lane operands: Q and dO rows as B fragments, row statistics
  bf16x8 qf[KK], dof[KV];
  {
    const uint16_t* qp = (const uint16_t*)p.q.ptr + b * p.q.sb + g * p.q.sg + h * p.q.sh + (int64_t)ic * p.q.ss;
    const uint16_t* dp = (const uint16_t*)p.dout.ptr + b * p.dout.sb + g * p.dout.sg + h * p.dout.sh + (int64_t)ic * p.dout.ss;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[kk] = *(const bf16x8*)(qp + 16 * kk + 8 * w.half);
#pragma unroll
    for (int kk = 0; kk < KV; ++kk) dof[kk] = *(const bf16x8*)(dp + 16 * kk + 8 * w.half);
  }
  // Row statistics: delta = rowsum(dO * O) and lse * log2(e), +inf for rows without a visible key (their P is exactly 0).  Where the
  // host gives O this kernel works them out from the dO it holds, two lanes per row, and writes them for the dK/dV kernel; a
  // pass of its own over dO and O took 58 us of 2 x 32 heads x 8192 rows at D = 128 and 14.6 of 8 x 16 x 2048 at 64 (window and
  // documents; training step 327 -> 318 us, causal 16 x 16 x 1000 321 -> 307).  (The composed
  // pass has them from its elementwise kernel.)
  float lse2, delta;
  if (p.o.ptr != nullptr) {                        // uniform
    const uint16_t* op = (const uint16_t*)p.o.ptr + b * p.o.sb + g * p.o.sg + h * p.o.sh + (int64_t)ic * p.o.ss;
    float s = 0.f;
#pragma unroll
    for (int kk = 0; kk < KV; ++kk) {
      const i32x4 ov = __builtin_bit_cast(i32x4, *(const bf16x8*)(op + 16 * kk + 8 * w.half)), dv = __builtin_bit_cast(i32x4, dof[kk]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s = fmaf(__uint_as_float((uint32_t)ov[e] << 16), __uint_as_float((uint32_t)dv[e] << 16), s);
        s = fmaf(__uint_as_float((uint32_t)ov[e] & 0xFFFF0000u), __uint_as_float((uint32_t)dv[e] & 0xFFFF0000u), s);
      }
    }
    delta = half_swap_sum(s);
    const float l = p.lse[b * p.lse_sb + g * p.lse_sg + h * p.lse_sh + ic];
    lse2 = l == -INFINITY ? INFINITY : l * kLog2e;
    if (w.half == 0 && i < p.Sq) {
      p.delta[srow] = delta;
      p.lse2[srow] = lse2;
    }
  } else {
    lse2 = p.lse2[srow];
    delta = p.delta[srow];
  }
  const float c_scale = p.scale * kLog2e;
  const float slope2 = C::MOD == kModAlibi ? p.alibi_slopes[h] * kLog2e : 0.f;
  int qdoc = 0;
  if constexpr ((MASK & kMaskDoc) != 0) qdoc = p.q_doc[(int64_t)b * p.Sq + ic];
  BiasHead<C::NBIAS> bh_;
  bh_.set(p, b, g, h);
  const bool bias_vec4 = C::NBIAS > 0 && bh_.rows_vec4(p);

  f32x16 acc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) acc[d] = W::zero16();

  // visible key range and tile skipping
  const int i_last = (i0 + C::BM < p.Sq ? i0 + C::BM : p.Sq) - 1;
  int k_lo, k_hi;
  key_range(MASK, i0 + p.q_off, i_last + p.q_off, p.Sk, p.window, p.prefix, k_lo, k_hi);   // rows by their positions
  const int t_lo = k_lo / BN, t_hi = (k_hi + BN - 1) / BN;
  const int nks = (p.Sk + kSumBlock - 1) / kSumBlock;
  int2 qs_wg = make_int2(0, 0), qs_wave = make_int2(0, 0);
  TileWindow win = {t_lo, make_int2(0, 0), 0};
  auto load_window = [&](int t) __attribute__((always_inline)) {   // what the skipper knows about tiles t .. t + 63
    win.base = t;
    win.ids = merge_summaries<NB>(p.kv_sum + (int64_t)b * nks, (t + lane) * NB, nks);
  };
  auto scan_window = [&]() __attribute__((always_inline)) {
    const int tt = win.base + lane;
    win.vis = __builtin_amdgcn_ballot_w64(
        tt < t_hi && classify_block(MASK, i0 + p.q_off, i_last + p.q_off, tt * BN, tt * BN + BN - 1, p.Sk, p.window, p.prefix, qs_wg, win.ids) != kSkip);
  };
  if (C::DOC && t_lo < t_hi) {                     // (without keys there are no summaries)
    const int nqs = (p.Sq + kSumBlock - 1) / kSumBlock;
    const int2* qsum = p.q_sum + (int64_t)b * nqs;
    load_window(t_lo);
    qs_wg = merge_summaries<C::BM / kSumBlock>(qsum, i0 / kSumBlock, nqs);
    qs_wave = qsum[min(iw / kSumBlock, nqs - 1)];
    scan_window();
  }
  // first tile at or after t that holds something visible to the workgroup's rows (t_hi if none), and its id range
  auto next_tile = [&](int t, int2& ks) __attribute__((always_inline)) -> int {
    if constexpr (C::DOC) {
      while (t < t_hi) {
        if (t >= win.base + 64) {
          load_window(t);
          scan_window();
        }
        const unsigned long long rest = win.vis >> (t - win.base);
        if (rest != 0) {
          t += __builtin_ctzll(rest);
          ks = win.at(t);
          return t;
        }
        t = min(win.base + 64, t_hi);
      }
    }
    return t;
  };

  const unsigned char* kbase = (const unsigned char*)((const uint16_t*)p.k.ptr + b * p.k.sb + g * p.k.sg + hk * p.k.sh);
  const unsigned char* vbase = (const unsigned char*)((const uint16_t*)p.v.ptr + b * p.v.sb + g * p.v.sg + hk * p.v.sh);
  const int64_t kss = p.k.ss * 2, vss = p.v.ss * 2;
  auto load_tile = [&](int t, int stage) __attribute__((always_inline)) {
    const int nvalid = min(BN, p.Sk - t * BN);
    unsigned char* st = lds_raw + stage * C::STAGE_DQ;
#pragma unroll
    for (int u = 0; u < (C::TILE_INSTR > C::TILEV_INSTR ? C::TILE_INSTR : C::TILEV_INSTR) / C::NW; ++u) {
      if (u < C::TILE_INSTR / C::NW) tile_load_instr<C::D>(kbase + (int64_t)(t * BN) * kss, kss, nvalid, wave + u * C::NW, lane, st);
      if (u < C::TILEV_INSTR / C::NW)
        tile_load_instr<C::DV>(vbase + (int64_t)(t * BN) * vss, vss, nvalid, wave + u * C::NW, lane, st + C::TILE);
    }
    if constexpr (C::DOC) {
      if (wave == 0) {
        lds_void* dst = (lds_void*)(st + C::TILE + C::TILEV);
        __builtin_amdgcn_global_load_lds((global_cvoid*)(p.kv_doc + (int64_t)b * p.Sk + t * BN + (lane < nvalid ? lane : nvalid - 1)), dst, 4, 0, 0);
      }
    }
  };

  const KeyBounds bounds = key_bounds(POS, iw + p.q_off, iw + 31 + p.q_off, p.Sk, p.window, p.prefix);
  // (tn: the tile to request into the other stage while this one is worked on; with biases its loads are issued behind
  // the first block's bias loads, so that waiting for those -- vector loads return in order -- leaves them in flight)
  auto compute = [&](auto stage_c, int t, int tn, int2 ks) __attribute__((always_inline)) {   // ks: the id range of tile t
    constexpr int ST = decltype(stage_c)::value * C::STAGE_DQ;
    const bool doc_mask = C::DOC && !same_document(qs_wave, ks), doc_skip = C::DOC && no_common_document(qs_wave, ks);   // uniform
    if constexpr (C::NBIAS == 0) load_tile(tn, 1 - decltype(stage_c)::value);
    const int j0 = t * BN;
    static_for<0, NB>([&](auto nbc) __attribute__((always_inline)) {
      constexpr int nb = decltype(nbc)::value;
      // the wave's 32 rows against this block's 32 keys under the positional masks (uniform)
      if (bounds.hidden(j0 + 32 * nb, j0 + 32 * nb + 31) || doc_skip) {   // nothing visible: dS = 0
        if constexpr (C::NBIAS > 0 && nb == 0) load_tile(tn, 1 - decltype(stage_c)::value);
        return;
      }
      const bool need_mask = doc_mask || (MASK & kMaskCustom) != 0 || iw + 31 >= p.Sq || !bounds.whole(j0 + 32 * nb, j0 + 32 * nb + 31);
      // This lane's bias values of the block: requested before the matrix work and left untouched until after it (a
      // conversion right here would put the wait for them, and for the tile loads issued before them, in front of the
      // MFMAs); four keys per load where the rows allow it.
      constexpr int NBR = C::NBIAS > 0 ? C::NBIAS : 1;
      uint2 bq[NBR][4];
      uint16_t b1[NBR][16];
      const bool bvec = C::NBIAS > 0 && bias_vec4 && j0 + 32 * nb + 32 <= p.Sk;   // uniform
      if constexpr (C::NBIAS > 0) {
        if (bvec) {
#pragma unroll
          for (int n = 0; n < C::NBIAS; ++n)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) bq[n][q4] = bh_.raw4(p, n, ic, j0 + 32 * nb + 4 * w.half + 8 * q4);
        } else {
#pragma unroll
          for (int n = 0; n < C::NBIAS; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int jj = j0 + 32 * nb + 4 * w.half + 8 * (r >> 2) + (r & 3);
              b1[n][r] = bh_.raw1(p, n, ic, jj < p.Sk ? jj : p.Sk - 1);
            }
        }
      }
      if constexpr (C::NBIAS > 0 && nb == 0) load_tile(tn, 1 - decltype(stage_c)::value);
      i32x4 kd[4];                                 // the block's key ids, covered by the waits of the streams below
      if constexpr (C::DOC)
        static_for<0, 4>([&](auto qc) __attribute__((always_inline)) {
          W::template read_b128<ST + C::TILE + C::TILEV + (32 * nb + 8 * decltype(qc)::value) * 4>(kd[decltype(qc)::value], 16 * w.half);
        });
      f32x16 s = W::zero16(), dp = W::zero16();
      w.template row_stream<ST + nb * 32 * ROW>(w.ra, [&](auto kk, bf16x8 a) __attribute__((always_inline)) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], s, 0, 0, 0);
      });
      w.template row_stream<ST + C::TILE + nb * 32 * ROWV>(w.rv, [&](auto kk, bf16x8 a) __attribute__((always_inline)) {
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, dof[kk], dp, 0, 0, 0);
      });
      if constexpr (C::DOC) {
        W::landed(kd[0], kd[1]);
        W::landed(kd[2], kd[3]);
      }
      const int jb = j0 + 32 * nb + 4 * w.half;    // key of register 0
      float bl[C::NBIAS > 0 ? 16 : 1];             // sum of the biases of each score, log2 units
      if constexpr (C::NBIAS > 0) {
        // the first block's values are older than the next tile's loads: all but those have to have landed
        if constexpr (nb == 0) __builtin_amdgcn_s_waitcnt(0x0F70 | ((C::TILE_INSTR + C::TILEV_INSTR) / C::NW));
        if (bvec) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            float sum = 0.f;
#pragma unroll
            for (int n = 0; n < C::NBIAS; ++n) {
              const uint32_t wd = (r & 2) ? bq[n][r >> 2].y : bq[n][r >> 2].x;
              sum += __uint_as_float((r & 1) ? (wd & 0xFFFF0000u) : (wd << 16));
            }
            bl[r] = bias_log2(sum);
          }
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            float sum = 0.f;
#pragma unroll
            for (int n = 0; n < C::NBIAS; ++n) sum += bf16_to_f32(b1[n][r]);
            bl[r] = bias_log2(sum);
          }
        }
      }
      // dsw: the gradient of the raw scaled score (what dQ contracts with K); dbw: the gradient of the score after the
      // score_mod, which is the bias gradient (biases follow the score_mod) -- the two differ by the soft-cap derivative
      // The row's visible keys, formed for each block that needs them from an opaque copy of the row: held across the tiles they took
      // the last registers of the kernels at four waves per SIMD.
      Span span = {0, 0u};
      if (need_mask) {
        int row = i;
        asm volatile("" : "+v"(row));
        span = visible_keys(MASK, row, p.Sq, p.Sk, p.q_off, p.window, p.prefix);
      }
      constexpr bool kSplit = C::NBIAS > 0 && C::MOD == kModSoftcap;
      uint32_t dsw[8], dbw[8];                   // (dbw is only written and read when the two differ)
#pragma unroll
      for (int r2 = 0; r2 < 8; ++r2) {
        float dsv[2], dbv[2], pr[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int r = 2 * r2 + e;
          const int j = jb + 8 * (r >> 2) + (r & 3);
          float fac;
          float a;
          if constexpr (C::MOD == kModCustom) a = replay_user<C::MOD>(s[r], p, uctx, lse2, b, g, h, i, j, fac);
          else a = replay_score<C::MOD>(s[r], c_scale, lse2, p.softcap, slope2, (float)(i + p.q_off - j), fac);
          if constexpr (C::NBIAS > 0) a = biased_exponent(a, bl[r]);
          pr[e] = fast_exp2(a);
          dbv[e] = dp[r] - delta;
          dsv[e] = (C::MOD == kModSoftcap || C::MOD == kModCustom) ? dbv[e] * fac : dbv[e];
        }
        if (need_mask) {                           // uniform; kept a branch: most tiles need no mask
          asm volatile("");
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int r = 2 * r2 + e;
            const int j = jb + 8 * (r >> 2) + (r & 3);
            if (hidden<MASK>(span.outside(j), i, j, p, uctx, b, g, h, qdoc, C::DOC ? kd[r >> 2][r & 3] : 0)) pr[e] = 0.f;
          }
        }
        dsv[0] *= pr[0];
        dsv[1] *= pr[1];
        dsw[r2] = pack_bf16(dsv[0], dsv[1]);
        if constexpr (kSplit) dbw[r2] = pack_bf16(dbv[0] * pr[0], dbv[1] * pr[1]);
      }
      if constexpr (C::NBIAS > 0) {                // staged for the host's reduction over the axes each bias broadcasts along
        auto staged = [&](int n) __attribute__((always_inline)) { return kSplit ? dbw[n] : dsw[n]; };
        if (p.ds_stage != nullptr && iw < p.Sq) {    // (rows past Sq and keys past Sk inside the block are zeros)
          const int nqb = (p.Sq + 31) / 32, nkb = (p.Sk + 31) / 32;
          const int64_t blk = (((int64_t)(b * p.G + g) * p.H + h) * nqb + iw / 32) * nkb + (j0 / 32 + nb);
          if (p.Sq >= 32) {                        // uniform; whole blocks, with nothing to work out per lane
#pragma unroll
            for (int u = 0; u < 2; ++u)
              *(uint4*)(p.ds_stage + blk * 1024 + u * 512 + lane * 8) = make_uint4(staged(4 * u), staged(4 * u + 1), staged(4 * u + 2), staged(4 * u + 3));
          } else if (w.col < p.Sq) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
              *(uint4*)(p.ds_stage + blk * ds_block(p.Sq) + ((2 * u + w.half) * p.Sq + w.col) * 8) =
                  make_uint4(staged(4 * u), staged(4 * u + 1), staged(4 * u + 2), staged(4 * u + 3));
          }
        }
      }
      w.template tr_stream<ST + nb * 32 * ROW>([&](auto fc, bf16x8 a) __attribute__((always_inline)) {
        constexpr int f = decltype(fc)::value, d = f % DB, ks = f / DB;
        const bf16x8 bop = __builtin_bit_cast(
            bf16x8, (i32x4){(int)dsw[4 * ks], (int)dsw[4 * ks + 1], (int)dsw[4 * ks + 2], (int)dsw[4 * ks + 3]});
        acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bop, acc[d], 0, 0, 0);
      });
    });
  };

  int2 ks = make_int2(0, 0), ks_n = make_int2(0, 0);
  int t = next_tile(t_lo, ks);
  if (t < t_hi) {
    load_tile(t, 0);
    __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0)
    __syncthreads();
    while (true) {
      bool done = false;
      static_for<0, 2>([&](auto sc) __attribute__((always_inline)) {
        if (!done) {
          const int tn = next_tile(t + 1, ks_n);
          compute(sc, t, tn < t_hi ? tn : t, ks);  // (past the last tile: the current one again, into the stage nobody reads)
          __builtin_amdgcn_s_waitcnt(0x0F70);
          __syncthreads();
          t = tn;
          ks = ks_n;
          done = t >= t_hi;
        }
      });
      if (done) break;
    }
  }

  if (i < p.Sq) {
    const int64_t orow = b * p.dq.sb + g * p.dq.sg + h * p.dq.sh + (int64_t)i * p.dq.ss;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int ch = 32 * d + 8 * r4 + 4 * w.half;
        const float x0 = acc[d][4 * r4] * p.scale, x1 = acc[d][4 * r4 + 1] * p.scale;
        const float x2 = acc[d][4 * r4 + 2] * p.scale, x3 = acc[d][4 * r4 + 3] * p.scale;
        if (p.dq_f32) *(float4*)((float*)p.dq.ptr + orow + ch) = make_float4(x0, x1, x2, x3);
        else *(uint2*)((uint16_t*)p.dq.ptr + orow + ch) = make_uint2(pack_bf16(x0, x1), pack_bf16(x2, x3));
      }
  }
}

// ------------------------------------------------------------------------------------------------
// dK, dV
// ------------------------------------------------------------------------------------------------
template <class C>
__global__ void __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::WPE, C::WPE)))
bwd_dkdv_kernel(const BwdParams p) {
  constexpr int BN = C::BN, NB = C::NB, KK = C::KK, KV = C::KV, DB = C::DB, ROW = C::ROW, ROWV = C::ROWV;
  constexpr uint32_t MASK = C::MASK;
  constexpr uint32_t POS = MASK & ~kMaskDoc;
  typedef BwdWave<C> W;
#ifdef FL_LDS_STATIC   // instantiated at run time: the size is part of the code object (a launch through the module API
                       // cannot ask for more than 64 KiB of dynamic LDS)
  __shared__ __attribute__((aligned(16))) unsigned char lds_raw[3 * C::STAGE_KV];
#else
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
#endif

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  W w;
  w.init(tid & 63);
  const int lane = w.lane;

  // grid decode: key tiles in increasing order (under a causal mask the first ones see the most rows)
  int kt, bh;
  if (p.order_k == 1) {                            // whole key/value heads per XCD: their Q / dO tiles stay in one L2
    tile_of(p.step_k, blockIdx.x >> 3, p.k_tiles, bh, kt);
    bh = bh * 8 + (blockIdx.x & 7);
  } else {
    tile_of(p.step_k, blockIdx.x, p.k_tiles, bh, kt);
  }
  const KeyProblem kp = key_problem(p, bh);
  const int split = kp.split, hk = kp.hk, g = kp.g, b = kp.b, h_first = kp.h_first;
  const int group = p.heads_wg;                    // query heads this workgroup sums over
  const int j0 = kt * C::BM, jw = j0 + 32 * wave;
  const int j = jw + w.col, jc = j < p.Sk ? j : p.Sk - 1;
  const Span span = C::NBIAS > 0 ? Span{0, 0u} : seeing_rows(MASK, j, p.Sq, p.Sk, p.q_off, p.window, p.prefix);
  const FwdParams uctx = user_context(p);          // what a compiled variant's expressions read (unused otherwise)

  bf16x8 kf[KK], vf[KV];
  {
    const uint16_t* kp = (const uint16_t*)p.k.ptr + b * p.k.sb + g * p.k.sg + hk * p.k.sh + (int64_t)jc * p.k.ss;
    const uint16_t* vp = (const uint16_t*)p.v.ptr + b * p.v.sb + g * p.v.sg + hk * p.v.sh + (int64_t)jc * p.v.ss;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[kk] = *(const bf16x8*)(kp + 16 * kk + 8 * w.half);
#pragma unroll
    for (int kk = 0; kk < KV; ++kk) vf[kk] = *(const bf16x8*)(vp + 16 * kk + 8 * w.half);
  }
  const float c_scale = p.scale * kLog2e;
  int kdoc = 0;
  if constexpr ((MASK & kMaskDoc) != 0) kdoc = p.kv_doc[(int64_t)b * p.Sk + jc];

  constexpr int DBV = C::DBV;
  f32x16 dk[DB], dv[DBV];
#pragma unroll
  for (int d = 0; d < DB; ++d) dk[d] = W::zero16();
#pragma unroll
  for (int d = 0; d < DBV; ++d) dv[d] = W::zero16();

  // query rows that can see the workgroup's keys; q-tile skipping for document masks
  const int j_last = (j0 + C::BM < p.Sk ? j0 + C::BM : p.Sk) - 1;
  int q_lo, q_hi;
  query_range(MASK, j0, j_last, p.Sq + p.q_off, p.window, p.prefix, q_lo, q_hi);   // as positions; row = position - q_off
  q_lo = max(q_lo - p.q_off, 0);
  q_hi = max(q_hi - p.q_off, 0);
  const int t_lo = q_lo / BN, t_hi = (q_hi + BN - 1) / BN;
  const int nt = t_hi - t_lo;                      // q-tiles per head
  // items, head-major: q-tile r (from t_lo) of query head h of the group; h == group: none.  A pair, because a division per use
  // stood in the chain of every step.
  struct Item { int r, h; };
  const int nqs = (p.Sq + kSumBlock - 1) / kSumBlock;
  int2 ks_wg = make_int2(0, 0), ks_wave = make_int2(0, 0);
  TileWindow win = {0, make_int2(0, 0), 0};        // over the q-tiles t_lo + 0, 1, ... of a head: the ids do not depend on it
  auto load_window = [&](int t) __attribute__((always_inline)) {
    win.base = t;
    win.ids = merge_summaries<NB>(p.q_sum + (int64_t)b * nqs, (t_lo + t + lane) * NB, nqs);
  };
  auto scan_window = [&]() __attribute__((always_inline)) {
    const int tt = t_lo + win.base + lane;
    const int q_last = (tt * BN + BN < p.Sq ? tt * BN + BN : p.Sq) - 1;
    win.vis = __builtin_amdgcn_ballot_w64(
        win.base + lane < nt && classify_block(MASK, tt * BN + p.q_off, q_last + p.q_off, j0, j0 + C::BM - 1, p.Sk, p.window, p.prefix, win.ids, ks_wg) != kSkip);
  };
  if (C::DOC && nt > 0) {                     // (without rows there are no summaries)
    const int nks = (p.Sk + kSumBlock - 1) / kSumBlock;
    const int2* ksum = p.kv_sum + (int64_t)b * nks;
    load_window(0);
    ks_wg = merge_summaries<C::BM / kSumBlock>(ksum, j0 / kSumBlock, nks);
    ks_wave = ksum[min(jw / kSumBlock, nks - 1)];
    scan_window();
  }
  // first item at or after `it` whose q-tile holds a row that sees any of the workgroup's keys, and what its document ids say
  // about the wave's keys (Docs)
  enum Docs { kDocsSame, kDocsMask, kDocsNone };   // all of one document; some; no row sees any of them
  auto next_item = [&](Item it, int& docs) __attribute__((always_inline)) -> Item {
    docs = kDocsSame;
    if constexpr (C::DOC) {
      while (it.h < group) {
        if (it.r < win.base || it.r >= win.base + 64) {
          load_window(it.r);
          scan_window();
        }
        const unsigned long long rest = win.vis >> (it.r - win.base);
        if (rest != 0) {
          it.r += __builtin_ctzll(rest);
          docs = same_document(win.at(it.r), ks_wave) ? kDocsSame : no_common_document(win.at(it.r), ks_wave) ? kDocsNone : kDocsMask;
          return it;
        }
        it.r = win.base + 64;
        if (it.r >= nt) it = Item{0, it.h + 1};
      }
    }
    return it;
  };
  auto item_after = [&](Item it, int& docs) __attribute__((always_inline)) -> Item {
    docs = kDocsSame;
    if (it.h >= group) return it;
    return next_item(it.r + 1 < nt ? Item{it.r + 1, it.h} : Item{0, it.h + 1}, docs);
  };

  // A whole tile's addresses: a uniform base and what this lane adds to it, the same for each of its load instructions (their rows
  // are a multiple of 16 apart, which leaves the swizzle as it is).  64 rows fit 32 bits: the host refuses negative row strides and those of
  // 2^23 elements and more.  Not with bias values in registers, where there is no room for it.  (Causal training step
  // 4 x 16 x 4096, D = 64: 778 -> 772 us; with the items as pairs, earlier, 830 -> 818)
  const uint32_t q_lane = tile_lane_offset<C::D>(wave, lane, (uint32_t)p.q.ss * 2), d_lane = tile_lane_offset<C::DV>(wave, lane, (uint32_t)p.dout.ss * 2);
  auto load_item = [&](Item it, int stage) __attribute__((always_inline)) {
    const int t = t_lo + it.r, h = h_first + it.h;
    const int nvalid = min(BN, p.Sq - t * BN);
    unsigned char* st = lds_raw + stage * C::STAGE_KV;
    const unsigned char* qb = (const unsigned char*)((const uint16_t*)p.q.ptr + b * p.q.sb + g * p.q.sg + h * p.q.sh + (int64_t)(t * BN) * p.q.ss);
    const unsigned char* db = (const unsigned char*)((const uint16_t*)p.dout.ptr + b * p.dout.sb + g * p.dout.sg + h * p.dout.sh + (int64_t)(t * BN) * p.dout.ss);
    constexpr int NU = (C::TILE_INSTR > C::TILEV_INSTR ? C::TILE_INSTR : C::TILEV_INSTR) / C::NW;
    if (C::NBIAS == 0 && nvalid == BN) {
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if (u < C::TILE_INSTR / C::NW)
          __builtin_amdgcn_global_load_lds((global_cvoid*)(qb + (int64_t)(u * C::NW * C::RPI) * 2 * p.q.ss + q_lane),
                                           (lds_void*)(st + (wave + u * C::NW) * 1024), 16, 0, 0);
        if (u < C::TILEV_INSTR / C::NW)
          __builtin_amdgcn_global_load_lds((global_cvoid*)(db + (int64_t)(u * C::NW * (1024 / ROWV)) * 2 * p.dout.ss + d_lane),
                                           (lds_void*)(st + C::TILE + (wave + u * C::NW) * 1024), 16, 0, 0);
      }
    } else {
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if (u < C::TILE_INSTR / C::NW) tile_load_instr<C::D>(qb, p.q.ss * 2, nvalid, wave + u * C::NW, lane, st);
        if (u < C::TILEV_INSTR / C::NW) tile_load_instr<C::DV>(db, p.dout.ss * 2, nvalid, wave + u * C::NW, lane, st + C::TILE);
      }
    }
    // row statistics: 64 rows per instruction, 4 bytes per lane
    const int64_t srow = ((int64_t)(b * p.G + g) * p.H + h) * p.Sq;
    if constexpr (C::DOC) {
      if (wave == 2) {                             // document ids of the rows
        lds_void* dst = (lds_void*)(st + C::STATS + 2 * C::STAT);
        __builtin_amdgcn_global_load_lds((global_cvoid*)(p.q_doc + (int64_t)b * p.Sq + t * BN + (lane < nvalid ? lane : nvalid - 1)), dst, 4, 0, 0);
      }
    }
    for (int u = wave; u < 2 * (BN / 64 > 0 ? BN / 64 : 1); u += C::NW) {
      const int which = u % 2, blk = u / 2;        // 0: lse2, 1: delta
      const int r = blk * 64 + lane;
      const int row = t * BN + (r < nvalid ? r : nvalid - 1);
      const float* src = (which == 0 ? p.lse2 : p.delta) + srow + row;
      if (BN >= 64 || lane < BN) {
        lds_void* dst = (lds_void*)(st + C::STATS + which * C::STAT + blk * 256);
        __builtin_amdgcn_global_load_lds((global_cvoid*)src, dst, 4, 0, 0);
      }
    }
  };

  // ---- software pipeline over 32-row query blocks.  Step n owns block n (scores and dP in
  // registers) and its successor:
  //   phase A:  S, dP of block n + 1 on the matrix core   ||   P, dS of the first 16 rows of block n
  //   phase B:  dV += dO^T P, dK += Q^T dS of block n, rows 0..15 first   ||   P, dS of rows 16..31
  // so the matrix core and the vector ALU of a wave have independent work at the same time.  The
  // Q / dO tiles cycle through a ring of three LDS stages: the tile after next is requested when
  // every wave has left the tile before the current one.
  constexpr int NBR = C::NBIAS > 0 ? C::NBIAS : 1;
  struct Blk {
    f32x16 s, dp;
    uint16_t bias[NBR][16];                        // this lane's bias values of the block, as loaded
  };
  // Bias values of query block Q of item it (rows past Sq: the last one's): requested a step before they are used, so that
  // their latency, and that of the tile loads in flight before them, lies behind a whole block's matrix work -- where two
  // blocks' values fit the registers (two biases at head dim 64 spilled 40 of them), else at the start of their own step.
  constexpr bool kBiasAhead = C::WPE == 1 || (C::D + C::DV) * C::NBIAS <= 128;
  auto load_bias = [&](Item it, int Q, Blk& blk) __attribute__((always_inline)) {
    if constexpr (C::NBIAS > 0) {
      BiasHead<C::NBIAS> bh_;
      bh_.set(p, b, g, h_first + it.h);
      const int i0 = (t_lo + it.r) * BN + 32 * Q + 4 * w.half;
#pragma unroll
      for (int n = 0; n < C::NBIAS; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) blk.bias[n][r] = bh_.raw1(p, n, min(i0 + 8 * (r >> 2) + (r & 3), p.Sq - 1), jc);
    }
  };
  constexpr int NSTAGE = 3;
  const RowBounds bounds = row_bounds(POS, jw, jw + 31, p.Sk, p.window, p.prefix);
  // one step: block QB of the tile in the LDS stage at byte offset base_c is current, block QN of
  // the tile at base_n is next (the same tile, or row block 0 of the following one)
  auto step = [&](auto qb_c, auto qn_c, uint32_t base_c, uint32_t base_n, Item it, Item it_n, bool doc_mask, bool first, Blk& cur, Blk& nxt) __attribute__((always_inline)) {
    constexpr int QB = decltype(qb_c)::value, QN = decltype(qn_c)::value;
    const int t = t_lo + it.r, h = h_first + it.h;
    const int ib = t * BN + 32 * QB;
    const float slope2 = C::MOD == kModAlibi ? p.alibi_slopes[h] * kLog2e : 0.f;
    const bool need_mask = doc_mask || (MASK & kMaskCustom) != 0 || ib + 31 >= p.Sq || (POS == 0 ? jw + 31 >= p.Sk : !bounds.whole(ib + p.q_off, ib + 31 + p.q_off));
    // lane addresses: row reads of the next block (Q fragments, then dO), transposing reads of the current one (dO, then Q)
    uint32_t ra_n[KK + KV], ta_c[DBV + DB][2];
#pragma unroll
    for (int f = 0; f < KK + KV; ++f) ra_n[f] = (f < KK ? w.ra[f < KK ? f : 0] : w.rv[f < KK ? 0 : f - KK]) + base_n;
#pragma unroll
    for (int d = 0; d < DBV + DB; ++d)
#pragma unroll
      for (int u = 0; u < 2; ++u) ta_c[d][u] = (d < DBV ? w.tv[d < DBV ? d : 0][u] : w.ta[d < DBV ? 0 : d - DBV][u]) + base_c;
    // row statistics of the current block's 16 rows of this half: quads of lse2 and of delta, read
    // shortly before the element pairs that use them
    const uint32_t stat_addr = (uint32_t)(4 * w.half) * 4 + base_c;
    i32x4 st_l[4], st_d[4], qd[4];                 // (qd: the rows' document ids)
    auto read_stats = [&](auto q_lo, auto q_hi) __attribute__((always_inline)) {   // quads [q_lo, q_hi): rows 8*q .. 8*q + 3 (+ 4*half)
      static_for<decltype(q_lo)::value, decltype(q_hi)::value>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q4 = decltype(qc)::value;
        W::template read_b128<C::STATS + (32 * QB + 8 * q4) * 4>(st_l[q4], stat_addr);
        W::template read_b128<C::STATS + C::STAT + (32 * QB + 8 * q4) * 4>(st_d[q4], stat_addr);
        if constexpr (C::DOC) W::template read_b128<C::STATS + 2 * C::STAT + (32 * QB + 8 * q4) * 4>(qd[q4], stat_addr);
      });
    };
    if (first) {                                   // the very first block: its scores are not there yet
      if constexpr (kBiasAhead) load_bias(it, QB, cur);
      cur.s = W::zero16();
      cur.dp = W::zero16();
      w.template row_stream_g<RowPair<QB * 32 * ROW, C::TILE + QB * 32 * ROWV, KK>, KK + KV, 2>(
          [&](auto fc) __attribute__((always_inline)) {
            constexpr int f = decltype(fc)::value;
            if constexpr (f < KK) return w.ra[f] + base_c;
            else return w.rv[f - KK] + base_c;
          },
          [&](auto fc, bf16x8 a) __attribute__((always_inline)) {
            constexpr int f = decltype(fc)::value;
            if constexpr (f < KK) cur.s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kf[f], cur.s, 0, 0, 0);
            else cur.dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, vf[f - KK], cur.dp, 0, 0, 0);
          });
    }
    read_stats(std::integral_constant<int, 0>(), std::integral_constant<int, 2>());   // for the pairs of phase A
    const int irow = ib + 4 * w.half;              // query row of register 0
    if constexpr (kBiasAhead) load_bias(it_n, QN, nxt);
    else load_bias(it, QB, cur);
    Span sp = span;
    if (C::NBIAS > 0 && need_mask) {               // formed again: with bias values in registers there is no room to hold it
      int key = j;
      asm volatile("" : "+v"(key));
      sp = seeing_rows(MASK, key, p.Sq, p.Sk, p.q_off, p.window, p.prefix);
    }
    uint32_t pw[8], dsw[8];
    auto ew_pair = [&](int r2) __attribute__((always_inline)) {      // P and dS of registers 2*r2, 2*r2 + 1
      float pv[2], dsv[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int r = 2 * r2 + e;
        const int i = irow + 8 * (r >> 2) + (r & 3);
        const float lse2 = __int_as_float(st_l[r >> 2][r & 3]), delta = __int_as_float(st_d[r >> 2][r & 3]);
        float fac;
        float a;
        if constexpr (C::MOD == kModCustom) a = replay_user<C::MOD>(cur.s[r], p, uctx, lse2, b, g, h, i, j, fac);
        else a = replay_score<C::MOD>(cur.s[r], c_scale, lse2, p.softcap, slope2, (float)(i + p.q_off - j), fac);
        if constexpr (C::NBIAS > 0) {
          float sum = bf16_to_f32(cur.bias[0][r]);
          if constexpr (C::NBIAS > 1) sum += bf16_to_f32(cur.bias[NBR - 1][r]);
          a = biased_exponent(a, bias_log2(sum));
        }
        pv[e] = fast_exp2(a);
        dsv[e] = cur.dp[r] - delta;
        if constexpr (C::MOD == kModSoftcap || C::MOD == kModCustom) dsv[e] *= fac;
      }
      if (need_mask) {                             // uniform; kept a branch: most blocks need no mask
        asm volatile("");
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int r = 2 * r2 + e;
          const int i = irow + 8 * (r >> 2) + (r & 3);
          if (hidden<MASK>(sp.outside(i), i, j, p, uctx, b, g, h, C::DOC ? qd[r >> 2][r & 3] : 0, kdoc)) pv[e] = 0.f;
        }
      }
      dsv[0] *= pv[0];
      dsv[1] *= pv[1];
      pw[r2] = pack_bf16(pv[0], pv[1]);
      dsw[r2] = pack_bf16(dsv[0], dsv[1]);
      asm volatile("" : "+v"(pw[r2]), "+v"(dsw[r2]));               // stays where it is scheduled
    };
    // phase A
    nxt.s = W::zero16();
    nxt.dp = W::zero16();
    w.template row_stream_g<RowPair<QN * 32 * ROW, C::TILE + QN * 32 * ROWV, KK>, KK + KV, C::GR>(
        [&](auto fc) __attribute__((always_inline)) { return ra_n[decltype(fc)::value]; }, [&](auto fc, bf16x8 a) __attribute__((always_inline)) {
          constexpr int f = decltype(fc)::value;
          if constexpr (f < KK) nxt.s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kf[f], nxt.s, 0, 0, 0);
          else nxt.dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, vf[f - KK], nxt.dp, 0, 0, 0);
          static_for<4 * f / (KK + KV), 4 * (f + 1) / (KK + KV)>([&](auto r2) __attribute__((always_inline)) { ew_pair(r2); });   // pairs 0..3
          __builtin_amdgcn_sched_barrier(0);
        });
    if constexpr (C::DOC) W::landed(qd[0], qd[1]);
    // phase B
    read_stats(std::integral_constant<int, 2>(), std::integral_constant<int, 4>());   // covered by the first wait below
    constexpr int NT = DBV + DB;                   // transposed fragments per 16 rows
    w.template tr_stream_g<TrQuad<C::TILE + QB * 32 * ROWV, QB * 32 * ROW, DBV, DB, ROWV, ROW>, 2 * NT, C::GT>(
        [&](auto fc, int u) __attribute__((always_inline)) { return ta_c[decltype(fc)::value % NT][u]; },
        [&](auto fc, bf16x8 a) __attribute__((always_inline)) {
          constexpr int f = decltype(fc)::value, ks = f / NT;
          if constexpr (f % NT < DBV) {
            constexpr int d = f % NT;
            const bf16x8 bop = __builtin_bit_cast(
                bf16x8, (i32x4){(int)pw[4 * ks], (int)pw[4 * ks + 1], (int)pw[4 * ks + 2], (int)pw[4 * ks + 3]});
            dv[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bop, dv[d], 0, 0, 0);
          } else {
            constexpr int d = f % NT - DBV;
            const bf16x8 bop = __builtin_bit_cast(
                bf16x8, (i32x4){(int)dsw[4 * ks], (int)dsw[4 * ks + 1], (int)dsw[4 * ks + 2], (int)dsw[4 * ks + 3]});
            dk[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bop, dk[d], 0, 0, 0);
          }
          if constexpr (f < NT)                    // pairs 4..7 during the rows-0..15 half
            static_for<4 + 4 * f / NT, 4 + 4 * (f + 1) / NT>([&](auto r2) __attribute__((always_inline)) { ew_pair(r2); });
          __builtin_amdgcn_sched_barrier(0);
        });
    if constexpr (C::DOC) W::landed(qd[2], qd[3]);
  };
  static_assert(NB == 2, "a tile is two row blocks: the two score register sets swap roles twice per tile");

  int dm0 = 0, dm1 = 0, dm2 = 0;                   // Docs of it0, it1, it2
  Item it0 = nt > 0 ? next_item(Item{0, 0}, dm0) : Item{0, group};
  if (it0.h < group) {
    Item it1 = item_after(it0, dm1), it2 = item_after(it1, dm2);
    load_item(it0, 0);
    if (it1.h < group) load_item(it1, 1);
    __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0)
    __syncthreads();
    if (it2.h < group) load_item(it2, 2);
    Blk ba, bb;
    int stage = 0;                                 // ring stage of the current tile
    bool first = true;
    while (it0.h < group) {
      const int stage_n = stage + 1 == NSTAGE ? 0 : stage + 1;
      const uint32_t base_c = stage * C::STAGE_KV, base_n = stage_n * C::STAGE_KV;
      // A tile of which this wave's keys are hidden is passed over (the workgroup's four waves walk one list, but the last wave's
      // keys start 96 rows later, and may be of another document); the next one's first scores are then formed on entry.
      // (windows and packed documents, 8 x 16 heads x 2048 rows, D = 64: 124 -> 121 us)
      const int pos0 = (t_lo + it0.r) * BN + p.q_off;
      const bool none = dm0 == kDocsNone || bounds.hidden(pos0, pos0 + BN - 1);
      if (!none) {
        step(std::integral_constant<int, 0>(), std::integral_constant<int, 1>(), base_c, base_c, it0, it0, dm0 != kDocsSame, first, ba, bb);
        step(std::integral_constant<int, 1>(), std::integral_constant<int, 0>(), base_c, base_n, it0, it1.h < group ? it1 : it0, dm0 != kDocsSame, false, bb, ba);
      }
      first = none;
      __builtin_amdgcn_s_waitcnt(0x0F70);          // the tile after next has landed ...
      __syncthreads();                             // ... for everyone, and everyone has left this tile
      it0 = it1;
      dm0 = dm1;
      it1 = it2;
      dm1 = dm2;
      it2 = item_after(it2, dm2);
      if (it2.h < group) load_item(it2, stage);
      stage = stage_n;
    }
  }

  if (j < p.Sk) {
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int ch = 32 * d + 8 * r4 + 4 * w.half;
        store_kv_grad<false, C::D>(p, split, b, g, hk, j, ch, dk[d][4 * r4] * p.scale, dk[d][4 * r4 + 1] * p.scale,
                                   dk[d][4 * r4 + 2] * p.scale, dk[d][4 * r4 + 3] * p.scale);
      }
#pragma unroll
    for (int d = 0; d < DBV; ++d)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int ch = 32 * d + 8 * r4 + 4 * w.half;
        store_kv_grad<true, C::DV>(p, split, b, g, hk, j, ch, dv[d][4 * r4], dv[d][4 * r4 + 1], dv[d][4 * r4 + 2], dv[d][4 * r4 + 3]);
      }
  }
}

// ------------------------------------------------------------------------------------------------
// dK, dV with specialised waves: the same contractions as bwd_dkdv_kernel, for head dims whose
// accumulators (32 keys x D channels x two gradients in fp32) leave no room for a second wave on
// the SIMD.  Eight waves per workgroup; waves w and w + 4 own the same 32 keys and share a SIMD:
//   wave w     ("P wave"):   S = Q K^T, P = exp2(..), dV += dO^T P one block later; hands P (times
//                            the soft-cap derivative) to its partner through LDS, fp32
//   wave w + 4 ("dS wave"):  dP = dO V^T, dS = P * (dP - delta) one block later, dK += Q^T dS
// Each does half of the matrix work of a block and holds one accumulator set, so both fit the
// register budget of two waves per SIMD and fill each other's stalls.  One workgroup barrier per
// 32-row block hands the P blocks over (two exchange buffers per wave pair).
// ------------------------------------------------------------------------------------------------
template <class C>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
bwd_dkdv_ws_kernel(const BwdParams p) {
  constexpr int BN = C::BN, NB = C::NB, KK = C::KK, KV = C::KV, DB = C::DB, ROW = C::ROW, ROWV = C::ROWV;
  constexpr uint32_t MASK = C::MASK;
  constexpr uint32_t POS = MASK & ~kMaskDoc;
  static_assert(C::MOD != kModCustom && (MASK & kMaskCustom) == 0, "compiled variants run the plain dK/dV kernel");
  constexpr int NWS = 8;                           // waves of the workgroup
  constexpr int NSTAGE = 3;
  constexpr int XBUF = 64 * 16 * 4;                // one exchange buffer: 16 floats per lane, [quad][lane][4]
  constexpr int XCH = NSTAGE * C::STAGE_KV;        // exchange buffers [key group][2] follow the tile ring
  constexpr int DBV = C::DBV;
  static_assert(NB == 2 && BN == 64, "two row blocks per tile");
  static_assert(C::TILE_INSTR % NWS == 0 && C::TILEV_INSTR % NWS == 0, "every wave issues the same number of loads");
  typedef BwdWave<C> W;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int role = wave >> 2, kg = wave & 3;       // 0: P wave, 1: dS wave; key group
  W w;
  w.init(tid & 63);
  const int lane = w.lane;

  int kt, bh;
  if (p.order_k == 1) {                            // whole key/value heads per XCD: their Q / dO tiles stay in one L2
    tile_of(p.step_k, blockIdx.x >> 3, p.k_tiles, bh, kt);
    bh = bh * 8 + (blockIdx.x & 7);
  } else {
    tile_of(p.step_k, blockIdx.x, p.k_tiles, bh, kt);
  }
  const KeyProblem kp = key_problem(p, bh);
  const int split = kp.split, hk = kp.hk, g = kp.g, b = kp.b, h_first = kp.h_first;
  const int group = p.heads_wg;                    // query heads this workgroup sums over
  const int j0 = kt * C::BM, jw = j0 + 32 * kg;
  const int j = jw + w.col, jc = j < p.Sk ? j : p.Sk - 1;
  const Span span = seeing_rows(MASK, j, p.Sq, p.Sk, p.q_off, p.window, p.prefix);
  const float c_scale = p.scale * kLog2e;

  // query rows that can see the workgroup's keys; q-tile skipping for document masks
  const int j_last = (j0 + C::BM < p.Sk ? j0 + C::BM : p.Sk) - 1;
  int q_lo, q_hi;
  query_range(MASK, j0, j_last, p.Sq + p.q_off, p.window, p.prefix, q_lo, q_hi);   // as positions; row = position - q_off
  q_lo = max(q_lo - p.q_off, 0);
  q_hi = max(q_hi - p.q_off, 0);
  const int t_lo = q_lo / BN, t_hi = (q_hi + BN - 1) / BN;
  const int nt = t_hi - t_lo;                      // q-tiles per head
  const int n_items = nt > 0 ? nt * group : 0;     // (head of the group, q-tile), head-major
  const int nqs = (p.Sq + kSumBlock - 1) / kSumBlock;
  int2 ks_wg = make_int2(0, 0), ks_wave = make_int2(0, 0);
  TileWindow win = {0, make_int2(0, 0), 0};        // over the q-tiles t_lo + 0, 1, ... of a head: the ids do not depend on it
  auto load_window = [&](int t) __attribute__((always_inline)) {
    win.base = t;
    win.ids = merge_summaries<NB>(p.q_sum + (int64_t)b * nqs, (t_lo + t + lane) * NB, nqs);
  };
  auto scan_window = [&]() __attribute__((always_inline)) {
    const int tt = t_lo + win.base + lane;
    const int q_last = (tt * BN + BN < p.Sq ? tt * BN + BN : p.Sq) - 1;
    win.vis = __builtin_amdgcn_ballot_w64(
        win.base + lane < nt && classify_block(MASK, tt * BN + p.q_off, q_last + p.q_off, j0, j0 + C::BM - 1, p.Sk, p.window, p.prefix, win.ids, ks_wg) != kSkip);
  };
  if (C::DOC && n_items > 0) {                     // (without rows there are no summaries)
    const int nks = (p.Sk + kSumBlock - 1) / kSumBlock;
    const int2* ksum = p.kv_sum + (int64_t)b * nks;
    load_window(0);
    ks_wg = merge_summaries<C::BM / kSumBlock>(ksum, j0 / kSumBlock, nks);
    ks_wave = ksum[min(jw / kSumBlock, nks - 1)];
    scan_window();
  }
  // first item at or after `it` whose q-tile holds a row that sees any of the workgroup's keys (n_items if none), and whether
  // the wave's keys need the document mask in it
  auto next_item = [&](int it, bool& doc_mask) __attribute__((always_inline)) -> int {
    doc_mask = false;
    if constexpr (C::DOC) {
      while (it < n_items) {
        const int r = it % nt;
        if (r < win.base || r >= win.base + 64) {
          load_window(r);
          scan_window();
        }
        const unsigned long long rest = win.vis >> (r - win.base);
        if (rest != 0) {
          const int step = __builtin_ctzll(rest);
          doc_mask = !same_document(win.at(r + step), ks_wave);
          return it + step;
        }
        it += min(win.base + 64, nt) - r;
      }
    }
    return it;
  };

  auto load_item = [&](int it, int stage) __attribute__((always_inline)) {
    const int t = t_lo + it % nt, h = h_first + it / nt;
    const int nvalid = min(BN, p.Sq - t * BN);
    unsigned char* st = lds_raw + stage * C::STAGE_KV;
    const unsigned char* qb = (const unsigned char*)((const uint16_t*)p.q.ptr + b * p.q.sb + g * p.q.sg + h * p.q.sh + (int64_t)(t * BN) * p.q.ss);
    const unsigned char* db = (const unsigned char*)((const uint16_t*)p.dout.ptr + b * p.dout.sb + g * p.dout.sg + h * p.dout.sh + (int64_t)(t * BN) * p.dout.ss);
#pragma unroll
    for (int u = 0; u < (C::TILE_INSTR > C::TILEV_INSTR ? C::TILE_INSTR : C::TILEV_INSTR) / NWS; ++u) {
      if (u < C::TILE_INSTR / NWS) tile_load_instr<C::D>(qb, p.q.ss * 2, nvalid, wave + u * NWS, lane, st);
      if (u < C::TILEV_INSTR / NWS) tile_load_instr<C::DV>(db, p.dout.ss * 2, nvalid, wave + u * NWS, lane, st + C::TILE);
    }
    if (wave < 2) {                                // row statistics, 4 bytes per lane: wave 0 lse2, wave 1 delta
      const int64_t srow = ((int64_t)(b * p.G + g) * p.H + h) * p.Sq;
      const int row = t * BN + (lane < nvalid ? lane : nvalid - 1);
      const float* src = (wave == 0 ? p.lse2 : p.delta) + srow + row;
      lds_void* dst = (lds_void*)(st + C::STATS + wave * C::STAT);
      __builtin_amdgcn_global_load_lds((global_cvoid*)src, dst, 4, 0, 0);
    }
    if constexpr (C::DOC) {
      if (wave == 2) {                             // document ids of the rows
        lds_void* dst = (lds_void*)(st + C::STATS + 2 * C::STAT);
        __builtin_amdgcn_global_load_lds((global_cvoid*)(p.q_doc + (int64_t)b * p.Sq + t * BN + (lane < nvalid ? lane : nvalid - 1)), dst, 4, 0, 0);
      }
    }
  };
  // end of an iteration: this wave's LDS traffic (and, when `loads`, its tile loads) is complete, then
  // the workgroup barrier.  No fence beyond that: every LDS access of the loop is issued by hand.
  auto iteration_end = [&](bool loads) __attribute__((always_inline)) {
    if (loads) __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
    else __builtin_amdgcn_s_waitcnt(0xC07F);         // lgkmcnt(0)
    asm volatile("" ::: "memory");                   // no memory access moves across the barrier at compile time
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // window of the tile list: items at list positions P - 1, P, P + 1, P + 2 (n_items = none)
  bool dm0 = false, dmp1 = false, dmp2 = false;    // do the items at P, P + 1, P + 2 need the document mask?
  int itm1 = n_items, it0 = next_item(0, dm0);
  int itp1 = it0 < n_items ? next_item(it0 + 1, dmp1) : n_items;
  int itp2 = itp1 < n_items ? next_item(itp1 + 1, dmp2) : n_items;
  if (it0 < n_items) load_item(it0, 0);
  if (itp1 < n_items) load_item(itp1, 1);
  if (itp2 < n_items) load_item(itp2, 2);
  iteration_end(true);
  int s0 = 0;                                      // ring stage of position P
  const uint32_t xaddr = XCH + kg * (2 * XBUF) + lane * 16;   // this lane's slot in exchange buffer 0 of its wave pair
  const uint32_t stat_addr = (uint32_t)(4 * w.half) * 4;

  if (role == 0) {
    // ================= P wave =================
    bf16x8 kf[KK];
    {
      const uint16_t* kp = (const uint16_t*)p.k.ptr + b * p.k.sb + g * p.k.sg + hk * p.k.sh + (int64_t)jc * p.k.ss;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kf[kk] = *(const bf16x8*)(kp + 16 * kk + 8 * w.half);
    }
    int kdoc = 0;
    if constexpr ((MASK & kMaskDoc) != 0) kdoc = p.kv_doc[(int64_t)b * p.Sk + jc];
    f32x16 dv[DBV];
#pragma unroll
    for (int d = 0; d < DBV; ++d) dv[d] = W::zero16();
    f32x16 sa = W::zero16(), sb = W::zero16();
    uint32_t pw[8] = {0, 0, 0, 0, 0, 0, 0, 0};     // bf16 pairs of the last block's P, consumed one iteration later
    auto scores = [&](auto off_c, uint32_t base, f32x16& dst) __attribute__((always_inline)) {   // S of one block, no overlap
      dst = W::zero16();
      w.template row_stream_g<RowOne<decltype(off_c)::value>, KK, 2>([&](auto fc) __attribute__((always_inline)) {
        return w.ra[decltype(fc)::value] + base;
      }, [&](auto fc, bf16x8 a) __attribute__((always_inline)) {
        dst = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kf[decltype(fc)::value], dst, 0, 0, 0);
      });
    };
    const RowBounds bounds = row_bounds(POS, jw, jw + 31, p.Sk, p.window, p.prefix);
    // block QB of item `it` (stage offset base_c) is current (scores in cur); the scores of block QN at
    // base_n go to nxt; P of the current block goes to exchange buffer XB
    auto p_iter = [&](auto qb_c, auto qn_c, auto xb_c, uint32_t base_c, uint32_t base_n, int it, f32x16& cur, f32x16& nxt) __attribute__((always_inline)) {
      constexpr int QB = decltype(qb_c)::value, QN = decltype(qn_c)::value, XB = decltype(xb_c)::value;
      const int t = t_lo + it % nt, h = h_first + it / nt;
      const int ib = t * BN + 32 * QB;
      const float slope2 = C::MOD == kModAlibi ? p.alibi_slopes[h] * kLog2e : 0.f;
      const bool need_mask = dm0 || ib + 31 >= p.Sq || (POS == 0 ? jw + 31 >= p.Sk : !bounds.whole(ib + p.q_off, ib + 31 + p.q_off));
      uint32_t ra_n[KK];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) ra_n[kk] = w.ra[kk] + base_n;
      i32x4 st_l[4], qd[4];                        // lse2 and document ids of the block's 16 rows of this half
      static_for<0, 4>([&](auto qc) __attribute__((always_inline)) {
        W::template read_b128<C::STATS + (32 * QB + 8 * decltype(qc)::value) * 4>(st_l[decltype(qc)::value], stat_addr + base_c);
        if constexpr (C::DOC)
          W::template read_b128<C::STATS + 2 * C::STAT + (32 * QB + 8 * decltype(qc)::value) * 4>(qd[decltype(qc)::value], stat_addr + base_c);
      });
      const int irow = ib + 4 * w.half;            // query row of register 0
      float bl[C::NBIAS > 0 ? 16 : 1];             // bias values of the current block's scores of this lane
      if constexpr (C::NBIAS > 0) {
        BiasHead<C::NBIAS> bh_;
        bh_.set(p, b, g, h);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = irow + 8 * (r >> 2) + (r & 3);
          bl[r] = bh_.value(p, i < p.Sq ? i : p.Sq - 1, jc);
        }
      }
      float pf[4];
      auto ew_pair = [&](auto r2c) __attribute__((always_inline)) {
        constexpr int r2 = decltype(r2c)::value;
        float pv[2], fc2[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int r = 2 * r2 + e;
          const int i = irow + 8 * (r >> 2) + (r & 3);
          const float lse2 = __int_as_float(st_l[r >> 2][r & 3]);
          float a = replay_score<C::MOD>(cur[r], c_scale, lse2, p.softcap, slope2, (float)(i + p.q_off - j), fc2[e]);
          if constexpr (C::NBIAS > 0) a = biased_exponent(a, bl[r]);
          pv[e] = fast_exp2(a);
        }
        if (need_mask) {                           // uniform; kept a branch: most blocks need no mask
          asm volatile("");
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int r = 2 * r2 + e;
            const int i = irow + 8 * (r >> 2) + (r & 3);
            if (span.outside(i) || (C::DOC && qd[r >> 2][r & 3] != kdoc)) pv[e] = 0.f;
          }
        }
        pw[r2] = pack_bf16(pv[0], pv[1]);
        asm volatile("" : "+v"(pw[r2]));
        pf[2 * (r2 & 1)] = C::MOD == kModSoftcap ? pv[0] * fc2[0] : pv[0];
        pf[2 * (r2 & 1) + 1] = C::MOD == kModSoftcap ? pv[1] * fc2[1] : pv[1];
        if constexpr (r2 % 2 == 1)                 // registers 4q .. 4q + 3 are complete: quad q = r2 / 2
          W::template write_b128<XB * XBUF + (r2 / 2) * 1024>(
              xaddr, (i32x4){__float_as_int(pf[0]), __float_as_int(pf[1]), __float_as_int(pf[2]), __float_as_int(pf[3])});
      };
      // phase 1: scores of the next block  ||  P of the current block
      nxt = W::zero16();
      w.template row_stream_g<RowOne<QN * 32 * ROW>, KK, 2>([&](auto fc) __attribute__((always_inline)) {
        return ra_n[decltype(fc)::value];
      }, [&](auto fc, bf16x8 a) __attribute__((always_inline)) {
        constexpr int f = decltype(fc)::value;
        nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kf[f], nxt, 0, 0, 0);
        static_for<8 * f / KK, 8 * (f + 1) / KK>([&](auto r2c) __attribute__((always_inline)) { ew_pair(r2c); });
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (C::DOC) {
        W::landed(qd[0], qd[1]);
        W::landed(qd[2], qd[3]);
      }
    };
    // dV += dO^T P for the block whose P (bf16 pairs in pw) the previous iteration formed: it runs
    // first in an iteration, while the partner wave is in its mixed phase, and the mixed phase above
    // runs while the partner is in its pure matrix phase
    auto dv_phase = [&](auto qb_c, uint32_t base_c) __attribute__((always_inline)) {
      constexpr int QB = decltype(qb_c)::value;
      uint32_t ta_c[DBV][2];
#pragma unroll
      for (int d = 0; d < DBV; ++d) {
        ta_c[d][0] = w.tv[d][0] + base_c;
        ta_c[d][1] = w.tv[d][1] + base_c;
      }
      w.template tr_stream_g<TrOne<C::TILE + QB * 32 * ROWV, DBV, ROWV>, 2 * DBV, 2>([&](auto fc, int u) __attribute__((always_inline)) {
        return ta_c[decltype(fc)::value % DBV][u];
      }, [&](auto fc, bf16x8 a) __attribute__((always_inline)) {
        constexpr int f = decltype(fc)::value, d = f % DBV, ks = f / DBV;
        const bf16x8 bop = __builtin_bit_cast(
            bf16x8, (i32x4){(int)pw[4 * ks], (int)pw[4 * ks + 1], (int)pw[4 * ks + 2], (int)pw[4 * ks + 3]});
        dv[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bop, dv[d], 0, 0, 0);
      });
    };
    if (it0 < n_items) scores(std::integral_constant<int, 0>(), 0u, sa);
    while (true) {
      const bool vp = it0 < n_items, vm = itm1 < n_items;
      if (!vp && !vm) break;
      const uint32_t b0 = s0 * C::STAGE_KV, b1 = (s0 + 1 == NSTAGE ? 0 : s0 + 1) * C::STAGE_KV;
      const int s2 = s0 + 2 >= NSTAGE ? s0 + 2 - NSTAGE : s0 + 2;
      // even iteration: dV of block (P - 1, 1); block (P, 0) current, (P, 1) next
      if (vm) dv_phase(std::integral_constant<int, 1>(), (uint32_t)(s2 * C::STAGE_KV));
      if (vp) p_iter(std::integral_constant<int, 0>(), std::integral_constant<int, 1>(), std::integral_constant<int, 0>(), b0, b0, it0, sa, sb);
      iteration_end(true);
      if (!vp) break;
      // odd iteration: dV of block (P, 0); block (P, 1) current, (P + 1, 0) next; the tile at P + 2
      // replaces the one at P - 1
      if (vm && itp2 < n_items) load_item(itp2, s2);
      dv_phase(std::integral_constant<int, 0>(), b0);
      p_iter(std::integral_constant<int, 1>(), std::integral_constant<int, 0>(), std::integral_constant<int, 1>(), b0, b1, it0, sb, sa);
      iteration_end(false);
      itm1 = it0;
      it0 = itp1;
      dm0 = dmp1;
      itp1 = itp2;
      dmp1 = dmp2;
      itp2 = itp2 < n_items ? next_item(itp2 + 1, dmp2) : n_items;
      s0 = s0 + 1 == NSTAGE ? 0 : s0 + 1;
    }
    if (j < p.Sk) {
#pragma unroll
      for (int d = 0; d < DBV; ++d)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          store_kv_grad<true, C::DV>(p, split, b, g, hk, j, 32 * d + 8 * r4 + 4 * w.half, dv[d][4 * r4], dv[d][4 * r4 + 1],
                                     dv[d][4 * r4 + 2], dv[d][4 * r4 + 3]);
    }
  } else {
    // ================= dS wave =================
    bf16x8 vf[KV];
    {
      const uint16_t* vp = (const uint16_t*)p.v.ptr + b * p.v.sb + g * p.v.sg + hk * p.v.sh + (int64_t)jc * p.v.ss;
#pragma unroll
      for (int kk = 0; kk < KV; ++kk) vf[kk] = *(const bf16x8*)(vp + 16 * kk + 8 * w.half);
    }
    f32x16 dk[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d) dk[d] = W::zero16();
    f32x16 da = W::zero16(), db = W::zero16();
    auto dscores = [&](auto off_c, uint32_t base, f32x16& dst) __attribute__((always_inline)) {  // dP of one block, no overlap
      dst = W::zero16();
      w.template row_stream_g<RowOne<decltype(off_c)::value>, KV, 2>([&](auto fc) __attribute__((always_inline)) {
        return w.rv[decltype(fc)::value] + base;
      }, [&](auto fc, bf16x8 a) __attribute__((always_inline)) {
        dst = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, vf[decltype(fc)::value], dst, 0, 0, 0);
      });
    };
    // block QP at stage offset base_p was handed over in exchange buffer XB (its dP in cur); the dP of
    // block QN at base_n goes to nxt
    auto ds_iter = [&](auto qp_c, auto qn_c, auto xb_c, uint32_t base_p, uint32_t base_n, f32x16& cur, f32x16& nxt) __attribute__((always_inline)) {
      constexpr int QP = decltype(qp_c)::value, QN = decltype(qn_c)::value, XB = decltype(xb_c)::value;
      uint32_t ra_n[KV], ta_p[DB][2];
#pragma unroll
      for (int kk = 0; kk < KV; ++kk) ra_n[kk] = w.rv[kk] + base_n;
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        ta_p[d][0] = w.ta[d][0] + base_p;
        ta_p[d][1] = w.ta[d][1] + base_p;
      }
      i32x4 pq[4], st_d[4];                        // P of the block (fp32) and delta of its rows, by register quad
      static_for<0, 4>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q4 = decltype(qc)::value;
        W::template read_b128<XB * XBUF + q4 * 1024>(pq[q4], xaddr);
        W::template read_b128<C::STATS + C::STAT + (32 * QP + 8 * q4) * 4>(st_d[q4], stat_addr + base_p);
      });
      uint32_t dsw[8];
      auto ew_pair = [&](auto r2c) __attribute__((always_inline)) {
        constexpr int r2 = decltype(r2c)::value;
        float dsv[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int r = 2 * r2 + e;
          dsv[e] = __int_as_float(pq[r >> 2][r & 3]) * (cur[r] - __int_as_float(st_d[r >> 2][r & 3]));
        }
        dsw[r2] = pack_bf16(dsv[0], dsv[1]);
        asm volatile("" : "+v"(dsw[r2]));
      };
      // phase 1: dP of the next block  ||  dS of the handed-over block
      nxt = W::zero16();
      w.template row_stream_g<RowOne<C::TILE + QN * 32 * ROWV>, KV, 2>([&](auto fc) __attribute__((always_inline)) {
        return ra_n[decltype(fc)::value];
      }, [&](auto fc, bf16x8 a) __attribute__((always_inline)) {
        constexpr int f = decltype(fc)::value;
        nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, vf[f], nxt, 0, 0, 0);
        static_for<8 * f / KV, 8 * (f + 1) / KV>([&](auto r2c) __attribute__((always_inline)) { ew_pair(r2c); });
        __builtin_amdgcn_sched_barrier(0);
      });
      // phase 2: dK += Q^T dS
      w.template tr_stream_g<TrOne<QP * 32 * ROW, DB, ROW>, 2 * DB, 2>([&](auto fc, int u) __attribute__((always_inline)) {
        return ta_p[decltype(fc)::value % DB][u];
      }, [&](auto fc, bf16x8 a) __attribute__((always_inline)) {
        constexpr int f = decltype(fc)::value, d = f % DB, ks = f / DB;
        const bf16x8 bop = __builtin_bit_cast(
            bf16x8, (i32x4){(int)dsw[4 * ks], (int)dsw[4 * ks + 1], (int)dsw[4 * ks + 2], (int)dsw[4 * ks + 3]});
        dk[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bop, dk[d], 0, 0, 0);
      });
    };
    if (it0 < n_items) dscores(std::integral_constant<int, C::TILE>(), 0u, da);
    while (true) {
      const bool vp = it0 < n_items, vm = itm1 < n_items;
      if (!vp && !vm) break;
      const uint32_t b0 = s0 * C::STAGE_KV;
      const int s2 = s0 + 2 >= NSTAGE ? s0 + 2 - NSTAGE : s0 + 2;
      const uint32_t b2 = s2 * C::STAGE_KV;        // stage of position P - 1
      // even iteration: block (P - 1, 1) was handed over in buffer 1; dP of block (P, 0) is next
      if (vm) ds_iter(std::integral_constant<int, 1>(), std::integral_constant<int, 0>(), std::integral_constant<int, 1>(), b2, b0, db, da);
      iteration_end(true);
      if (!vp) break;
      // odd iteration: block (P, 0) was handed over in buffer 0; dP of block (P, 1) is next
      if (vm && itp2 < n_items) load_item(itp2, s2);
      ds_iter(std::integral_constant<int, 0>(), std::integral_constant<int, 1>(), std::integral_constant<int, 0>(), b0, b0, da, db);
      iteration_end(false);
      itm1 = it0;
      it0 = itp1;
      dm0 = dmp1;
      itp1 = itp2;
      dmp1 = dmp2;
      itp2 = itp2 < n_items ? next_item(itp2 + 1, dmp2) : n_items;
      s0 = s0 + 1 == NSTAGE ? 0 : s0 + 1;
    }
    if (j < p.Sk) {
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          store_kv_grad<false, C::D>(p, split, b, g, hk, j, 32 * d + 8 * r4 + 4 * w.half, dk[d][4 * r4] * p.scale,
                                     dk[d][4 * r4 + 1] * p.scale, dk[d][4 * r4 + 2] * p.scale, dk[d][4 * r4 + 3] * p.scale);
    }
  }
}

}  // namespace fl
