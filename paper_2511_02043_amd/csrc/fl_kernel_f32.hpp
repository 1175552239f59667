// fp32 attention-variant forward kernel: fp32 storage, scores, softmax state and accumulators; both contractions over three bf16
// parts of each operand (v_mfma_f32_32x32x16_bf16), or on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32): variants above head dim
// 64 and with few key tiles, and values that the parts do not hold.
//
// This is the fp32-storage specialisation of the fused pass; tanh, the logarithm and the gate use the
// accurate math-library routines, and the result is meant to stay within 1e-5 of an fp64 evaluation.
// Every variant feature is available here, as runtime switches; calls without any (F32Cfg::PLAIN) have instances without the
// switches.  It follows the same structure as the bf16 kernel: a workgroup owns a tile of query rows, walks the visible key tiles
// (skipper), keeps (m, l, O) in registers and never stores a score (Sec. 3.2 dimension demotion; Sec. 3.4 running max / sum
// with the exp(m_old - m_new) correction).
//
// Orientation as in the bf16 kernel: S^T = K Q^T with the query in the lane (lane % 32) and sixteen keys
// n(r) = 8 (r / 4) + 4 (lane / 32) + r % 4 in the registers, so a softmax row is two lanes, and the registers of P are, as they
// stand, the B operand of O^T += V^T P^T (register r of the step over the key pair n(r); registers 8 s ... 8 s + 7, split, of the
// s-th step of sixteen keys).  Both operands of a step may take the channels (or keys) in any common order: a lane
// reads K in 16-byte pieces, and V^T row c of channel block d is channel DVB c + d, so that one LDS read of 4 DVB bytes feeds
// DVB channel blocks.
//
// Contractions on parts: x = h + m + l, each the bf16 rounding of what the ones before leave, holds 24 bits; six of the nine products
// of two such sums (all above 2^-27 of the largest) cost 6 x 32 clocks for 16 channels where the fp32 instruction takes 8 x 64.  The error
// against fp64 is lower than the fp32 instruction's (fewer roundings of the sum: 2 x 8 heads x 1024 rows, D = 64, relative 4.2e-7 before,
// 2.9e-7).  A bf16 part holds nothing below 2^-134, so that a value below 2^-110 loses bits, and a value may round to infinity.  What is lost
// of K comes to 2^-27 of a score at most while |Q| < 2^100 / max(scale, 1); of Q nothing from 2^-100 on: both are checked as Q is split (sums of
// products below 2^-126 meet a scale of 2^64 at most).  What is lost of P and V shows in the accumulators beside the largest value
// (f32_most), overflows as infinity or NaN there.  A wave (where waves share tiles: a workgroup) that finds such a value takes the pass again
// on the fp32 instruction, so that infinities, NaN and tiny values give what they gave there; but beside ordinary values, a channel
// whose values are all below 2^-134 gives zero.
//
// What bounds it: issue of vector instructions, 10.8 for each matrix instruction of a call at D = 64, about nine of them in the key loop (eleven per
// pair of values split, one per pair of V for its magnitude; four run beside a matrix instruction).  So a wave takes two row blocks (K and V are split once for both) wherever registers allow, the split of
// the next operands stands between the matrix instructions of the present ones (f32_stage), and where the call has fewer than two waves
// per SIMD the key tiles of a row group are dealt to KS waves, which merge through LDS by the rescale rule of Sec. 3.3.  K / V tiles
// of 32 keys go to LDS by direct loads.
// Measured against the fp32 instruction in both contractions, one row block per wave: 2 x 8 heads, 1024 rows and keys, D = 32 / 64 / 128: 30 / 53 /
// 107 -> 21 / 33 / 65 us, 8 x 16 heads x 2048 rows, D = 64: 1260 -> 732 us (188 TFLOP/s); the same pass on plain VALU arithmetic
// took 508 us for the first at D = 64.  Variants (PARTS) 2 x 8 x 1024, ALiBi / bias / gate / differential, D = 32: 31 / 60 / 31 / 55 -> 28 / 55 / 29 / 51,
// D = 64: 48 / 75 / 50 / 89 -> 42 / 65 / 43 / 76; at D = 128 they run on the fp32 instruction: 107 / 138 / 121 / 212 and 105 / 135 / 116 / 205.
#pragma once
#include "fl_kernel_bf16.hpp"

namespace fl {

constexpr int kF32Keys = 32;     // keys per LDS tile (= kSumBlock)

template <int DMAX_, int RB_, int RG_, int KS_, bool PLAIN_>
struct F32Cfg {
  static constexpr bool PLAIN = PLAIN_;            // no score_mod, bias, document mask, epilogue or second stream: nothing of those in the code
  static constexpr bool PARTS = PLAIN_ || DMAX_ <= 64;   // contractions on bf16 parts (the switches of the variants leave no registers for them at 128)
  static constexpr int DMAX = DMAX_;               // head dims up to this one; smaller ones compute on channels that are zero in Q
  static constexpr int RB = RB_;                   // 32-row blocks of a wave
  static constexpr int RG = RG_, KS = KS_;         // row groups (32 RB query rows each) and key splits of the workgroup
  static constexpr int NT = RG * KS * 64;
  static constexpr int WPE = RB * DMAX > 128 ? 1 : 2;    // waves per SIMD that the registers are cut for
  static constexpr int WROWS = 32 * RB, BM = RG * WROWS;
  static constexpr int ROW = DMAX * 4;             // bytes of a tile row in LDS
  static constexpr int CH = DMAX / 4;              // 16-byte chunks of a tile row
  static constexpr int TILE = kF32Keys * ROW;
  static constexpr int STAGE = 2 * TILE;           // K, V
  static constexpr int NBUF = RG == 1 ? 1 : 2;     // buffers per key split (see the loops)
  static constexpr int RING = KS * NBUF * STAGE;   // [key split][buffer][K, V]
  static constexpr int DVB = DMAX / 32;            // 32-channel blocks of the output
  static constexpr int NINSTR = TILE / 1024;       // direct-load instructions per tile
  static constexpr int OBYTES = RB * DVB * 16 * 64 * 4;   // one wave's accumulators
  static constexpr int MLBYTES = RB * 2 * 64 * 4;  // ... running maxima and sums
  // Every split of a row group hands its accumulators over, and each wave sums and stores its share of them.  An epilogue or a
  // second stream needs whole rows: the other splits hand over to the first.
  static constexpr bool SHARE = PLAIN_ && KS_ > 1;
  static constexpr int MERGE = RG * (SHARE ? KS : KS - 1) * (OBYTES + MLBYTES);
  // The third (and second) parts of Q's fragments wait in LDS where two waves per SIMD have no registers for them: [row group][step]
  // [block][part], 1 KiB each.
  static constexpr int QP = !PARTS ? 0 : DMAX == 128 && RG > 1 ? 1 : RB * DMAX >= 128 ? 2 : 0;   // parts in LDS: the third, the second
  static constexpr int QBYTES = QP * RG * RB * (DMAX / 16) * 1024;
  static constexpr int LDS = RING + QBYTES > MERGE ? RING + QBYTES : MERGE;
  static constexpr int QBASE = RING;
  static_assert(DMAX == 32 || DMAX == 64 || DMAX == 128, "head dims of the fp32 kernel");
};

// chunk swizzle of a K row: sixteen consecutive rows read the same chunk through sixteen different bank groups
template <int CH>
__device__ __forceinline__ int swz_f32(int r) {
  if constexpr (CH == 8) return (r >> 1) & 7;
  else return r & 15;
}

// N floats of a lane and the LDS read that fetches them.  The reads are issued by hand with explicit lgkmcnt waits, so that
// the compiler cannot tie one to the direct global->LDS loads of the next tile.
template <int N>
struct F32Vec {
  typedef __attribute__((ext_vector_type(N))) float type;
  static __device__ __forceinline__ float at(const type& v, int d) { return v[d]; }
  template <int OFF>
  static __device__ __forceinline__ void read(type& v, uint32_t addr) {
    if constexpr (N == 4) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
    else asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  }
};
template <>
struct F32Vec<1> {
  typedef float type;
  static __device__ __forceinline__ float at(const type& v, int) { return v; }
  template <int OFF>
  static __device__ __forceinline__ void read(type& v, uint32_t addr) {
    asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  }
};

// 16 zero bytes to LDS, in order with this wave's reads
__device__ __forceinline__ void f32_clear16(uint32_t addr) {
  const F32Vec<4>::type z = {0.f, 0.f, 0.f, 0.f};
  asm volatile("ds_write_b128 %0, %1" : : "v"(addr), "v"(z) : "memory");
}
static __device__ const float4 kF32Zero = {0.f, 0.f, 0.f, 0.f};

// until at most N younger vector memory operations of this wave are in flight
template <int N>
__device__ __forceinline__ void f32_wait_mem() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}
template <int N>
__device__ __forceinline__ void f32_wait_lds() {
  asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(N) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Three bf16 parts of eight fp32 values, each the rounded rest of the one before: 24 bits of the value, exact unless it is below
// 2^-100 or rounds to infinity.  (A rest by v_dot2_f32_bf16 would take three instructions less per pair, but that runs on the matrix
// unit: four of them beside a matrix instruction of 32 clocks make it 56, eight ordinary ones 43.)
struct F32Split {
  i32x4 h, m, l;
};
template <int E>   // values 2 E and 2 E + 1 of the eight
__device__ __forceinline__ void f32_split(float a, float b, F32Split& out) {
  auto rest = [&](uint32_t u) __attribute__((always_inline)) {
    a -= __uint_as_float(u << 16);
    b -= __uint_as_float(u & 0xffff0000u);
  };
  const uint32_t h = pack_bf16(a, b);
  rest(h);
  const uint32_t m = pack_bf16(a, b);
  rest(m);
  out.h[E] = (int)h;
  out.m[E] = (int)m;
  out.l[E] = (int)pack_bf16(a, b);
}
// The N-th of the six products of parts above 2^-27 of the largest, small ones first: acc += a b over one 16-element step
template <int N>
__device__ __forceinline__ f32x16 f32_mfma(const F32Split& a, const F32Split& b, f32x16 acc) {
  const i32x4& x = N == 0 ? a.l : N == 2 || N == 3 ? a.m : a.h;
  const i32x4& y = N == 1 ? b.l : N == 2 || N == 4 ? b.m : b.h;
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), acc, 0, 0, 0);
}
// N matrix instructions with W pieces of vector work spread between them, in this order: a wave issues in order, and the matrix unit
// is free for its next instruction 32 clocks after the last
template <int N, int W, class M, class J>
__device__ __forceinline__ void f32_stage(M&& mfma, J&& job) {
  static_for<0, N>([&](auto i) __attribute__((always_inline)) {
    mfma(i);
    static_for<i * W / N, (i + 1) * W / N>(job);
    __builtin_amdgcn_sched_barrier(0);
  });
}
// Magnitudes of the values taken: the least other than zero, and the largest
struct F32Range {
  uint32_t least = 0xffffffffu, most = 0u;
  __device__ __forceinline__ void take(float x) {
    const uint32_t v = __float_as_uint(x) & 0x7fffffffu;
    least = min(least, v - 1u);                    // (zero: the largest)
    most = max(most, v);
  }
  // all zero or in [lo, hi), lo > 0; a NaN is not
  __device__ __forceinline__ bool inside(float lo, float hi) const { return least >= __float_as_uint(lo) - 1u && most < __float_as_uint(hi); }
};
// most = max(most, |a|, |b|), one instruction (fmaxf would make each value canonical first); a NaN stays one, and shows in the accumulators, too
__device__ __forceinline__ void f32_most(float& most, float a, float b) {
  most = __builtin_elementwise_maximum(__builtin_elementwise_maximum(__builtin_fabsf(a), __builtin_fabsf(b)), most);
}

template <class C>
__global__ void __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::WPE)))
fwd_f32_kernel(const FwdParams p) {
  constexpr int DMAX = C::DMAX, RB = C::RB, RG = C::RG, KS = C::KS, DVB = C::DVB, ROW = C::ROW, NU = DMAX / 8, NK = DMAX / 16;
  const int MOD = C::PLAIN ? kModNone : p.mod, NBIAS = C::PLAIN ? 0 : p.n_bias;
  const uint32_t MASK = C::PLAIN ? p.mask & ~kMaskDoc : p.mask, EPI = C::PLAIN ? 0 : p.epi;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];

  const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rg = wave % RG, ks = wave / RG;        // this wave's row group and key split

  // grid decode: whole (b, g, h) problems per XCD where their number allows it, longest causal tiles first
  const int nq = p.n_qtiles;
  int qt, bh;
  if (p.order == 1) {
    p.by_tiles.split(blockIdx.x >> 3, bh, qt);
    bh = bh * 8 + (int)(blockIdx.x & 7);
  } else {
    p.by_tiles.split(blockIdx.x, bh, qt);
  }
  qt = nq - 1 - qt;
  int bg, h, b, g;
  p.by_heads.split(bh, bg, h);
  p.by_g.split(bg, b, g);
  const int hk = p.by_group.div(h);
  const int i0 = qt * C::BM, iw = i0 + C::WROWS * rg;    // first query row of the workgroup / of the wave
  const int ns = !C::PLAIN && p.diff ? 2 : 1;                   // softmax streams, one after the other

  const float slope = MOD == kModAlibi ? p.alibi_slopes[h] : 0.f;

  // ---- visible key range of the workgroup (positional masks, rows by their positions); document summaries of its rows
  const int i_max = min(i0 + C::BM, p.Sq) - 1, iw_max = min(iw + C::WROWS, p.Sq) - 1;
  int k_lo, k_hi;
  key_range(MASK, i0 + p.q_off, i_max + p.q_off, p.Sk, p.window, p.prefix, k_lo, k_hi);
  const int t_lo = k_lo / kF32Keys, t_hi = (k_hi + kF32Keys - 1) / kF32Keys;
  const int n_iter = t_hi > t_lo ? (t_hi - t_lo + KS - 1) / KS : 0;   // the same for every wave: they meet at barriers
  int2 qs_wg = make_int2(0, 0), qs_w = qs_wg;
  const int nks = (p.Sk + kSumBlock - 1) / kSumBlock;
  if ((MASK & kMaskDoc) != 0) {
    const int nqs = (p.Sq + kSumBlock - 1) / kSumBlock;
    const int2* s = p.q_sum + (int64_t)b * nqs;
    auto range = [&](int first, int n) __attribute__((always_inline)) -> int2 {
      int2 r = s[min(first / kSumBlock, nqs - 1)];
      for (int u = 1; u < n; ++u) {
        const int2 x = s[min(first / kSumBlock + u, nqs - 1)];
        r.x = min(r.x, x.x);
        r.y = max(r.y, x.y);
      }
      return r;
    };
    qs_wg = range(i0, RG * RB);
    qs_w = range(iw, RB);
  }
  auto tile_ids = [&](int t) __attribute__((always_inline)) -> int2 {   // document-id range of tile t's keys
    return (MASK & kMaskDoc) != 0 ? p.kv_sum[(int64_t)b * nks + t] : make_int2(0, 0);
  };
  auto classify = [&](int t, int r_lo, int r_hi, int2 qs, int2 kd) __attribute__((always_inline)) -> int {
    return classify_block(MASK, r_lo + p.q_off, r_hi + p.q_off, t * kF32Keys, t * kF32Keys + kF32Keys - 1, p.Sk, p.window, p.prefix,
                          qs, kd);
  };

  // ---- per-lane LDS offsets (see the header comment)
  const uint32_t ka = (uint32_t)(ks * C::NBUF * C::STAGE + col * ROW + ((half ^ swz_f32<C::CH>(col)) << 4));
  const uint32_t va = (uint32_t)(ks * C::NBUF * C::STAGE + C::TILE + 4 * half * ROW + col * (4 * DVB));

  for (int s = 0; s < ns; ++s) {
    const View& qv = s == 0 ? p.q : p.q2;
    const View& kv = s == 0 ? p.k : p.k2;
    f32x16 o[RB][DVB];
    float m[RB], l[RB];                            // log2-domain running max; this lane's part of the running sum

    const float* kp = (const float*)kv.ptr + b * kv.sb + g * kv.sg + hk * kv.sh;
    const float* vp = (const float*)p.v.ptr + b * p.v.sb + g * p.v.sg + hk * p.v.sh;
    // K or V tile t of this wave's split into its buffer `buf`: the split's RG waves share the load instructions.  A chunk
    // past the head dim is replaced by the row's first (V's end in channels nobody stores), a row past Sk by the last one (its
    // scores are masked).
    // (The offsets inside a tile are formed again for every tile, from an opaque copy of the lane id: hoisted out of the loop
    // they would hold the registers that two waves per SIMD do not have.)
    auto load_tile = [&](const float* head, int64_t ss, int dim, auto is_k, int t, int lds_off) __attribute__((always_inline)) {
      constexpr bool kKeys = decltype(is_k)::value;   // K rows are swizzled
      const int last = p.Sk - 1 - t * kF32Keys;    // last row of the tile that exists (uniform)
      const unsigned char* base = (const unsigned char*)(head + (int64_t)(t * kF32Keys) * ss);
      // Whole tile: a lane's offsets differ between the instructions in their chunk only.  (Not in kernels with document masks whose waves share
      // tiles: beside the general loads the compiler keeps an offset in a register that it also loads tile summaries into, and
      // waits there for the loads just issued.  8 x 16 heads x 512 rows, ALiBi, D = 64 / 128: 83 / 178 us with it, 80 / 173 without.)
      if ((C::PLAIN || RG == 1) && last >= kF32Keys - 1 && dim == DMAX) {
        constexpr int RPI = 64 / C::CH;            // rows of an instruction; the swizzle of a row is that of its instruction's first ^ its own
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int row = ln / C::CH, pos = ln % C::CH;
        const uint32_t chunk = (uint32_t)(kKeys ? pos ^ swz_f32<C::CH>(row) : pos) << 4, first = (uint32_t)row * (uint32_t)ss * 4u;
#pragma unroll
        for (int u = 0; u < (C::NINSTR + RG - 1) / RG; ++u) {
          const int inst = (rg + u * RG) % C::NINSTR;
          const uint32_t off = (chunk ^ (kKeys ? (uint32_t)swz_f32<C::CH>(inst * RPI) << 4 : 0u)) + first;
          __builtin_amdgcn_global_load_lds((global_cvoid*)(base + (int64_t)(inst * RPI) * ss * 4 + off),
                                           (lds_void*)(lds_raw + lds_off + inst * 1024), 16, 0, 0);
        }
        return;
      }
      auto issue = [&](auto zeros) __attribute__((always_inline)) {
        int ln = lane;
#pragma unroll
        for (int u = 0; u < (C::NINSTR + RG - 1) / RG; ++u) {
          asm volatile("" : "+v"(ln));
          const int inst = (rg + u * RG) % C::NINSTR;
          const int row = inst * (64 / C::CH) + ln / C::CH, pos = ln % C::CH;
          const int c = (kKeys ? pos ^ swz_f32<C::CH>(row) : pos) * 4;
          const uint32_t off = ((uint32_t)min(row, last) * (uint32_t)ss + (uint32_t)(c < dim ? c : 0)) * 4u;
          const unsigned char* src = base + off;
          if (decltype(zeros)::value && c >= dim) src = (const unsigned char*)&kF32Zero;
          __builtin_amdgcn_global_load_lds((global_cvoid*)src, (lds_void*)(lds_raw + lds_off + inst * 1024), 16, 0, 0);
        }
      };
      if (kKeys && RG == 1 && dim < DMAX) issue(std::integral_constant<bool, true>());
      else issue(std::integral_constant<bool, false>());
    };
    // Stand-ins that would meet a zero: K's chunks past D the zeros of Q, V's rows past Sk a weight of zero.  What they stand in
    // for may be infinite, so each lane clears those that it loaded, once they have landed and before anyone reads them.  (One
    // wave per split has a whole tile to clear, and reads K's from zeros instead: 2 x 8 heads of 1000 rows at D = 68 take 102
    // us with the stand-ins as they are, 106 us read from zeros and 114 us cleared; two and more waves 1 % either way.)
    auto clear_tile = [&](auto is_k, int t, int lds_off) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < (C::NINSTR + RG - 1) / RG; ++u) {
        const int inst = (rg + u * RG) % C::NINSTR;
        const int row = inst * (64 / C::CH) + lane / C::CH, pos = lane % C::CH;
        if (decltype(is_k)::value ? (pos ^ swz_f32<C::CH>(row)) * 4 >= p.D : t * kF32Keys + row >= p.Sk)
          f32_clear16(lds_off + inst * 1024 + lane * 16);
      }
    };
    auto clear_k = [&](int t, int buf) __attribute__((always_inline)) {
      if (RG > 1 && p.D < DMAX) clear_tile(std::integral_constant<bool, true>(), t, (ks * C::NBUF + buf) * C::STAGE);
    };
    auto clear_v = [&](int t, int buf) __attribute__((always_inline)) {
      if ((t + 1) * kF32Keys > p.Sk) clear_tile(std::integral_constant<bool, false>(), t, (ks * C::NBUF + buf) * C::STAGE + C::TILE);
    };
    auto load_k = [&](int t, int buf) __attribute__((always_inline)) { load_tile(kp, kv.ss, p.D, std::integral_constant<bool, true>(), t, (ks * C::NBUF + buf) * C::STAGE); };
    auto load_v = [&](int t, int buf) __attribute__((always_inline)) { load_tile(vp, p.v.ss, p.Dv, std::integral_constant<bool, false>(), t, (ks * C::NBUF + buf) * C::STAGE + C::TILE); };
    auto wanted = [&](int t) __attribute__((always_inline)) -> bool {
      return t < t_hi && classify(t, i0, i_max, qs_wg, tile_ids(t)) != kSkip;
    };

    // One pass over the keys.  EXACT = 0: both contractions on the bf16 matrix instruction, over the three parts of each operand;
    // EXACT = 1: on the fp32 one.  Returns whether the parts may have lost something (EXACT = 0 only).
    auto pass = [&](auto exact) __attribute__((always_inline)) -> bool {
      constexpr bool EXACT = decltype(exact)::value;
      float4 qf[EXACT ? RB : 1][EXACT ? NU : 1];   // B fragments of S^T = K Q^T; channels past D are zero
      F32Split qp[EXACT ? 1 : RB][EXACT ? 1 : NK];
      F32Range range;
      float vmost = 0.f;                           // largest magnitude of this lane's values
      {
        int ql = lane;                             // (opaque, as in the epilogue below)
        asm volatile("" : "+v"(ql));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          const float* qrow = (const float*)qv.ptr + b * qv.sb + g * qv.sg + h * qv.sh + (int64_t)min(iw + 32 * rb + (ql & 31), p.Sq - 1) * qv.ss;
          float4 x[NU];
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            const int c = 8 * u + 4 * (ql >> 5);
            x[u] = c < p.D ? *(const float4*)(qrow + c) : make_float4(0.f, 0.f, 0.f, 0.f);
          }
          if constexpr (EXACT) {
#pragma unroll
            for (int u = 0; u < NU; ++u) qf[rb][u] = x[u];
          } else {
#pragma unroll
            for (int kk = 0; kk < NK; ++kk) {
              const float v[8] = {x[2 * kk].x, x[2 * kk].y, x[2 * kk].z, x[2 * kk].w,
                                  x[2 * kk + 1].x, x[2 * kk + 1].y, x[2 * kk + 1].z, x[2 * kk + 1].w};
#pragma unroll
              for (int e = 0; e < 8; ++e) range.take(v[e]);
              // (the waves of a row group hold the same rows: the ks-th stores every KS-th fragment)
              if (C::QP < 2 || (kk * RB + rb) % KS == ks) {
                static_for<0, 4>([&](auto e) __attribute__((always_inline)) { f32_split<e>(v[2 * e], v[2 * e + 1], qp[rb][kk]); });
                if (C::QP > 0 && (kk * RB + rb) % KS == ks) {
                  i32x4* dst = (i32x4*)(lds_raw + C::QBASE + ((rg * NK + kk) * RB + rb) * C::QP * 1024 + lane * 16);
                  dst[0] = qp[rb][kk].l;
                  if (C::QP > 1) dst[64] = qp[rb][kk].m;
                }
              } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) qp[rb][kk].h[e] = (int)pack_bf16(v[2 * e], v[2 * e + 1]);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
      auto load_first = [&]() __attribute__((always_inline)) {
        if (wanted(t_lo + ks)) {
          load_k(t_lo + ks, 0);
          load_v(t_lo + ks, 0);
        }
      };
      if (RG > 1 && C::PLAIN) load_first();
      if constexpr (!EXACT) {                      // a row that the parts do not hold: none of the keys is looked at
        bool outside = __builtin_amdgcn_ballot_w64(!range.inside(0x1p-100f, 0x1p100f / fmaxf(fabsf(p.scale), 1.f))) != 0;
        if (RG > 1) {                              // (in the first split's second buffer, which is free until the loop's first barrier)
          int* flags = (int*)(lds_raw + C::STAGE);
          if (lane == 0) flags[wave] = outside ? 1 : 0;
          f32_wait_lds<0>();
          __syncthreads();
#pragma unroll
          for (int w = 0; w < RG * KS; ++w) outside = outside || flags[w] != 0;
          outside = __builtin_amdgcn_readfirstlane(outside ? 1 : 0) != 0;
        } else if (C::QP > 0) {
          f32_wait_lds<0>();
          if (KS > 1) __syncthreads();
        }
        if (outside) {
          if (RG > 1 && C::PLAIN) f32_wait_mem<0>();
          return true;
        }
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        m[rb] = -INFINITY;
        l[rb] = 0.f;
#pragma unroll
        for (int d = 0; d < DVB; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[rb][d][r] = 0.f;
      }

      const bool plain = MOD == kModNone && NBIAS == 0 && p.scale > 0.f;   // then scale and log2(e) are one factor under the exponent's FMA
      const float fe = plain ? p.scale * kLog2e : 1.f;
      // variant transform of a block's scores (Eq. 3, Eq. 4, biases, masks), log2 domain unless plain; register r holds key jl + 8 (r / 4) + r % 4
      auto transform = [&](f32x16& x, int rb, int t, int cls) __attribute__((always_inline)) {
        const int jl = t * kF32Keys + 4 * half;
        const int i = iw + 32 * rb + col, ic = min(i, p.Sq - 1);
        auto key = [&](int r) __attribute__((always_inline)) { return jl + 8 * (r >> 2) + (r & 3); };
        if (!plain) {
#pragma unroll
          for (int r = 0; r < 16; ++r) x[r] *= p.scale;
          if (MOD == kModSoftcap) {
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = p.softcap * tanhf(x[r] / p.softcap);
          }
          if (MOD == kModAlibi) {
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] -= slope * fabsf((float)(i + p.q_off - key(r)));
          }
          for (int nb = 0; nb < NBIAS; ++nb) {
            const BiasView& bv = p.bias[nb];
            int bl = ic;
            asm volatile("" : "+v"(bl));
            const int64_t row = b * bv.sb + g * bv.sg + h * bv.sh + (int64_t)bl * bv.si;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int64_t off = row + (int64_t)min(key(r), p.Sk - 1) * bv.sj;
              x[r] += bv.is_f32 ? ((const float*)bv.ptr)[off] : bf16_to_f32(((const uint16_t*)bv.ptr)[off]);
            }
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) x[r] *= kLog2e;
        }
        if (cls == kPartial) {                     // the positional masks and the end of the keys as two bounds on the key
          const int ip = i + p.q_off;
          int last = p.Sk - 1, first = 0;
          if ((MASK & kMaskPrefix) != 0) last = min(last, max(ip, p.prefix - 1));
          else if ((MASK & (kMaskCausal | kMaskWindow)) != 0) last = min(last, ip);
          if ((MASK & kMaskWindow) != 0) first = ip - p.window;
          const int d_hi = last - jl, d_lo = first - jl;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int c = 8 * (r >> 2) + (r & 3);
            x[r] = (c > d_hi) | (c < d_lo) ? -INFINITY : x[r];
          }
          if ((MASK & kMaskDoc) != 0) {
            const int32_t* kdoc = p.kv_doc + (int64_t)b * p.Sk;
            const int qdoc = p.q_doc[(int64_t)b * p.Sq + ic];
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = kdoc[min(key(r), p.Sk - 1)] != qdoc ? -INFINITY : x[r];
          }
        }
      };
      // online softmax (Alg. 2): the running max moves to the block's, the sums follow; returns the exponent's reference
      auto advance = [&](const f32x16& x, int rb) __attribute__((always_inline)) -> float {
        float mx = x[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, x[r]);
        mx = fmaxf(m[rb], half_swap_max(mx) * fe);
        const float ms = mx == -INFINITY ? 0.f : mx;
        if (__builtin_amdgcn_ballot_w64(mx != m[rb]) != 0) {       // uniform: some row's maximum moved
          const float alpha = fast_exp2(m[rb] - ms);
          l[rb] *= alpha;
          m[rb] = mx;
#pragma unroll
          for (int d = 0; d < DVB; ++d)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[rb][d][r] *= alpha;
        }
        return ms;
      };
      // (v_exp_f32: 1 ulp; results below 2^-126 are zero beside a row sum of at least 1)
      auto weight = [&](f32x16& x, int r, float ms, float& sum) __attribute__((always_inline)) {
        x[r] = fast_exp2(fmaf(x[r], fe, -ms));
        sum = r == 0 ? x[r] : sum + x[r];
      };

      // One tile.  k_free() runs when the K tile has been read, v_ready() before V is, v_free() when V has been read.
      auto tile = [&](int t, int cls, uint32_t buf, auto&& k_free, auto&& v_ready, auto&& v_free) __attribute__((always_inline)) {
        f32x16 sc[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int r = 0; r < 16; ++r) sc[rb][r] = 0.f;
        typename F32Vec<DVB>::type vf[16];
        const uint32_t a = va + buf;
        auto read_v = [&](auto rc) __attribute__((always_inline)) {          // one key, DVB channels
          constexpr int r = decltype(rc)::value, OFF = (8 * (r >> 2) + (r & 3)) * ROW;
          F32Vec<DVB>::template read<OFF>(vf[r], a);
        };
        F32Vec<4>::type kf[NU];
        auto read_k = [&](auto uc) __attribute__((always_inline)) {          // four channels
          constexpr int u = decltype(uc)::value;
          F32Vec<4>::template read<0>(kf[u], (ka ^ (uint32_t)(u << 5)) + buf);
        };

        if constexpr (EXACT) {
          // S^T = K Q^T: one LDS read per four steps, four reads ahead
          constexpr int G = 4 < NU ? 4 : NU, NG = NU / G;
          static_for<0, G>(read_k);
          static_for<0, NG>([&](auto gc) __attribute__((always_inline)) {
            constexpr int gg = decltype(gc)::value;
            if constexpr (gg + 1 < NG) static_for<(gg + 1) * G, (gg + 2) * G>(read_k);
            f32_wait_lds<gg + 1 < NG ? G : 0>();
            static_for<gg * G, (gg + 1) * G>([&](auto uc) __attribute__((always_inline)) {
              constexpr int u = decltype(uc)::value;
#pragma unroll
              for (int rb = 0; rb < RB; ++rb) {
                sc[rb] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u][0], qf[rb][u].x, sc[rb], 0, 0, 0);
                sc[rb] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u][1], qf[rb][u].y, sc[rb], 0, 0, 0);
                sc[rb] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u][2], qf[rb][u].z, sc[rb], 0, 0, 0);
                sc[rb] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u][3], qf[rb][u].w, sc[rb], 0, 0, 0);
              }
            });
          });
          k_free();
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            transform(sc[rb], rb, t, cls);
            const float ms = advance(sc[rb], rb);
            float sum;
#pragma unroll
            for (int r = 0; r < 16; ++r) weight(sc[rb], r, ms, sum);
            l[rb] += sum;
          }
          v_ready();
          // O^T += V^T P^T: one LDS read per key pair, four ahead
          static_for<0, 4>(read_v);
          static_for<0, 4>([&](auto gc) __attribute__((always_inline)) {
            constexpr int gg = decltype(gc)::value;
            if constexpr (gg + 1 < 4) static_for<(gg + 1) * 4, (gg + 2) * 4>(read_v);
            f32_wait_lds<gg + 1 < 4 ? 4 : 0>();
            static_for<gg * 4, gg * 4 + 4>([&](auto rc) __attribute__((always_inline)) {
              constexpr int r = decltype(rc)::value;
#pragma unroll
              for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int d = 0; d < DVB; ++d)
                  o[rb][d] = __builtin_amdgcn_mfma_f32_32x32x2f32(F32Vec<DVB>::at(vf[r], d), sc[rb][r], o[rb][d], 0, 0, 0);
            });
          });
          v_free();
        } else {
          // S^T = K Q^T, a step of sixteen channels per stage: its matrix instructions beside the split of the next step's K (of V's
          // first piece in the last one); LDS reads one stage further ahead
          constexpr int QP = C::QP;
          F32Vec<4>::type qx[QP > 0 ? NK * RB * QP : 1];
          uint32_t qa = (uint32_t)lane;
          if (QP > 0) {
            asm volatile("" : "+v"(qa));
            qa = (uint32_t)(C::QBASE + rg * NK * RB * QP * 1024) + qa * 16u;
          }
          auto read_q = [&](auto kc) __attribute__((always_inline)) {
            static_for<kc * RB * QP, (kc + 1) * RB * QP>([&](auto n) __attribute__((always_inline)) { F32Vec<4>::template read<n * 1024>(qx[n], qa); });
          };
          F32Split kp[2], vp[2], pp[2][RB];        // K and V: of this stage and the next; P: of either half of the keys
          auto split_k = [&](auto kc, auto e) __attribute__((always_inline)) {
            constexpr int kk = decltype(kc)::value, n = 2 * (e % 2);
            f32_split<e>(kf[2 * kk + e / 2][n], kf[2 * kk + e / 2][n + 1], kp[kk % 2]);
          };
          auto split_v = [&](auto uc, auto e) __attribute__((always_inline)) {             // unit: half of the keys, channel block
            constexpr int u = decltype(uc)::value, k0 = 8 * (u / DVB) + 2 * e, d = u % DVB;
            f32_most(vmost, F32Vec<DVB>::at(vf[k0], d), F32Vec<DVB>::at(vf[k0 + 1], d));
            f32_split<e>(F32Vec<DVB>::at(vf[k0], d), F32Vec<DVB>::at(vf[k0 + 1], d), vp[u % 2]);
          };
          read_k(std::integral_constant<int, 0>());
          read_k(std::integral_constant<int, 1>());
          read_q(std::integral_constant<int, 0>());
          read_k(std::integral_constant<int, 2>());
          read_k(std::integral_constant<int, 3>());
          f32_wait_lds<2>();
          static_for<0, 4>([&](auto e) __attribute__((always_inline)) { split_k(std::integral_constant<int, 0>(), e); });
          static_for<0, NK>([&](auto kc) __attribute__((always_inline)) {
            constexpr int kk = decltype(kc)::value;
            constexpr bool last = kk + 1 == NK;
            if constexpr (!last) read_q(std::integral_constant<int, kk + 1>());
            if constexpr (kk + 2 < NK) static_for<2 * kk + 4, 2 * kk + 6>(read_k);
            if constexpr (last) {
              k_free();
              v_ready();
              static_for<0, 8>(read_v);
            }
            f32_wait_lds<last ? 0 : QP * RB + (kk + 2 < NK ? 2 : 0)>();
            f32_stage<6 * RB, 4>(
                [&](auto i) __attribute__((always_inline)) {
                  constexpr int rb = i % RB, n = i / RB;
                  F32Split q = qp[rb][kk];
                  if (QP > 0) q.l = __builtin_bit_cast(i32x4, qx[(kk * RB + rb) * QP]);
                  if (QP > 1) q.m = __builtin_bit_cast(i32x4, qx[(kk * RB + rb) * QP + QP - 1]);
                  sc[rb] = f32_mfma<n>(kp[kk % 2], q, sc[rb]);
                },
                [&](auto e) __attribute__((always_inline)) {
                  if constexpr (last) split_v(std::integral_constant<int, 0>(), e);
                  else split_k(std::integral_constant<int, kk + 1>(), e);
                });
          });

          // the tile's maxima; the weights of the first half of its keys and their parts
          float ms[RB], sum[RB];
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            transform(sc[rb], rb, t, cls);
            ms[rb] = advance(sc[rb], rb);
          }
          auto weights = [&](auto jc) __attribute__((always_inline)) {       // job 2 n: weights of the n-th pair, 2 n + 1: their parts
            constexpr int hf = jc / (8 * RB), n = jc / 2 % (4 * RB), rb = n / 4, e = n % 4, r = 8 * hf + 2 * e;
            if constexpr (jc % 2 == 0) {
              weight(sc[rb], r, ms[rb], sum[rb]);
              weight(sc[rb], r + 1, ms[rb], sum[rb]);
              if (r + 2 == 16) l[rb] += sum[rb];
            } else {
              f32_split<e>(sc[rb][r], sc[rb][r + 1], pp[hf][rb]);
            }
          };
          static_for<0, 8 * RB>(weights);
          __builtin_amdgcn_sched_barrier(0);

          // O^T += V^T P^T in units of (half of the keys, channel block): the matrix instructions of a unit beside the split of the next
          // one's V, and beside the weights of the second half of the keys in the units of the first
          static_for<0, 2 * DVB>([&](auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value, hf = u / DVB, d = u % DVB;
            constexpr int NP = hf == 0 ? 8 * RB / DVB : 0, NV = u + 1 < 2 * DVB ? 4 : 0;
            if constexpr (u + 1 == DVB) static_for<8, 16>(read_v);           // (the first half's values are split)
            f32_stage<6 * RB, NP + NV>(
                [&](auto i) __attribute__((always_inline)) {
                  constexpr int rb = i % RB, n = i / RB;
                  o[rb][d] = f32_mfma<n>(vp[u % 2], pp[hf][rb], o[rb][d]);
                },
                [&](auto j) __attribute__((always_inline)) {
                  if constexpr (j < NP) {
                    weights(std::integral_constant<int, 8 * RB + d * NP + j>());
                  } else {
                    if constexpr (j == NP && u + 1 == DVB) {
                      f32_wait_lds<0>();
                      v_free();
                    }
                    split_v(std::integral_constant<int, u + 1>(), std::integral_constant<int, j - NP>());
                  }
                });
          });
        }
      };

      if constexpr (RG == 1) {
        // One wave per split: nobody shares its tiles, so it never meets another wave inside the loop.  One buffer is enough:
        // K of the next tile is requested when the scores are formed, V when P V is, each has the other contraction's time
        // to arrive, and vector memory completes in order, so that the wait for one leaves the other in flight.
        auto next = [&](int t) __attribute__((always_inline)) {
          while (t < t_hi && !wanted(t)) t += KS;
          return t;
        };
        int t = next(t_lo + ks);
        if (t < t_hi) {
          load_k(t, 0);
          load_v(t, 0);
        }
        while (t < t_hi) {
          const int tn = next(t + KS);
          f32_wait_mem<C::NINSTR>();
          tile(t, classify(t, iw, iw_max, qs_w, tile_ids(t)), 0u,
               [&]() __attribute__((always_inline)) { if (tn < t_hi) load_k(tn, 0); },
               [&]() __attribute__((always_inline)) {
                 if (tn < t_hi) f32_wait_mem<C::NINSTR>();
                 else f32_wait_mem<0>();
                 clear_v(t, 0);
               },
               [&]() __attribute__((always_inline)) { if (tn < t_hi) load_v(tn, 0); });
          t = tn;
        }
      } else {
        if (!C::PLAIN) load_first();
        for (int it = 0; it < n_iter; ++it) {
          const int t = t_lo + it * KS + ks;
          f32_wait_mem<0>();                       // this wave's loads of tile t have landed ...
          clear_k(t, it & 1);
          clear_v(t, it & 1);
          f32_wait_lds<0>();
          __syncthreads();                         // ... and everyone's; the other buffer is free
          if (it + 1 < n_iter && wanted(t + KS)) {
            load_k(t + KS, (it + 1) & 1);
            load_v(t + KS, (it + 1) & 1);
          }
          if (t >= t_hi) continue;
          const int cls = iw < p.Sq ? classify(t, iw, iw_max, qs_w, tile_ids(t)) : kSkip;
          if (cls == kSkip) continue;              // (uniform over the wave)
          tile(t, cls, (uint32_t)((it & 1) * C::STAGE), []() __attribute__((always_inline)) {}, []() __attribute__((always_inline)) {},
               []() __attribute__((always_inline)) {});
        }
      }
      if constexpr (EXACT) {
        return false;
      } else {
        // A weight below 2^-110 loses up to 2^-134 of itself: an accumulator from 2^-98 of the largest value on holds 2^-24 of its own
        // beside up to 2^12 of them.  Where no value reaches 2^-88, zero in an accumulator may be what bf16 made of them.
        float lo = 0x1p-88f;
        if (__builtin_amdgcn_ballot_w64(vmost > 0x1p10f) != 0) {
#pragma unroll
          for (int x = 32; x >= 1; x >>= 1) vmost = fmaxf(vmost, __shfl_xor(vmost, x));
          lo = vmost * 0x1p-98f;
        }
        const bool tiny = __builtin_amdgcn_ballot_w64(vmost >= 0x1p-88f) == 0 && __builtin_amdgcn_ballot_w64(vmost > 0.f) != 0;
        F32Range sums;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int d = 0; d < DVB; ++d)
#pragma unroll
            for (int r = 0; r < 16; ++r) sums.take(o[rb][d][r]);
        return tiny || __builtin_amdgcn_ballot_w64(!sums.inside(lo, INFINITY)) != 0;
      }
    };

    if (s > 0) __syncthreads();                    // LDS is reused by the second stream
    bool again = true;
    // The variants take the parts where there are tiles enough to earn what they cost beside the tiles (the split of Q, the check and the
    // agreement of the waves).  16 x 16 heads x 32 / 64 / 96 / 128 / 160 rows and keys, on parts and not: ALiBi, D = 32 8.5 / 10.5 / 12.7 / 15.2 / 20.1 and
    // 7.8 / 9.8 / 12.2 / 14.7 / 21.0 us, gate, D = 64 12.9 / 16.0 / 18.9 / 22.3 / 32.0 and 11.9 / 15.5 / 18.8 / 22.5 / 36.2; the second stream, 4 x 16 x 256,
    // D = 32 / 64 (two tiles for each of four splits) 22.7 / 34.4 and 21.4 / 35.0.  With one wave per split parts are as fast from the first tile on.
    const int least = RG == 1 ? 0 : KS > 1 ? (DMAX == 32 ? 2 : 0) : DMAX == 32 ? 4 : 3;
    if constexpr (C::PARTS)
      if (fabsf(p.scale) <= 0x1p64f && (C::PLAIN || n_iter > least)) again = pass(std::integral_constant<bool, false>());
    if constexpr (C::PARTS && RG > 1) {                        // waves that share tiles take the second pass together
      int* flags = (int*)lds_raw;
      __syncthreads();
      if (lane == 0) flags[wave] = again ? 1 : 0;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < RG * KS; ++w) again = again || flags[w] != 0;
      again = __builtin_amdgcn_readfirstlane(again ? 1 : 0) != 0;
      __syncthreads();
    }
    if (again) pass(std::integral_constant<bool, true>());

    // ---- the splits of a row group merge in split 0 (rescale rule of Sec. 3.3), in the order of the splits
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) l[rb] = half_swap_sum(l[rb]);
    if constexpr (C::SHARE) {
      __syncthreads();                             // the tile ring is free
      float* mo = (float*)(lds_raw + rg * KS * C::OBYTES) + lane * 4;               // [split][block][register group][channel block]
      float* ml = (float*)(lds_raw + RG * KS * C::OBYTES + rg * KS * C::MLBYTES) + lane;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
#pragma unroll
          for (int d = 0; d < DVB; ++d)
            *(float4*)(mo + ks * (C::OBYTES / 4) + ((rb * 4 + r4) * DVB + d) * 256) =
                make_float4(o[rb][d][4 * r4], o[rb][d][4 * r4 + 1], o[rb][d][4 * r4 + 2], o[rb][d][4 * r4 + 3]);
        ml[(ks * RB + rb) * 128] = m[rb];
        ml[(ks * RB + rb) * 128 + 64] = l[rb];
      }
      __syncthreads();
      int el = lane;                               // (opaque, as in the epilogue below)
      asm volatile("" : "+v"(el));
      const int eh = el >> 5;
      for (int n = ks; n < 4 * RB; n += KS) {      // block n / 4, register group n % 4
        const int rb = n / 4, r4 = n % 4, er = iw + 32 * rb + (el & 31);
        float f[KS], mall = -INFINITY, lt = 0.f;
#pragma unroll
        for (int u = 0; u < KS; ++u) mall = fmaxf(mall, ml[(u * RB + rb) * 128]);
        const float ms = mall == -INFINITY ? 0.f : mall;
#pragma unroll
        for (int u = 0; u < KS; ++u) {
          f[u] = fast_exp2(ml[(u * RB + rb) * 128] - ms);
          lt += ml[(u * RB + rb) * 128 + 64] * f[u];
        }
        float x[DVB][4] = {};
#pragma unroll
        for (int u = 0; u < KS; ++u)
#pragma unroll
          for (int d = 0; d < DVB; ++d) {
            const float4 y = *(const float4*)(mo + u * (C::OBYTES / 4) + (n * DVB + d) * 256);
            x[d][0] += y.x * f[u];
            x[d][1] += y.y * f[u];
            x[d][2] += y.z * f[u];
            x[d][3] += y.w * f[u];
          }
        if (er < p.Sq) {
          const float inv = lt > 0.f ? 1.f / lt : 0.f;
          float* op = (float*)p.out.ptr + b * p.out.sb + g * p.out.sg + h * p.out.sh + (int64_t)er * p.out.ss;
          if (p.lse != nullptr && eh == 0 && r4 == 0)
            p.lse[b * p.lse_sb + (int64_t)g * p.lse_sg + h * p.lse_sh + er] = lt > 0.f ? mall * kLn2 + logf(lt) : -INFINITY;
#pragma unroll
          for (int e4 = 0; e4 < DVB; ++e4) {       // (channel DVB i + d is element i of channel block d)
            const int c = DVB * (8 * r4 + 4 * eh) + 4 * e4;
            auto at = [&](int e) __attribute__((always_inline)) { return x[(4 * e4 + e) % DVB][(4 * e4 + e) / DVB] * inv; };
            if (c < p.Dv) *(float4*)(op + c) = make_float4(at(0), at(1), at(2), at(3));
          }
        }
      }
      return;
    } else if constexpr (KS > 1) {
      __syncthreads();                             // the tile ring is free
      float* mo = (float*)(lds_raw + (rg * (KS - 1) + ks - 1) * C::OBYTES) + lane * 4;
      float* ml = (float*)(lds_raw + RG * (KS - 1) * C::OBYTES) + (rg * (KS - 1) + ks - 1) * (128 * RB) + lane;
      if (ks > 0) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
          for (int d = 0; d < DVB; ++d)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
              *(float4*)(mo + ((rb * DVB + d) * 4 + r4) * 256) =
                  make_float4(o[rb][d][4 * r4], o[rb][d][4 * r4 + 1], o[rb][d][4 * r4 + 2], o[rb][d][4 * r4 + 3]);
          ml[rb * 128] = m[rb];
          ml[rb * 128 + 64] = l[rb];
        }
      }
      __syncthreads();
      if (ks == 0) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          const float* mr = ml + rb * 128;
          float f[KS], mall = m[rb];
#pragma unroll
          for (int u = 1; u < KS; ++u) mall = fmaxf(mall, mr[u * 128 * RB]);
          const float ms = mall == -INFINITY ? 0.f : mall;
          f[0] = fast_exp2(m[rb] - ms);
          float lt = l[rb] * f[0];
#pragma unroll
          for (int u = 1; u < KS; ++u) {
            f[u] = fast_exp2(mr[u * 128 * RB] - ms);
            lt += mr[u * 128 * RB + 64] * f[u];
          }
          m[rb] = mall;
          l[rb] = lt;
#pragma unroll
          for (int d = 0; d < DVB; ++d)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
              f32x16& a = o[rb][d];
#pragma unroll
              for (int e = 0; e < 4; ++e) a[4 * r4 + e] *= f[0];
#pragma unroll
              for (int u = 1; u < KS; ++u) {
                const float4 x = *(const float4*)(mo + u * (C::OBYTES / 4) + ((rb * DVB + d) * 4 + r4) * 256);
                a[4 * r4] += x.x * f[u];
                a[4 * r4 + 1] += x.y * f[u];
                a[4 * r4 + 2] += x.z * f[u];
                a[4 * r4 + 3] += x.w * f[u];
              }
            }
        }
      }
    }

    // ---- epilogue: normalise, combine, RMSNorm, gate, store.  Of two streams the first one's normalised rows wait in
    // `out`, where the same lanes pick them up.
    // (Row and channels come from an opaque copy of the lane id: their addresses would otherwise be formed before the key loop
    // and hold registers through it.)
    int el = lane;
    asm volatile("" : "+v"(el));
    const int eh = el >> 5;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int er = iw + 32 * rb + (el & 31);
      if (ks != 0 || er >= p.Sq) continue;
      f32x16 (&x)[DVB] = o[rb];
      const float inv = l[rb] > 0.f ? 1.f / l[rb] : 0.f;
      float* op = (float*)p.out.ptr + b * p.out.sb + g * p.out.sg + h * p.out.sh + (int64_t)er * p.out.ss;
      if (p.lse != nullptr && eh == 0)
        p.lse[b * p.lse_sb + (int64_t)(ns * g + s) * p.lse_sg + h * p.lse_sh + er] = l[rb] > 0.f ? m[rb] * kLn2 + logf(l[rb]) : -INFINITY;
      const float lam = s == 1 ? p.lambda[h] : 0.f;
      const bool last = s + 1 == ns;
      float ssq = 0.f;
      // register group r4 holds 4 DVB consecutive channels, in DVB pieces of four; element e of piece e4 sits in ...
      auto chan = [&](int r4, int e4) __attribute__((always_inline)) { return DVB * (8 * r4 + 4 * eh) + 4 * e4; };
      auto at = [&](int r4, int e4, int e) __attribute__((always_inline)) -> float { return x[(4 * e4 + e) % DVB][4 * r4 + (4 * e4 + e) / DVB]; };
#pragma unroll
      for (int d = 0; d < DVB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) x[d][r] *= inv;
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
#pragma unroll
        for (int e4 = 0; e4 < DVB; ++e4) {
          const int c = chan(r4, e4);
          if (c >= p.Dv) continue;
          if (s == 1) {
            const float4 first = *(const float4*)(op + c);
            const float f4[4] = {first.x, first.y, first.z, first.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int d = (4 * e4 + e) % DVB, r = 4 * r4 + (4 * e4 + e) / DVB;
              x[d][r] = f4[e] - lam * x[d][r];
            }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) ssq += at(r4, e4, e) * at(r4, e4, e);
        }
      float rn = 1.f;
      if (last && (EPI & kEpiRms) != 0) {
        ssq = half_swap_sum(ssq);
        rn = 1.f / sqrtf(ssq / (float)p.Dv + p.rms_eps);
      }
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
#pragma unroll
        for (int e4 = 0; e4 < DVB; ++e4) {
          const int c = chan(r4, e4);
          if (c >= p.Dv) continue;
          float4 a = make_float4(at(r4, e4, 0), at(r4, e4, 1), at(r4, e4, 2), at(r4, e4, 3));
          if (last && (EPI & kEpiRms) != 0) {
            float4 w = make_float4(1.f, 1.f, 1.f, 1.f);
            if (p.rms_weight) w = make_float4(p.rms_weight[c], p.rms_weight[c + 1], p.rms_weight[c + 2], p.rms_weight[c + 3]);
            a.x *= rn * w.x; a.y *= rn * w.y; a.z *= rn * w.z; a.w *= rn * w.w;
          }
          if (last && (EPI & kEpiGate) != 0) {
            const float* gp = (const float*)p.gate.ptr + b * p.gate.sb + g * p.gate.sg + h * p.gate.sh + (int64_t)er * p.gate.ss;
            const float4 gg = *(const float4*)(gp + c);
            a.x *= 1.f / (1.f + expf(-gg.x));
            a.y *= 1.f / (1.f + expf(-gg.y));
            a.z *= 1.f / (1.f + expf(-gg.z));
            a.w *= 1.f / (1.f + expf(-gg.w));
          }
          *(float4*)(op + c) = a;
        }
    }
  }
}

}  // namespace fl
