// dK, dV with 64 keys per wave (bwd_dkdv_wide_kernel): the contractions of bwd_dkdv_ws_kernel without its specialised waves.
//
// A wave owns 64 keys, and every fragment of Q and dO that it reads from LDS feeds two MFMAs; there is no second wave to hand P over to, and a
// workgroup meets once per 64-row tile instead of once per 32 rows.  bwd_dkdv_ws_kernel spent as long on LDS as on its matrix work (144 KB read, 32 KB
// written per 32 rows of 128 keys), and its matrix cores were busy 45 % of the time.  The price is the whole register file for one wave per SIMD: two fp32
// accumulators of 64 x 128 are all 256 accumulation registers, K and V of the keys 128 vector registers, and a lone wave has to hide every latency by itself:
//   * the 32 fragments of a 32-row block are one stream, read four ahead across its four products (dP, dV, dK, the next block's S);
//   * the elementwise work is cut into units of one score and put behind single MFMAs, P behind those of dP and half of dV, dS behind the rest of dV and half of dK;
//   * delta is the accumulator that dP starts from (V is negated, the product is delta - dP), so dS takes one multiplication;
//   * scores are hidden once, before their exponentials, in the few blocks that a mask cuts.
// Matrix cores 64 % busy (46 % at D = 64, Dv = 128), at the lower clock that this leaves under the power cap.
// Measured, us, one card, 128 keys per workgroup with specialised waves / this kernel, D = 128: causal 2 x 32/8 x 8192 2280 / 1812, 4 x 16 x 4096
// 610 / 501, no mask 4 x 16 x 4096 1137 / 872, ALiBi 2 x 16 x 4096 599 / 453, soft-cap 639 / 544, prefix 4 x 16 x 4096 605 / 499; D = 64, Dv = 128,
// one stream of 2 x 16 x 4096 290 / 223.  Windows and documents, of which few blocks are whole, gain nothing (241 / 235, 374 / 379), and D = 64 on
// long sequences only (causal 8 x 16 x 1999 218 / 241, 4 x 16 x 4096 354 / 310): they have no such kernel.
#pragma once
#include "fl_bwd_bf16.hpp"

namespace fl {

// D: channels of Q and K, DV: of V and dO.
template <class C>
struct WideCfg {
  static constexpr int NW = 4, KEYS = 64, BM = NW * KEYS;          // waves, keys per wave, keys per workgroup
  static constexpr int NSTAGE = 3;
  static constexpr int STAGE = (C::STAGE_KV + 255) & ~255;
  static constexpr int LDS = NSTAGE * STAGE;
  static constexpr int N1 = C::KV, N2 = 2 * C::DBV, N3 = 2 * C::DB, N4 = C::KK, NS = N1 + N2 + N3 + N4;   // fragments per 32-row block
  static constexpr int PD = C::D == 128 && C::MOD == kModSoftcap ? 2 : 4;   // fragments read ahead (the soft-cap's steps are longer, and need registers)
  static_assert(NS % PD == 0, "every block begins at the same place of the ring");
};

constexpr uint32_t kHiddenBits = 0xff7ffffdu;     // -3.4e38

// acc += a b on accumulation registers.  The accumulators live there for the whole kernel and only these instructions touch them;
// left to the compiler, every MFMA result of a kernel with more than 256 registers goes there and is copied back (or, told to leave results in
// vector registers, it moves the accumulators through them: 178 registers in scratch).  The compiler keeps no wait states for an instruction that it cannot see, so
// they are part of the statement: two where the vector ALU may have written b just before (FRESH), else one.  Nothing else can be needed: a has
// come from LDS behind a wait, the results go to registers that no other instruction reads or writes before the loop has ended, and an
// accumulator's next product comes several MFMAs later, which the hardware would hold back anyway.  A copy of a or b that the compiler put in front
// would need two as well (two everywhere: 1 % of the kernel); there is none, and the build looks for one in the assembly (check_wide.py).
template <bool FRESH>
__device__ __forceinline__ void mfma_acc(f32x16& acc, bf16x8 a, bf16x8 b) {
  asm volatile("s_nop %3\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b), "n"(FRESH ? 1 : 0));
}

template <class C>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
bwd_dkdv_wide_kernel(const BwdParams p) {
  typedef WideCfg<C> X;
  typedef BwdWave<C> W;
  constexpr int BN = C::BN, KK = C::KK, KV = C::KV, DB = C::DB, DBV = C::DBV, ROW = C::ROW, ROWV = C::ROWV;
  constexpr uint32_t MASK = C::MASK;
  static_assert(C::MOD != kModCustom && (MASK & (kMaskCustom | kMaskDoc)) == 0 && C::NBIAS == 0 && BN == 64, "what the kernel is written for");
  extern __shared__ __attribute__((aligned(256))) unsigned char lds_raw[];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, half = lane >> 5, col = lane & 31;

  // tile by tile through all problems, the longest (under a causal mask) first: with one workgroup per compute unit the launch is a few rounds
  int kt, bh;
  if (p.order_k == 1) {                            // whole key/value heads per XCD: their Q / dO tiles stay in one L2
    p.k_tiles.split(blockIdx.x >> 3, kt, bh);
    bh = bh * 8 + (blockIdx.x & 7);
  } else {
    p.k_tiles.split(blockIdx.x, kt, bh);
  }
  const KeyProblem kp = key_problem(p, bh);
  const int split = kp.split, hk = kp.hk, g = kp.g, b = kp.b, h_first = kp.h_first;
  const int group = p.heads_wg;                    // query heads this workgroup sums over
  const int j0 = kt * X::BM, jw = j0 + X::KEYS * wave;
  const float c_scale = p.scale * kLog2e;

  const int j_last = (j0 + X::BM < p.Sk ? j0 + X::BM : p.Sk) - 1;
  int q_lo, q_hi;
  query_range(MASK, j0, j_last, p.Sq + p.q_off, p.window, p.prefix, q_lo, q_hi);   // as positions; row = position - q_off
  q_lo = max(q_lo - p.q_off, 0);
  q_hi = max(q_hi - p.q_off, 0);
  const int t_lo = q_lo / BN, t_hi = (q_hi + BN - 1) / BN;
  const int nt = max(t_hi - t_lo, 0);              // q-tiles per head
  // What the workgroup goes through: (head of the group, q-tile), head-major.  h == group: none left.
  struct Item { int h, r; };
  auto after = [&](Item a) __attribute__((always_inline)) -> Item {
    const bool wrap = a.r + 1 >= nt;
    return Item{a.h + (wrap ? 1 : 0), wrap ? 0 : a.r + 1};
  };

  const uint32_t q_stride = (uint32_t)p.q.ss * 2, do_stride = (uint32_t)p.dout.ss * 2;   // (below 2^24, the host sees to it)
  const unsigned char* const q_base = (const unsigned char*)((const uint16_t*)p.q.ptr + b * p.q.sb + g * p.q.sg + h_first * p.q.sh);
  const unsigned char* const do_base = (const unsigned char*)((const uint16_t*)p.dout.ptr + b * p.dout.sb + g * p.dout.sg + h_first * p.dout.sh);
  const unsigned char* const st_base = (const unsigned char*)((wave == 0 ? p.lse2 : p.delta) + ((int64_t)(b * p.G + g) * p.H + h_first) * p.Sq);
  auto load_item = [&](Item it, uint32_t stage) __attribute__((always_inline)) {
    const int t = t_lo + it.r;
    const int last = min(BN, p.Sq - t * BN) - 1;
    int ln = lane;
    asm volatile("" : "+v"(ln));                   // the lane's row and chunk are formed anew: no registers for them across the loop
    const int lq_row = wave * (512 / C::D) + ln / (C::D / 8), lv_row = wave * (512 / C::DV) + ln / (C::DV / 8);
    const uint32_t lq_ch = ((ln % (C::D / 8)) ^ swz_u<C::D>(lq_row)) * 16, lv_ch = ((ln % (C::DV / 8)) ^ swz_u<C::DV>(lv_row)) * 16;
    unsigned char* st = lds_raw + stage + wave * 1024;
    const unsigned char* qb = q_base + ((int64_t)it.h * p.q.sh + (int64_t)(t * BN) * p.q.ss) * 2;
    const unsigned char* db = do_base + ((int64_t)it.h * p.dout.sh + (int64_t)(t * BN) * p.dout.ss) * 2;
#pragma unroll
    for (int u = 0; u < C::TILE_INSTR / 4; ++u) {
      const uint32_t off = __umul24(min(lq_row + u * 4 * (512 / C::D), last), q_stride) + lq_ch;
      __builtin_amdgcn_global_load_lds((global_cvoid*)(qb + off), (lds_void*)(st + u * 4096), 16, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < C::TILEV_INSTR / 4; ++u) {
      const uint32_t off = __umul24(min(lv_row + u * 4 * (512 / C::DV), last), do_stride) + lv_ch;
      __builtin_amdgcn_global_load_lds((global_cvoid*)(db + off), (lds_void*)(st + C::TILE + u * 4096), 16, 0, 0);
    }
    if (wave < 2) {                                // row statistics, 4 bytes per lane: wave 0 lse2, wave 1 delta
      const unsigned char* src = st_base + ((int64_t)it.h * p.Sq + t * BN) * 4 + (uint32_t)min(ln, last) * 4;
      lds_void* dst = (lds_void*)(lds_raw + stage + C::STATS + wave * C::STAT);
      __builtin_amdgcn_global_load_lds((global_cvoid*)src, dst, 4, 0, 0);
    }
  };
  auto meet = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0x0070);            // vmcnt(0) lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  Item it0 = Item{nt > 0 ? 0 : group, 0};
  Item it1 = after(it0), it2 = after(it1);
  if (it0.h < group) load_item(it0, 0);
  if (it1.h < group) load_item(it1, X::STAGE);

  // K and -V of this lane's keys as B operands: with -V the second product is delta - dP, its accumulator starting from delta
  bf16x8 kf[2][KK], vf[2][KV];
#pragma unroll
  for (int kh = 0; kh < 2; ++kh) {
    const int j = jw + 32 * kh + col, jc = j < p.Sk ? j : p.Sk - 1;
    const uint16_t* kp = (const uint16_t*)p.k.ptr + b * p.k.sb + g * p.k.sg + hk * p.k.sh + (int64_t)jc * p.k.ss;
    const uint16_t* vp = (const uint16_t*)p.v.ptr + b * p.v.sb + g * p.v.sg + hk * p.v.sh + (int64_t)jc * p.v.ss;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[kh][kk] = *(const bf16x8*)(kp + 16 * kk + 8 * half);
#pragma unroll
    for (int kk = 0; kk < KV; ++kk) {
      i32x4 x = *(const i32x4*)(vp + 16 * kk + 8 * half);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] ^= (int)0x80008000;
      vf[kh][kk] = __builtin_bit_cast(bf16x8, x);
    }
  }

  // lane offsets of the row reads and of the transposing reads; the fragments' chunks differ from the first one's by an XOR
  const uint32_t rq0 = col * ROW + ((half ^ swz_u<C::D>(col)) * 16), rv0 = col * ROWV + ((half ^ swz_u<C::DV>(col)) * 16);
  const int s16 = lane & 15, r0 = 4 * half + (s16 >> 2), ch0 = 16 * ((lane >> 4) & 1) + 4 * (s16 & 3);
  const uint32_t tq0 = r0 * ROW + (((ch0 >> 3) ^ swz_u<C::D>(r0)) * 16) + (ch0 & 7) * 2;
  const uint32_t tv0 = r0 * ROWV + (((ch0 >> 3) ^ swz_u<C::DV>(r0)) * 16) + (ch0 & 7) * 2;

  f32x16 dk[DB][2], dv[DBV][2];
#pragma unroll
  for (int d = 0; d < DB; ++d) dk[d][0] = dk[d][1] = W::zero16();
#pragma unroll
  for (int d = 0; d < DBV; ++d) dv[d][0] = dv[d][1] = W::zero16();
  f32x16 s[2], dp[2];                              // scores, then P; delta - dP
  // fragments in flight: by rows, transposed (two reads each, put together behind their wait: until then the compiler has no use of either)
  i32x4 fr[X::PD];
  i32x2 lo[X::PD], hi[X::PD];
  i32x4 lse[4], del[4];
  uint32_t pw[2][8], dw[2][8];                     // bf16 pairs of P and of -dS

  // fragment f of the block QB at stage offset `cur` (f >= NS: of the next block, QN at `nxt`) into its ring slot
  auto issue = [&](auto fc, auto qb_c, auto qn_c, uint32_t cur, uint32_t nxt) __attribute__((always_inline)) {
    constexpr int F = decltype(fc)::value;
    constexpr bool NEXT = F >= X::NS;
    constexpr int f = NEXT ? F - X::NS : F, QB = NEXT ? decltype(qn_c)::value : decltype(qb_c)::value, QN = decltype(qn_c)::value;
    const uint32_t base = NEXT ? nxt : cur;
    constexpr int slot = F % X::PD;
    if constexpr (f < X::N1) {
      W::template read_b128<C::TILE + QB * 32 * ROWV>(fr[slot], (rv0 + base) ^ (f * 32));
    } else if constexpr (f < X::N1 + X::N2) {
      constexpr int d = (f - X::N1) % DBV, ks = (f - X::N1) / DBV, off = C::TILE + (QB * 32 + ks * 16) * ROWV;
      W::template read_tr<off>(lo[slot], (tv0 + base) ^ (d * 64));
      W::template read_tr<off + 8 * ROWV>(hi[slot], (tv0 + base) ^ (d * 64 + 32));
    } else if constexpr (f < X::N1 + X::N2 + X::N3) {
      constexpr int d = (f - X::N1 - X::N2) % DB, ks = (f - X::N1 - X::N2) / DB, off = (QB * 32 + ks * 16) * ROW;
      W::template read_tr<off>(lo[slot], (tq0 + base) ^ (d * 64));
      W::template read_tr<off + 8 * ROW>(hi[slot], (tq0 + base) ^ (d * 64 + 32));
    } else {
      constexpr int kk = f - X::N1 - X::N2 - X::N3;
      W::template read_b128<QN * 32 * ROW>(fr[slot], (rq0 + nxt) ^ (kk * 32));
    }
  };
  // LDS instructions of fragment F
  constexpr auto cost = [](int F) constexpr {
    const int f = F % X::NS;
    return f >= X::N1 && f < X::N1 + X::N2 + X::N3 ? 2 : 1;
  };
  // statistics of the next block: quad x of delta (x < 4), of lse2 (x - 4) at step STAT0 + x
  constexpr int STAT0 = X::NS - X::PD - 7;
  static_assert(STAT0 > 0 && STAT0 + 4 >= X::N1 + X::N2 / 2, "the current block's statistics are done with");

  auto block = [&](auto qb_c, auto qn_c, uint32_t cur, uint32_t nxt, Item it) __attribute__((always_inline)) {
    constexpr int QB = decltype(qb_c)::value, QN = decltype(qn_c)::value;
    const int ib = (t_lo + it.r) * BN + 32 * QB;
    const int cls = classify_block(MASK, ib + p.q_off, ib + 31 + p.q_off, jw, jw + X::KEYS - 1, p.Sk, p.window, p.prefix, make_int2(0, 0), make_int2(0, 0));
    // Hidden scores, in the few blocks that have any: -inf, of which the positive scale makes P = 0, or for the soft-cap, of which
    // tanh makes -1, one particular number at the end of the range whose P is replaced by 0.  A row whose lse is NaN gives NaN where it sees a key and 0 elsewhere.
    if (ib + 31 >= p.Sq || cls != kFull) {
      int ln = lane;
      uint32_t hidden = C::MOD == kModSoftcap ? kHiddenBits : 0xff800000u;
      asm volatile("" : "+v"(ln), "+v"(hidden));   // (nothing of this is worth a register outside the branch)
      W::template wait_lds<0>();                   // lse2 may still be on its way
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) {
        Span span = seeing_rows(MASK, jw + 32 * kh + (ln & 31), p.Sq, p.Sk, p.q_off, p.window, p.prefix);
        span.first -= ib + 4 * (ln >> 5);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float l = __int_as_float(lse[r >> 2][r & 3]);
          if (C::MOD != kModSoftcap) s[kh][r] = l != l ? l : s[kh][r];
          s[kh][r] = span.outside(8 * (r >> 2) + (r & 3)) ? __uint_as_float(hidden) : s[kh][r];
          __builtin_amdgcn_sched_barrier(0);       // one after the other: the conditions would take the scalar registers of the loop
        }
      }
      if constexpr (C::MOD != kModSoftcap) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float l = __int_as_float(lse[r >> 2][r & 3]);
          lse[r >> 2][r & 3] = l != l ? 0x7f800000 : lse[r >> 2][r & 3];
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    // ALiBi: the distance of register 0's row from the lane's first key (a whole number, like the registers' offsets to it), the slope
    const float slope2 = C::MOD == kModAlibi ? p.alibi_slopes[h_first + it.h] * kLog2e : 0.f;
    float dist = 0.f;
    if constexpr (C::MOD == kModAlibi) {
      int ln = lane;
      asm volatile("" : "+v"(ln));
      dist = (float)(ib + p.q_off + 4 * (ln >> 5) - (jw + (ln & 31)));
    }
    // the elementwise work in small units, one after the other: score u of the block (registers in pairs, key halves in turn), pair u of dS
    float pv0 = 0.f;
    auto p_unit = [&](auto uc) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value, e = u % 2, kh = u / 2 % 2, r2 = u / 4, r = 2 * r2 + e;
      float fac;
      float pv = fast_exp2(replay_score<C::MOD>(s[kh][r], c_scale, __int_as_float(lse[r >> 2][r & 3]), p.softcap, slope2,
                                             dist + (float)(8 * (r >> 2) + (r & 3) - 32 * kh), fac));
      if (C::MOD == kModSoftcap && __float_as_uint(s[kh][r]) == kHiddenBits) pv = 0.f;
      s[kh][r] = C::MOD == kModSoftcap ? pv * fac : pv;
      if constexpr (e == 0) pv0 = pv;
      else pw[kh][r2] = pack_bf16(pv0, pv);
    };
    auto ds_unit = [&](auto uc) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value, r2 = u / 2, kh = u % 2;
      dw[kh][r2] = pack_bf16(s[kh][2 * r2] * dp[kh][2 * r2], s[kh][2 * r2 + 1] * dp[kh][2 * r2 + 1]);
    };
    // units of P done before MFMA x (phase 1 and the first half of phase 2), of dS (second half of phase 2, first half of phase 3)
    constexpr auto p_at = [](int x) constexpr { const int n = 2 * X::N1 + X::N2 - 2; return x <= 0 ? 0 : x >= n ? 32 : 32 * x / n; };
    constexpr auto ds_at = [](int x) constexpr {
      const int x0 = 2 * X::N1 + X::N2, n = X::N2 + X::N3 - 2;
      return x <= x0 ? 0 : x - x0 >= n ? 16 : 16 * (x - x0) / n;
    };
    static_assert(p_at(2 * X::N1) >= 16 && p_at(2 * X::N1 + X::N2) == 32, "P before its product");
    static_assert(ds_at(2 * (X::N1 + X::N2)) >= 8 && ds_at(2 * (X::N1 + X::N2) + X::N3) == 16, "dS before its product");
    auto units = [&](auto xc) __attribute__((always_inline)) {        // behind MFMA x
      constexpr int x = decltype(xc)::value;
      static_for<p_at(x), p_at(x + 1)>([&](auto u) __attribute__((always_inline)) { p_unit(u); });
      static_for<ds_at(x), ds_at(x + 1)>([&](auto u) __attribute__((always_inline)) { ds_unit(u); });
      __builtin_amdgcn_sched_barrier(0);
    };
    uint32_t st_n = 0;                             // (formed where it is needed)
    static_for<0, X::NS>([&](auto fc) __attribute__((always_inline)) {
      constexpr int f = decltype(fc)::value;
      if constexpr (f >= STAT0 && f < STAT0 + 8) {
        constexpr int x = f - STAT0, q = x % 4;
        if constexpr (x == 0) {
          int ln = lane;
          asm volatile("" : "+v"(ln));
          st_n = nxt + (ln >> 5) * 16;
        }
        if constexpr (x < 4) W::template read_b128<C::STATS + C::STAT + (32 * QN + 8 * q) * 4>(del[q], st_n);
        else W::template read_b128<C::STATS + (32 * QN + 8 * q) * 4>(lse[q], st_n);
      }
      // fragment f has landed when no more than what was issued behind it is outstanding
      constexpr auto behind = [=](int f) constexpr {
        int n = 0;
        for (int i = 1; i < X::PD; ++i) {
          n += cost(f + i);
          const int at = f + i - X::PD;            // the step that issued it
          const int st = (at + X::NS) % X::NS;
          n += st >= STAT0 && st < STAT0 + 8 ? 1 : 0;
        }
        return n;
      };
      static_assert(behind(f) <= 15, "lgkmcnt is a 4-bit counter");
      constexpr int extra = f >= STAT0 && f < STAT0 + 8 ? 1 : 0;
      W::template wait_lds<behind(f) + extra>();
      constexpr int slot = f % X::PD;
      constexpr bool tr = f >= X::N1 && f < X::N1 + X::N2 + X::N3;
      const bf16x8 a = __builtin_bit_cast(bf16x8, tr ? (i32x4){lo[slot][0], lo[slot][1], hi[slot][0], hi[slot][1]} : fr[slot]);
      static_for<0, 2>([&](auto khc) __attribute__((always_inline)) {
        constexpr int kh = decltype(khc)::value;
        if constexpr (f < X::N1) {
          if constexpr (f == 0) {
            f32x16 c0;
#pragma unroll
            for (int r = 0; r < 16; ++r) c0[r] = __int_as_float(del[r >> 2][r & 3]);
            dp[kh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, vf[kh][f], c0, 0, 0, 0);
          } else {
            dp[kh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, vf[kh][f], dp[kh], 0, 0, 0);
          }
        } else if constexpr (f < X::N1 + X::N2) {
          constexpr int d = (f - X::N1) % DBV, ks = (f - X::N1) / DBV;
          mfma_acc<d == 0>(dv[d][kh], a, __builtin_bit_cast(bf16x8, (i32x4){(int)pw[kh][4 * ks], (int)pw[kh][4 * ks + 1], (int)pw[kh][4 * ks + 2], (int)pw[kh][4 * ks + 3]}));
        } else if constexpr (f < X::N1 + X::N2 + X::N3) {
          constexpr int d = (f - X::N1 - X::N2) % DB, ks = (f - X::N1 - X::N2) / DB;
          mfma_acc<d == 0>(dk[d][kh], a, __builtin_bit_cast(bf16x8, (i32x4){(int)dw[kh][4 * ks], (int)dw[kh][4 * ks + 1], (int)dw[kh][4 * ks + 2], (int)dw[kh][4 * ks + 3]}));
        } else {
          constexpr int kk = f - X::N1 - X::N2 - X::N3;
          s[kh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kf[kh][kk], kk == 0 ? W::zero16() : s[kh], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kh == 1) issue(std::integral_constant<int, f + X::PD>(), qb_c, qn_c, cur, nxt);   // into the slot just read
        units(std::integral_constant<int, 2 * f + kh>());
      });
    });
  };

  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  // scores of the first block of the tile at `base`, its statistics, its first fragments
  auto start = [&](uint32_t base) __attribute__((always_inline)) {
    const uint32_t st = base + 16 * half;
    static_for<0, 4>([&](auto q) __attribute__((always_inline)) {
      W::template read_b128<C::STATS + C::STAT + 8 * decltype(q)::value * 4>(del[decltype(q)::value], st);
      W::template read_b128<C::STATS + 8 * decltype(q)::value * 4>(lse[decltype(q)::value], st);
    });
    static_for<0, KK>([&](auto kc) __attribute__((always_inline)) {
      constexpr int kk = decltype(kc)::value;
      i32x4 a;
      W::template read_b128<0>(a, (rq0 + base) ^ (kk * 32));
      W::template wait_lds<0>();
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
        s[kh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), kf[kh][kk], kk == 0 ? W::zero16() : s[kh], 0, 0, 0);
    });
    static_for<0, X::PD>([&](auto f) __attribute__((always_inline)) { issue(f, I0(), I0(), base, base); });
    W::template wait_lds<0>();
  };

  meet();
  uint32_t b0 = 0, b1 = X::STAGE, b2 = 2 * X::STAGE;
  if (it0.h < group) {
    start(b0);
    while (true) {
      if (it2.h < group) load_item(it2, b2);
      block(I0(), I1(), b0, b0, it0);
      block(I1(), I0(), b0, b1, it0);
      W::template wait_lds<0>();                   // no read in flight past the loop
      if (it1.h >= group) break;
      meet();
      it0 = it1;
      it1 = it2;
      it2 = after(it2);
      const uint32_t x = b0;
      b0 = b1;
      b1 = b2;
      b2 = x;
    }
  }
  // The accumulators are read by the vector ALU from here on: past the last MFMA's results
#pragma unroll
  for (int d = 0; d < DBV; ++d) asm volatile("s_nop 15\n\ts_nop 15" : "+a"(dv[d][0]), "+a"(dv[d][1]));
#pragma unroll
  for (int d = 0; d < DB; ++d) asm volatile("s_nop 15\n\ts_nop 15" : "+a"(dk[d][0]), "+a"(dk[d][1]));
  int ln = lane;
  asm volatile("" : "+v"(ln));                     // (no addresses kept through the loop)
#pragma unroll
  for (int kh = 0; kh < 2; ++kh) {
    const int j = jw + 32 * kh + (ln & 31);
    if (j < p.Sk) {
#pragma unroll
      for (int d = 0; d < DBV; ++d)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          store_kv_grad<true, C::DV>(p, split, b, g, hk, j, 32 * d + 8 * r4 + 4 * (ln >> 5), dv[d][kh][4 * r4], dv[d][kh][4 * r4 + 1],
                                     dv[d][kh][4 * r4 + 2], dv[d][kh][4 * r4 + 3]);
      const float m = -p.scale;
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          store_kv_grad<false, C::D>(p, split, b, g, hk, j, 32 * d + 8 * r4 + 4 * (ln >> 5), dk[d][kh][4 * r4] * m, dk[d][kh][4 * r4 + 1] * m,
                                     dk[d][kh][4 * r4 + 2] * m, dk[d][kh][4 * r4 + 3] * m);
    }
  }
}

}  // namespace fl
