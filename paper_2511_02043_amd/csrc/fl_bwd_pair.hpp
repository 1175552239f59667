// bf16 backward kernels of attention with a pair bias shared by many row problems, for gfx950 (Evoformer row-wise attention,
// Sec. 4.1): scores of (b, g, h) take a bias [b, h, Sq, Sk] that does not depend on the row axis g, and optionally a key bias
// that does not depend on the query row; no mask, no score_mod, Sq and Sk of at most 512 (head
// dim 32) or 384 (64).
//
// The general kernels of fl_bwd_bf16.hpp give a workgroup one (b, g, h) problem.  There the bias values dominate: every
// problem reads the whole [Sq, Sk] bias again, in 2-byte (dK/dV) or 8-byte (dQ) pieces per lane, and the bias gradient is staged
// as dS of every score and summed over g afterwards.  Here the bias stays where it is instead: a workgroup owns 64 rows of one
// axis (queries in the dQ kernel, keys in the dK/dV kernel) of one (b, h), each of its waves keeps the bias of its 32 x 32
// blocks in registers, and the problems g go by -- the other axis in steps of 128 rows through a ring of LDS stages.
//   * dQ kernel: the bias gradient of a block is the running sum of dS in fp32 registers, written once per workgroup;
//   * dK/dV kernel: the key bias gradient is the sum of dS over the registers of a lane.
// Wave (rg, kq) = (wave % 2, wave / 2) takes owned rows 32 * rg .. + 31 and, of each step, streamed rows 32 * kq .. + 31.  Its
// streamed rows are its own: it fetches them into a private ring and waits for nobody, so that the two waves of a SIMD drift apart
// and fill each other's gaps; the workgroup only meets once or twice per problem.  (With tiles shared by the workgroup and a
// barrier per step the kernels were no slower at head dim 32 but 1.3 x at 64, 256 x 8 heads x 120; four waves of 512 registers,
// two blocks each, took 110 / 107 us where this took 76 / 85, before lse met the biases in log2 units: dQ / dK, dV of 128 x 8 heads x
// 384, D = 32, which now take 88 / 104.)
// What bounds them there: instruction issue (two waves of a SIMD issue in 75 % of the clocks; dQ: 27 matrix, 48 exp2, 287 other vector
// and 104 scalar instructions per wave and problem of three steps) and, for the rest, the start of a workgroup (7 us).  The
// general kernels took 140 + 64 (reduction of the staged dS) / 146 us.
// The accumulators of a problem are partial over kq: the four waves of a row group meet in LDS, each sums and stores a quarter of
// the channels, in a fixed order (bitwise reproducible, no atomics).
// delta comes folded into the accumulator's starting value, dp = <v, dO> - delta.  lse does not: it meets the bias in log2 units, as
// in the general kernels (biased_exponent).
#pragma once
#include "fl_decode_bf16.hpp"

namespace fl {

struct PairParams {
  BwdParams b;                     // bias[0]: the pair bias (sg unused); delta: -delta
  const float* key;                // key bias in fp32, [.., n_key] (n_key: Sk rounded up to 128), or null
  int64_t key_sb, key_sg, key_sh;
  float* bias_part;                // dQ kernel, or null: partial bias gradients [chunks][B][H][ceil(Sq / 32)][ceil(Sk / 32)][1024]
  float* key_part;                 // dK/dV kernel, or null: sums of dS over the query rows, [B, G, H, Sk]
  int32_t chunks;                  // the problems g of a (b, h) are cut into this many ranges, one workgroup each
  int32_t n_own;                   // ceil(rows of the owned axis / 64)
  int32_t xcd;                     // 1: the tiles of a (b, h, chunk) run on one XCD (chunks * B * H % 8 == 0)
  Divisor by_own, by_chunks, by_h; // n_own, chunks, H
};

// ROLE 0: dQ and the pair bias gradient (streams K, V); 1: dK, dV and the key bias gradient (streams Q, dO).
// NBLK: steps of 128 streamed rows per problem.
template <int D_, int NBLK_, int ROLE_, bool KEYB_>
struct PairCfg : BwdCfg<D_, kModNone, 0, 128, 2, 1> {
  typedef BwdCfg<D_, kModNone, 0, 128, 2, 1> Base;
  static constexpr int NBLK = NBLK_, ROLE = ROLE_;
  static constexpr bool KEYB = KEYB_;
  static constexpr int NACC = ROLE == 0 ? 1 : 2;
  // A wave's ring: a stage is refilled as soon as its fragments are in registers, which is one step ahead of a ring that waits
  // for the end of the step.  Two stages at head dim 32 (one: 91 / 105 us instead of 88 / 104); at 64 the LDS holds one.
  static constexpr int NSTG = D_ == 32 ? 2 : 1;
  static constexpr int STEP_TILE = 32 * Base::ROW;                   // 32 rows of one streamed tensor
  static constexpr int STEP_STAT = 2 * STEP_TILE;                    // role 1: lse2, -delta of the rows
  static constexpr int STEP = STEP_STAT + (ROLE == 1 ? 256 : 0);
  static constexpr int WAVE_RING = NSTG * STEP;
  static constexpr int OWN_TILE = 64 * Base::ROW;                    // the owned rows of a problem: Q, dO (role 0) or K, V
  static constexpr int OWN_STAT = 2 * OWN_TILE;                      // role 0: lse2, -delta of the rows
  static constexpr int OWN_KEY = OWN_STAT + (ROLE == 0 ? 2 * 64 * 4 : 0);
  static constexpr int OWN = OWN_KEY + (KEYB ? (ROLE == 0 ? NBLK * 128 * 4 : 64 * 4) : 0);
  static constexpr int OWN_RING = 8 * WAVE_RING;
  static constexpr int XCH = OWN_RING + 2 * OWN;
  // Hand-over of one 32-channel block of one accumulator: [row group][owner][source wave][lane] float4
  static constexpr int XBLK = 2 * 4 * 4 * 1024;
  static constexpr int NX = NACC * Base::DB;                         // channel blocks to hand over (dV's, then dQ's or dK's)
  // spaces for them: all of them twice (a problem's are read while the next one's are written), all of them, or one that they pass
  // through one after the other
  static constexpr bool XTWICE = D_ == 32 && ROLE == 0;
  static constexpr int NSPACE = D_ == 32 ? NX : 1;
  static constexpr int XSUM = XCH + (XTWICE ? 2 : 1) * NSPACE * XBLK;
  static constexpr int LDS = XSUM + (ROLE == 1 && KEYB ? 8 * 256 : 0);
  // the bias in fp32, in log2 units unless a key bias is added first, where the registers allow it; else as bf16 pairs (one or two
  // instructions more per score)
  static constexpr bool BIAS_F32 = ROLE == 1 ? D_ == 32 || NBLK <= (KEYB ? 1 : 2) : NBLK <= (D_ == 32 ? 3 : 2);
  static constexpr bool OWN_REGS = D_ == 32;                         // the owned rows' fragments stay in registers for a problem
  static constexpr int STEP_INSTR = 2 * (STEP_TILE / 1024) + (ROLE == 1 ? 1 : 0);   // vector memory loads per wave and step
};

// Fragment -> LDS offset map of pairs (owned fragment, streamed fragment): KK pairs at OWN0 / STR0, then KK at OWN1 / STR1
template <int OWN0, int OWN1, int STR0, int STR1, int KK>
struct OwnPair {
  static constexpr int off(int f) { return f % 2 == 0 ? (f < 2 * KK ? OWN0 : OWN1) : (f < 2 * KK ? STR0 : STR1); }
};

template <int OFF>
__device__ __forceinline__ void read_b32(float& dst, uint32_t addr) {   // by hand, as BwdWave's reads
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
}
__device__ __forceinline__ void write_b32(uint32_t addr, float v) { asm volatile("ds_write_b32 %0, %1" : : "v"(addr), "v"(v) : "memory"); }

template <class C>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
bwd_pair_kernel(const PairParams pp) {
  constexpr int D = C::D, KK = C::KK, DB = C::DB, ROW = C::ROW, NBLK = C::NBLK, NSTG = C::NSTG, ROLE = C::ROLE;
  typedef BwdWave<C> W;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const BwdParams& p = pp.b;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = wave & 1, kq = wave >> 1;
  W w;
  w.init(tid & 63);
  const int lane = w.lane;

  // ---- (b, h, chunk of the problems g), tile of 64 owned rows
  // The tiles of a unit (b, h, chunk) stream the same rows: they run on one XCD (consecutive workgroup ids go round-robin to the
  // 8 XCDs; the host checks that the number of units is a multiple of 8).
  int unit, ot;
  if (pp.xcd == 1) {
    pp.by_own.split(blockIdx.x >> 3, unit, ot);
    unit = unit * 8 + (int)(blockIdx.x & 7);
  } else {
    pp.by_own.split(blockIdx.x, unit, ot);
  }
  int bh, chunk, h, b;
  pp.by_chunks.split(unit, bh, chunk);
  pp.by_h.split(bh, b, h);
  auto first_problem = [&](int c) __attribute__((always_inline)) -> int {
    const int64_t n = (int64_t)p.G * c;
    return n <= 0x7fffffff ? pp.by_chunks.div((int)n) : (int)(n / pp.chunks);
  };
  const int g_lo = first_problem(chunk), g_hi = first_problem(chunk + 1);
  const int n_prob = g_hi - g_lo;                  // (at least one: chunks <= G)
  const int S_own = ROLE == 0 ? p.Sq : p.Sk, S_str = ROLE == 0 ? p.Sk : p.Sq;
  const int o0 = ot * 64;                          // first owned row of the workgroup
  const int own = o0 + 32 * rg + w.col;            // this lane's owned row
  const float c_scale = p.scale * kLog2e;

  // ---- the bias of this wave's blocks: register r of step t is streamed row 128 t + 32 kq + 8 (r / 4) + 4 half + r % 4
  constexpr int NBF = C::BIAS_F32 ? NBLK : 1, NBP = C::BIAS_F32 ? 1 : NBLK;
  float blf[NBF][16];
  uint32_t blp[NBP][8];
  {
    const BiasView& bv = p.bias[0];
    const int64_t so = ROLE == 0 ? bv.si : bv.sj, ss = ROLE == 0 ? bv.sj : bv.si;
    // (dQ kernel: a lane's four consecutive keys in one load where the rows allow it)
    const bool vec = ROLE == 0 && ss == 1 && ((uint64_t)bv.ptr) % 8 == 0 && ((bv.sb | bv.sh | so) & 3) == 0;   // uniform
    const uint16_t* brow = (const uint16_t*)bv.ptr + b * bv.sb + h * bv.sh + (int64_t)min(own, S_own - 1) * so;
    // all loads first: their latency is most of a workgroup's start-up
    uint32_t raw[NBLK][8];                         // bf16 pairs
#pragma unroll
    for (int t = 0; t < NBLK; ++t) {
      const int j0 = 128 * t + 32 * kq + 4 * w.half;
      if (vec && 128 * t + 32 * kq + 32 <= S_str) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const uint2 v = *(const uint2*)(brow + j0 + 8 * q4);
          raw[t][2 * q4] = v.x;
          raw[t][2 * q4 + 1] = v.y;
        }
      } else {                                     // streamed rows past the end: -inf, their P is 0
        uint16_t e[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) e[r] = brow[(int64_t)min(j0 + 8 * (r >> 2) + (r & 3), S_str - 1) * ss];
#pragma unroll
        for (int r = 0; r < 16; ++r) e[r] = j0 + 8 * (r >> 2) + (r & 3) < S_str ? e[r] : (uint16_t)0xFF80;
#pragma unroll
        for (int r2 = 0; r2 < 8; ++r2) raw[t][r2] = (uint32_t)e[2 * r2] | ((uint32_t)e[2 * r2 + 1] << 16);
      }
    }
#pragma unroll
    for (int t = 0; t < NBLK; ++t)
#pragma unroll
      for (int r2 = 0; r2 < 8; ++r2) {
        if constexpr (C::BIAS_F32) {
          const float x0 = __uint_as_float(raw[t][r2] << 16), x1 = __uint_as_float(raw[t][r2] & 0xFFFF0000u);
          blf[t][2 * r2] = C::KEYB ? x0 : bias_log2(x0);
          blf[t][2 * r2 + 1] = C::KEYB ? x1 : bias_log2(x1);
          asm volatile("" : "+v"(blf[t][2 * r2]), "+v"(blf[t][2 * r2 + 1]));   // (worked out here, not again in every step)
        } else {
          blp[t][r2] = raw[t][r2];
          asm volatile("" : "+v"(blp[t][r2]));
        }
      }
  }

  // ---- loads: streamed tensors X, Y (K, V or Q, dO), owned ones U, V (Q, dO or K, V).  Uniform 64-bit bases move from step to
  // step and from problem to problem; a lane's offset inside a tile is fixed and fits 32 bits (the host bounds the row stride).
  const View& xv = ROLE == 0 ? p.k : p.q;
  const View& yv = ROLE == 0 ? p.v : p.dout;
  const View& uv = ROLE == 0 ? p.q : p.k;
  const View& vv = ROLE == 0 ? p.dout : p.v;
  auto first = [&](const View& v, int row) __attribute__((always_inline)) {
    return (const unsigned char*)((const uint16_t*)v.ptr + b * v.sb + g_lo * v.sg + h * v.sh + (int64_t)row * v.ss);
  };
  auto lane_off = [&](int inst, int nvalid, uint32_t row_bytes) __attribute__((always_inline)) {
    const int dst_row = inst * (512 / D) + lane / (D / 8);
    return (uint32_t)min(dst_row, nvalid - 1) * row_bytes + (uint32_t)(((lane % (D / 8)) ^ swz_u<D>(dst_row)) * 16);
  };
  auto fetch = [&](const unsigned char* base, uint32_t off, unsigned char* dst, int bytes4) __attribute__((always_inline)) {
    if (bytes4) __builtin_amdgcn_global_load_lds((global_cvoid*)(base + off), (lds_void*)dst, 4, 0, 0);
    else __builtin_amdgcn_global_load_lds((global_cvoid*)(base + off), (lds_void*)dst, 16, 0, 0);
  };
  constexpr int XI = C::STEP_TILE / 1024;          // load instructions per streamed tile of a wave
  const uint32_t xss = (uint32_t)(xv.ss * 2), yss = (uint32_t)(yv.ss * 2);
  // [1]: of a problem's last step, which may be ragged: rows past the end repeat the last one (a block that lies past the end
  // altogether takes the last row throughout: its P is 0)
  const int r_last = min(128 * (NBLK - 1) + 32 * kq, S_str - 1);
  uint32_t x_off[2][XI], y_off[2][XI];
#pragma unroll
  for (int u = 0; u < XI; ++u) {
    x_off[0][u] = lane_off(u, 32, xss);
    y_off[0][u] = lane_off(u, 32, yss);
    x_off[1][u] = lane_off(u, min(32, S_str - r_last), xss);
    y_off[1][u] = lane_off(u, min(32, S_str - r_last), yss);
  }
  constexpr bool kHalfOwn = C::OWN_TILE == 4096;   // four instructions per owned tile: waves 0 .. 3 take U, 4 .. 7 V
  const uint32_t u_off = lane_off(kHalfOwn ? wave & 3 : wave, S_own - o0, (uint32_t)((kHalfOwn && wave >= 4 ? vv.ss : uv.ss) * 2));
  const uint32_t v_off = lane_off(wave, S_own - o0, (uint32_t)(vv.ss * 2));
  const unsigned char *xg = first(xv, 0), *yg = first(yv, 0);                       // problem `ig`, row 0
  const unsigned char *ug = first(uv, o0), *vg = first(vv, o0);                     // the problem whose owned rows are next
  const int64_t stat0 = ((int64_t)(b * p.G + g_lo) * p.H + h) * p.Sq + (ROLE == 0 ? o0 : 0), stat_step = (int64_t)p.H * p.Sq;
  // role 0: the owned rows' lse / delta by even / odd waves; role 1: of problem `ig`, lse for lanes 0 .. 31, delta for 32 .. 63
  const unsigned char* sg = (const unsigned char*)(((ROLE == 0 ? (wave & 1) == 0 : w.half == 0) ? p.lse2 : p.delta) + stat0);
  const unsigned char* kg = nullptr;
  if constexpr (C::KEYB) kg = (const unsigned char*)(pp.key + b * pp.key_sb + g_lo * pp.key_sg + h * pp.key_sh + (ROLE == 0 ? 64 * (wave % (2 * NBLK)) : o0));
  const uint32_t lane4 = lane * 4;
  unsigned char* const ring = lds_raw + wave * C::WAVE_RING;
  // the tiles of step tc of the problem whose row 0 is at xg, yg (sg)
  auto load_step = [&](auto tc, uint32_t base) __attribute__((always_inline)) {   // base: the stage
    constexpr int t = decltype(tc)::value, L = t == NBLK - 1 ? 1 : 0;
    const int r0 = L ? r_last : 128 * t + 32 * kq;
    const unsigned char *xb = xg + (uint64_t)(uint32_t)r0 * xss, *yb = yg + (uint64_t)(uint32_t)r0 * yss;
#pragma unroll
    for (int u = 0; u < XI; ++u) {
      fetch(xb, x_off[L][u], ring + base + u * 1024, 0);
      fetch(yb, y_off[L][u], ring + base + C::STEP_TILE + u * 1024, 0);
    }
    if constexpr (ROLE == 1) fetch(sg, (uint32_t)(r0 + (L ? min(w.col, S_str - r_last - 1) : w.col)) * 4, ring + base + C::STEP_STAT, 1);
  };
  auto load_own = [&](int slot) __attribute__((always_inline)) {
    unsigned char* st = lds_raw + C::OWN_RING + slot * C::OWN;
    if constexpr (kHalfOwn) {
      fetch(wave < 4 ? ug : vg, u_off, st + (wave < 4 ? 0 : C::OWN_TILE) + (wave & 3) * 1024, 0);
    } else {
      fetch(ug, u_off, st + wave * 1024, 0);
      fetch(vg, v_off, st + C::OWN_TILE + wave * 1024, 0);
    }
    if constexpr (ROLE == 0) fetch(sg, (uint32_t)min(lane, S_own - o0 - 1) * 4, st + C::OWN_STAT + (wave & 1) * 256, 1);
    // (the key bias array is padded to whole steps of 128 keys)
    if constexpr (C::KEYB) fetch(kg, lane4, st + C::OWN_KEY + (ROLE == 0 ? wave % (2 * NBLK) : 0) * 256, 1);
  };
  // this wave's LDS traffic is complete and all but its newest N vector memory operations have landed; then the workgroup meets.
  // (Every LDS access is issued by hand: no fence beyond that.)
  auto meet = [&](auto nc) __attribute__((always_inline)) {
    constexpr int N = decltype(nc)::value;
    static_assert(N < 16, "the low four bits of vmcnt");
    __builtin_amdgcn_s_waitcnt(0x0070 | N);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  typedef std::integral_constant<int, (NSTG < NBLK ? NSTG : NBLK) * C::STEP_INSTR> IN;   // the next steps may stay in flight

  // lane addresses inside a stage of this wave's ring / inside the owned rows
  uint32_t xr[KK], xt[DB][2], ur[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    xr[kk] = w.ra[kk] + wave * C::WAVE_RING;
    ur[kk] = w.ra[kk] + C::OWN_RING + rg * 32 * ROW;
  }
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int u = 0; u < 2; ++u) xt[d][u] = w.ta[d][u] + wave * C::WAVE_RING;

  // Pair bias gradient of this wave's blocks: dS (rounded to bf16, as the contraction takes it) times the identity, summed in
  // fp32 on the matrix core, which is idle most of the time, while the vector ALU is not.
  f32x16 db[ROLE == 0 ? NBLK : 1];
  if constexpr (ROLE == 0)
#pragma unroll
    for (int t = 0; t < NBLK; ++t) db[t] = W::zero16();
  // A operands: the identity over rows 0 .. 15 and 16 .. 31 of a block (element e of half h is row 8 (e / 4) + 4 h + e % 4 of
  // the sixteen), and ones in contraction indices 0 .. 2, which adds the three bf16 parts of -delta to every dP.
  bf16x8 eye[2], ones;
  if constexpr (ROLE == 0) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      i32x4 v;
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        const int k0 = 16 * ks + 8 * (e2 >> 1) + 4 * w.half + 2 * (e2 & 1);
        v[e2] = w.col == k0 ? 0x3F80 : (w.col == k0 + 1 ? 0x3F800000 : 0);
      }
      eye[ks] = __builtin_bit_cast(bf16x8, v);
    }
    ones = __builtin_bit_cast(bf16x8, (i32x4){w.half == 0 ? 0x3F803F80 : 0, w.half == 0 ? 0x3F80 : 0, 0, 0});
  }
  // x as the sum of three bf16 values of eight bits each, cut and not rounded (rounded, the first could overflow), in contraction
  // indices 0 .. 2 of the B operand.  An infinity or NaN leaves NaN in the sum.
  auto three = [&](float x) __attribute__((always_inline)) -> bf16x8 {
    const uint32_t hi = __float_as_uint(x) & 0xFFFF0000u;
    const float r1 = x - __uint_as_float(hi);
    const uint32_t mid = __float_as_uint(r1) & 0xFFFF0000u;
    const uint32_t lo = __float_as_uint(r1 - __uint_as_float(mid)) >> 16;
    const bool on = w.half == 0;
    return __builtin_bit_cast(bf16x8, (i32x4){on ? (int)((hi >> 16) | mid) : 0, on ? (int)lo : 0, 0, 0});
  };

  // ---- hand-over at the end of a problem: register quad o of every channel block goes to wave o of the row group
  f32x16 acc[C::NACC][DB];                         // [0]: X^T dS (dQ or dK); [1], role 1: dO^T P (dV)
  float ksum = 0.f;
  const uint32_t xch_w = C::XCH + rg * 16384 + kq * 1024 + lane * 16, xch_r = C::XCH + rg * 16384 + kq * 4096 + lane * 16;
  // channel block x of the NX to hand over: dV's first, then dQ's or dK's.  par: the problem's parity (XTWICE)
  auto put = [&](auto xc, uint32_t par) __attribute__((always_inline)) {
    constexpr int x = decltype(xc)::value, N = C::NACC - 1 - x / DB, d = x % DB, SPACE = C::NSPACE > 1 ? x : 0;
    static_for<0, 4>([&](auto oc) __attribute__((always_inline)) {
      constexpr int o = decltype(oc)::value;
      const f32x16& a = acc[N][d];
      W::template write_b128<SPACE * C::XBLK + o * 4096>(
          xch_w + (C::XTWICE ? par * C::XBLK : 0), (i32x4){__float_as_int(a[4 * o]), __float_as_int(a[4 * o + 1]), __float_as_int(a[4 * o + 2]), __float_as_int(a[4 * o + 3])});
    });
  };
  // this lane's first channel of the next problem to store, in each output
  const View& ov0 = ROLE == 0 ? p.dq : p.dk;
  const int of0 = ROLE == 0 ? p.dq_f32 : p.dk_f32;
  unsigned char* optr[C::NACC];
  auto out_first = [&](const View& v, int f32) __attribute__((always_inline)) {
    const int64_t e = b * v.sb + g_lo * v.sg + h * v.sh + (int64_t)own * v.ss + 8 * kq + 4 * w.half;
    return (unsigned char*)v.ptr + e * (f32 ? 4 : 2);
  };
  optr[0] = out_first(ov0, of0);
  if constexpr (ROLE == 1) optr[1] = out_first(p.dv, p.dv_f32);
  auto take = [&](auto xc, uint32_t par) __attribute__((always_inline)) {
    constexpr int x = decltype(xc)::value, N = C::NACC - 1 - x / DB, d = x % DB, SPACE = C::NSPACE > 1 ? x : 0;
    i32x4 v[4];
    static_for<0, 4>([&](auto uc) __attribute__((always_inline)) {
      W::template read_b128<SPACE * C::XBLK + decltype(uc)::value * 1024>(v[decltype(uc)::value], xch_r + (C::XTWICE ? par * C::XBLK : 0));
    });
    W::template wait_lds<0>();
    const View& ov = N == 0 ? ov0 : p.dv;
    const int f32 = N == 0 ? of0 : p.dv_f32;
    const float scale = N == 0 ? p.scale : 1.f;
    float y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      y[e] = (((__int_as_float(v[0][e]) + __int_as_float(v[1][e])) + __int_as_float(v[2][e])) + __int_as_float(v[3][e])) * scale;
    if (own < S_own) {
      if (f32) *(float4*)(optr[N] + 128 * d) = make_float4(y[0], y[1], y[2], y[3]);
      else *(uint2*)(optr[N] + 64 * d) = make_uint2(pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3]));
    }
    if constexpr (d == DB - 1) optr[N] += ov.sg * (f32 ? 4 : 2);
  };
  // The end of a problem.  Its last blocks stay in the space(s) until the next problem's first step (take_all).
  auto put_all = [&](uint32_t par) __attribute__((always_inline)) {
    // The hand-written LDS stores below read matrix results.  Nothing interlocks that, and the compiler, which otherwise keeps the
    // distance (19 wait states after a 16-pass instruction), does not look into asm statements: keep it here.
#pragma unroll
    for (int N = 0; N < C::NACC; ++N)
#pragma unroll
      for (int d = 0; d < DB; ++d) asm volatile("" : "+v"(acc[N][d]));
    asm volatile("s_nop 15\n\ts_nop 7" : "+v"(acc[0][DB - 1]));
    if constexpr (!C::XTWICE) meet(IN());          // everyone has taken the previous problem's
    static_for<0, C::NX>([&](auto xc) __attribute__((always_inline)) {
      constexpr int x = decltype(xc)::value;
      if constexpr (C::NSPACE == 1 && x > 0) {
        meet(IN());
        take(std::integral_constant<int, x - 1>(), par);
        meet(IN());
      }
      put(xc, par);
    });
    if constexpr (ROLE == 1 && C::KEYB) write_b32(C::XSUM + wave * 256 + lane * 4, half_swap_sum(ksum));
    meet(IN());
  };
  auto take_all = [&](int g, uint32_t par) __attribute__((always_inline)) {
    static_for<C::NX - C::NSPACE, C::NX>([&](auto xc) __attribute__((always_inline)) { take(xc, par); });
    if constexpr (ROLE == 1 && C::KEYB) {
      if (kq == 0 && pp.key_part != nullptr) {     // uniform
        float v[4];
        static_for<0, 4>([&](auto qc) __attribute__((always_inline)) {
          read_b32<decltype(qc)::value * 512>(v[decltype(qc)::value], C::XSUM + rg * 256 + lane * 4);
        });
        W::template wait_lds<0>();
        if (w.half == 0 && own < S_own) pp.key_part[((int64_t)(b * p.G + g) * p.H + h) * p.Sk + own] = ((v[0] + v[1]) + v[2]) + v[3];
      }
    }
  };

  // ---- prologue: the first problem's owned rows, the first NSTG steps
  int ig = g_lo, io = g_lo;                        // problems that the next loads take (past the end: the last one again)
  auto next_load = [&](auto tc, uint32_t base) __attribute__((always_inline)) {
    load_step(tc, base);
    if constexpr (decltype(tc)::value == NBLK - 1) {
      if (ig + 1 < g_hi) {
        ++ig;
        xg += xv.sg * 2;
        yg += yv.sg * 2;
        if constexpr (ROLE == 1) sg += stat_step * 4;
      }
    }
  };
  auto next_own = [&](int slot) __attribute__((always_inline)) {
    load_own(slot);
    if (io + 1 < g_hi) {
      ++io;
      ug += uv.sg * 2;
      vg += vv.sg * 2;
      if constexpr (ROLE == 0) sg += stat_step * 4;
      if constexpr (C::KEYB) kg += pp.key_sg * 4;
    }
  };
  next_own(0);
  static_for<0, NSTG>([&](auto sc) __attribute__((always_inline)) {
    next_load(std::integral_constant<int, decltype(sc)::value % NBLK>(), decltype(sc)::value * C::STEP);
  });
  meet(std::integral_constant<int, 0>());

  uint32_t base = 0;                               // the current step's stage
#pragma nounroll
  for (int n = 0; n < n_prob; ++n) {
    const int g = g_lo + n;
    const uint32_t par = n & 1, ob = par * C::OWN;
    bf16x8 uf[C::OWN_REGS ? KK : 1], vf[C::OWN_REGS ? KK : 1];         // the owned rows as B operands
    bf16x8 d3;                                     // role 0: -delta of this lane's row
    float st0 = 0.f;                               // role 0: lse2 of this lane's row; 1: the bias of its key
    static_for<0, NBLK>([&](auto tc) __attribute__((always_inline)) {
      constexpr int t = decltype(tc)::value;
      if constexpr (t == 0) {
        next_own((n + 1) & 1);
        i32x4 fr[C::OWN_REGS ? 2 * KK : 1];
        if constexpr (C::OWN_REGS)
          static_for<0, KK>([&](auto kc) __attribute__((always_inline)) {
            constexpr int kk = decltype(kc)::value;
            W::template read_b128<0>(fr[kk], ur[kk] + ob);
            W::template read_b128<C::OWN_TILE>(fr[KK + kk], ur[kk] + ob);
          });
        float st1 = 0.f;
        const uint32_t sa = C::OWN_RING + ob + (32 * rg + w.col) * 4;
        if constexpr (ROLE == 0) {
          read_b32<C::OWN_STAT>(st0, sa);
          read_b32<C::OWN_STAT + 256>(st1, sa);
        } else if constexpr (C::KEYB) {
          read_b32<C::OWN_KEY>(st0, sa);
        }
        W::template wait_lds<0>();
        if constexpr (C::OWN_REGS)
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) {
            uf[kk] = __builtin_bit_cast(bf16x8, fr[kk]);
            vf[kk] = __builtin_bit_cast(bf16x8, fr[KK + kk]);
          }
        if constexpr (ROLE == 0) d3 = three(st1);
        ksum = 0.f;
        if (n > 0) take_all(g - 1, par ^ 1);
      }
      wait_vm<(NSTG - 1) * C::STEP_INSTR>();       // the step's tiles have landed
      asm volatile("" ::: "memory");
      {
        i32x4 ql[4], qd[4], fx[C::OWN_REGS ? 2 * KK : 1];
        const uint32_t stat_a = wave * C::WAVE_RING + base + w.half * 16;
        if constexpr (ROLE == 1)                   // the rows' -delta
          static_for<0, 4>([&](auto qc) __attribute__((always_inline)) {
            W::template read_b128<C::STEP_STAT + 128 + decltype(qc)::value * 32>(qd[decltype(qc)::value], stat_a);
          });
        // role 1: the rows' lse2; 0: the keys' biases.  Behind the matrix work: there is no room for them beside its operands
        auto read_terms = [&]() __attribute__((always_inline)) {
          __builtin_amdgcn_sched_barrier(0);
          const uint32_t key_a = C::OWN_RING + ob + (32 * kq + 4 * w.half) * 4;
          static_for<0, 4>([&](auto qc) __attribute__((always_inline)) {
            constexpr int q = decltype(qc)::value;
            if constexpr (ROLE == 1) W::template read_b128<C::STEP_STAT + q * 32>(ql[q], stat_a);
            else if constexpr (C::KEYB) W::template read_b128<C::OWN_KEY + t * 512 + q * 32>(ql[q], key_a);
          });
        };
        f32x16 sc = W::zero16(), dp = W::zero16();
        auto start = [&]() __attribute__((always_inline)) {             // behind the wait that covers qd: dp starts at -delta
          if constexpr (ROLE == 1) {
#pragma unroll
            for (int r = 0; r < 16; ++r) dp[r] = __int_as_float(qd[r >> 2][r & 3]);
          } else {
            asm volatile("" : "+v"(ones));         // (formed anew for every block: a copy of sixteen registers costs more)
            dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, d3, dp, 0, 0, 0);
          }
        };
        // fragments of X^T (and, role 1, Y^T first), rows 0 .. 15 of the block, then 16 .. 31
        constexpr int DY = ROLE == 1 ? DB : 0, NT = DB + DY;
        typedef TrQuad<C::STEP_TILE, 0, DY, DB, ROW, ROW> TrOff;
        i32x2 tlo[2 * NT], thi[2 * NT];
        auto read_transposed = [&]() __attribute__((always_inline)) {
          static_for<0, 2 * NT>([&](auto fc) __attribute__((always_inline)) {
            constexpr int f = decltype(fc)::value;
            W::template read_tr<TrOff::off(f)>(tlo[f], xt[f % NT % DB][0] + base);
            W::template read_tr<TrOff::off(f)>(thi[f], xt[f % NT % DB][1] + base);
          });
        };
        if constexpr (C::OWN_REGS) {
          static_for<0, 2 * KK>([&](auto fc) __attribute__((always_inline)) {
            constexpr int f = decltype(fc)::value;
            W::template read_b128<f < KK ? 0 : C::STEP_TILE>(fx[f], xr[f % KK] + base);
          });
          W::template wait_lds<0>();
          read_transposed();
          start();
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fx[kk]), uf[kk], sc, 0, 0, 0);
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fx[KK + kk]), vf[kk], dp, 0, 0, 0);
        } else {
          bf16x8 u;
          w.template row_stream_g<OwnPair<0, C::OWN_TILE, 0, C::STEP_TILE, KK>, 4 * KK, 4>(
              [&](auto fc) __attribute__((always_inline)) {
                constexpr int f = decltype(fc)::value;
                if constexpr (f % 2 == 0) return ur[f / 2 % KK] + ob;
                else return xr[f / 2 % KK] + base;
              },
              [&](auto fc, bf16x8 a) __attribute__((always_inline)) {
                constexpr int f = decltype(fc)::value;
                if constexpr (f == 0) start();
                if constexpr (f % 2 == 0) u = a;
                else if constexpr (f / 2 < KK) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, u, sc, 0, 0, 0);
                else dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, u, dp, 0, 0, 0);
              });
          read_transposed();
        }
        read_terms();
        W::template wait_lds<0>();                 // every fragment is in registers: the stage takes the step NSTG ahead
        next_load(std::integral_constant<int, (t + NSTG) % NBLK>(), base);
        if constexpr (NSTG > 1) base = base == (NSTG - 1) * C::STEP ? 0 : base + C::STEP;
        uint32_t pw[8], dsw[8];
#pragma unroll
        for (int r2 = 0; r2 < 8; ++r2) {
          float pv[2], ds[2];
          // (opaque: the compiler would unpack all of them in front of the loop over the problems and run out of registers.  The unpacking
          // itself is left to it: it does not see what asm statements need behind matrix instructions)
          if constexpr (!C::BIAS_F32) asm volatile("" : "+v"(blp[C::BIAS_F32 ? 0 : t][r2]));
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int r = 2 * r2 + e;
            float bl;
            if constexpr (C::BIAS_F32) bl = blf[C::BIAS_F32 ? t : 0][r];
            else bl = __uint_as_float(e ? (blp[C::BIAS_F32 ? 0 : t][r2] & 0xFFFF0000u) : (blp[C::BIAS_F32 ? 0 : t][r2] << 16));
            const float st_r = ROLE == 1 || C::KEYB ? __int_as_float(ql[r >> 2][r & 3]) : 0.f;
            if constexpr (C::KEYB) bl += ROLE == 0 ? st_r : st0;
            if constexpr (C::KEYB || !C::BIAS_F32) bl = bias_log2(bl);
            pv[e] = fast_exp2(biased_exponent(fmaf(sc[r], c_scale, ROLE == 0 ? -st0 : -st_r), bl));
            ds[e] = pv[e] * dp[r];
            if constexpr (ROLE == 1 && C::KEYB) ksum += ds[e];
          }
          if constexpr (ROLE == 1) pw[r2] = pack_bf16(pv[0], pv[1]);
          dsw[r2] = pack_bf16(ds[0], ds[1]);
        }
        static_for<0, 2 * NT>([&](auto fc) __attribute__((always_inline)) {
          constexpr int f = decltype(fc)::value, ks = f / NT, d = f % NT % DB;
          const bf16x8 a = __builtin_bit_cast(bf16x8, (i32x4){tlo[f][0], tlo[f][1], thi[f][0], thi[f][1]});
          if constexpr (f % NT < DY) {
            const bf16x8 bop = __builtin_bit_cast(
                bf16x8, (i32x4){(int)pw[4 * ks], (int)pw[4 * ks + 1], (int)pw[4 * ks + 2], (int)pw[4 * ks + 3]});
            acc[C::NACC - 1][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bop, t == 0 && ks == 0 ? W::zero16() : acc[C::NACC - 1][d], 0, 0, 0);
          } else {
            const bf16x8 bop = __builtin_bit_cast(
                bf16x8, (i32x4){(int)dsw[4 * ks], (int)dsw[4 * ks + 1], (int)dsw[4 * ks + 2], (int)dsw[4 * ks + 3]});
            acc[0][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bop, t == 0 && ks == 0 ? W::zero16() : acc[0][d], 0, 0, 0);
            if constexpr (ROLE == 0 && d == 0)
              db[ROLE == 0 ? t : 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(eye[ks], bop, db[ROLE == 0 ? t : 0], 0, 0, 0);
          }
        });
      }
    });
    // (the next problem's owned rows were requested before this problem's NBLK steps of loads: they have landed too)
    put_all(par);
  }
  take_all(g_hi - 1, (n_prob - 1) & 1);
  __builtin_amdgcn_s_waitcnt(0x0070);              // nothing of the rings is in flight when the workgroup ends

  if constexpr (ROLE == 0) {
    if (pp.bias_part != nullptr) {
      const int nqb = (p.Sq + 31) / 32, nkb = (p.Sk + 31) / 32, qb = 2 * ot + rg;
#pragma unroll
      for (int t = 0; t < NBLK; ++t) {
        const int kb2 = 4 * t + kq;
        if (qb < nqb && kb2 < nkb) {               // uniform
          float* dst = pp.bias_part + (((((int64_t)chunk * p.B + b) * p.H + h) * nqb + qb) * nkb + kb2) * 1024 + lane * 4;
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4)
            *(float4*)(dst + q4 * 256) = make_float4(db[t][4 * q4], db[t][4 * q4 + 1], db[t][4 * q4 + 2], db[t][4 * q4 + 3]);
        }
      }
    }
  }
}

}  // namespace fl
