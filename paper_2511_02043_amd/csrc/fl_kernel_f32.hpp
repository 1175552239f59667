// fp32 attention-variant forward kernel: both contractions on the fp32 matrix instruction
// (v_mfma_f32_32x32x2_f32), fp32 scores, softmax state and accumulators.
//
// This is the fp32-storage specialisation of the fused pass; tanh, the logarithm and the gate use the
// accurate math-library routines, and the result is meant to stay within 1e-5 of an fp64 evaluation.
// Every variant feature is available here, as runtime switches.  It follows the same structure as the
// bf16 kernel: a workgroup owns a tile of query rows, walks the visible key tiles (skipper), keeps
// (m, l, O) in registers and never stores a score (Sec. 3.2 dimension demotion; Sec. 3.4 running max / sum
// with the exp(m_old - m_new) correction).
//
// Orientation as in the bf16 kernel: S^T = K Q^T with the query in the lane (lane % 32) and sixteen keys
// n(r) = 8 (r / 4) + 4 (lane / 32) + r % 4 in the registers, so a softmax row is two lanes, and register r
// of P is, as it stands, the B operand of the contraction step over the key pair n(r) of
// O^T += V^T P^T.  Both operands of a step may take the channels (or keys) in any common order: a lane
// reads K in 16-byte pieces (four steps per LDS read), and V^T row c of channel block d is channel
// DVB c + d, so that one LDS read of 4 DVB bytes feeds the DVB steps of a key pair.
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s; a 32x32x2 step takes 64 cycles of a SIMD, in which it
// issues sixteen other instructions).  It has to be kept supplied by every SIMD: a wave takes 32 query rows, and where the
// call has fewer than two such waves per SIMD the key tiles of a row group are dealt to KS waves, which merge through LDS by
// the rescale rule of Sec. 3.3.  K / V tiles of 32 keys go to LDS by direct loads.
// Measured, 2 x 8 heads, 1024 rows and keys, D = 64: 48 us, 89 TFLOP/s; the same pass on plain VALU arithmetic (four lanes per
// row, LDS broadcasts) took 508 us.  Large launches (8 x 16 heads, 2048 rows) run at 112 TFLOP/s: the softmax of the two
// waves of a SIMD falls between the same two barriers.
#pragma once
#include "fl_kernel_bf16.hpp"

namespace fl {

constexpr int kF32Keys = 32;     // keys per LDS tile (= kSumBlock)

template <int DMAX_, int RG_, int KS_>
struct F32Cfg {
  static constexpr int DMAX = DMAX_;               // head dims up to this one; smaller ones compute on channels that are zero in Q
  static constexpr int RG = RG_, KS = KS_;         // row groups (32 query rows each) and key splits of the workgroup
  static constexpr int NT = RG * KS * 64;
  static constexpr int BM = RG * 32;
  static constexpr int ROW = DMAX * 4;             // bytes of a tile row in LDS
  static constexpr int CH = DMAX / 4;              // 16-byte chunks of a tile row
  static constexpr int TILE = kF32Keys * ROW;
  static constexpr int STAGE = 2 * TILE;           // K, V
  static constexpr int NBUF = RG == 1 ? 1 : 2;     // buffers per key split (see the loops)
  static constexpr int RING = KS * NBUF * STAGE;   // [key split][buffer][K, V]
  static constexpr int DVB = DMAX / 32;            // 32-channel blocks of the output
  static constexpr int NINSTR = TILE / 1024;       // direct-load instructions per tile
  static constexpr int OBYTES = DVB * 16 * 64 * 4; // one wave's accumulators
  static constexpr int MERGE = RG * (KS - 1) * (OBYTES + 2 * 64 * 4);
  static constexpr int LDS = RING > MERGE ? RING : MERGE;
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

template <class C>
__global__ void __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2)))
fwd_f32_kernel(const FwdParams p) {
  constexpr int DMAX = C::DMAX, RG = C::RG, KS = C::KS, DVB = C::DVB, ROW = C::ROW, NU = DMAX / 8;
  const int MOD = p.mod, NBIAS = p.n_bias;
  const uint32_t MASK = p.mask, EPI = p.epi;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];

  const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rg = wave % RG, ks = wave / RG;        // this wave's row group and key split

  // grid decode: whole (b, g, h) problems per XCD where their number allows it, longest causal tiles first
  const int nq = p.n_qtiles;
  int qt, bh;
  if (p.order == 1) {
    const int idx = blockIdx.x >> 3;
    bh = (idx / nq) * 8 + (blockIdx.x & 7);
    qt = nq - 1 - idx % nq;
  } else {
    bh = blockIdx.x / nq;
    qt = nq - 1 - (int)(blockIdx.x % nq);
  }
  const int h = bh % p.H, g = (bh / p.H) % p.G, b = bh / (p.H * p.G);
  const int hk = h / (p.H / p.Hkv);
  const int i0 = qt * C::BM, iw = i0 + 32 * rg;    // first query row of the workgroup / of the wave
  const int i = iw + col, ic = i < p.Sq ? i : p.Sq - 1;
  const int ns = p.diff ? 2 : 1;                   // softmax streams, one after the other

  const int qdoc = (MASK & kMaskDoc) ? p.q_doc[(int64_t)b * p.Sq + ic] : 0;
  const float slope = MOD == kModAlibi ? p.alibi_slopes[h] : 0.f;

  // ---- visible key range of the workgroup (positional masks, rows by their positions); document summaries of its rows
  const int i_max = min(i0 + C::BM, p.Sq) - 1, iw_max = min(iw + 32, p.Sq) - 1;
  int k_lo, k_hi;
  key_range(MASK, i0 + p.q_off, i_max + p.q_off, p.Sk, p.window, p.prefix, k_lo, k_hi);
  const int t_lo = k_lo / kF32Keys, t_hi = (k_hi + kF32Keys - 1) / kF32Keys;
  const int n_iter = t_hi > t_lo ? (t_hi - t_lo + KS - 1) / KS : 0;   // the same for every wave: they meet at barriers
  int2 qs_wg = make_int2(0, 0), qs_w = qs_wg;
  const int nks = (p.Sk + kSumBlock - 1) / kSumBlock;
  if ((MASK & kMaskDoc) != 0) {
    const int nqs = (p.Sq + kSumBlock - 1) / kSumBlock;
    const int2* s = p.q_sum + (int64_t)b * nqs;
    qs_wg = s[min(i0 / kSumBlock, nqs - 1)];
    for (int u = 1; u < RG; ++u) {
      const int2 x = s[min(i0 / kSumBlock + u, nqs - 1)];
      qs_wg.x = min(qs_wg.x, x.x);
      qs_wg.y = max(qs_wg.y, x.y);
    }
    qs_w = s[min(iw / kSumBlock, nqs - 1)];
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
    float4 qf[NU];                                 // B fragments of S^T = K Q^T; channels past D are zero
    {
      int ql = lane;                               // (opaque, as in the epilogue below)
      asm volatile("" : "+v"(ql));
      const float* qp = (const float*)qv.ptr + b * qv.sb + g * qv.sg + h * qv.sh + (int64_t)min(iw + (ql & 31), p.Sq - 1) * qv.ss;
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int c = 8 * u + 4 * (ql >> 5);
        qf[u] = c < p.D ? *(const float4*)(qp + c) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    f32x16 o[DVB];
#pragma unroll
    for (int d = 0; d < DVB; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
    float m = -INFINITY, l = 0.f;                  // log2-domain running max; this lane's part of the running sum

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

    // one tile: scores, softmax update, P V.  before_softmax() runs when the K tile has been read, before_pv() before V is.
    auto tile = [&](int t, int cls, uint32_t buf, auto&& before_softmax, auto&& before_pv) __attribute__((always_inline)) {
      // S^T = K Q^T: one LDS read per four steps, four reads ahead
      f32x16 sc;
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[r] = 0.f;
      {
        constexpr int G = 4 < NU ? 4 : NU, NG = NU / G;
        F32Vec<4>::type kf[NU];
        auto read = [&](auto uc) __attribute__((always_inline)) {
          constexpr int u = decltype(uc)::value;
          F32Vec<4>::template read<0>(kf[u], (ka ^ (uint32_t)(u << 5)) + buf);
        };
        static_for<0, G>(read);
        static_for<0, NG>([&](auto gc) __attribute__((always_inline)) {
          constexpr int gg = decltype(gc)::value;
          if constexpr (gg + 1 < NG) static_for<(gg + 1) * G, (gg + 2) * G>(read);
          f32_wait_lds<gg + 1 < NG ? G : 0>();
          static_for<gg * G, (gg + 1) * G>([&](auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value;
            sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u][0], qf[u].x, sc, 0, 0, 0);
            sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u][1], qf[u].y, sc, 0, 0, 0);
            sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u][2], qf[u].z, sc, 0, 0, 0);
            sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u][3], qf[u].w, sc, 0, 0, 0);
          });
        });
      }

      before_softmax();
      // variant transform (Eq. 3, Eq. 4, biases, masks); register r holds key jl + 8 (r / 4) + r % 4
      const int jl = t * kF32Keys + 4 * half;
      auto key = [&](int r) __attribute__((always_inline)) { return jl + 8 * (r >> 2) + (r & 3); };
      const bool plain = MOD == kModNone && NBIAS == 0;   // then scale and log2(e) are one factor
      const float f1 = plain ? p.scale * kLog2e : p.scale;
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[r] *= f1;
      if (MOD == kModSoftcap) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = p.softcap * tanhf(sc[r] / p.softcap);
      }
      if (MOD == kModAlibi) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] -= slope * fabsf((float)(i + p.q_off - key(r)));
      }
      for (int nb = 0; nb < NBIAS; ++nb) {
        const BiasView& bv = p.bias[nb];
        int bl = ic;
        asm volatile("" : "+v"(bl));
        const int64_t row = b * bv.sb + g * bv.sg + h * bv.sh + (int64_t)bl * bv.si;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int64_t off = row + (int64_t)min(key(r), p.Sk - 1) * bv.sj;
          sc[r] += bv.is_f32 ? ((const float*)bv.ptr)[off] : bf16_to_f32(((const uint16_t*)bv.ptr)[off]);
        }
      }
      if (cls == kPartial) {                       // the positional masks and the end of the keys as two bounds on the key
        const int ip = i + p.q_off;
        int last = p.Sk - 1, first = 0;
        if ((MASK & kMaskPrefix) != 0) last = min(last, max(ip, p.prefix - 1));
        else if ((MASK & (kMaskCausal | kMaskWindow)) != 0) last = min(last, ip);
        if ((MASK & kMaskWindow) != 0) first = ip - p.window;
        const int d_hi = last - jl, d_lo = first - jl;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int c = 8 * (r >> 2) + (r & 3);
          sc[r] = (c > d_hi) | (c < d_lo) ? -INFINITY : sc[r];
        }
        if ((MASK & kMaskDoc) != 0) {
          const int32_t* kdoc = p.kv_doc + (int64_t)b * p.Sk;
#pragma unroll
          for (int r = 0; r < 16; ++r) sc[r] = kdoc[min(key(r), p.Sk - 1)] != qdoc ? -INFINITY : sc[r];
        }
      }

      // online softmax update with the tile (Alg. 2), log2 domain
      if (!plain) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] *= kLog2e;
      }
      float mx = m;
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[r]);
      mx = half_swap_max(mx);
      const float ms = mx == -INFINITY ? 0.f : mx;
      if (__builtin_amdgcn_ballot_w64(mx != m) != 0) {     // uniform: some row's maximum moved
        const float alpha = fast_exp2(m - ms);
        l *= alpha;
        m = mx;
#pragma unroll
        for (int d = 0; d < DVB; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
      }
      float psum = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sc[r] = fast_exp2(sc[r] - ms);             // (v_exp_f32: 1 ulp; results below 2^-126 are zero beside a row sum of at least 1)
        psum += sc[r];
      }
      l += psum;

      before_pv();
      // O^T += V^T P^T: one LDS read per key pair, four ahead
      {
        typename F32Vec<DVB>::type vf[16];
        const uint32_t a = va + buf;
        auto read = [&](auto rc) __attribute__((always_inline)) {
          constexpr int r = decltype(rc)::value, OFF = (8 * (r >> 2) + (r & 3)) * ROW;
          F32Vec<DVB>::template read<OFF>(vf[r], a);
        };
        static_for<0, 4>(read);
        static_for<0, 4>([&](auto gc) __attribute__((always_inline)) {
          constexpr int gg = decltype(gc)::value;
          if constexpr (gg + 1 < 4) static_for<(gg + 1) * 4, (gg + 2) * 4>(read);
          f32_wait_lds<gg + 1 < 4 ? 4 : 0>();
          static_for<gg * 4, gg * 4 + 4>([&](auto rc) __attribute__((always_inline)) {
            constexpr int r = decltype(rc)::value;
#pragma unroll
            for (int d = 0; d < DVB; ++d) o[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(F32Vec<DVB>::at(vf[r], d), sc[r], o[d], 0, 0, 0);
          });
        });
      }
    };

    if (s > 0) __syncthreads();                    // LDS is reused by the second stream
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
             });
        if (tn < t_hi) load_v(tn, 0);
        t = tn;
      }
    } else {
      if (wanted(t_lo + ks)) {
        load_k(t_lo + ks, 0);
        load_v(t_lo + ks, 0);
      }
      for (int it = 0; it < n_iter; ++it) {
        const int t = t_lo + it * KS + ks;
        f32_wait_mem<0>();                         // this wave's loads of tile t have landed ...
        clear_k(t, it & 1);
        clear_v(t, it & 1);
        f32_wait_lds<0>();
        __syncthreads();                           // ... and everyone's; the other buffer is free
        if (it + 1 < n_iter && wanted(t + KS)) {
          load_k(t + KS, (it + 1) & 1);
          load_v(t + KS, (it + 1) & 1);
        }
        if (t >= t_hi) continue;
        const int cls = iw < p.Sq ? classify(t, iw, iw_max, qs_w, tile_ids(t)) : kSkip;
        if (cls == kSkip) continue;                // (uniform over the wave)
        tile(t, cls, (uint32_t)((it & 1) * C::STAGE), []() __attribute__((always_inline)) {}, []() __attribute__((always_inline)) {});
      }
    }

    // ---- the splits of a row group merge in split 0 (rescale rule of Sec. 3.3), in the order of the splits
    l = half_swap_sum(l);
    if constexpr (KS > 1) {
      __syncthreads();                             // the tile ring is free
      float* mo = (float*)(lds_raw + (rg * (KS - 1) + ks - 1) * C::OBYTES) + lane * 4;
      float* ml = (float*)(lds_raw + RG * (KS - 1) * C::OBYTES) + (rg * (KS - 1) + ks - 1) * 128 + lane;
      if (ks > 0) {
#pragma unroll
        for (int d = 0; d < DVB; ++d)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4)
            *(float4*)(mo + (d * 4 + r4) * 256) = make_float4(o[d][4 * r4], o[d][4 * r4 + 1], o[d][4 * r4 + 2], o[d][4 * r4 + 3]);
        ml[0] = m;
        ml[64] = l;
      }
      __syncthreads();
      if (ks == 0) {
        float f[KS], mall = m;
#pragma unroll
        for (int u = 1; u < KS; ++u) mall = fmaxf(mall, ml[u * 128]);
        const float ms = mall == -INFINITY ? 0.f : mall;
        f[0] = fast_exp2(m - ms);
        float lt = l * f[0];
#pragma unroll
        for (int u = 1; u < KS; ++u) {
          f[u] = fast_exp2(ml[u * 128] - ms);
          lt += ml[u * 128 + 64] * f[u];
        }
        m = mall;
        l = lt;
#pragma unroll
        for (int d = 0; d < DVB; ++d)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[d][4 * r4 + e] *= f[0];
#pragma unroll
            for (int u = 1; u < KS; ++u) {
              const float4 x = *(const float4*)(mo + u * (C::OBYTES / 4) + (d * 4 + r4) * 256);
              o[d][4 * r4] += x.x * f[u];
              o[d][4 * r4 + 1] += x.y * f[u];
              o[d][4 * r4 + 2] += x.z * f[u];
              o[d][4 * r4 + 3] += x.w * f[u];
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
    const int er = iw + (el & 31), eh = el >> 5;
    if (ks == 0 && er < p.Sq) {
      const float inv = l > 0.f ? 1.f / l : 0.f;
      float* op = (float*)p.out.ptr + b * p.out.sb + g * p.out.sg + h * p.out.sh + (int64_t)er * p.out.ss;
      if (p.lse != nullptr && eh == 0)
        p.lse[b * p.lse_sb + (int64_t)(ns * g + s) * p.lse_sg + h * p.lse_sh + er] = l > 0.f ? m * kLn2 + logf(l) : -INFINITY;
      const float lam = s == 1 ? p.lambda[h] : 0.f;
      const bool last = s + 1 == ns;
      float ssq = 0.f;
      // register group r4 holds 4 DVB consecutive channels, in DVB pieces of four; element e of piece e4 sits in ...
      auto chan = [&](int r4, int e4) __attribute__((always_inline)) { return DVB * (8 * r4 + 4 * eh) + 4 * e4; };
      auto at = [&](int r4, int e4, int e) __attribute__((always_inline)) -> float { return o[(4 * e4 + e) % DVB][4 * r4 + (4 * e4 + e) / DVB]; };
#pragma unroll
      for (int d = 0; d < DVB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] *= inv;
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
              o[d][r] = f4[e] - lam * o[d][r];
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
