// Launch of the stationary-bias backward kernels by head dim, steps per problem, role and key bias.
#pragma once
#include "fl_bwd_pair.hpp"
#include "fl_bwd_registry.hpp"

namespace fl {

template <class C>
hipError_t launch_pair(const PairParams& p, int nblocks, hipStream_t stream) {
  static_assert(C::LDS <= kMaxLdsBytes, "rings exceed the LDS of a compute unit");
  hipError_t e = raise_lds_limit(bwd_pair_kernel<C>);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(bwd_pair_kernel<C>, dim3(nblocks), dim3(512), C::LDS, stream, p);
  return hipGetLastError();
}

template <int D, int NBLK>
hipError_t launch_pair_steps(int role, bool keyb, const PairParams& p, int nblocks, hipStream_t stream) {
  if (role == 0) return keyb ? launch_pair<PairCfg<D, NBLK, 0, true>>(p, nblocks, stream) : launch_pair<PairCfg<D, NBLK, 0, false>>(p, nblocks, stream);
  return keyb ? launch_pair<PairCfg<D, NBLK, 1, true>>(p, nblocks, stream) : launch_pair<PairCfg<D, NBLK, 1, false>>(p, nblocks, stream);
}

template <int D>
hipError_t launch_pair_any(int nblk, int role, bool keyb, const PairParams& p, int nblocks, hipStream_t stream) {
  switch (nblk) {
    case 1: return launch_pair_steps<D, 1>(role, keyb, p, nblocks, stream);
    case 2: return launch_pair_steps<D, 2>(role, keyb, p, nblocks, stream);
  }
  if constexpr (D == 32) {
    if (nblk == 3) return launch_pair_steps<D, 3>(role, keyb, p, nblocks, stream);
    if (nblk == 4) return launch_pair_steps<D, 4>(role, keyb, p, nblocks, stream);
  } else if (nblk == 3 && !keyb) {
    return role == 0 ? launch_pair<PairCfg<D, 3, 0, false>>(p, nblocks, stream) : launch_pair<PairCfg<D, 3, 1, false>>(p, nblocks, stream);
  }
  return hipErrorInvalidValue;
}

// role 0: dQ and bias_part; 1: dK, dV and key_part.  nblk: ceil(streamed rows / 128): 1 .. 4 at head dim 32, 1 .. 3 (with a key bias
// 1 .. 2) at 64.
hipError_t launch_pair32(int nblk, int role, bool keyb, const PairParams& p, int nblocks, hipStream_t stream);
hipError_t launch_pair64(int nblk, int role, bool keyb, const PairParams& p, int nblocks, hipStream_t stream);

}  // namespace fl
