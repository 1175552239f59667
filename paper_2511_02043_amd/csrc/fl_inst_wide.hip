// dK/dV kernels with 64 keys per wave.
#include "fl_bwd_wide.hpp"
#include "fl_bwd_registry.hpp"
namespace fl {

template <class C>
static hipError_t launch_wide(const BwdParams& p, int nblocks, hipStream_t stream) {
  hipError_t e = raise_lds_limit(bwd_dkdv_wide_kernel<C>);
  if (e != hipSuccess) return e;
  static_assert(WideCfg<C>::LDS <= kMaxLdsBytes, "LDS of the dK/dV kernel");
  hipLaunchKernelGGL(bwd_dkdv_wide_kernel<C>, dim3(nblocks), dim3(256), WideCfg<C>::LDS, stream, p);
  return hipGetLastError();
}
#define E(D, DV, MOD, MASK) {BwdKey{D, MOD, (int)(MASK), 0, DV}, WideCfg<BwdCfg<D, MOD, MASK, 64, 1, 0, DV>>::BM, &launch_wide<BwdCfg<D, MOD, MASK, 64, 1, 0, DV>>}
static const WideEntry kEntries[] = {
    E(128, 128, kModNone, 0), E(128, 128, kModNone, kMaskCausal), E(128, 128, kModNone, kMaskPrefix), E(128, 128, kModAlibi, 0),
    E(128, 128, kModSoftcap, 0), E(64, 128, kModNone, 0), E(64, 128, kModNone, kMaskCausal),
};
#undef E
const WideEntry* find_wide(const BwdKey& k) {
  for (const WideEntry& e : kEntries)
    if (e.key.D == k.D && e.key.Dv == k.Dv && e.key.mod == k.mod && e.key.mask == k.mask && e.key.nbias == k.nbias) return &e;
  return nullptr;
}
}  // namespace fl
