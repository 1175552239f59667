// fp32-storage kernels: variant switches are runtime values here, only the register budget for the head dim and the
// workgroup's shape (row groups x key splits) are compile-time.
#include "fl_registry.hpp"
#include "fl_kernel_f32.hpp"
namespace fl {
template <class C>
static hipError_t launch_f32(const FwdParams& call, int nblocks, hipStream_t stream) {
  FwdParams p = call;
  p.order_heads = 1;                               // (its tiles go out one problem after the other)
  p.tile_step = 0;
  set_divisors(p, 1);
  static std::atomic<bool> done[64];               // the dynamic-LDS limit is per device and sticky, as in launch_bf16
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64 || !done[dev].load(std::memory_order_acquire)) {
    e = hipFuncSetAttribute((const void*)fwd_f32_kernel<C>, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64) done[dev].store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(fwd_f32_kernel<C>, dim3(nblocks), dim3(C::NT), C::LDS, stream, p);
  return hipGetLastError();
}
template <int DMAX, int RB, int RG, int KS, bool PLAIN>
static constexpr KernelEntry entry() {
  typedef F32Cfg<DMAX, RB, RG, KS, PLAIN> C;
  static_assert(C::LDS <= kMaxLdsBytes, "LDS of a compute unit");
  return KernelEntry{KernelKey{2, DMAX, DMAX, PLAIN ? 0 : -1, -1, -1, -1, -1, RG * KS, KS, kF32Keys, 0, 0, 0, 1}, C::BM, C::LDS, &launch_f32<C>};
}
// Per head dim in the order of the key splits (find_entry takes the first one that fills the chip): <head dim, row blocks per wave, row groups,
// key splits, plain>.  Two row blocks where 256 registers hold them; at head dim 128 only where LDS leaves one wave per SIMD in any case
// (2 x 8 heads x 1024 rows: 63 us, 73 with one).  The variants keep one: their switches take the registers.
static const KernelEntry kEntries[] = {
    entry<32, 2, 8, 1, true>(), entry<32, 2, 4, 2, true>(), entry<32, 2, 2, 4, true>(), entry<32, 2, 1, 8, true>(), entry<32, 1, 1, 8, true>(),
    entry<64, 2, 8, 1, true>(), entry<64, 2, 4, 2, true>(), entry<64, 2, 2, 4, true>(), entry<64, 2, 1, 8, true>(), entry<64, 1, 1, 8, true>(),
    entry<128, 1, 8, 1, true>(), entry<128, 1, 4, 2, true>(), entry<128, 2, 1, 4, true>(), entry<128, 1, 1, 4, true>(),
    entry<32, 1, 8, 1, false>(), entry<32, 1, 4, 2, false>(), entry<32, 1, 2, 4, false>(), entry<32, 1, 1, 8, false>(),
    entry<64, 1, 8, 1, false>(), entry<64, 1, 4, 2, false>(), entry<64, 1, 2, 4, false>(), entry<64, 1, 1, 8, false>(),
    entry<128, 1, 8, 1, false>(), entry<128, 1, 4, 2, false>(), entry<128, 1, 1, 4, false>(),
};
const KernelEntry* entries_f32(int* n) {
  *n = (int)(sizeof(kEntries) / sizeof(kEntries[0]));
  return kEntries;
}
}  // namespace fl
