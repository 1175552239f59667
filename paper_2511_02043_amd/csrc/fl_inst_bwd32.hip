// Backward kernels of head dim 32 (Evoformer) and of D = 64 with Dv = 128 (differential attention, whose values are twice
// as wide as a stream's queries and keys).  Variants outside this table run at the next head dim of the other tables, on
// zero-padded copies of their tensors.  Measured against those copies: Evoformer rows (128 x 8 heads x 384, one bias, gate)
// dQ 218 -> 200 us (143 since), dK / dV 185 -> 147 us and 106 us of copies less; differential training (2 x 16 heads, 4096 rows) dQ
// 256 -> 191 us and dK / dV 366 -> 337 us per stream, 143 us of copies less.
#include "fl_bwd_registry.hpp"
namespace fl {
static const BwdEntry kEntries[] = {
    bwd_entry<32, kModNone, 0, 64, 4, 64, 3, false>(), bwd_entry<32, kModNone, kMaskCausal, 64, 4, 64, 3, false>(),
    bwd_entry<32, kModNone, 0, 64, 4, 64, 2, false, 1>(), bwd_entry<32, kModNone, 0, 64, 3, 64, 2, false, 2>(),
    // two specialised waves per SIMD: a wave's matrix work per 32 rows is 4 + 8 instructions in either role (scores and dV,
    // dP and dK)
    bwd_entry<64, kModNone, 0, 64, 3, 64, 2, true, 0, 128>(), bwd_entry<64, kModNone, kMaskCausal, 64, 3, 64, 2, true, 0, 128>(),
};
const BwdEntry* entries_bwd32(int* n) {
  *n = (int)(sizeof(kEntries) / sizeof(kEntries[0]));
  return kEntries;
}
}  // namespace fl
