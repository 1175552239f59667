// Backward kernels of attention with a stationary pair bias, head dim 64: one to three steps of 128 streamed rows per problem, one
// or two with a key bias.
#include "fl_pair_registry.hpp"
namespace fl {
hipError_t launch_pair64(int nblk, int role, bool keyb, const PairParams& p, int nblocks, hipStream_t stream) {
  return launch_pair_any<64>(nblk, role, keyb, p, nblocks, stream);
}
}  // namespace fl
