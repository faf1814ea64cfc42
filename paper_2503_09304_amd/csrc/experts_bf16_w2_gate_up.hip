// Instantiation of one bf16 expert kernel for one weight format (a translation unit of its own so
// that they compile in parallel).
#include "experts_bf16_tile.h"

namespace qmoe {
namespace bf16k {
template void launch_expert_kernel<WF_MXFP4, true>(int, bool, const BArgs &, hipStream_t);
}  // namespace bf16k
}  // namespace qmoe
