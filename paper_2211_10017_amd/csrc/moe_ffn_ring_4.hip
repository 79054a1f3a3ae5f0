// Grouped GEMM kernels with an LDS ring for 4-bit weights.  The forms that keep group scales out of the FP16 weights are one here:
// exact codes, sums folded once per group, for every group size (a multiple of the K step).
#include "moe_ffn_ring_kernel.h"

namespace moe {
void launch_ring_4(const GemmArgs &p, int smode, int bm, dim3 grid, hipStream_t s)
{
    if (smode == SCALE_CHANNEL) launch_ring_variants<4, SCALE_CHANNEL>(p, bm, grid, s);
    else if (smode == SCALE_CHANNEL_BF16) launch_ring_variants<4, SCALE_CHANNEL_BF16>(p, bm, grid, s);
    else if (smode == SCALE_GROUP) launch_ring_variants<4, SCALE_GROUP>(p, bm, grid, s);
    else launch_ring_variants<4, SCALE_GROUP_ACC>(p, bm, grid, s);
}
}  // namespace moe
