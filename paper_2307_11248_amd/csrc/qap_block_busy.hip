// qap_block_busy.hip -- block form of the searches: the kernels held to 64 VGPRs (n up to
// 128), for launches of more searches than compute units: two and more searches share one and
// fill each other's waits (us per iteration and compute unit at n = 96 1.30 and 0.96, n = 128
// symmetric 1.48 and 1.13), where one search alone is 9 % slower for the operands it cannot
// hold.  Above n = 128 the accumulators leave no such budget.
#include "qap_block.h"

namespace qapk {

hipError_t launch_block_busy(bool tabu, int form, const SearchArgs &a, const BatchArgs &b, int grid, size_t smem,
                             hipStream_t st) {
    return tabu ? launch_any<true, true>(form, a, b, grid, smem, st) : launch_any<false, true>(form, a, b, grid, smem, st);
}

}  // namespace qapk
