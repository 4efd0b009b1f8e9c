// qap_block_busy.hip -- block form of the searches: the kernels held to 64 VGPRs (n up to
// 128), for launches of more searches than compute units.
#include "qap_block.h"

namespace qapk {

hipError_t launch_block_busy(bool tabu, int form, const SearchArgs &a, const BatchArgs &b, int grid, size_t smem,
                             hipStream_t st) {
    return tabu ? launch_any<true, true>(form, a, b, grid, smem, st) : launch_any<false, true>(form, a, b, grid, smem, st);
}

}  // namespace qapk
