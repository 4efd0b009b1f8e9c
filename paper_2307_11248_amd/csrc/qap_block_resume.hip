// qap_block_resume.hip -- block form of the searches: chunked runs (serving).  The slots (as
// they are, tabu offsets included) and the ring of moves are saved between chunks; everything
// else is made again from the permutation.  64 requests of n = 30 .. 256 took 80.2 ms in the
// tile kernels and take 27.2 ms here.
#include "qap_block.h"

namespace qapk {

namespace {

// Chunked runs: block i runs one chunk of items[i], of any form (waves a form does not need
// end at once).
__global__ void __launch_bounds__(1024) resume_block_kernel(const Item *items) {
    extern __shared__ __align__(16) unsigned char sm[];
    __shared__ __align__(16) BlkShared sh;
    const Item it = items[blockIdx.x];
    switch ((it.n + 31) / 32 * 2 + (it.sym ? 1 : 0)) {
        case 2: block_body<1, false, true, true, false, false>(it, sm, sh); break;
        case 3: block_body<1, true, true, true, false, false>(it, sm, sh); break;
        case 4: block_body<2, false, true, true, false, false>(it, sm, sh); break;
        case 5: block_body<2, true, true, true, false, false>(it, sm, sh); break;
        case 6: block_body<3, false, true, true, false, false>(it, sm, sh); break;
        case 7: block_body<3, true, true, true, false, false>(it, sm, sh); break;
        case 8: block_body<4, false, true, true, false, false>(it, sm, sh); break;
        case 9: block_body<4, true, true, true, false, false>(it, sm, sh); break;
        case 10: block_body<5, false, true, true, false, false>(it, sm, sh); break;
        case 11: block_body<5, true, true, true, false, false>(it, sm, sh); break;
        case 12: block_body<6, false, true, true, false, false>(it, sm, sh); break;
        case 13: block_body<6, true, true, true, false, false>(it, sm, sh); break;
        case 14: block_body<7, false, true, true, false, false>(it, sm, sh); break;
        case 15: block_body<7, true, true, true, false, false>(it, sm, sh); break;
        case 16: block_body<8, false, true, true, false, false>(it, sm, sh); break;
        default: block_body<8, true, true, true, false, false>(it, sm, sh); break;
    }
}

}  // namespace

hipError_t launch_resume_block(const Item *d_items, int count, size_t smem, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(resume_block_kernel, dim3(count), dim3(1024), smem, st, d_items);
    return report(hipGetLastError(), "resume kernel launch");
}

}  // namespace qapk
