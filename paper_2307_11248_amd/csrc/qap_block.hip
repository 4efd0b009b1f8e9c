// qap_block.hip -- block form of the searches: what it serves, and its kernels for launches
// of at most one search a compute unit.
#include "qap_block.h"

namespace qapk {

static_assert(sizeof(BlkShared) <= 1024, "the kernels' own LDS, as block_ok counts it");

int block_form(int n, int sym) { return 2 * ((n + 31) / 32 - 1) + (sym ? 1 : 0); }

size_t block_smem_bytes(int n, int sym, int hi, bool tabu) {
    return (size_t)blk_plan(n, (n + 31) / 32, sym, hi, tabu).total;
}

size_t block_ring_bytes(int hi) { return (size_t)blk_ring(hi) * 4; }

int block_ok(int n, int sym, int blk, bool tabu, int lo, int hi, size_t max_smem) {
    if (!blk || n > WIDE_N) return 0;
    if (tabu && (hi - lo >= 64 || hi > BLOCK_MAX_TENURE)) return 0;
    return block_smem_bytes(n, sym, hi, tabu) + 1024 <= max_smem ? 1 : 0;
}

hipError_t launch_block_busy(bool tabu, int form, const SearchArgs &a, const BatchArgs &b, int grid, size_t smem,
                             hipStream_t st);   // qap_block_busy.hip
hipError_t launch_block_freq(int form, const SearchArgs &a, int grid, size_t smem, hipStream_t st);   // qap_block_freq.hip

hipError_t launch_block(bool tabu, int form, bool busy, size_t smem, const SearchArgs *a, const BatchArgs *b, int grid,
                        hipStream_t st) {
    if (grid <= 0) return hipSuccess;
    const SearchArgs sa = a ? *a : SearchArgs{};
    const BatchArgs ba = b ? *b : BatchArgs{};
    if (sa.freq) return launch_block_freq(form, sa, grid, smem, st);
    if (busy && form < 2 * 4) return launch_block_busy(tabu, form, sa, ba, grid, smem, st);
    return tabu ? launch_any<true, false>(form, sa, ba, grid, smem, st)
                : launch_any<false, false>(form, sa, ba, grid, smem, st);
}

}  // namespace qapk
