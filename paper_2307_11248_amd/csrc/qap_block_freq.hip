// qap_block_freq.hip -- block form of the tabu search with the frequency memory.
//
// Served are tabu pairs and marked units (attr 0, 1) without the diversification move and
// without a step record; those, and the unit-location table (attr 2), stay with the tile
// kernels.  (A diversification move that scanned the blocks' free slots behind two more
// barriers was taken out: it chose another pair than the tiles in about one search of 500 when
// 300 ran at once.  In those kernels the housekeeping wave, and for symmetric n = 65 .. 96 the
// task waves too, came to B1 without the wait that block_sync now asks for.)  The counts add one
// vector atomic a move by the housekeeping wave.  Marked units need no expiry lists: the block waves read their rows'
// and columns' marks in the select.  us per iteration, tile kernels and here, pairs / marked
// units: n = 64 2.26 / 2.59 and 1.03 / 1.02, n = 128 symmetric 2.93 / 4.15 and 1.33 / 1.40,
// n = 150 4.21 / 5.68 and 1.90 / 2.12, n = 256 13.5 / 18.2 and 3.67 / 4.60 (one start; 700
// starts gain as much).
#include "qap_block.h"

namespace qapk {

hipError_t launch_block_freq(int form, const SearchArgs &a, int grid, size_t smem, hipStream_t st) {
    return launch_any<true, false, true>(form, a, BatchArgs{}, grid, smem, st);
}

}  // namespace qapk
