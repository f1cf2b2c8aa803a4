// Launchers of the root-MUSIC kernels for line windows and for block windows
// up to 8 x 8; the larger block windows are instantiated in bm_bigblock.hip.
#include "bm_block_kernels.h"

namespace bm {

int rootmusic_windows_per_block(int L, int block) { return line_windows_per_block(L, block); }

hipError_t launch_rootmusic(int L, const RmBatch& b, int block, int grid, hipStream_t s) {
    if (b.total <= 0 || b.njobs <= 0) return hipSuccess;
    if (block != 128 && block != 256) return hipErrorInvalidValue;
    if (grid <= 0 || grid > b.total) grid = b.total;
    if (L > kMaxL) return launch_big_block_window(L, b, s);
    return b.jacobi ? launch_rootmusic_jacobi(L, b, block, grid, s) : launch_rootmusic_J<false>(L, b, block, grid, s);
}

}  // namespace bm
