// Block windows of 15 x 15 and 17 x 17 (the paper's experimental window and
// the top of its window-size table, Sec. 3 and 4): the largest instantiations,
// in a translation unit of their own.
#include "bm_block_kernels.h"

namespace bm {

hipError_t launch_big_block_window_15_17(int L, const RmBatch& b, hipStream_t s) {
    switch (L) {
        case 15: return launch_big_block<15>(b, s);
        case 17: return launch_big_block<17>(b, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace bm
