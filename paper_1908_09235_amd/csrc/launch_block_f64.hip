// Several steps per launch, FP64 storage and arithmetic.
#include "launch_block.hpp"

namespace lbm {

void launch_block_f64(const Ctx& c, const BlockKernarg& k, int lanes, unsigned lds) {
    block_any<double, double, 0>(c, k, lanes, lds);
}

void launch_block_batch_f64(const BlockBatchLaunch& L) { block_batch_any<double, double, 0>(L); }

}  // namespace lbm
