// Several steps per launch, FP64 storage and arithmetic.
#include "launch_block.hpp"

namespace lbm {

void launch_block_f64(const Ctx& c, const BlockArgs& a, bool wide, unsigned lds) {
    block_any<double, double, 0>(c, a, wide, lds);
}

}  // namespace lbm
