// Several steps per launch, FP32 and FP16 storage with one reference density.
#include "launch_block.hpp"

namespace lbm {

void launch_block_f32(const Ctx& c, const BlockKernarg& k, int lanes, unsigned lds) {
    switch (c.storage) {
    case 2: block_any<float, float, 0>(c, k, lanes, lds); break;
    case 3: block_any<float, float, 1>(c, k, lanes, lds); break;
    case 4: block_any<_Float16, float, 1>(c, k, lanes, lds); break;
    default: block_any<float, double, 0>(c, k, lanes, lds);
    }
}

void launch_block_batch_f32(const BlockBatchLaunch& L) {
    switch (L.storage) {
    case 2: block_batch_any<float, float, 0>(L); break;
    case 3: block_batch_any<float, float, 1>(L); break;
    case 4: block_batch_any<_Float16, float, 1>(L); break;
    default: block_batch_any<float, double, 0>(L);
    }
}

}  // namespace lbm
