// Several steps per launch, FP32 and FP16 storage with one reference density.
#include "launch_block.hpp"

namespace lbm {

void launch_block_f32(const Ctx& c, const BlockArgs& a, bool wide, unsigned lds) {
    switch (c.storage) {
    case 2: block_any<float, float, 0>(c, a, wide, lds); break;
    case 3: block_any<float, float, 1>(c, a, wide, lds); break;
    case 4: block_any<_Float16, float, 1>(c, a, wide, lds); break;
    default: block_any<float, double, 0>(c, a, wide, lds);
    }
}

}  // namespace lbm
