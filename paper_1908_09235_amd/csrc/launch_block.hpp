// Launcher body of the several-steps kernel, instantiated per storage form.
#pragma once

#include "launch.hpp"

namespace lbm {

// Two workgroups of 512 lanes share a CU where there are enough tiles; with at
// most one tile a CU, 1024 lanes on it have twice the wavefronts to hide the
// latency of each phase (droplet 128^2 FP64, 6 steps per launch: 4.40 us a
// step with 512 lanes, 4.03 with 1024; at 2048^2, 2 steps: 96 and 138).
template <typename S, typename R, int EOS, int DEV>
void block_t(const Ctx& c, const BlockArgs& a, bool wide, unsigned lds) {
    if (wide)
        hipLaunchKernelGGL((k_block<S, R, EOS, DEV, kBlockW, kBlockH, 2 * kBlockThreads>),
                           dim3(a.ntiles + 1), dim3(2 * kBlockThreads), lds, c.stream, a,
                           phys_as<R>(c.ph));
    else
        hipLaunchKernelGGL((k_block<S, R, EOS, DEV, kBlockW, kBlockH, kBlockThreads>),
                           dim3(a.ntiles + 1), dim3(kBlockThreads), lds, c.stream, a,
                           phys_as<R>(c.ph));
}

template <typename S, typename R, int DEV>
void block_any(const Ctx& c, const BlockArgs& a, bool wide, unsigned lds) {
    if (c.eos == EOS_NONE) block_t<S, R, EOS_NONE, DEV>(c, a, wide, lds);
    else if (c.eos == EOS_EXP) block_t<S, R, EOS_EXP, DEV>(c, a, wide, lds);
    else block_t<S, R, EOS_CS, DEV>(c, a, wide, lds);
}

}  // namespace lbm
