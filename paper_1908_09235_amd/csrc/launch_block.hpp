// Launcher body of the several-steps kernel, instantiated per storage form.
#pragma once

#include "launch.hpp"

namespace lbm {

// Two workgroups of 512 lanes share a CU where there are enough tiles; with at
// most one tile a CU, 1024 lanes on it have twice the wavefronts to hide the
// latency of each phase (droplet 128^2 FP64, 6 steps per launch: 3.82 us a
// step with 512 lanes, 3.49 with 1024; at 400^2, 3 steps, 400 tiles: 6.82 and
// 7.38).  A single-phase lattice that regions of 24 x 24 cover with at most one
// tile a CU takes those: as many steps a launch, half the nodes a step (static
// channel 100 x 50 FP64, 8 steps: 2.81 us a step with 32 x 32, 2.39 with 24 x
// 24).  The two-phase step's halo is twice as wide, so that they would make two
// steps fewer a launch: droplet 128^2 FP64 3.47 with 4 steps, 64^2 3.19 with 5
// against 3.28 with 7; not used there.
template <typename S, typename R, int EOS, int DEV>
void block_t(const Ctx& c, const BlockKernarg& k, int lanes, unsigned lds) {
    const dim3 grid(k.a.ntiles + 1);
    if constexpr (EOS == EOS_NONE)
        if (lanes == kBlockSmall) {
            hipLaunchKernelGGL((k_block<S, R, EOS, DEV, kBlockSmall>), grid, dim3(kBlockSmall),
                               lds, c.stream, k);
            return;
        }
    if (lanes > kBlockThreads)
        hipLaunchKernelGGL((k_block<S, R, EOS, DEV, 2 * kBlockThreads>), grid,
                           dim3(2 * kBlockThreads), lds, c.stream, k);
    else
        hipLaunchKernelGGL((k_block<S, R, EOS, DEV, kBlockThreads>), grid, dim3(kBlockThreads),
                           lds, c.stream, k);
}

template <typename S, typename R, int DEV>
void block_any(const Ctx& c, const BlockKernarg& k, int lanes, unsigned lds) {
    if (c.eos == EOS_NONE) block_t<S, R, EOS_NONE, DEV>(c, k, lanes, lds);
    else if (c.eos == EOS_EXP) block_t<S, R, EOS_EXP, DEV>(c, k, lanes, lds);
    else block_t<S, R, EOS_CS, DEV>(c, k, lanes, lds);
}

template <typename S, typename R, int DEV>
void block_batch_any(const BlockBatchLaunch& L) {
    const dim3 grid(L.ntiles), block(kBlockThreads);
    if (L.eos == EOS_NONE)
        hipLaunchKernelGGL((k_block_batch<S, R, EOS_NONE, DEV>), grid, block, L.lds, L.stream,
                           L.args);
    else if (L.eos == EOS_EXP)
        hipLaunchKernelGGL((k_block_batch<S, R, EOS_EXP, DEV>), grid, block, L.lds, L.stream,
                           L.args);
    else
        hipLaunchKernelGGL((k_block_batch<S, R, EOS_CS, DEV>), grid, block, L.lds, L.stream,
                           L.args);
    hipLaunchKernelGGL(k_block_reduce<0>, dim3(L.red_grid), dim3(256), 0, L.stream, L.args);
}

}  // namespace lbm
