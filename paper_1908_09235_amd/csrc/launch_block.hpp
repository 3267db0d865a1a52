// Launcher body of the several-steps kernel, instantiated per storage form.
#pragma once

#include "launch.hpp"

namespace lbm {

// Two workgroups of 512 lanes share a CU where there are enough tiles; with at
// most one tile a CU, 1024 lanes on it have twice the wavefronts to hide the
// latency of each phase (droplet 128^2 FP64, 6 steps per launch: 4.40 us a
// step with 512 lanes, 4.03 with 1024; at 2048^2, 2 steps: 96 and 138).
template <typename S, typename R, int EOS, int DEV>
void block_t(const Ctx& c, const BlockKernarg& k, bool wide, unsigned lds) {
    const dim3 grid(k.a.ntiles + 1);
    if (wide)
        hipLaunchKernelGGL((k_block<S, R, EOS, DEV, 2 * kBlockThreads>), grid,
                           dim3(2 * kBlockThreads), lds, c.stream, k);
    else
        hipLaunchKernelGGL((k_block<S, R, EOS, DEV, kBlockThreads>), grid, dim3(kBlockThreads),
                           lds, c.stream, k);
}

template <typename S, typename R, int DEV>
void block_any(const Ctx& c, const BlockKernarg& k, bool wide, unsigned lds) {
    if (c.eos == EOS_NONE) block_t<S, R, EOS_NONE, DEV>(c, k, wide, lds);
    else if (c.eos == EOS_EXP) block_t<S, R, EOS_EXP, DEV>(c, k, wide, lds);
    else block_t<S, R, EOS_CS, DEV>(c, k, wide, lds);
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
