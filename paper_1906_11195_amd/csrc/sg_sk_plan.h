// How the sweeps of SK chains are cut into launches.
#pragma once
#include <algorithm>
#include <cstdint>

namespace sg {

// Blocks of 64 spins that one launch runs of a chain: the sweep kernels count blocks
// in 31 bits and a launch's accepted flips, up to 64 a block, in 32.
constexpr int64_t kSkLaunchBlocks = ((int64_t)1 << 26) - 1;

// Sweeps of the next launch: of the `left` ones, up to the next recomputation
// (`to_check` sweeps away), of chains of up to `blocks` blocks.
inline int64_t sk_launch_sweeps(int64_t left, int64_t to_check, int32_t blocks)
{
    return std::min(std::min(left, to_check), std::max<int64_t>(1, kSkLaunchBlocks / blocks));
}

}  // namespace sg
