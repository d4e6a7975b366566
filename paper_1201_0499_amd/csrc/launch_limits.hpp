// Limits of a launch's grid, shared by the launch code and the CPU tests
// (pure C++, no HIP dependency).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace pe {

// Largest number of workgroups of `threads` work-items in one dimension of a
// grid: HIP refuses 2^32 work-items or more there.
inline int64_t max_workgroups(int threads) { return (((int64_t)1 << 32) - 1) / threads; }

// Workgroups for `work` items (a multiple of 8) of a kernel whose workgroups
// stride over them: all at once as far as a grid holds them, and a multiple of
// 8, so that an item's XCD (item mod 8) stays that of its workgroup.
inline int64_t strided_grid(int64_t work, int threads)
{
    return std::min(work, max_workgroups(threads) / 8 * 8);
}

}  // namespace pe
