// Workgroups of a launch (host code, no HIP, so that it can be checked on the CPU).
#pragma once
#include <stdint.h>

namespace agile {

// HIP refuses a launch of 2^32 threads or more in a dimension of its grid.
inline uint32_t max_workgroups(uint32_t threads) { return 0xFFFFFFFFu / threads; }

// Workgroups of `threads` threads for `items`, `per_group` each, at least one and at most `cap` and what a
// grid holds: kernels that use it loop over what is left.
inline uint32_t workgroups(uint64_t items, uint64_t per_group, uint32_t threads, uint64_t cap = ~0ull) {
    const uint64_t most = max_workgroups(threads) < cap ? max_workgroups(threads) : cap;
    uint64_t want = items / per_group + (items % per_group ? 1 : 0);
    if (want < 1) want = 1;
    return (uint32_t)(want < most ? want : most);
}

}  // namespace agile
