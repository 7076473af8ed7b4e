// Splitting a call's blocks into launches.  Host logic without HIP.
#pragma once

#include <algorithm>
#include <cstdint>

namespace sparkcl {

// launch(first, count) for all `blocks` blocks of `threads` threads, a launch
// at a time, until one does not return 0: a dispatch counts its grid in
// work-items, in 32 bits.
template <class Launch>
int in_launches(uint64_t blocks, uint32_t threads, Launch launch)
{
    const uint64_t most = 0xFFFFFFFFull / threads;
    for (uint64_t at = 0; at < blocks; at += most) {
        const int rc = launch(at, (uint32_t)std::min(blocks - at, most));
        if (rc != 0)
            return rc;
    }
    return 0;
}

} // namespace sparkcl
