// Launch sizes, host code only, so that they can be tested without a device.
#pragma once

#include <algorithm>
#include <cstdint>

namespace dfpr {

// Workgroups of `threads` for a kernel whose threads stride over `items`: a
// thread an item, up to a number that fills the device many times over.  A launch
// may have fewer than 2^32 threads, and an edge list can be longer.
inline unsigned stride_blocks(uint64_t items, unsigned threads, unsigned most = 1u << 16)
{
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((items + threads - 1) / threads, most));
}

}  // namespace dfpr
