// Order key of a work entry of a near-field list by its estimated cost, heaviest first, in
// 8 bits: the cost's binary exponent and its next two bits (within 25%, which is what an
// order of dispatch needs).  One sort pass instead of four or five over the whole number.
// Plain constexpr: the host and the device builds sort by the same key.
#pragma once

#include <cstdint>

namespace fmm {

constexpr uint64_t cost_order(uint64_t cost)
{
    const int msb = 63 - __builtin_clzll(cost | 1);
    const int e = msb > 2 ? msb - 2 : 0;  // cost >> e < 8
    return 255 - (4 * (uint64_t)e + (cost >> e));
}

}  // namespace fmm
