// How the workgroups of one group find out which of them ends last, without a clear of the count between launches and whatever
// ran before.  Every workgroup adds a share of its own to the group's 32-bit count; the shares of n workgroups add up to 2^32, so
// a launch leaves the count as it found it, modulo 2^32, also one that shared the count with other launches at the same
// time and also a replay of a captured one.  Plain C++, so that it can be checked without a GPU.
#pragma once
#include <stdint.h>

namespace space {

// What workgroup i of n adds.
constexpr uint32_t arrival_share(int n, int i) {
    const uint32_t each = UINT32_MAX / (uint32_t)n;
    return n < 2 ? 0u : i ? each : 0u - each * (uint32_t)(n - 1);
}
// Whether the workgroup that found the count at `before` and added `share` is the last one: the shares of fewer than all
// add up to something between 0 and 2^32, of all to 2^32.
constexpr bool arrival_is_last(uint32_t before, uint32_t share) { return before + share == 0u; }

}  // namespace space
