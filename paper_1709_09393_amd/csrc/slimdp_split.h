// How the passes over the candidates of a core selection split the tiles: contiguous groups, one block each.  Plain C++
// (no HIP), so that the rule can be checked over every size on a CPU.
#pragma once
#include <cstdint>

namespace slimdp {

constexpr uint32_t GROUP_MAX = 1024;       // tiles per group at most (LDS counters of k_core_count)
constexpr uint32_t CORE_GROUPS = 2048;     // groups at most (eight blocks on each of 256 compute units)

// Groups for T tiles on a device of cus compute units: a tile per wave at least, eight blocks per compute unit at most, and
// on a small device as many as it takes to keep to GROUP_MAX.
constexpr uint32_t core_groups(uint32_t T, uint32_t cus)
{
    const uint32_t waves = (T + 3u) / 4u, blocks = cus < CORE_GROUPS / 8u ? cus * 8u : CORE_GROUPS;
    const uint32_t want = waves < blocks ? waves : blocks, least = (T + GROUP_MAX - 1u) / GROUP_MAX;
    return want > least ? want : least;
}

// First tile of group g, and the group that holds tile t.
constexpr uint32_t group_first(uint32_t g, uint32_t T, uint32_t groups) { return (uint32_t)((uint64_t)T * g / groups); }
constexpr uint32_t group_of(uint32_t t, uint32_t T, uint32_t groups)
{
    return (uint32_t)((((uint64_t)t + 1u) * groups - 1u) / T);
}

}  // namespace slimdp
