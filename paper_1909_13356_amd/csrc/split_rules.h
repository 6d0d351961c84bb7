// Rules on counts alone, without HIP types: how work lists are cut.
#pragma once
#include <cstdint>

namespace lss {

// The M2L plan holds pair indices in 32 bits (tiles, blocks, each box's pairs);
// a longer list is run class by class, whose segments are 64-bit.
inline bool m2l_plan_holds(int64_t npairs) { return npairs <= INT32_MAX; }

}  // namespace lss
