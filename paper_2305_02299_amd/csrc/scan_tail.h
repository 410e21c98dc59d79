// How the passes of an update share out a layer (plain C++: the bounds are tested on the host).
#pragma once
#include <cstdint>

namespace srigl {

// Worker `worker` of `workers` visits its share of the elements [4 n4, n) in steps of `workers`.  A layer may have up to 2^32 - 1
// elements and a step is up to 2^18: the counter has 64 bits, a 32-bit one would wrap instead of reaching n.
template <typename Element>
constexpr void each_of_tail(uint32_t n, uint32_t n4, uint32_t worker, uint32_t workers, Element element) {
    for (uint64_t i = 4 * (uint64_t)n4 + worker; i < n; i += workers) element((uint32_t)i);
}

// Workgroups of a launch over all rows, `rows_each` rows to one: the same number on every die.  The last ones may have no row: a part's rows are counted
// without a sign, as a layer of one column may have up to 2^31 - 1 of them and the parts go beyond that.
constexpr uint32_t kDies = 8;
constexpr uint32_t row_workgroups(int32_t d_out, uint32_t rows_each) {
    return (((uint32_t)d_out + rows_each - 1) / rows_each + kDies - 1) / kDies * kDies;
}
constexpr bool is_row(uint32_t r, int32_t d_out) { return r < (uint32_t)d_out; }

}  // namespace srigl
