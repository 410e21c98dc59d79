// The elements of a flat layer that the layer-wide passes of an update take one by one (plain C++: the bounds are tested on the host).
#pragma once
#include <cstdint>

namespace srigl {

// Worker `worker` of `workers` visits its share of the elements [4 n4, n) in steps of `workers`.  A layer may have up to 2^32 - 1
// elements and a step is up to 2^18: the counter has 64 bits, a 32-bit one would wrap instead of reaching n.
template <typename Element>
constexpr void each_of_tail(uint32_t n, uint32_t n4, uint32_t worker, uint32_t workers, Element element) {
    for (uint64_t i = 4 * (uint64_t)n4 + worker; i < n; i += workers) element((uint32_t)i);
}

}  // namespace srigl
