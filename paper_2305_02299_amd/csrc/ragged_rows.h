// Rows that are staged with loads of four elements at any alignment: where a load that would run past the last element starts earlier,
// and how its values move back to their places (plain C++: tested on the host).
#pragma once
#include <cstdint>

namespace srigl {

// The load at element e of `total` starts this many elements earlier: more than three where none of the four elements is there.
constexpr int ragged_shift(unsigned e, int total) { return (int)e > total - 4 ? (int)e - (total - 4) : 0; }

// Four 16-bit values, the lowest-addressed one lowest, moved by `places`.  From four places on nothing of what was loaded belongs there and
// the result stands for columns that no index names; the shift stays below the width of the word all the same.
constexpr uint64_t move_halves(uint64_t four, int places) { return four >> (16 * (places < 3 ? places : 3)); }

}  // namespace srigl
