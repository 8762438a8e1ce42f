// Orders whose ranks are used as places in an array: total for any values, so
// that the counts of what comes before are a permutation. (constexpr: for the
// kernels and for the host alike.)
#pragma once

namespace zh {

// whether (a, i) comes before (b, j) from the largest value down: what is not a
// number after every number, equal values by index
constexpr bool before_desc(double a, int i, double b, int j) {
    return (a != a) != (b != b) ? b != b : a > b || (!(a < b) && i < j);
}

}  // namespace zh
