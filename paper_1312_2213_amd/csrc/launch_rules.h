// launch_rules.h -- how work is cut and which kernels take it, as plain
// arithmetic with no HIP dependency: the kernels and the runtime include it,
// and a check program builds it on its own (with sanitizers).
#pragma once

#include <stdint.h>

namespace muca {

// Calls f(done, n) for consecutive segments of n <= at_most of `total` sweeps,
// done sweeps behind each.  Counts what is left: done + at_most may lie
// beyond the type's range.
template <class F>
__attribute__((always_inline)) constexpr void for_segments(int32_t total, int32_t at_most, F f)
{
    for (int32_t left = total; left > 0;) {
        const int32_t n = left < at_most ? left : at_most;
        f(total - left, n);
        left -= n;
    }
}

} // namespace muca
