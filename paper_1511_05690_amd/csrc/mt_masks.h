// Bit masks over the powers of a family (at most 32 of them: bit q stands for
// power q).  Plain C++ without a dependency, for host and device code alike
// (constexpr functions are both).
#pragma once

#include <stdint.h>

namespace mt {

// The bits of powers 0 .. n - 1, 0 <= n <= 32 (a shift by 32 is undefined).
constexpr uint32_t family_bits(int n) { return n >= 32 ? ~0u : (1u << n) - 1u; }

// f(q, wanted) for every power q from 0 up to the mask's highest one, in
// ascending order; wanted: bit q of the mask.
template <class F>
constexpr void each_power(uint32_t mask, F&& f) {
    const int end = mask == 0u ? 0 : 32 - __builtin_clz(mask);
    for (int q = 0; q < end; ++q) f(q, ((mask >> q) & 1u) != 0u);
}

}  // namespace mt
