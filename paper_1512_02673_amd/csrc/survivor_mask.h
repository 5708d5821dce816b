// Survivor sets as bit masks: bit w of the 128 bits (m0 the lower 64) is set
// when worker w survived.  Plain C++, so the host checks run the same code.
#pragma once
#include <cstdint>

namespace coded {

// Bits below position i, 0 <= i <= 128 (i = 128 in a code of 128 blocks: a
// shift of ones down, so that no word is ever shifted by its own width).
constexpr int bits_below(uint64_t m0, uint64_t m1, int i) {
    const uint64_t b0 = i >= 64 ? ~uint64_t{0} : (uint64_t{1} << i) - 1;
    const uint64_t b1 = i > 64 ? ~uint64_t{0} >> (128 - i) : 0;
    return __builtin_popcountll(m0 & b0) + __builtin_popcountll(m1 & b1);
}

}  // namespace coded
