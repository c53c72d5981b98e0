// Division of a 31-bit index by a number that stays the same for a whole launch
// (a box's row length, its number of rows): one high multiplication and a shift
// instead of the 64-bit division that no instruction does.
#pragma once

#include <cstdint>

namespace fd6 {

// n / d for n < 2^31, 2 <= d <= 2^30.  With l = ceil(log2 d) and m = ceil(2^(31 + l) / d)
// the excess of m n / 2^(31 + l) over n / d is below n / 2^(31 + l) < 1 / 2^l <= 1 / d,
// so the integer part is that of n / d; m < 2^32 because 2^l < 2 d.
struct DivConst {
    uint32_t d, m, shift;
};

inline DivConst div_const(uint32_t d) {
    uint32_t l = 1;
    while ((1u << l) < d) ++l;
    return DivConst{d, (uint32_t)(((1ull << (31 + l)) + d - 1) / d), l - 1};
}

#if defined(__HIPCC__)
__host__ __device__
#endif
inline uint32_t operator/(uint32_t n, const DivConst& c) {
    return (uint32_t)(((uint64_t)n * c.m) >> 32) >> c.shift;
}

}  // namespace fd6
