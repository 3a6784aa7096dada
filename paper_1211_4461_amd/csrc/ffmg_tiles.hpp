// ffmg_tiles.hpp -- tile heights chosen by rule (host only).
#pragma once

#include <cstddef>

namespace ffmg {

// Rows of the one-pass pre-smoothing tile on a finest level of N points, by
// FFMG_TUNE_PRE variant: 8, in FP32 from 2^21 points 16 (variant 0), or the other
// height (variant 2).  FP32, two sweeps from a guess, 8 rows and 16: 255^2 5.6 us
// and 7.0, 511^2 6.3 and 7.6, 1023^2 12.2 and 12.1, 2047^2 31.6 and 30.3; from
// zero 5.0 and 6.0, 5.7 and 6.6, 10.5 and 11.2, 28.8 and 27.2.
constexpr int presmooth_rows(bool fp32, std::size_t N, int variant)
{
    const int rows = fp32 && N >= (std::size_t)1 << 21 ? 16 : 8;
    return variant == 2 ? 24 - rows : rows;
}

}  // namespace ffmg
