// Fixed-point scale of the capacity loss's probability sums.  Plain C++, so that it can be checked on the host.
#pragma once

namespace slicemoe {

// Fraction bits f with which up to Na probabilities, each at most 1, can be added as integers p * 2^f without leaving 64 bits: 38, one less
// for every doubling from 2^26 assignments on (Na < 2^(64 - f), so the sum stays below 2^64 also if one expert gets all of them with p = 1).
constexpr int capacity_fraction_bits(long long Na)
{
    int f = 38;
    while (f > 0 && (Na >> (64 - f)) != 0) --f;
    return f;
}

}  // namespace slicemoe
