// Seal of the flag words that the device writes to host memory and the host
// polls for.  The words, their number and the seal leave the device in one
// store, but may reach memory in parts: the host takes a set only if the seal
// is that of the words it read.  Each word is mixed with its place (the
// finalizer of the SplitMix64 generator, a bijection of 64 bits) before the
// exclusive or, so that words of two sets match the seal of one of them with
// chance 2^-64.  A plain exclusive or of the words would also match where two
// stale words differ from the new ones by the same bits, as the steps that ran
// (4 to 5) and the mark of a stop (0 to 1) do.
#pragma once

#include <cstdint>

namespace md {

// (constexpr: for the host and the device)
constexpr uint64_t seal_mix(uint64_t word, int place)
{
    uint64_t x = word + (uint64_t)(place + 1) * 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

}  // namespace md
