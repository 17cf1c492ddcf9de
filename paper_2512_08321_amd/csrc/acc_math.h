// Arithmetic on INT32 accumulators modulo 2^32.  Accumulators start at 2^31 (the offset that
// put_residue's byte dot product expects), and p = 256 may wrap by itself, so differences and sums of
// them pass the signed range for a large share of the outputs; signed overflow is undefined, so
// everything is formed on the unsigned bit patterns.
#pragma once

#include <cstdint>

namespace ozc {

constexpr int kAccBias = (int)0x80000000;  // accumulators' start, as the signed type of the accumulators

constexpr uint32_t acc_add(int x, int y) { return (uint32_t)x + (uint32_t)y; }
constexpr uint32_t acc_sub(int x, int y) { return (uint32_t)x - (uint32_t)y; }
constexpr uint32_t acc_flip(int x) { return (uint32_t)x ^ 0x80000000u; }  // x + 2^31
// A folded accumulator: the symmetric residue s, given as s + 128 in [0, 255], with the offset or not.
constexpr int acc_refill(uint32_t s128, bool biased) {
    return (int)(s128 - 128u + (biased ? 0x80000000u : 0u));
}

}  // namespace ozc
