// Home slots of the group-bys' LDS tables.  Plain C++ (no HIP), so that the
// spread is checked on the host.
#pragma once

#include <cstdint>

// Hash of a group key (key32 is 0, or a 32-bit key alone is key64's low word)
// for a table of 2^p slots, whose home slot is the top p bits.  Every row is
// looked up, so it is a few 32-bit operations.  Each word of the key has an odd
// multiplier of its own: with one for two words the keys (i, c - i) all have
// the same slot, find no slot in reach and take device atomics.  The product
// x * 0x9E3779B1 alone spreads runs of consecutive codes as evenly as can be,
// but gives keys at some strides (1597, 10946) neighbouring slots; so runs of
// 256 keep it, and each run is turned by a stronger hash of its number.
// 5M rows, with one product of the summed words, with the stronger hash of all
// bits, and so: 512 consecutive codes 578, 807, 586 us; 400 keys at stride 1597
// 3867, 564, 559; 20 x 25 pairs 1376, 862, 813; pairs (i, 511 - i) 5497, 1294, 1133.
constexpr uint32_t gq_slot_hash(uint64_t key64, uint32_t key32)
{
    const uint32_t x =
        static_cast<uint32_t>(key64) + static_cast<uint32_t>(key64 >> 32) * 0x85EBCA6Bu + key32 * 0x9E3779B1u;
    uint32_t run = (x >> 8) * 0x9E3779B1u;
    run ^= run >> 15;
    return (x * 0x9E3779B1u) ^ (run * 0x85EBCA6Bu);
}
