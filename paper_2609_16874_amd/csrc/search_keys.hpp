// search_keys.hpp -- the keys of the assignment's candidate search (search_tile
// in k_mfma.hpp): the bits of a batch's binary32 distance sum with the batch's
// step in the low bits.
#pragma once

#include <cstdint>

namespace cpe {

// Bits that a key needs for the step of one of nbat batches, eight a step.
// They are taken from the sums, so no more than the frame needs: a pixel is
// decided only if its two smallest sums differ by key_gap() above those bits,
// which takes a gap of 17 to 32 binary32 steps with the 4 bits of 128 batches, 9
// to 16 with the 3 of 64.
constexpr int step_bits(int nbat)
{
    int bits = 0;
    while ((8 << bits) < nbat) bits++;
    return bits;
}

// Difference of two sums, each shifted right by `bits`, from which on the sums
// themselves are at least `gap` steps apart.
constexpr uint32_t key_gap(uint32_t gap, int bits)
{
    return (gap + 2u * ((1u << bits) - 1u)) >> bits;
}

}  // namespace cpe
