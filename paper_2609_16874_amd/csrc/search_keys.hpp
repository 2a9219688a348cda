// search_keys.hpp -- rules of the assignment's candidate search (search_tile in
// k_mfma.hpp): its keys, the bits of a batch's binary32 distance sum with the
// batch's step in the low bits, and the frames that the fast search serves.
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
    return nbat > 8 ? 32 - __builtin_clz((uint32_t)(nbat - 1) >> 3) : 0;
}

// Difference of two sums, each shifted right by `bits`, from which on the sums
// themselves are at least `gap` steps apart.
constexpr uint32_t key_gap(uint32_t gap, int bits)
{
    return (gap + 2u * ((1u << bits) - 1u)) >> bits;
}

// Frames from this many pixels on take the fast search when only labels are
// requested (elem: bytes of an input element, F: harmonics, plane: there is a
// foreground plane): where a wave has more than a tile or two its shorter
// instruction stream pays, below the longer code fetched cold and a near tie's
// second pass cost more.  The line lies above the last size at which it measured
// slower.  Time of a whole frame with the fast search over that with the exact
// one, 32 x 32 bins, 30 to 60 % of the pixels foreground:
//   up to 4 harmonics, both types, from 256 x 256 to 2160 x 3840: 0.94 .. 1.00;
//   fp32, 5 to 8: 512 x 513 1.02 .. 1.03, 640 x 640 0.99 .. 1.02, 720 x 1024
//     1.00, 900 x 900 0.98 .. 1.01, 1024 x 1024 0.98 .. 0.99;
//   fp16, 5 to 9: 512 x 513 0.97 .. 1.01, 512 x 600 0.97 .. 0.98;
//   fp16, 10 to 16: 640 x 640 0.99 .. 1.02, 720 x 1024 0.99 .. 1.02, 900 x 900
//     0.98 .. 1.01, 1024 x 1024 0.97 .. 1.00, 1024 x 2048 0.95 .. 0.97;
//   fp32, 9 to 16: 1.04 .. 1.24 at every size from 479 x 641 to 1500 x 1500
//     (its registers spill), so it has no such kernel.
// On 40 x 40 to 96 x 96 bins the ratios at these lines are 0.97 .. 1.00.
// Without a plane every pixel is searched, twice the tiles or more: 256 x 256 0.98
// .. 1.03, 512 x 513 and above 0.93 .. 1.00 for every harmonic count.
constexpr int64_t fast_search_pixels(int elem, int F, bool plane)
{
    if (elem == 4 && F > 8) return INT64_MAX;
    if (F <= 4 || !plane) return 1LL << 18;
    return elem == 2 && F <= 9 ? 9LL << 15 : 1LL << 20;
}

}  // namespace cpe
