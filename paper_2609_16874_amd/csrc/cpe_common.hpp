// cpe_common.hpp -- constants, device tables and arithmetic helpers shared by
// the decoder's kernels.  Every helper implements one step of the fixed-point
// contract stated in include/cpe_decode.h.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "cpe_decode.h"

namespace cpe {

constexpr int kWMant = 8;             // weight bucket: top 8 mantissa bits of fl32(S+1)
constexpr int kWKeys = 32 << kWMant;  // 8192 weight buckets (32 binades)
constexpr int kReplicas = 4;          // replicated global histograms (spread of the atomics)
constexpr int kMaxF = 16;             // harmonics per axis
constexpr int kMaxBins = 128;
constexpr int kCountCap = 1024;       // centroids whose pixel counts are privatised in LDS
constexpr int kMfmaBins = 32;         // side of a block of bins; grids of one block are assigned without a peak kernel
constexpr int kDistBase = 158;        // palette split of the matrix-core distances (head of k_mfma.hpp)
constexpr int kPopKinds = 7;          // binary16 palette operand kinds per axis (Tables::pop)
constexpr int kMaxBinBlocks = (kMaxBins + kMfmaBins - 1) / kMfmaBins;   // blocks of 32 bins per axis
constexpr int kMaxSlices = 256;       // workgroups of the compaction (slices of the pixel list)
constexpr int64_t kFusedMaxPixels = 1LL << 21;   // frames the vote launch compacts itself (two launches)
constexpr int kFusedMaxSeg = 8192;               // listed pixels per workgroup of that launch (LDS)

typedef short v2s __attribute__((ext_vector_type(2)));

// Device-resident constants built once by cpe_decode_create.
struct Tables {
    const float *cx;          // [Bw] bin centres (pixels)
    const float *cy;          // [Bh]
    // matrix-core path
    const uint32_t *pop;      // [axis][block][kind][64 lanes][4 words]: the binary16 palette operand of
                              //   lane l (bin 32 block + (l & 31), K slots 8 (l >> 5) .. + 7); kinds:
                              //   norms of A, norms of R for S, for S + 1, then hi and lo of channels
                              //   0 .. 15 and of 16 .. 31; see k_mfma.hpp
    const uint16_t *wt_pk;    // [kWKeys] weight q = lo - 256 nh as int8 limbs lo | nh << 8 (lo >= -128, nh <= 0),
                              //          at LDS position ((e + 17) & 31) * 256 + t
};

// The correctly rounded binary32 square root of x, 0 or at least 2^-20: the
// Eq4 distance from x = fl32(S), also scaled by 2^-14.  y is the hardware's
// reciprocal root; s = x y is corrected to first order by its residual x - s^2
// times y / 2, with one rounding of each multiply-add.  No bound on the
// hardware's root proves the result: that it is correctly rounded for every
// input rests on trial alone, cpe_check_sqrt tries them all.  For x = 0, s and
// the residual are 0.  (The hardware root with its
// two neighbours tested by residuals takes three instructions more: 28.5 against
// 27.7 us for a 640 x 640 fp16 frame with 16 harmonics, 92.2 against 89.4 us for
// 1024 x 2048 with the score map.)
__device__ __forceinline__ float sqrt_cr(float x)
{
    const float y = __builtin_amdgcn_rsqf(fmaxf(x, 0x1p-20f));
    const float s = x * y;
    return __builtin_fmaf(__builtin_fmaf(-s, s, x), 0.5f * y, s);
}

// min of two binary64 values that are never NaN (one instruction; the
// library's min also canonicalises its operands).
__device__ __forceinline__ double min_f64(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ __forceinline__ float half_bits_to_float(uint32_t bits)
{
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
}

template <typename T> __device__ __forceinline__ float load_scalar(const T *p);
template <> __device__ __forceinline__ float load_scalar<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ float load_scalar<_Float16>(const _Float16 *p) { return (float)*p; }

// Inclusive prefix sum of x over the 64 lanes of a wave with DPP moves:
// shifts by 1, 2, 4, 8 within each row of 16 lanes, then the last lane of
// row 0 added to row 1 (and of row 2 to row 3), then the last lane of row 1
// added to rows 2 and 3.  Every lane must be active.
__device__ __forceinline__ int wave_incl_sum(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
    return x;
}

// Bitwise or of x over the first 32 lanes of a wave (every lane active).
__device__ __forceinline__ uint32_t wave_or32(uint32_t x)
{
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);   // row_shr:1
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);   // row_shr:2
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);   // row_shr:4
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);   // row_shr:8
    return (uint32_t)(__builtin_amdgcn_readlane((int)x, 15) | __builtin_amdgcn_readlane((int)x, 31));
}

// Bitwise or of x over a wave (every lane active).
__device__ __forceinline__ uint32_t wave_or64(uint32_t x)
{
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);
    return (uint32_t)(__builtin_amdgcn_readlane((int)x, 15) | __builtin_amdgcn_readlane((int)x, 31) |
                      __builtin_amdgcn_readlane((int)x, 47) | __builtin_amdgcn_readlane((int)x, 63));
}

__device__ __forceinline__ int lane_prefix(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

}  // namespace cpe
