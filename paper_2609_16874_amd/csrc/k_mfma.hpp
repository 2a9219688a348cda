// k_mfma.hpp -- matrix-core decoder kernels: the vote for every bin grid (above
// 32 x 32 in passes of two x blocks and one y block of 32 bins), the assignment
// for grids up to 32 x 32.
//
// Both passes stream a compact list of participating pixels (or every
// pixel, when the frame has no foreground channel), cut into tiles of 32
// consecutive entries.  The assignment, and the vote of frames above
// kFusedMaxPixels, read the list in global memory (written by k_compact, or by
// the vote launch of smaller frames): every workgroup gets a contiguous run
// of tiles of the same length to within one.  In smaller frames the vote
// lists its own share of the pixels in LDS (FusedArgs).  The waves take
// their tiles one at a time from a counter in LDS (so that they finish
// together however the SIMDs favour older waves), always loading the
// embedding rows of the next tile (and the list entries of the one after)
// before computing the current one.  Every tile but the last is full.
//
// Per-axis distances (Eq4/Eq10).  With the input X = rint(4096 v) (|X| <=
// 6144) and the palette split as -2P = 158 hi + lo (|lo| <= 79), both limbs
// whole binary16 numbers,
//   S = |X|^2 + |P|^2 - 2 X.P = 158 A + R,  A = X.hi + a,  R = X.lo + b
// where a and b hold the norms, |X|^2 + |P|^2 = 158 a + b.  A and R come from
// dense [pixels x channels] x [channels x bins] contractions on
// v_mfma_f32_32x32x16_f16, the norms from one more K-step (norm_operand:
// |X|^2 = f0 + 2^10 f1 + 2^20 f2, with 2^10 = 158 6 + 76 and 2^20 = 158 6636 +
// 88).  Every product and every partial sum, in any order, is a whole number
// below 2^24 in magnitude (times the scale), so the binary32 accumulation is
// exact.  With 32 channels |X| <= 34756, |P| <= 16387, and
//   R: sum |X lo| <= 32 6144 79 = 15.53 10^6, norms <= 0.58 10^6;
//   A: |X| |hi| <= 34756 (2 |P| + 79 sqrt 32) / 158 = 7.31 10^6, |X|^2 part
//      <= 7.65 10^6, |P|^2 part <= 1.70 10^6, together 16.68 10^6 < 2^24
//      (a base of 128 would let A reach 20.5 10^6, one of 172 R pass 2^24).
// One fused multiply-add 158 A + R then rounds the exact S once: it is
// fl32(S).  (Three int8 limb products with int32 accumulation, shifts, adds
// and a conversion took 8 VALU instructions per result up to the weight's
// packing instead of 4 and 11 instead of 6 per pair of input channels; at
// 1024 x 2048, 16 harmonics, fp16, the vote goes from 38.1 to 32.8 us and the
// assignment from 49.6 to 44.7 us.)
//
// Pass 1, k_vote_mfma (recovery + soft voting, Eq5/Eq6/Eq11).  With pixels
// as the MFMA rows, the distance result leaves in each lane one bin and 16
// pixels -- exactly the operand layout of the vote contraction
// H = Qx^T Qy over pixels, so the weights feed the second MFMA without any
// data exchange between lanes.  A weight q <= 2^15 is split into int8 limbs
// q = lo - 256 nh, -128 <= lo < 128 and nh = -hi in [-128, 0]; a tile's 32
// pixels take one v_mfma_i32_32x32x32_i8 for each of the four limb products,
// whose int32 sums hold for kFoldTiles tiles and are then added into a 64-bit
// histogram in LDS.  (fp16 limbs, 16 pixels per instruction, took twice the
// MFMAs, and their fp32 sums had to be folded every 8 tiles: 32.8 against
// 31.5 us at 1024 x 2048, 86.7 against 78.3 us at 2160 x 3840 with 8
// harmonics.)
//
// Pass 2, k_assign_mfma (assignment, Eq7, and label write-out).  Only the
// candidate columns and rows are needed: they are numbered in ascending
// order (slots), the MFMA rows are the slots' palette entries, each lane
// holds one pixel and 16 slots, and distances are computed for the groups of
// 8 slots that hold candidates: r = sqrtf(fl32(S)) correctly rounded, stored
// in LDS as binary32 bits (which order like the distances, r >= 0).  The
// candidate search walks batches of 4 columns of one row, in (row, column)
// order: the smallest x distance of the batch plus the row's y distance, in
// binary32, with the second smallest sum telling whether rounding could have
// decided; near ties are searched again with exact binary64 sums.  Slots keep
// the bins' order, so the result is the lowest centroid index among the
// smallest sums.
#pragma once

#include <type_traits>

#include "cpe_common.hpp"
#include "k_compact.hpp"
#include "k_peaks.hpp"
#include "search_keys.hpp"

namespace cpe {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x16 __attribute__((ext_vector_type(16)));

// The distance contraction (see the head of this file) splits -2P = kBase hi
// + lo and carries every product scaled by kScale, which keeps all operands
// normal binary16 numbers and shifts only the exponents of its results.
constexpr float kBaseF = (float)kDistBase;
constexpr float kScale = 0x1p-14f;

// Operands of one axis of a tile: per K-step of 16 channels a hi and a lo
// palette operand, after the constants of the A and the R accumulator.
template <int F>
constexpr int kSteps = (2 * F + 15) / 16;
template <int F>
constexpr int kAxisKinds = 2 + 2 * kSteps<F>;
template <int F>
constexpr int kPopBytes = 2 * kAxisKinds<F> * 64 * 16;   // LDS palette operands of both axes

// The binary16 pixel operands of one axis: the K slots 8 g .. 8 g + 7 of step
// j (lane half g) hold kScale X of the channels 16 j + 8 g + b (channels past
// 2F are zero).  A binary16 input's X has at most 11 significant bits (its
// spacing exceeds 1/4096 where |X| > 1024), so one number holds it; a
// binary32 input's 13-bit X takes two, its leading 11 bits and the rest.
template <typename T, int F>
struct AxisOp {
    static constexpr int NL = sizeof(T) == 2 ? 1 : 2;
    f16x8 a[NL][kSteps<F>];
};

__device__ __forceinline__ i32x16 mfma8(i32x4 a, i32x4 b, i32x16 c)
{
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 mfma16(f16x8 a, f16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Steps (binary32 units in the last place) by which the fast assignment
// search needs the second smallest batch sum to exceed the smallest: at
// least 7 by its error bound (see k_assign_mfma).
constexpr int kFastGap = 8;
// Low bits of the search's keys that hold the step of a lane's batch: as many
// as the frame's batches need (step_bits), at most this for grids up to 32 x 32.
constexpr int kStepBits = 4;
static_assert(step_bits(kMaxBatchLds) == kStepBits, "eight batches per step");

// Exchanges between the lanes of a wave: the upper half (the odd rows of 16
// lanes) of a and the lower half (the even rows) of b swap places, so that a
// lane of the lower half (an even row) gets both halves' a, the others both
// halves' b; and x of the lane 8 further in the row.
__device__ __forceinline__ u32x2 swap32(uint32_t a, uint32_t b)
{
    return __builtin_amdgcn_permlane32_swap(a, b, false, false);
}
__device__ __forceinline__ u32x2 swap16(uint32_t a, uint32_t b)
{
    return __builtin_amdgcn_permlane16_swap(a, b, false, false);
}
__device__ __forceinline__ uint32_t row_ror8(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, true);
}

// Row of the 32 x 32 MFMA result held by register r of a lane in group g.
__device__ __forceinline__ constexpr int acc_row(int r, int g) { return 8 * (r >> 2) + 4 * g + (r & 3); }

// Two channels of a binary16 input as kScale X, X = rint(4096 clamp(v, -1.5,
// 1.5)): 2^-12 v is subnormal where X needs rounding (|v| < 1/4), and the
// spacing 2^-24 of the subnormals is that of X 2^-24, so the product rounds
// exactly as rint; the clamp commutes with it, and the second product is
// exact.  A NaN clamps to -1.5 (max returns the non-NaN operand).
__device__ __forceinline__ f16x2 scaled_pair(uint32_t w)
{
    const f16x2 down = {(_Float16)0x1p-12f, (_Float16)0x1p-12f}, up = {(_Float16)0x1p10f, (_Float16)0x1p10f};
    const f16x2 lo = {(_Float16)-0x1.8p-12f, (_Float16)-0x1.8p-12f}, hi = {(_Float16)0x1.8p-12f, (_Float16)0x1.8p-12f};
    f16x2 c = __builtin_bit_cast(f16x2, w) * down;
    c = __builtin_elementwise_max(c, lo);
    c = __builtin_elementwise_min(c, hi);
    return c * up;
}

// Both halves of x = kScale X as the int16 pair 2X: rint(32767 x) = rint(2X -
// X / 2^14), and |X / 2^14| < 3/8.
__device__ __forceinline__ v2s twice_x(f16x2 x)
{
    uint32_t r;
    asm("v_cvt_pknorm_i16_f16 %0, %1, %1 op_sel:[0,1,0]" : "=v"(r) : "v"(x));
    return __builtin_bit_cast(v2s, r);
}

// Raw input words of one lane's operand slices: for each axis and K-step j
// the 8 channels [16 j + 8 g, 16 j + 8 g + 8) of one pixel's axis block.
// Loaded one tile ahead of their use, so the load only moves them: a lane of
// half 1 whose channels lie past the block holds those of half 0 instead, which
// convert() leaves out of |X|^2 and the palette's zeros out of
// the products.  (Zeroing them here makes the load wait for its data at once:
// 165.6 against 149.4 us per frame at 1500 x 1600 fp32 with 12 harmonics, 80.7
// against 76.5 at fp16 with 4, 31.9 against 31.2 at 704 x 704 fp32 with 4.)
template <typename T, int F>
struct RawSlices {
    static constexpr int C = 2 * F;
    static constexpr int KS = kSteps<F>;
    static constexpr int kWords = 2 * (int)sizeof(T);      // of a slice
    // channels per load: the widest group that divides the axis block and is
    // aligned in it (16-byte loads for whole slices and F even fp32, else 8
    // bytes, or 4 for odd F in fp16), so that a group is a part of the block
    // or lies past it
    static constexpr int kG = C % 16 == 0 || C == 8 ? 8 : F % 2 == 0 ? 4 : 2;
    static constexpr int kGB = kG * (int)sizeof(T);        // its bytes
    static constexpr int kLoad = kGB < 16 ? kGB : 16;      // bytes of one load
    uint32_t w[2][KS][kWords];

    // `row` = first channel of the pixel, `yoff` = first channel of its y
    // block.  The embedding is 16-byte aligned, and so are the row and the y
    // block where D > 4F; where D = 4F their offsets are multiples of 2F
    // channels, so of kLoad bytes.
    __device__ __forceinline__ void load(const T *__restrict__ row, int yoff, int g)
    {
#pragma unroll
        for (int ax = 0; ax < 2; ax++)
#pragma unroll
            for (int j = 0; j < KS; j++)
#pragma unroll
                for (int q = 0; q < 8 / kG; q++) {
                    const int c0 = 16 * j + kG * q;            // of half 0; half 1's is 8 further
                    if (c0 >= C) continue;                     // of neither half: never read
                    uint32_t *dst = &w[ax][j][q * kGB / 4];
                    const T *src = row + ax * yoff + (c0 + 8 < C ? c0 + 8 * g : c0);
#pragma unroll
                    for (int k = 0; k < kGB / kLoad; k++) {
                        typedef uint32_t vec __attribute__((ext_vector_type(kLoad / 4)));
                        if constexpr (kLoad == 4) {
                            dst[0] = *reinterpret_cast<const uint32_t *>(__builtin_assume_aligned(src, 4));
                        } else {
                            const vec v =
                                reinterpret_cast<const vec *>(__builtin_assume_aligned(src, kLoad))[k];
#pragma unroll
                            for (int i = 0; i < kLoad / 4; i++) dst[k * kLoad / 4 + i] = v[i];
                        }
                    }
                }
    }

    // Operands of one axis (finite for any input); n2: this lane's part of
    // |X|^2 over its channels, times 4 for a binary16 input (below 2^32).
    __device__ __forceinline__ void convert(int ax, int g, AxisOp<T, F> &op, int &n2) const
    {
        int all = 0, half0 = 0;         // sums over channels of both halves, and over those that only half 0 has
#pragma unroll
        for (int j = 0; j < KS; j++) {
            if constexpr (sizeof(T) == 2) {
                u32x4 t = {};
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int c = 16 * j + 2 * q;
                    if (c >= C) continue;
                    const f16x2 x = scaled_pair(w[ax][j][q]);
                    const v2s x2 = twice_x(x);
                    int &sum = c + 8 < C ? all : half0;
                    sum = __builtin_amdgcn_sdot2(x2, x2, sum, false);
                    t[q] = __builtin_bit_cast(uint32_t, x);
                }
                op.a[0][j] = __builtin_bit_cast(f16x8, t);
            } else {
                // 768 = 1.5 2^9 has the spacing 2^-14 of kScale X, so the
                // multiply-add rounds 4096 v to X, and its low 16 bits are X
                constexpr float kM = 768.0f;
                u32x4 t = {}, u = {};
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int c = 16 * j + 2 * q;
                    if (c >= C) continue;
                    float x[2], r[2];
                    uint32_t b[2];
#pragma unroll
                    for (int i = 0; i < 2; i++) {
                        const float v = fminf(fmaxf(__uint_as_float(w[ax][j][2 * q + i]), -1.5f), 1.5f);
                        const float m = __builtin_fmaf(v, 4096.0f * kScale, kM);
                        b[i] = __float_as_uint(m);
                        x[i] = m - kM;
                    }
                    const v2s xi = __builtin_bit_cast(v2s, __builtin_amdgcn_perm(b[1], b[0], 0x05040100u));
                    int &sum = c + 8 < C ? all : half0;
                    sum = __builtin_amdgcn_sdot2(xi, xi, sum, false);
                    const auto lead = __builtin_amdgcn_cvt_pkrtz(x[0], x[1]);
                    r[0] = x[0] - (float)lead[0];
                    r[1] = x[1] - (float)lead[1];
                    t[q] = __builtin_bit_cast(uint32_t, lead);
                    u[q] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(r[0], r[1]));
                }
                op.a[0][j] = __builtin_bit_cast(f16x8, t);
                op.a[1][j] = __builtin_bit_cast(f16x8, u);
            }
        }
        n2 = C % 16 == 0 ? all : all + (g == 0 ? half0 : 0);
    }
};

// The operand that adds the norms: this lane's parts n of |X|^2 (convert) of
// both axes in fields of 10, 10 and the rest of the bits, as the binary16
// numbers 1024 + field (the two low ones, packed by or-ing the field into
// the mantissa) and the field itself (at most 576), then two ones for the
// palette's constants: slots x0 x1 y0 y1 x2 y2 1 1.
template <typename T>
__device__ __forceinline__ f16x8 norm_operand(uint32_t nx, uint32_t ny)
{
    constexpr int SH = sizeof(T) == 2 ? 2 : 0;
    auto low = [](uint32_t n) {
        return ((n >> SH) & 0x3ffu) | ((n << (6 - SH)) & 0x03ff0000u) | 0x64006400u;
    };
    const u32x4 w = {low(nx), low(ny),
                     __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz((float)(nx >> (20 + SH)),
                                                                             (float)(ny >> (20 + SH)))),
                     0x3c003c00u};
    return __builtin_bit_cast(f16x8, w);
}

// Operands of both axes of one tile.
template <typename T, int F>
struct PixOps {
    AxisOp<T, F> ax[2];
    f16x8 e;

    // Empty asm statements that take the converted operands, the last one
    // clobbering memory: the next tile's row loads, which follow it, issue
    // after the conversion and reuse the input registers (otherwise the
    // compiler hoists them above the conversion and copies 16 registers per
    // tile).
    __device__ __forceinline__ void from(const RawSlices<T, F> &raw, int g)
    {
        int nx, ny;
        raw.convert(0, g, ax[0], nx);
        raw.convert(1, g, ax[1], ny);
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
            for (int l = 0; l < AxisOp<T, F>::NL; l++)
#pragma unroll
                for (int j = 0; j < kSteps<F>; j++) __asm__ volatile("" : "+v"(ax[a].a[l][j]));
        __asm__ volatile("" : "+v"(nx), "+v"(ny) : : "memory");
        e = norm_operand<T>((uint32_t)nx, (uint32_t)ny);
    }
};

// Palette operand k of axis ax for lane `lane` (bin lane & 31, K slots 8 g ..
// 8 g + 7, g = lane >> 5).
template <int F>
__device__ __forceinline__ f16x8 palette_operand(const uint32_t *__restrict__ pop, int ax, int k, int lane)
{
    return *reinterpret_cast<const f16x8 *>(pop + (((ax * kAxisKinds<F> + k) * 64 + lane) * 4));
}

// Word group i (16 bytes) of the LDS palette operands [NX + 1][kAxisKinds]
// [64][16] for the x bins of the NX blocks from bx on (the last one again past
// the table) and the y bins of block by, from the table [axis]
// [kMaxBinBlocks][kPopKinds][64][16]; PLUS1: with the constants of S + 1
// instead of S.
template <int F, int NX, bool PLUS1>
__device__ __forceinline__ u32x4 pop_block(const uint32_t *__restrict__ pop, int i, int bx, int by)
{
    constexpr int kAxis = kAxisKinds<F> * 64;             // 16-byte groups per block
    const int part = i / kAxis, r = i % kAxis, k = r >> 6, ax = part == NX ? 1 : 0;
    const int blk = ax ? by : min(bx + part, kMaxBinBlocks - 1);
    const int kind = k == 0 ? 0 : k == 1 ? (PLUS1 ? 2 : 1) : k + 1;
    return reinterpret_cast<const u32x4 *>(pop)[((ax * kMaxBinBlocks + blk) * kPopKinds + kind) * 64 + (r & 63)];
}

// The accumulators A and R of one axis, kDistBase A + R = kScale S (or kScale
// (S + 1)).  PIX_ROWS: pixels are the MFMA rows (pass 1) or its columns
// (pass 2).
template <typename T, int F, bool PIX_ROWS>
__device__ __forceinline__ void axis_products(const AxisOp<T, F> &X, f16x8 e, const f16x8 (&P)[kAxisKinds<F>],
                                              f32x16 &A, f32x16 &R)
{
    const f32x16 z = {};
    auto mm = [](f16x8 px, f16x8 pal, f32x16 c) { return PIX_ROWS ? mfma16(px, pal, c) : mfma16(pal, px, c); };
    A = mm(e, P[0], z);
    R = mm(e, P[1], z);
#pragma unroll
    for (int j = 0; j < kSteps<F>; j++)
#pragma unroll
        for (int l = 0; l < AxisOp<T, F>::NL; l++) {
            A = mm(X.a[l][j], P[2 + 2 * j], A);
            R = mm(X.a[l][j], P[3 + 2 * j], R);
        }
}

// kScale fl32(S) (or S + 1): one rounding of the exact sum.
__device__ __forceinline__ float assemble(float A, float R) { return __builtin_fmaf(kBaseF, A, R); }

// Tiles [first, last) of workgroup b of nb when ntiles tiles are shared out
// in contiguous runs.
__device__ __forceinline__ void block_run(int ntiles, int b, int nb, int &first, int &last)
{
    first = (int)((int64_t)ntiles * b / nb);
    last = (int)((int64_t)ntiles * (b + 1) / nb);
}

// Tiles of a workgroup's run: wave w starts with tile first + w, later
// tiles come from an LDS counter (zeroed before the run) in taking order,
// tile first + waves + k for the k-th taker (wave-uniform).
__device__ __forceinline__ int take_tile(int *next, int lane, int first, int waves)
{
    int k = 0;
    if (lane == 0) k = atomicAdd(next, 1);
    return first + waves + __builtin_amdgcn_readfirstlane(k);
}

// ---------------------------------------------------------------------------
// Pass 1: recovery + soft voting
// ---------------------------------------------------------------------------
// Row stride (in 64-bit words) of the vote kernel's LDS histogram: one word
// of padding per row puts the 32 rows that one fold instruction touches
// (lanes = y bins, fixed x bin) into distinct banks.
constexpr int kHStride = kMfmaBins + 1;

// Tiles between two folds of a wave's limb sums: |nh lo| <= 2^14, so the
// middle accumulator grows by at most 2^15 per pixel, 2^20 per tile.
constexpr int kFoldTiles = 2047;

// LDS bytes of k_vote_mfma (nx x blocks per pass): the weight table, the 64-bit histograms,
// the palette operands, the slice prefix sums and counters; with the
// compaction folded in (FUSED), the workgroup's own participating pixels.
template <int F>
constexpr size_t kVoteLds(int nx, bool fused)
{
    return (size_t)kWKeys * 2 + nx * kMfmaBins * kHStride * 8 + (nx + 1) * (kPopBytes<F> / 2) + (kMaxSlices + 1) * 4 + 16 + (fused ? (size_t)kFusedMaxSeg * 4 : 0);
}

// Eight foreground values from pixel p0 on (p0 a multiple of 8), in two
// parts: load8_raw issues one (fp16) or two (fp32) 16-byte loads when the
// plane is 16-byte aligned and the eight lie below lim (zero words
// otherwise); load8_values gives the values, loading pixel by pixel below
// lim (0 beyond) where the vector loads do not apply.
template <typename T>
struct Raw8 {
    uint4 w[sizeof(T) / 2];
};
template <typename T>
__device__ __forceinline__ Raw8<T> load8_raw(const T *fg, int p0, int lim, bool vec)
{
    Raw8<T> r = {};
    if (vec && p0 + 8 <= lim) {
#pragma unroll
        for (int k = 0; k < (int)(sizeof(T) / 2); k++) r.w[k] = reinterpret_cast<const uint4 *>(fg + p0)[k];
    }
    return r;
}
template <typename T>
__device__ __forceinline__ void load8_values(const T *fg, int p0, int lim, bool vec, const Raw8<T> &r, float v[8])
{
    if (vec && p0 + 8 <= lim) {
        if constexpr (sizeof(T) == 2) {
            const uint32_t ww[4] = {r.w[0].x, r.w[0].y, r.w[0].z, r.w[0].w};
#pragma unroll
            for (int i = 0; i < 4; i++) {
                v[2 * i] = half_bits_to_float(ww[i] & 0xffffu);
                v[2 * i + 1] = half_bits_to_float(ww[i] >> 16);
            }
        } else {
#pragma unroll
            for (int k = 0; k < 2; k++) {
                v[4 * k] = __uint_as_float(r.w[k].x);
                v[4 * k + 1] = __uint_as_float(r.w[k].y);
                v[4 * k + 2] = __uint_as_float(r.w[k].z);
                v[4 * k + 3] = __uint_as_float(r.w[k].w);
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] = fg && p0 + i < lim ? load_scalar<T>(fg + p0 + i) : 0.0f;
    }
}

// The compaction folded into the vote launch (frames of up to kFusedMaxPixels
// pixels).  Workgroup b lists the participating pixels
// twice: those of its range b * seg_cap .. (b + 1) * seg_cap - 1 of the
// frame (seg_cap a multiple of 8) into list[b * seg_cap ..], their number
// into counts[b] -- the assignment launch reads these segments as its slices,
// in the frame's order -- and those of the slices of `slice` pixels (a
// multiple of 64) dealt to it in turn, in LDS, in any order: the pixels it
// votes on, spread over the frame so that the workgroups' shares of votes
// stay even.  Round r deals the slices G r .. G r + G - 1, slice G r + c to
// workgroup c, or with a rotation rot > 0 (G = 256, whole rounds) slice
// G r + ((b + rot r) mod G) to workgroup b, which moves a workgroup's slices
// across the columns of the frame from round to round.  The pixels outside the list
// get their final outputs here.  The launch also clears `hnext`, the
// histograms of the next frame.
struct FusedArgs {
    const void *fg;              // foreground plane (element type of the embedding), or null: every pixel
    float fg_thr;
    int32_t slice, seg_cap, rot;
    int32_t *list, *counts;
    int32_t *labels;
    float *score;
    unsigned long long *hnext;
    int32_t nnext;
};

// Waves per SIMD the register allocation must allow: three (one workgroup of
// 12 waves per compute unit) for fp16 inputs and fp32 ones with up to 8
// harmonics (1500 x 1500 fp32 with 8: 77.3 against 79.1 us per frame with two;
// 900 x 900 fp16 with 10: 38.7 against 40.0), two otherwise and for two
// blocks' accumulators (multi), which would spill.  Without a bound the
// compiler keeps the accumulators in a separate AGPR allocation and the
// kernel drops to one wave per SIMD.
template <typename T, int F>
constexpr int vote_waves(bool multi)
{
    return !multi && (F <= 8 || sizeof(T) == 2) ? 3 : 2;
}
// Waves per workgroup of the vote kernel: one workgroup per compute unit.
template <typename T, int F>
constexpr int vote_wpb(bool multi)
{
    return 4 * vote_waves<T, F>(multi);
}
//
// Every workgroup adds its histogram into one of the kReplicas vote
// histograms `hrep` (clear when the frame starts: an earlier launch cleared
// them); the assignment launch that follows sums them and extracts the
// peaks.  Workgroup 0 also resets the pixel counts of the centroid records,
// which the assignment launch accumulates.
// MULTI: grids above 32 x 32 bins, in passes over the workgroup's tiles of
// two x blocks and one y block each (a single block is compiled without the
// pass loop).  Each pass converts the input and weighs the y block anew, so
// two x blocks per pass take 3 weight sets and one conversion where single
// blocks take 4 and 2 (704 x 704 fp32 with 4 harmonics, 64 x 64 bins: 31.3
// against 40.3 us on a list made before the launch; 34.2 with the compaction).
// FUSED: the launch lists the participating pixels itself (FusedArgs); list
// and counts are then unused.
template <typename T, int F, bool MULTI, bool FUSED>
__global__ __launch_bounds__((vote_wpb<T, F>(MULTI) * 64)) __attribute__((amdgpu_waves_per_eu(vote_waves<T, F>(MULTI)))) void k_vote_mfma(
    const T *__restrict__ emb, int32_t dstride, int32_t yoff, const int32_t *__restrict__ list,
    const int32_t *__restrict__ counts, int32_t nslices, int32_t slice_px, int32_t npix, Tables tb, int32_t Bw,
    int32_t Bh, unsigned long long *__restrict__ hrep,
    cpe_centroid *__restrict__ cents, int32_t cap, FusedArgs fz)
{
    constexpr int kWpb = vote_wpb<T, F>(MULTI), NX = MULTI ? 2 : 1;
    constexpr int kBlockH = kMfmaBins * kHStride, kPopWords = (NX + 1) * (kPopBytes<F> / 2) / 4;
    // passes over the workgroup's tiles: NX x blocks and one y block each
    const int nbx = MULTI ? (Bw + kMfmaBins - 1) / kMfmaBins : 1, nby = MULTI ? (Bh + kMfmaBins - 1) / kMfmaBins : 1;
    const int npx = MULTI ? (nbx + NX - 1) / NX : 1;
    // All LDS is static, so that table addresses are compile-time constants.
    __shared__ __align__(16) unsigned char smem[kVoteLds<F>(NX, FUSED)];
    uint16_t *s_wt = reinterpret_cast<uint16_t *>(smem);                              // [kWKeys] int8 limb pairs
    unsigned long long *s_h = reinterpret_cast<unsigned long long *>(s_wt + kWKeys);  // [NX][32][kHStride], b * kHStride + a
    uint32_t *s_pop = reinterpret_cast<uint32_t *>(s_h + NX * kBlockH);              // palette operands: x blocks, y
    int *s_pref = reinterpret_cast<int *>(s_pop + kPopWords);                         // [kMaxSlices + 1]
    int *s_next = s_pref + kMaxSlices + 1;                                            // next tile of the run
    int *s_cnt = s_next + 1;                                                          // FUSED: [2] pixels listed (LDS, global)
    int *s_list = s_pref + kMaxSlices + 5;                                            // FUSED: [kFusedMaxSeg]

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int g = lane >> 5, ln = lane & 31;
    SliceLoad sl;
    int nlist = npix;
    if (!FUSED && list) slice_load(counts, nslices, sl);
    {
        constexpr int kThreads = kWpb * 64, kN = kWKeys / 8, kPer = (kN + kThreads - 1) / kThreads;
        u32x4 w[kPer];
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int i = k * kThreads + tid;
            w[k] = reinterpret_cast<const u32x4 *>(tb.wt_pk)[i < kN ? i : 0];
        }
        if constexpr (FUSED) {
            // While the table loads are in flight, two lists of the
            // participating pixels: (a) the assignment's, of this workgroup's
            // range lo .. hi-1 of the frame, in global memory, with the other
            // pixels' final outputs; (b) the vote's own, of its slices b,
            // b + G, ..., in LDS.  Both in steps of 64 lanes x 8 consecutive
            // pixels (b: slice r of the workgroup, chunk of 8 o, from lane
            // chunk 64 k + lane = r * slice / 8 + o), one step per wave at a
            // time (the code stays short: a launch fetches it cold, and
            // unrolling three steps measured 1.3 us slower per 640 x 640
            // frame); LDS counters hand out the positions.
            if (tid == 0) s_cnt[0] = s_cnt[1] = 0;
            __syncthreads();
            const int G = gridDim.x, b = blockIdx.x;
            const T *fgp = static_cast<const T *>(fz.fg);
            const bool vec = fgp && ((uintptr_t)fgp & 15u) == 0;
            const int lo = b * fz.seg_cap, hi = lo + fz.seg_cap < npix ? lo + fz.seg_cap : npix;
            const int steps_a = hi > lo ? (hi - lo + 511) >> 9 : 0;
            const int nsl = (npix + fz.slice - 1) / fz.slice;
            const int mine = b < nsl ? (nsl - 1 - b) / G + 1 : 0;
            const int csh = __builtin_ctz(fz.slice) - 3;                // log2 of the 8-pixel chunks per slice
            const int steps = steps_a + ((mine << csh) + 63) / 64;
            int32_t *seg = fz.list + (size_t)lo;
            // first pixel and limit of this lane's 8 in step j
            auto place = [&](int j, int &p0, int &lim) {
                if (j < steps_a) {
                    p0 = lo + j * 512 + lane * 8;
                    lim = hi;
                } else {
                    const int c = (j - steps_a) * 64 + lane, r = c >> csh;
                    const int sb = fz.rot ? (b + fz.rot * r) & (kMaxSlices - 1) : b;   // rot: G = kMaxSlices
                    p0 = (sb + G * r) * fz.slice + ((c & ((1 << csh) - 1)) << 3);
                    lim = r < mine ? npix : 0;
                }
            };
            // the next step's foreground words are loaded before this step's
            // are used
            int pn = 0, limn = 0;
            Raw8<T> rn = {};
            if (wv < steps) {
                place(wv, pn, limn);
                rn = load8_raw<T>(fgp, pn, limn, vec);
            }
            for (int j = wv; j < steps; j += kWpb) {
                const bool in_a = j < steps_a;                          // wave-uniform
                const int p0 = pn, lim = limn;
                const Raw8<T> rc = rn;
                if (j + kWpb < steps) {
                    place(j + kWpb, pn, limn);
                    rn = load8_raw<T>(fgp, pn, limn, vec);
                }
                float v[8];
                load8_values<T>(fgp, p0, lim, vec, rc, v);
                uint32_t m = 0, valid = 0;
#pragma unroll
                for (int i = 0; i < 8; i++) {
                    const bool in = p0 + i < lim;
                    valid |= (in ? 1u : 0u) << i;
                    m |= (in && (!fgp || v[i] > fz.fg_thr) ? 1u : 0u) << i;   // a NaN never exceeds it
                }
                const int c = __popc(m), incl = wave_incl_sum(c);
                const int tot = __builtin_amdgcn_readlane(incl, 63);
                int base = 0;
                if (lane == 0 && tot) base = atomicAdd(&s_cnt[in_a ? 1 : 0], tot);
                int off = __builtin_amdgcn_readfirstlane(base) + incl - c;
                if (in_a) {
#pragma unroll
                    for (int i = 0; i < 8; i++)
                        if ((m >> i) & 1u) seg[off++] = p0 + i;         // off < hi - lo <= seg_cap
                    const uint32_t bg = valid & ~m;
                    if (bg == 0xffu) {
                        const int4 z = {0, 0, 0, 0};
                        reinterpret_cast<int4 *>(fz.labels + p0)[0] = z;     // labels: 16-byte aligned
                        reinterpret_cast<int4 *>(fz.labels + p0)[1] = z;
                    } else if (bg) {
#pragma unroll
                        for (int i = 0; i < 8; i++)
                            if ((bg >> i) & 1u) fz.labels[p0 + i] = 0;
                    }
                    if (fz.score && bg) {
#pragma unroll
                        for (int i = 0; i < 8; i++)
                            if ((bg >> i) & 1u) fz.score[p0 + i] = 0.0f;
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; i++)
                        if ((m >> i) & 1u) s_list[off++] = p0 + i;      // off < the slices' pixels <= kFusedMaxSeg
                }
            }
            for (int i = b * kThreads + tid; i < fz.nnext; i += G * kThreads) fz.hnext[i] = 0ull;
        }
#pragma unroll
        for (int k = 0; k < kPer; k++) {
            const int i = k * kThreads + tid;
            if (i < kN) reinterpret_cast<u32x4 *>(s_wt)[i] = w[k];
        }
        for (int i = tid; i < NX * kBlockH; i += kThreads) s_h[i] = 0ull;
        for (int i = tid; i < kPopWords / 4; i += kThreads)
            reinterpret_cast<u32x4 *>(s_pop)[i] = pop_block<F, NX, true>(tb.pop, i, 0, 0);
        if (tid == 0) *s_next = 0;
        if (!FUSED && list) nlist = slice_scan(sl, nslices, s_pref);
    }
    __syncthreads();
    // the workgroup's run of tiles: a share of the list, or (FUSED) its own pixels
    const int n = FUSED ? *s_cnt : nlist, ntiles = (n + 31) >> 5;
    int t0, tend;
    if constexpr (FUSED) {
        t0 = 0;
        tend = ntiles;
        if (tid == 0) fz.counts[blockIdx.x] = s_cnt[1];
    } else {
        block_run(ntiles, blockIdx.x, gridDim.x, t0, tend);
    }

    i32x16 acc2[NX] = {}, acc1[NX] = {}, acc0[NX] = {};       // sums of nh nh, nh lo + lo nh, lo lo
    int ntile = 0;

    // Add the limb sums into the workgroup's histograms (this wave owns every
    // (a, b) exactly once, so its own atomics never collide).
    auto fold = [&]() {
#pragma unroll
        for (int x = 0; x < NX; x++)
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const long long v = (long long)acc2[x][r] * 65536 - (long long)acc1[x][r] * 256 + acc0[x][r];
                atomicAdd(&s_h[x * kBlockH + ln * kHStride + acc_row(r, g)], (unsigned long long)v);
                acc2[x][r] = acc1[x][r] = acc0[x][r] = 0;
            }
    };

    // Weight limbs (lo | nh << 8) of the 16 (pixel, bin) results of one block
    // (palette operands `part`): the binary32 bits of kScale (S + 1) give the
    // bucket.
    auto weights = [&](const AxisOp<T, F> &X, f16x8 e8, int part, uint32_t (&e)[16]) {
        f16x8 P[kAxisKinds<F>];
#pragma unroll
        for (int k = 0; k < kAxisKinds<F>; k++) P[k] = palette_operand<F>(s_pop, part, k, lane);
        f32x16 A, R;
        axis_products<T, F, true>(X, e8, P, A, R);
#pragma unroll
        for (int r = 0; r < 16; r++) e[r] = s_wt[(__float_as_uint(assemble(A[r], R[r])) >> 15) & (kWKeys - 1)];
    };
    // The 16 pixels of this lane as the bytes of two operands.
    struct Limbs {
        i32x4 lo, nh;
    };
    auto limbs = [](const uint32_t (&e)[16]) {
        u32x4 l, h;
#pragma unroll
        for (int s = 0; s < 4; s++) {
            const uint32_t w01 = e[4 * s] | e[4 * s + 1] << 16, w23 = e[4 * s + 2] | e[4 * s + 3] << 16;
            l[s] = __builtin_amdgcn_perm(w23, w01, 0x06040200u);
            h[s] = __builtin_amdgcn_perm(w23, w01, 0x07050301u);
        }
        return Limbs{__builtin_bit_cast(i32x4, l), __builtin_bit_cast(i32x4, h)};
    };

    // One tile of up to 32 pixels (queue slot m = lane & 31) from prefetched
    // input; `next` reuses the input registers once they are converted; nx: x
    // blocks of this pass.
    auto tile = [&](RawSlices<T, F> &raw, int nvalid, int nx, auto next) {
        PixOps<T, F> X;
        X.from(raw, g);
        next();
        uint32_t e[16];
        Limbs x[NX];
#pragma unroll
        for (int i = 0; i < NX; i++) {
            if (i > 0 && i >= nx) break;
            weights(X.ax[0], X.e, i, e);
            x[i] = limbs(e);
        }
        weights(X.ax[1], X.e, NX, e);
        if (nvalid < 32) {        // pixels past the end of the list vote nothing
            // (kept a real branch: only the last tile of a round is partial)
            __asm__ volatile("" ::: "memory");
#pragma unroll
            for (int r = 0; r < 16; r++)
                if (acc_row(r, g) >= nvalid) e[r] = 0u;
        }
        const Limbs y = limbs(e);
        // vote: K = the 16 pixels of this lane, one byte each
#pragma unroll
        for (int i = 0; i < NX; i++) {
            if (i > 0 && i >= nx) break;
            acc2[i] = mfma8(x[i].nh, y.nh, acc2[i]);
            acc1[i] = mfma8(x[i].nh, y.lo, acc1[i]);
            acc0[i] = mfma8(x[i].lo, y.lo, acc0[i]);
            acc1[i] = mfma8(x[i].lo, y.nh, acc1[i]);
        }
    };

    for (int blk = 0; blk < npx * nby; blk++) {
        const int bx = NX * (blk % npx), by = blk / npx, nx = min(NX, nbx - bx);
        if (MULTI && blk > 0) {
            // the next block: its palette operands, a clear histogram and tile
            // counter (the previous pass has flushed)
            for (int i = tid; i < NX * kBlockH; i += blockDim.x) s_h[i] = 0ull;
            for (int i = tid; i < kPopWords / 4; i += blockDim.x)
                reinterpret_cast<u32x4 *>(s_pop)[i] = pop_block<F, NX, true>(tb.pop, i, bx, by);
            if (tid == 0) *s_next = 0;
            __syncthreads();
        }
        int t = t0 + wv;
        ListCursor cur_list;
        if (!FUSED) cur_list.start(list, s_pref, nslices, slice_px, t < tend ? 32 * t : 0);
        // lane m of tile tt: entry 32 tt + m, or the tile's first entry past the end
        auto pixel = [&](int tt) {
            const int e = 32 * tt + ln < n ? 32 * tt + ln : 32 * tt;
            if constexpr (FUSED)
                return s_list[e];
            else
                return cur_list.pixel(e);
        };
        // the next tile's rows are loaded as soon as the current ones are converted
        RawSlices<T, F> raw;
        int tn = tend, idx = 0;                            // next tile, and this lane's pixel in it
        if (t < tend) {
            raw.load(emb + (size_t)pixel(t) * dstride, yoff, g);
            tn = take_tile(s_next, lane, t0, kWpb);
            if (tn < tend) idx = pixel(tn);
        }
        while (t < tend) {
            int tnn = tend;
            tile(raw, min(32, n - 32 * t), nx, [&]() {
                if (tn < tend) {
                    raw.load(emb + (size_t)idx * dstride, yoff, g);
                    tnn = take_tile(s_next, lane, t0, kWpb);
                    if (tnn < tend) idx = pixel(tnn);
                }
            });
            t = tn;
            tn = tnn;
            if (++ntile == kFoldTiles || t >= tend) {
                fold();
                ntile = 0;
            }
        }

        // one global atomic per bin of the block
        __syncthreads();
        const int nb = Bw * Bh;
        unsigned long long *dst = hrep + (size_t)(blockIdx.x % kReplicas) * nb;
        for (int i = tid; i < nx * kMfmaBins * kMfmaBins; i += blockDim.x) {
            const int x = i / (kMfmaBins * kMfmaBins), c = i % kMfmaBins, r = i / kMfmaBins % kMfmaBins;
            const int b = kMfmaBins * by + r, a = kMfmaBins * (bx + x) + c;
            const unsigned long long v = s_h[x * kBlockH + r * kHStride + c];
            if (a < Bw && b < Bh && v) atomicAdd(dst + b * Bw + a, v);
        }
        __syncthreads();
    }
    if (blockIdx.x == 0)
        for (int k = tid; k < cap; k += blockDim.x) cents[k].npix = 0;
}

// ---------------------------------------------------------------------------
// Pass 2: assignment + label write-out
// ---------------------------------------------------------------------------
// Distances of one tile and up to 32 slots (of which nslot hold candidates)
// from the accumulators into an array [slot][kKeyStride], scaled by 2^-7 (the
// root of kScale); dst: this lane's pixel in slot 4 g.
template <bool EXACT>
__device__ __forceinline__ void store_distances(const f32x16 &A, const f32x16 &R, int nslot, uint32_t *dst)
{
#pragma unroll
    for (int r4 = 0; r4 < 4; r4++) {
        if (8 * r4 >= nslot) break;                  // wave-uniform: no candidate in slots 8 r4 ..
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int r = 4 * r4 + i;
            const float x = assemble(A[r], R[r]);
            const float d = EXACT ? sqrt_cr(x) : __builtin_amdgcn_sqrtf(x);
            dst[kKeyStride * (8 * r4 + i)] = __float_as_uint(d);
        }
    }
}

// The candidate batches in LDS (k_peaks.hpp): n of them, padded to a multiple
// of 8 with batches of the far row, `real` before the padding.
struct Batches {
    const u32x4 *bo;
    const uint32_t *bh, *bk;
    int n, real;
};

// Where a tile's results go.  BIG: more candidates than cnt (LDS, kCountCap
// of them) may exist; the others are counted in their records.
template <bool BIG>
struct Labeller {
    int32_t *labels;
    float *score_map;
    double tau32;
    int32_t *cnt;
    cpe_centroid *cents;

    __device__ __forceinline__ void label(int pix, int k) const
    {
        labels[pix] = k + 1;
        if (!BIG || k < kCountCap)
            atomicAdd(cnt + k, 1);
        else
            atomicAdd(&cents[k].npix, 1);
    }
    // Label and score of pixel `pix`, whose nearest candidate k has the exact
    // distance sum D (Eq8).
    __device__ __forceinline__ void put(int pix, int k, double D) const
    {
        if (D < tau32) {
            label(pix, k);
            if (score_map) score_map[pix] = expf(-(float)(D * 0x1p-5));
        } else {
            labels[pix] = 0;
            if (score_map) score_map[pix] = 0.0f;
        }
    }
};

// Candidate search of one tile from the distance arrays; false, with
// nothing written, if a pixel is not decided.  Lane l serves the four
// pixels 4 q .. 4 q + 3 (q = l & 7) over the batches j, j + 8, ... (j =
// l >> 3): one 16-byte read fetches a column's distances of its four
// pixels, and the next batch's offsets are read ahead.  Per pixel it keeps
// the smallest binary32 sum s = fl(min x + y) of a batch and the second
// smallest, as keys: the bits of s (which order like the sums) with the
// batch's step in the low `bits`.  The first batch only initialises.
// The eight lanes of a pixel quad then merge in registers (half and row
// swaps that leave a lane two pixels, one, then a rotation within the row
// of 16), which leaves pixel m = 4 q + 2 (l >> 5) + (l >> 4 & 1) in lane l
// and the arrays intact.
//
// Let every x and y be within one binary32 step (at most 2^-23 of the
// value) of the correctly rounded root: the hardware's root is
// (cpe_check_sqrt tries every input).  Then x + y lies within relative 2^-23 of
// the exact sum, and s within g = 3 2^-24 + 2^-47 of the batch's true
// minimum D.  If every other batch's s exceeds the winner's s_w by
// kFastGap steps (each more than 2^-24 s_w), so by more than 2g / (1 - g)
// s_w, its D is strictly larger (a sum of 0 is exact: any other distance
// sum is at least 2^-7).  The keys show a gap of s less the step bits, hence as
// few of them as the frame's batches need (always 4: 0.30 % of the tiles of a
// 640 x 640 fp16 frame with outliers were undecided, with its 3 0.18 %; 1024 x
// 2048, 16 harmonics, 75.2 against 74.2 us).
// (Merging through LDS, with the batch in a register of its own per pixel
// and the binary64 sums in the exact kernel, took 43 VALU instructions per
// step instead of 31 and two LDS round trips more: 1024 x 2048, 16
// harmonics, fp16, 78.0 against 74.3 us per frame; 2160 x 3840 with 8
// 239 against 228.)
// Within the winning batch (one row, one y) a column 3 steps above the
// smallest is strictly farther.  So a decided pixel has the label of the
// exact sums.  EXACT (correctly rounded roots): the first column at the
// batch's smallest x is the nearest, and its D is exact.
template <bool EXACT, bool BIG>
__device__ __forceinline__ bool search_tile(const Batches &bt, const uint32_t *kx, const uint32_t *ky, int lane, int pix,
                                            int nvalid, int bits, int force_exact, const Labeller<BIG> &out)
{
    uint32_t sum_mask = ~0u << bits;
    __asm__ volatile("" : "+v"(sum_mask));  // a vector register: an instruction reads one scalar, the step
    __builtin_amdgcn_wave_barrier();
    int lo = lane;
    __asm__ volatile("" : "+v"(lo));        // recomputed per tile, not held across the loop
    const int q = lo & 7, j0 = lo >> 3;
    const unsigned char *kxq = reinterpret_cast<const unsigned char *>(kx + 4 * q);
    const unsigned char *kyq = reinterpret_cast<const unsigned char *>(ky + 4 * q);
    uint32_t b[4], s2[4];
    u32x4 o = bt.bo[j0];                     // j0 < 8 <= bt.n
    uint32_t hb = bt.bh[j0];
    // the sums of the batch at o, hb; then the offsets of batch `next`
    // (past the list: bytes of the arrays behind it, never used)
    auto keys = [&](int it, int next, uint32_t (&key)[4]) {
        const u32x4 v0 = *reinterpret_cast<const u32x4 *>(kxq + o.x);
        const u32x4 v1 = *reinterpret_cast<const u32x4 *>(kxq + o.y);
        const u32x4 v2 = *reinterpret_cast<const u32x4 *>(kxq + o.z);
        const u32x4 v3 = *reinterpret_cast<const u32x4 *>(kxq + o.w);
        const u32x4 yd = *reinterpret_cast<const u32x4 *>(kyq + hb);
        o = bt.bo[next];
        hb = bt.bh[next];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const uint32_t m = min(min(v0[e], v1[e]), min(v2[e], v3[e]));
            const uint32_t s = __float_as_uint(__uint_as_float(m) + __uint_as_float(yd[e]));
            key[e] = (s & sum_mask) | (uint32_t)it;
        }
    };
    keys(0, j0 + 8, b);
#pragma unroll
    for (int e = 0; e < 4; e++) s2[e] = 0x7f800000u;
    for (int it = 1; 8 * it < bt.n; it++) {
        uint32_t key[4];
        keys(it, 8 * it + 8 + j0, key);
#pragma unroll
        for (int e = 0; e < 4; e++) {
            s2[e] = max(min(b[e], s2[e]), min(max(b[e], s2[e]), key[e]));      // their median
            b[e] = min(b[e], key[e]);
        }
    }
    // merge (b, s2, lane j) of two parts of one pixel's batches
    struct Part {
        uint32_t b, s2, j;
    };
    auto merge = [](Part u, Part v) -> Part {
        Part r;
        r.j = v.b < u.b ? v.j : u.j;
        r.s2 = min(min(u.s2, v.s2), max(u.b, v.b));
        r.b = min(u.b, v.b);
        return r;
    };
    Part p[2];
#pragma unroll
    for (int e = 0; e < 2; e++) {           // pixel e in half 0, e + 2 in half 1; j bit 2
        const u32x2 bb = swap32(b[e], b[e + 2]), ss = swap32(s2[e], s2[e + 2]);
        p[e] = merge({bb[0], ss[0], (uint32_t)j0 & 3u}, {bb[1], ss[1], (uint32_t)j0 | 4u});
    }
    {                                       // pixel + 0 in even rows of 16, + 1 in odd ones; j bit 1
        const u32x2 bb = swap16(p[0].b, p[1].b), ss = swap16(p[0].s2, p[1].s2), jj = swap16(p[0].j, p[1].j);
        p[0] = merge({bb[0], ss[0], jj[0]}, {bb[1], ss[1], jj[1]});
    }
    p[0] = merge(p[0], {row_ror8(p[0].b), row_ror8(p[0].s2), row_ror8(p[0].j)});   // j bit 0
    const int m = 4 * q + 2 * (lo >> 5) + ((lo >> 4) & 1);
    const int pm = __shfl(pix, m);
    const int bi = (int)(8u * (p[0].b & ~sum_mask) + p[0].j);
    const u32x4 ow = bt.bo[bi];
    const int k0 = (int)bt.bk[bi];
    const unsigned char *kxl = reinterpret_cast<const unsigned char *>(kx + m);
    const uint32_t w0 = *reinterpret_cast<const uint32_t *>(kxl + ow.x);
    const uint32_t w1 = *reinterpret_cast<const uint32_t *>(kxl + ow.y);
    const uint32_t w2 = *reinterpret_cast<const uint32_t *>(kxl + ow.z);
    const uint32_t w3 = *reinterpret_cast<const uint32_t *>(kxl + ow.w);
    const uint32_t l01 = min(w0, w1), l23 = min(w2, w3), wm = min(l01, l23);
    const int k = k0 + (w0 == wm ? 0 : w1 == wm ? 1 : w2 == wm ? 2 : 3);
    bool amb = (p[0].s2 >> bits) - (p[0].b >> bits) < key_gap(kFastGap, bits);
    if constexpr (!EXACT) {
        const uint32_t second = min(min(max(w0, w1), max(w2, w3)), max(l01, l23));
        amb |= second - wm < 3u;
    }
    // one of the two lanes that hold the pixel
    const bool valid = (lo & 8) == 0 && m < nvalid;
    if (force_exact || __ballot(amb && valid)) return false;
    if (valid) {
        if constexpr (EXACT) {
            const uint32_t y = *reinterpret_cast<const uint32_t *>(
                reinterpret_cast<const unsigned char *>(ky + m) + bt.bh[bi]);
            const double D = (double)__uint_as_float(wm) + (double)__uint_as_float(y);
            out.put(pm, k, D);
        } else {
            out.label(pm, k);
        }
    }
    __builtin_amdgcn_wave_barrier();
    return true;
}

// The tiles that the search leaves undecided, from exact distances: lane
// m (either half: half g takes the batches g, g + 2, ...) scans every
// batch for pixel m.  The smallest x distance of a batch plus the row's y
// distance, summed exactly in binary64, has at least 12 zero bits at the
// bottom of its mantissa (both distances are 0 or binary32 values of at
// least 2^-7, so the sum is a multiple of 2^-30 below 2^10), which take the
// batch index (at most INDEX < 4096): one binary64 minimum selects the smallest sum and,
// on ties, the first batch, and its first column at the batch's minimum
// is the lowest candidate index.
template <uint32_t INDEX, bool BIG>
__device__ __forceinline__ void search_exact(const Batches &bt, const uint32_t *kx, const uint32_t *ky, int lane,
                                             int pix, int nvalid, const Labeller<BIG> &out)
{
    const int g = lane >> 5, ln = lane & 31;
    __builtin_amdgcn_wave_barrier();
    const unsigned char *kxl = reinterpret_cast<const unsigned char *>(kx + ln);
    const unsigned char *kyl = reinterpret_cast<const unsigned char *>(ky + ln);
    double best = __builtin_inf();
    for (int bi = g; bi < bt.real; bi += 2) {
        const u32x4 o = bt.bo[bi];
        const uint32_t w0 = *reinterpret_cast<const uint32_t *>(kxl + o.x);
        const uint32_t w1 = *reinterpret_cast<const uint32_t *>(kxl + o.y);
        const uint32_t w2 = *reinterpret_cast<const uint32_t *>(kxl + o.z);
        const uint32_t w3 = *reinterpret_cast<const uint32_t *>(kxl + o.w);
        const uint32_t yv = *reinterpret_cast<const uint32_t *>(kyl + bt.bh[bi]);
        const uint32_t m = min(min(w0, w1), min(w2, w3));
        const double sum = (double)__uint_as_float(m) + (double)__uint_as_float(yv);
        const unsigned long long sb = (unsigned long long)__double_as_longlong(sum);
        best = min_f64(best, __longlong_as_double((long long)((sb & ~0xffffffffull) | ((uint32_t)sb | (uint32_t)bi))));
    }
    best = min_f64(best, __shfl_xor(best, 32));
    const unsigned long long key = (unsigned long long)__double_as_longlong(best);
    const int bi = (int)((uint32_t)key & INDEX);
    const u32x4 o = bt.bo[bi];
    const uint32_t w0 = *reinterpret_cast<const uint32_t *>(kxl + o.x);
    const uint32_t w1 = *reinterpret_cast<const uint32_t *>(kxl + o.y);
    const uint32_t w2 = *reinterpret_cast<const uint32_t *>(kxl + o.z);
    const uint32_t w3 = *reinterpret_cast<const uint32_t *>(kxl + o.w);
    const uint32_t wm = min(min(w0, w1), min(w2, w3));
    if (g == 0 && ln < nvalid)
        out.put(pix, (int)bt.bk[bi] + (w0 == wm ? 0 : w1 == wm ? 1 : w2 == wm ? 2 : 3),
            __longlong_as_double((long long)(key & ~(unsigned long long)INDEX)));
    __builtin_amdgcn_wave_barrier();
}

// Waves per SIMD of the assignment kernel: four where the register
// allocation fits 128 registers without spilling (vector input slices and up
// to 9 harmonics, or fp16 with 16), three otherwise; one workgroup per
// compute unit.
template <typename T, int F>
constexpr int kAssignWaves = (F <= 9 || (sizeof(T) == 2 && F == 16)) ? 4 : 3;
template <typename T, int F>
constexpr int kAssignWpb = 4 * kAssignWaves<T, F>;

// LDS bytes of k_assign_mfma: palette operands, candidate batches, counts,
// per wave x and y distances [32 slots][kKeyStride] (u32) and the far row,
// then the peak-extraction state.  The summed vote histogram of
// the prologue (kPadHist counts, 9 KB) shares its bytes with the first waves'
// distance arrays, which are written only after it is no longer read.
constexpr int kWaveKeys = (2 * kMfmaBins + 1) * kKeyStride;    // words
template <int F>
constexpr size_t kAssignLdsCore(int wpb)
{
    return (size_t)kPopBytes<F> + (size_t)kMaxBatchLds * 24 + kMfmaBins * kMfmaBins * 4 +
           (size_t)wpb * kWaveKeys * 4 + sizeof(PeakLds) +
           (kMaxSlices + 1) * 4 + 16;
}
template <int F>
constexpr size_t kAssignLds(int wpb)
{
    return (kAssignLdsCore<F>(wpb) + 15) & ~(size_t)15;
}

// Every workgroup first sums the vote histograms `hcur` of the vote launch
// and extracts the peaks in LDS (identical in every workgroup); workgroup 0
// writes the centroid records (all fields but the pixel count), K and the
// summed histogram `hlast`.  This prologue is a chain of memory round trips
// and of code fetched cold, paid by every frame: with every wave scanning the
// slice counts for itself (its first list entries load before the first
// barrier), a bordered histogram instead of range checks and the candidates'
// indices kept with the batches (instead of a bin -> index table, two
// dependent LDS reads per labelled pixel) it takes 5.0 us at 640 x 640; the
// launch went from 9.8 to 7.9 us at 64 x 64 and from 18.7 to 17.1 us at 640 x
// 640, 16 harmonics, fp16.
//
// Then, per tile of 32 pixels, the distances of both axes for the candidate
// slots (palette entries of the slots' bins as the MFMA rows, so that each
// lane holds one pixel and 16 slots) go to LDS as binary32 bits, laid out
// [slot][kKeyStride] so that lane m finds pixel m's value of any slot at a
// fixed stride.
// The candidate search walks the batches of 4 columns of one row (see the
// search below).  A pixel is labelled iff its distance sum D (in units of
// 1/32, the scale of the distance arrays) is below tau32 = 32 tau (Eq8; +inf:
// every pixel).
template <typename T, int F, bool FAST>
__global__ __launch_bounds__((kAssignWpb<T, F> * 64)) __attribute__((amdgpu_waves_per_eu(kAssignWaves<T, F>))) void k_assign_mfma(
    const T *__restrict__ emb, int32_t dstride, int32_t yoff, const int32_t *__restrict__ list,
    const int32_t *__restrict__ counts, int32_t nslices, int32_t slice_px, int32_t npix, double tau32, Tables tb,
    const unsigned long long *__restrict__ hcur, unsigned long long *__restrict__ hlast, int32_t Bw, int32_t Bh, long long cut, int32_t cap,
    cpe_centroid *__restrict__ cents, int32_t *__restrict__ num, int32_t *__restrict__ labels,
    float *__restrict__ score_map, int32_t force_exact)
{
    constexpr int kWpb2 = kAssignWpb<T, F>;
    constexpr int kThreads = kWpb2 * 64;
    static_assert(kAssignLds<F>(kWpb2) <= 160 * 1024, "LDS of one compute unit");
    static_assert(kPadHist * 8 <= kWpb2 * kWaveKeys * 4, "the summed histogram fits in the waves' arrays");
    // All LDS is static, so that table addresses are compile-time constants.
    __shared__ __align__(16) unsigned char smem[kAssignLds<F>(kWpb2)];
    uint32_t *s_pop = reinterpret_cast<uint32_t *>(smem);                            // palette operands
    u32x4 *s_bo = reinterpret_cast<u32x4 *>(s_pop + kPopBytes<F> / 4);              // [kMaxBatchLds]
    uint32_t *s_bh = reinterpret_cast<uint32_t *>(s_bo + kMaxBatchLds);             // [kMaxBatchLds]
    uint32_t *s_bk = s_bh + kMaxBatchLds;                                            // [kMaxBatchLds]
    int32_t *s_cnt = reinterpret_cast<int32_t *>(s_bk + kMaxBatchLds);              // [1024]
    uint32_t *s_keys = reinterpret_cast<uint32_t *>(s_cnt + kMfmaBins * kMfmaBins); // [kWpb2][kWaveKeys]
    PeakLds &pl = *reinterpret_cast<PeakLds *>(s_keys + kWpb2 * kWaveKeys);
    int *s_pref = reinterpret_cast<int *>(&pl + 1);                                  // [kMaxSlices + 1]
    int *s_next = s_pref + kMaxSlices + 1;                                            // next tile of the run
    long long *s_h = reinterpret_cast<long long *>(s_keys);                          // [kPadHist] summed votes

    const int tid = threadIdx.x, lane = tid & 63;
    // a scalar in the fast kernel, which otherwise spills with fp32 inputs and 8
    // harmonics (704 x 704 without a plane: 45.6 against 45.2 us)
    const int wv = FAST ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
    const int g = lane >> 5, ln = lane & 31;

    // Loads, in the order in which they are waited for: the slice counts (on
    // which the first tile's list entries and then its rows depend), the
    // vote counts, the palette operands.
    SliceLoad sl;
    if (list) slice_load(counts, nslices, sl);
    PeakBins<kWpb2> pb;
    pb.load(hcur, Bw, Bh);
    // workgroup 0 writes the records: the bin centres it needs, loaded now
    float cx[PeakBins<kWpb2>::N], cy[PeakBins<kWpb2>::N];
#pragma unroll
    for (int u = 0; u < PeakBins<kWpb2>::N; u++) {
        int a, b;
        const bool in = PeakBins<kWpb2>::pair(u, a, b) && blockIdx.x == 0 && a < Bw && b < Bh;
        cx[u] = in ? tb.cx[a] : 0.0f;
        cy[u] = in ? tb.cy[b] : 0.0f;
    }
    constexpr int kPopPer = (kPopBytes<F> / 16 + kThreads - 1) / kThreads;
    u32x4 pop[kPopPer];
#pragma unroll
    for (int k = 0; k < kPopPer; k++) {
        const int i = k * kThreads + tid;
        pop[k] = pop_block<F, 1, false>(tb.pop, i < kPopBytes<F> / 16 ? i : 0, 0, 0);
    }
    // This wave's search arrays, [slot][kKeyStride] per axis: x key of column
    // slot j, pixel m at kx[j * kKeyStride + m], y distance of row slot j at
    // ky[...].
    uint32_t *kx = s_keys + wv * kWaveKeys;
    uint32_t *ky = kx + kMfmaBins * kKeyStride;
    for (int i = tid; i < kMfmaBins * kMfmaBins; i += kThreads) s_cnt[i] = 0;
    if (tid == 0) *s_next = 0;

    // the workgroup's run of tiles of 32 list entries; the first tile's list
    // entries and rows are loaded while the peaks are extracted
    const int n = list ? slice_scan(sl, nslices, s_pref) : npix, ntiles = (n + 31) >> 5;
    int t0, tend;
    block_run(ntiles, blockIdx.x, gridDim.x, t0, tend);
    int t = t0 + wv;
    ListCursor cur_list;
    cur_list.start(list, s_pref, nslices, slice_px, t < tend ? 32 * t : 0);
    // lane m of tile tt: entry 32 tt + m, or the tile's first entry past the end
    auto pixel = [&](int tt) { return cur_list.pixel(32 * tt + ln < n ? 32 * tt + ln : 32 * tt); };
    RawSlices<T, F> raw;
    int ip = t < tend ? pixel(t) : 0;                   // this lane's pixel in this tile
    pb.store(s_h, Bw, Bh);
#pragma unroll
    for (int k = 0; k < kPopPer; k++) {
        const int i = k * kThreads + tid;
        if (i < kPopBytes<F> / 16) reinterpret_cast<u32x4 *>(s_pop)[i] = pop[k];
    }
    __syncthreads();
    peaks_lds_find<kWpb2>(pb, cut, cap, s_h, pl, s_bo, s_bh, s_bk, [&]() {
        if (t < tend) raw.load(emb + (size_t)ip * dstride, yoff, g);
    });
    // s_h is read; its bytes become distance arrays, each with its far row
    if (lane < 32) kx[2 * kMfmaBins * kKeyStride + lane] = kFarBits;
    const int Kc = pl.Kc;
    if (blockIdx.x == 0) {
#pragma unroll
        for (int u = 0; u < PeakBins<kWpb2>::N; u++) {
            int a, b;
            if (!PeakBins<kWpb2>::pair(u, a, b) || a >= Bw || b >= Bh) continue;
            const uint32_t m = pl.rowmask[b];
            hlast[b * Bw + a] = (unsigned long long)pb.sum[u];
            if ((m >> a) & 1u) {
                // npix was reset by the vote launch and is counted below
                cpe_centroid *c = cents + pl.rowfirst[b] + __popc(m & ((1u << a) - 1u));
                c->bin_x = a;
                c->bin_y = b;
                c->x = cx[u];
                c->y = cy[u];
                c->score = (double)pb.sum[u] * 0x1p-30;
                c->reserved = 0;
            }
        }
        if (tid == 0) *num = pl.K;
    }

    if (Kc == 0) {              // no centroid: every participating pixel is unlabelled
        ListCursor c0;
        c0.start(list, s_pref, nslices, slice_px, 32 * t0 + 64 * wv < n ? 32 * t0 + 64 * wv : 0);
        for (int i = 32 * t0 + tid; i < min(32 * tend, n); i += kThreads) {
            const int p = c0.pixel(i);
            labels[p] = 0;
            if (score_map) score_map[p] = 0.0f;
        }
        return;
    }
    const int nbat = __builtin_amdgcn_readfirstlane(min(pl.nbat, kMaxBatchLds));    // a multiple of kBatchPad
    const int bits = step_bits(nbat);

    // The MFMA rows are the candidate slots: the palette operands of slot j's
    // bin, gathered once and kept in registers for the whole run; distances
    // are computed only for the groups of 8 slots that hold candidates.
    const int nslot[2] = {__builtin_amdgcn_readfirstlane(pl.ncol), __builtin_amdgcn_readfirstlane(pl.nrow)};
    // (the fast kernel reads them from LDS per tile: its search needs the
    // registers)
    const int slotbin[2] = {g * 32 + pl.colbin[ln], g * 32 + pl.rowbin[ln]};
    constexpr bool kPalRegs = !FAST && kSteps<F> == 1;
    f16x8 popr[2][kAxisKinds<F>];
    if constexpr (kPalRegs) {
#pragma unroll
        for (int ax = 0; ax < 2; ax++)
#pragma unroll
            for (int k = 0; k < kAxisKinds<F>; k++) popr[ax][k] = palette_operand<F>(s_pop, ax, k, slotbin[ax]);
    }

    // Distances of one tile (pixel m = lane & 31; this lane's 16 slots
    // acc_row(r, g) of each axis), scaled by 2^-7 (the root of kScale);
    // `next` reuses the input registers once they are converted.  EXACT: the
    // correctly rounded square root of fl32(S); otherwise the hardware square
    // root, within one binary32 step of it (the fast search below).
    auto distances = [&](auto exact, RawSlices<T, F> &raw, auto next) {
        PixOps<T, F> X;
        X.from(raw, g);
        next();
#pragma unroll
        for (int ax = 0; ax < 2; ax++) {
            f16x8 pop[kAxisKinds<F>];
#pragma unroll
            for (int k = 0; k < kAxisKinds<F>; k++)
                pop[k] = kPalRegs ? popr[ax][k] : palette_operand<F>(s_pop, ax, k, slotbin[ax]);
            f32x16 A, R;
            axis_products<T, F, false>(X.ax[ax], X.e, pop, A, R);
            store_distances<decltype(exact)::value>(A, R, nslot[ax], (ax ? ky : kx) + 4 * g * kKeyStride + ln);
        }
    };

    const Batches bt{s_bo, s_bh, s_bk, nbat, min(pl.nbat_real, kMaxBatchLds)};
    const Labeller<false> out{labels, score_map, tau32, s_cnt, nullptr};

    // the next tile's rows are loaded as soon as the current ones are converted
    int tn = tend, ipn = 0;                             // next tile; this lane's pixel in it
    if (t < tend) {
        tn = take_tile(s_next, lane, t0, kWpb2);
        if (tn < tend) ipn = pixel(tn);
    }
    while (t < tend) {
        int tnn = tend, ipnn = 0;
        auto next = [&]() {
            if (tn < tend) {
                raw.load(emb + (size_t)ipn * dstride, yoff, g);
                tnn = take_tile(s_next, lane, t0, kWpb2);
                if (tnn < tend) ipnn = pixel(tnn);
            }
        };
        const int nvalid = min(32, n - 32 * t);
        if constexpr (FAST) {
            distances(std::false_type{}, raw, next);
            if (!search_tile<false>(bt, kx, ky, lane, ip, nvalid, bits, force_exact, out)) {
                raw.load(emb + (size_t)ip * dstride, yoff, g);          // this tile's rows again
                distances(std::true_type{}, raw, []() {});
                if (tn < tend) raw.load(emb + (size_t)ipn * dstride, yoff, g);   // the next tile's rows again
                search_exact<127>(bt, kx, ky, lane, ip, nvalid, out);
            }
        } else {
            distances(std::true_type{}, raw, next);
            if (!search_tile<true>(bt, kx, ky, lane, ip, nvalid, bits, force_exact, out))
                search_exact<127>(bt, kx, ky, lane, ip, nvalid, out);
        }
        t = tn;
        tn = tnn;
        ip = ipn;
        ipn = ipnn;
    }
    __syncthreads();
    for (int i = tid; i < Kc && i < kMfmaBins * kMfmaBins; i += kThreads)
        if (s_cnt[i]) atomicAdd(&cents[i].npix, s_cnt[i]);
}

}  // namespace cpe
