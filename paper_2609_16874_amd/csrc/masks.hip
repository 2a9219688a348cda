// masks.hip -- binary instance masks M^_m (Eq8) from a label map.
//
// masks[m][p] = (labels[p] == first + m + 1) as one byte.  The work is one
// read of the labels per group of kMaskGroup masks and count * H * W bytes of
// mask stores, so it is bound by the HBM write rate.  A lane turns 16
// consecutive labels into 16 bytes whose bit i says "mask m0 + i", packed in
// four words; a mask's 16 bytes are then a shift and an `and` per word, and one
// 16-byte store.  The stores are non-temporal (the masks are not read back by
// this library).
//
// When H * W is no multiple of 16, mask m starts `off` bytes past a 128-byte
// line, another off for every mask.  A workgroup then stores whole lines of each
// mask (but for the mask's first and last, which it shares with its
// neighbours): it keeps the bytes of its pixels and of the 128 before them in
// LDS, and a lane cuts its 16 out of two aligned reads.
#include <hip/hip_runtime.h>

#include "cpe_decoder.hpp"

namespace cpe {
namespace {

constexpr int kMaskGroup = 8;     // masks per thread (grid.y = groups): the bits of a byte
constexpr int kMaskThreads = 256;

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4m __attribute__((ext_vector_type(4)));

constexpr int kLine = 128;
constexpr int kMaskSpan = 16 * kMaskThreads;     // bytes of a mask per workgroup

// byte j of the result = 1 << (v[j] - base), 0 if that is no bit of a byte
__device__ __forceinline__ uint32_t one_hot(i32x4 v, int32_t base)
{
    uint32_t b[4];
#pragma unroll
    for (int j = 0; j < 4; j++) b[j] = 1u << min((uint32_t)v[j] - (uint32_t)base, 8u);
    const uint32_t lo = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u), hi = __builtin_amdgcn_perm(b[3], b[2], 0x04000c0cu);
    return lo | hi;
}

// 16 labels from labels[p] on (0, no mask's, outside the map), and their bytes;
// bit i: label base + i.
struct Piece {
    i32x4 l[4];

    __device__ __forceinline__ void load(const int32_t *__restrict__ labels, int64_t p, int64_t npix)
    {
#pragma unroll
        for (int q = 0; q < 4; q++) l[q] = i32x4{};
        if (p < 0 || p >= npix) return;
        const int32_t *src = labels + p;
        if (p + 16 <= npix) {
#pragma unroll
            for (int q = 0; q < 4; q++) l[q] = reinterpret_cast<const i32x4 *>(src)[q];
        } else {
            // unconditional loads: behind a condition each would be waited
            // for before the next is issued
            const int last = (int)(npix - 1 - p);
#pragma unroll
            for (int i = 0; i < 16; i++) l[i >> 2][i & 3] = src[min(i, last)];
#pragma unroll
            for (int i = 0; i < 16; i++)
                if (i > last) l[i >> 2][i & 3] = 0;
        }
    }
    __device__ __forceinline__ u32x4m hot(int32_t base) const
    {
        u32x4m w;
#pragma unroll
        for (int q = 0; q < 4; q++) w[q] = one_hot(l[q], base);
        return w;
    }
};

__device__ __forceinline__ u32x4m mask_bytes(u32x4m w, int bit)
{
#pragma unroll
    for (int i = 0; i < 4; i++) w[i] = (w[i] >> bit) & 0x01010101u;
    return w;
}

// H W a multiple of 16
__global__ __launch_bounds__(kMaskThreads) void k_masks16(const int32_t *__restrict__ labels, int64_t npix,
                                                         int32_t first, int32_t count, uint8_t *__restrict__ masks)
{
    const int64_t p = ((int64_t)blockIdx.x * kMaskThreads + threadIdx.x) * 16;
    const int m0 = (int)blockIdx.y * kMaskGroup, m1 = min(m0 + kMaskGroup, (int)count);
    if (p >= npix) return;
    Piece l;
    l.load(labels, p, npix);
    const u32x4m w = l.hot(first + m0 + 1);
    for (int m = m0; m < m1; m++)
        __builtin_nontemporal_store(mask_bytes(w, m - m0), reinterpret_cast<u32x4m *>(masks + (int64_t)m * npix + p));
}

// Any H W: the workgroup's span starts kMaskSpan blockIdx.x bytes after the line
// that mask m starts in.  Bound by the instructions per 16 bytes as much as by
// the stores, so a wave whose pieces all lie inside every mask tests nothing.
// 1025 x 2047, 64 masks: 23.2 us against 37.4 with one pixel per thread.
__global__ __launch_bounds__(kMaskThreads) void k_masks_any(const int32_t *__restrict__ labels, int64_t npix,
                                                           int32_t first, int32_t count, uint8_t *__restrict__ masks)
{
    __shared__ u32x4m s_hot[(kLine + kMaskSpan) / 16 + 1];     // of the pixels from p0 - kLine on
    const int t = threadIdx.x;
    const int64_t p0 = (int64_t)blockIdx.x * kMaskSpan;
    const int m0 = (int)blockIdx.y * kMaskGroup, m1 = min(m0 + kMaskGroup, (int)count);
    if (p0 - kLine >= npix) return;
    Piece before, own;
    if (t < kLine / 16) before.load(labels, p0 - kLine + 16 * t, npix);
    own.load(labels, p0 + 16 * t, npix);
    if (t < kLine / 16) s_hot[t] = before.hot(first + m0 + 1);
    s_hot[kLine / 16 + t] = own.hot(first + m0 + 1);
    __syncthreads();
    const int lane = t & 63, w0 = 16 * (t - lane);                   // the wave's part of the span
    const bool inside = __builtin_amdgcn_readfirstlane((int)(p0 + w0 >= kLine && p0 + w0 + 16 * 64 <= npix)) != 0;
    const uint8_t *hot = reinterpret_cast<const uint8_t *>(s_hot) + kLine;   // of pixel p0
    for (int m = m0; m < m1; m++) {
        uint8_t *const dst = masks + (int64_t)m * npix;
        const int off = (int)((uintptr_t)dst & (kLine - 1));
        // 16 bytes from the span's byte 16 t - off on: the aligned words that
        // hold them, shifted by whole bytes (one word more than needed if
        // there is no shift: the array's last, never used)
        const uint32_t *w = reinterpret_cast<const uint32_t *>(hot + 16 * t) - ((off + 3) >> 2);
        u32x4m v;
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] = __builtin_amdgcn_alignbyte(w[i + 1], w[i], (uint32_t)-off & 3u);
        v = mask_bytes(v, m - m0);
        const int64_t at = p0 + 16 * t - off;                        // their first pixel
        if (inside || (at >= 0 && at + 16 <= npix))
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4m *>(dst - off + p0 + 16 * t));
        if (inside) continue;
        // the bytes before the mask's first aligned 16 and after its last, a lane each
        const int head = -off & 15, tail = (int)((off + npix) & 15);
        if (p0 + w0 == 0 && lane < head && lane < npix) dst[lane] = (hot[lane] >> (m - m0)) & 1;
        const int64_t last = npix - tail;
        if (last - (p0 - off + w0) >= 0 && last - (p0 - off + w0) < 16 * 64 && lane < tail && last + lane >= 0)
            dst[last + lane] = (hot[(int)(last - p0) + lane] >> (m - m0)) & 1;
    }
}

}  // namespace

cpe_status launch_masks(hipStream_t stream, const int32_t *labels, int64_t npix, int32_t first, int32_t count,
                        uint8_t *masks)
{
    const unsigned groups = (unsigned)((count + kMaskGroup - 1) / kMaskGroup);
    auto launch = [&](auto kernel, int64_t bytes) {
        // a multiple of eight workgroups per group of masks: workgroups go to
        // the eight XCDs in turn, so that every group's workgroup of a span
        // finds its labels in the same L2 (1025 x 2047, 64 masks: 28.2 us with
        // 513 workgroups, 23.1 with 520)
        const int64_t spans = (bytes + kMaskSpan - 1) / kMaskSpan;
        const dim3 grid((unsigned)((spans + 7) / 8 * 8), groups);
        hipLaunchKernelGGL(kernel, grid, dim3(kMaskThreads), 0, stream, labels, npix, first, count, masks);
    };
    if (npix % 16 == 0)
        launch(k_masks16, npix);
    else
        launch(k_masks_any, npix + kLine - 1);      // of a mask that starts at the end of a line
    return hipGetLastError() == hipSuccess ? CPE_OK : CPE_ERR_HIP;
}

}  // namespace cpe
