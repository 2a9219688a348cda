// k_peaks.hpp -- local-maxima search and compaction (Section 3.2, "Local
// Maxima Search").
//
// A bin is a candidate centroid when its vote count exceeds the threshold and
// every in-range 8-neighbour; candidates are numbered in ascending bin order
// b * B_w + a (wave ballots and a prefix sum over the waves).  Two forms:
//
//   peaks_lds     grids up to 32 x 32: run by every workgroup of the
//                 matrix-core assignment kernel in its prologue, entirely in
//                 LDS, as candidate masks of the rows and the candidate
//                 batches of the assignment search.
//   k_peaks       larger grids: a stand-alone kernel between the vote and
//                 the assignment kernels; it writes the records, K, the
//                 summed histogram and the assignment's plan to memory.
//
// Candidate batches.  The first min(K, cap) candidates are grouped by row b
// into batches of 4 columns (a row's last batch is filled with the far row,
// which never attains a minimum).  Batch i is bo[i] = the byte offsets
// 128 j of its 4 column slots j in the assignment kernel's [slot][32 pixels]
// x array, bh[i] the byte offset of its row's slot in the y array, and bk[i]
// the index of its first candidate.  The list is padded to a multiple of 8
// batches of the far row.
#pragma once

#include <type_traits>

#include "cpe_common.hpp"

namespace cpe {

typedef uint32_t u32x4_pk __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Grids up to 32 x 32: candidates in LDS, in the assignment kernel's prologue
// ---------------------------------------------------------------------------
// A wave owns pairs of rows: pair p (rows 2 p and 2 p + 1) belongs to wave p
// mod waves, lane l holding column l & 31 of row 2 p + (l >> 5), so that one
// ballot is the candidate mask of both rows.
constexpr int kLdsPeakBins = 32;
constexpr int kMaxBatchLds = 128;   // <= 16 strict maxima per row of 32 -> <= 4 batches per row
constexpr int kBatchPad = 8;        // the batch list is padded to a multiple of this
constexpr int kKeyStride = 32;      // words per bin row of the assignment kernel's key arrays
// Byte offsets of the far row, kFarBits (2^126) for every pixel, which follows
// the x and y arrays of 32 slots each: from the x and from the y array.
constexpr uint32_t kFarX = 2 * 32 * 4 * kKeyStride, kFarY = kFarX / 2;
constexpr uint32_t kFarBits = 0x7e800000u;
constexpr int kPadRow = kLdsPeakBins + 2;                  // the summed histogram in LDS: rows of 34 counts,
constexpr int kPadHist = kPadRow * (kLdsPeakBins + 2);     //   a border of -1 around the 32 x 32 bins

// LDS of peaks_lds (the summed histogram may alias any scratch the caller
// does not need until the peaks are known).
struct PeakLds {
    uint32_t rowmask[kLdsPeakBins];   // bit a of row b: (a, b) is one of the first min(K, cap) candidates
    int rowfirst[kLdsPeakBins];       // index of row b's first candidate
    int K, Kc, nbat;                  // nbat: batches, padded to a multiple of kBatchPad
    int nbat_real;                    // batches before the padding
    int ncol, nrow;                   // candidate columns and rows
    uint8_t colbin[kLdsPeakBins];     // column of column slot j (ascending; 0 past ncol)
    uint8_t rowbin[kLdsPeakBins];     // row of row slot j (ascending; 0 past nrow)
};

// This thread's bins (one per row pair of its wave, WAVES waves): the vote
// counts of the kReplicas histograms `hsrc` ([kReplicas][Bh][Bw], written by
// the previous launch), and their sum.  The loads are issued first, so that
// their latency overlaps the caller's table staging.
template <int WAVES>
struct PeakBins {
    static constexpr int N = (kLdsPeakBins / 2 + WAVES - 1) / WAVES;
    unsigned long long v[N][kReplicas];
    long long sum[N];

    __device__ __forceinline__ static bool pair(int u, int &a, int &b)
    {
        const int tid = threadIdx.x, p = (tid >> 6) + u * WAVES;
        a = tid & 31;
        b = 2 * p + ((tid >> 5) & 1);
        return p < kLdsPeakBins / 2;          // wave-uniform
    }
    __device__ __forceinline__ void load(const unsigned long long *__restrict__ hsrc, int Bw, int Bh)
    {
#pragma unroll
        for (int u = 0; u < N; u++) {
            int a, b;
            const bool in = pair(u, a, b) && a < Bw && b < Bh;
#pragma unroll
            for (int r = 0; r < kReplicas; r++) v[u][r] = in ? hsrc[(size_t)r * Bw * Bh + b * Bw + a] : 0ull;
        }
    }
    // The sums into s_h [kPadHist], -1 in the border and past the grid.
    __device__ __forceinline__ void store(long long *s_h, int Bw, int Bh)
    {
#pragma unroll
        for (int u = 0; u < N; u++) {
            int a, b;
            if (!pair(u, a, b)) continue;
            unsigned long long s = 0;
#pragma unroll
            for (int r = 0; r < kReplicas; r++) s += v[u][r];
            sum[u] = a < Bw && b < Bh ? (long long)s : -1;
            s_h[(b + 1) * kPadRow + a + 1] = sum[u];
        }
        const int i = threadIdx.x, c = i < 2 * kPadRow ? i % kPadRow : 0;
        if (i < 2 * kPadRow)
            s_h[(i < kPadRow ? 0 : (kPadRow - 1) * kPadRow) + c] = -1;
        else if (i < 2 * kPadRow + 2 * kLdsPeakBins)
            s_h[((i - 2 * kPadRow) / 2 + 1) * kPadRow + (i & 1) * (kPadRow - 1)] = -1;
    }
};

// The extraction, called by every thread of the block after a barrier that
// publishes s_h: the candidate masks of the rows, then the column and row
// slots and the candidate batches s_bo / s_bh / s_bk (pl.nbat of them, a
// multiple of kBatchPad; s_bk[i] = index of batch i's first candidate, so
// column c of the batch is candidate s_bk[i] + c).  Everything follows from
// the row masks: the candidates are in bin order, so a row's are consecutive.
// `mid` runs after the first barrier (the caller's independent work, e.g.
// loads whose latency the extraction hides).  A cold launch pays for the
// instruction fetch of this code about as much as for its execution, hence
// the border instead of range checks, and one bin per lane.
template <int WAVES, typename Mid>
__device__ __forceinline__ void peaks_lds_find(const PeakBins<WAVES> &pb, long long cut, int cap,
                                               const long long *s_h, PeakLds &pl, u32x4_pk *s_bo, uint32_t *s_bh,
                                               uint32_t *s_bk, Mid mid)
{
    const int tid = threadIdx.x, lane = tid & 63;
#pragma unroll
    for (int u = 0; u < PeakBins<WAVES>::N; u++) {
        int a, b;
        if (!PeakBins<WAVES>::pair(u, a, b)) continue;
        const long long v = pb.sum[u], *q = s_h + b * kPadRow + a;      // the corner of its neighbourhood
        bool f = v > cut;                                              // cut >= -1: false past the grid
#pragma unroll
        for (int n = 0; n < 9; n++)
            if (n != 4) f &= v > q[(n / 3) * kPadRow + n % 3];
        const unsigned long long m = __ballot(f);
        if (lane == 0) {
            pl.rowmask[b] = (uint32_t)m;
            pl.rowmask[b + 1] = (uint32_t)(m >> 32);
        }
    }
    __syncthreads();
    mid();
    // Slots: the candidate columns and rows, each numbered in ascending
    // order; the assignment computes distances for slots only, and its
    // arrays and batches are indexed by slot.  Lane b of the first wave owns
    // row b: it cuts the row's candidates off at `cap`, numbers column b and
    // row b and builds the row's batches (strict maxima are never
    // horizontally adjacent: <= 16 per row, <= 4 batches).
    if (tid < 64) {
        const int b = tid;
        uint32_t m = b < kLdsPeakBins ? pl.rowmask[b] : 0u;
        const int c = __popc(m), upto = wave_incl_sum(c), first = upto - c;    // the whole first wave is active
        const int K = __builtin_amdgcn_readlane(upto, kLdsPeakBins - 1);
        for (int over = min(upto - cap, c); over > 0; over--) m &= ~(0x80000000u >> __clz(m));
        const uint32_t cm = wave_or32(m);
        const unsigned long long rows = __ballot(m != 0u);
        const int rslot = lane_prefix(rows);                         // slot of row b if it holds candidates
        if (b < kLdsPeakBins) {
            pl.rowmask[b] = m;
            pl.rowfirst[b] = first;
            pl.colbin[b] = 0;
            pl.rowbin[b] = 0;
        }
        __builtin_amdgcn_wave_barrier();
        if (b < kLdsPeakBins && ((cm >> b) & 1u)) pl.colbin[__popc(cm & ((1u << b) - 1u))] = (uint8_t)b;
        if (m) pl.rowbin[rslot] = (uint8_t)b;
        const int nbt = (__popc(m) + 3) >> 2;
        const int incl = wave_incl_sum(nbt);
        const int start = incl - nbt, total = __builtin_amdgcn_readlane(incl, kLdsPeakBins - 1);
        const int padded = (total + kBatchPad - 1) & ~(kBatchPad - 1);
        const uint32_t hb = (uint32_t)rslot * (4u * kKeyStride);
        for (int j = 0; j < nbt; j++) {
            u32x4_pk o;
#pragma unroll
            for (int s4 = 0; s4 < 4; s4++) {
                o[s4] = kFarX;
                if (m) {
                    const int a = __builtin_ctz(m);
                    o[s4] = (uint32_t)__popc(cm & ((1u << a) - 1u)) * (4u * kKeyStride);
                    m &= m - 1u;
                }
            }
            s_bo[start + j] = o;
            s_bh[start + j] = hb;
            s_bk[start + j] = (uint32_t)(first + 4 * j);
        }
        if (b < padded - total) {
            s_bo[total + b] = u32x4_pk{kFarX, kFarX, kFarX, kFarX};
            s_bh[total + b] = kFarY;
            s_bk[total + b] = 0u;
        }
        if (tid == 0) {
            pl.K = K;
            pl.Kc = K < cap ? K : cap;
            pl.nbat = padded;
            pl.nbat_real = total;
            pl.ncol = __popc(cm);
            pl.nrow = __popcll(rows);
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Grids above 32 x 32: the stand-alone peak kernel
// ---------------------------------------------------------------------------
// What the assignment needs of the candidates, in global memory: this header,
// then the batches' column offsets (16 bytes each), row offsets and first
// candidates (4 bytes each), arrays of max_batches() + kBatchPad entries.
struct BigPlan {
    int32_t Kc;                   // min(K, cap) candidates
    int32_t nbat, nbat_real;      // batches with and without the padding
    int32_t ncol, nrow;           // candidate columns and rows
    int32_t reserved[3];
    uint8_t colbin[kMaxBins], rowbin[kMaxBins];   // bins of the column and row slots (ascending)
};
static_assert(sizeof(BigPlan) % 16 == 0, "the batch offsets follow, 16-byte aligned");

// Upper bound of the batches of a grid: strict maxima are never horizontally
// adjacent, so a row holds at most ceil(B_w / 2).
__host__ __device__ constexpr int max_batches(int Bw, int Bh) { return Bh * (((Bw + 1) / 2 + 3) / 4); }
__host__ __device__ constexpr size_t plan_bytes(int Bw, int Bh)
{
    return sizeof(BigPlan) + 24 * (size_t)(max_batches(Bw, Bh) + kBatchPad);
}
template <typename P>      // BigPlan, const or not
__device__ __forceinline__ auto plan_offsets(P *p)
{
    using V = std::conditional_t<std::is_const_v<P>, const u32x4_pk, u32x4_pk>;
    return reinterpret_cast<V *>(p + 1);
}
template <typename P>
__device__ __forceinline__ auto plan_rows(P *p, int max_bat)
{
    using V = std::conditional_t<std::is_const_v<P>, const uint32_t, uint32_t>;
    return reinterpret_cast<V *>(plan_offsets(p) + max_bat + kBatchPad);
}
template <typename P>
__device__ __forceinline__ auto plan_first(P *p, int max_bat)
{
    return plan_rows(p, max_bat) + max_bat + kBatchPad;
}

namespace {   // one private copy per translation unit that launches it

// One workgroup: sums the vote histograms into LDS (rows of B_w + 2 counts
// with a border of -1), tests the bins for candidates (a wave takes 64 columns
// of a row at a time, whose ballot is a word of the row's mask), builds the
// plan from the row masks (one wave, two rows per lane) and writes the
// centroid records, K and the summed histogram.  The launch is a chain of
// latencies: its loads are issued kUnroll bins at a time, and everything after
// the masks is local to a lane's rows.
__global__ __launch_bounds__(1024) __attribute__((unused)) void k_peaks(const unsigned long long *__restrict__ hrep,
                                                unsigned long long *__restrict__ hlast, int32_t Bw, int32_t Bh,
                                                long long cut, int32_t cap, const float *__restrict__ cx,
                                                const float *__restrict__ cy, cpe_centroid *__restrict__ cents,
                                                int32_t *__restrict__ num, BigPlan *__restrict__ plan,
                                                int32_t max_bat)
{
    constexpr int kUnroll = 4;
    extern __shared__ __align__(16) unsigned char smem[];
    long long *s_h = reinterpret_cast<long long *>(smem);                     // [Bh + 2][Bw + 2]
    __shared__ unsigned long long s_mask[kMaxBins][2];                        // candidate columns of a row
    __shared__ int s_first[kMaxBins];                                         // its first candidate
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nb = Bw * Bh, stride = Bw + 2;
    const int csh = Bw > 64 ? 1 : 0, words = Bh << csh;                       // 64-column words of the rows
    // word i: row i >> csh, columns 64 (i & csh) ..
    auto bin = [&](int i, int &a, int &b) {
        b = i >> csh;
        a = 64 * (i & csh) + lane;
        return i < words && a < Bw;
    };
    for (int w0 = wv; w0 < words; w0 += 16 * kUnroll) {
        unsigned long long v[kUnroll][kReplicas];
#pragma unroll
        for (int u = 0; u < kUnroll; u++) {
            int a, b;
            const bool in = bin(w0 + 16 * u, a, b);
#pragma unroll
            for (int r = 0; r < kReplicas; r++) v[u][r] = in ? hrep[(size_t)r * nb + b * Bw + a] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < kUnroll; u++) {
            int a, b;
            if (!bin(w0 + 16 * u, a, b)) continue;
            unsigned long long sum = 0;
#pragma unroll
            for (int r = 0; r < kReplicas; r++) sum += v[u][r];
            s_h[(b + 1) * stride + a + 1] = (long long)sum;
        }
    }
    for (int i = tid; i < 2 * stride + 2 * Bh; i += 1024) {
        const int j = i - 2 * stride;
        s_h[i < stride ? i : j < 0 ? (Bh + 1) * stride + i - stride : (j / 2 + 1) * stride + (j & 1) * (Bw + 1)] = -1;
    }
    if (tid < 2 * kMaxBins) s_mask[tid >> 1][tid & 1] = 0ull;
    __syncthreads();
    for (int i = wv; i < words; i += 16) {
        int a, b;
        bool f = bin(i, a, b);
        const long long *q = s_h + b * stride + (f ? a : 0);                  // the corner of its neighbourhood
        const long long v = q[stride + 1];
        f = f && v > cut;
#pragma unroll
        for (int n = 0; n < 9; n++)
            if (n != 4) f &= v > q[(n / 3) * stride + n % 3];
        const unsigned long long m = __ballot(f);
        if (lane == 0) s_mask[b][i & csh] = m;
    }
    __syncthreads();
    if (tid < 64) {
        // rows 2 lane and 2 lane + 1; c: candidates, cut off at `cap`
        unsigned long long m[2][2];
        int c[2], first[2], nbt[2];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            m[u][0] = s_mask[2 * lane + u][0];
            m[u][1] = s_mask[2 * lane + u][1];
            c[u] = __popcll(m[u][0]) + __popcll(m[u][1]);
        }
        const int upto = wave_incl_sum(c[0] + c[1]), K = __builtin_amdgcn_readlane(upto, 63);
        first[0] = upto - c[0] - c[1];
        first[1] = upto - c[1];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            int over = min(max(first[u] + c[u] - cap, 0), c[u]);
            c[u] -= over;
            for (; over > 0; over--) {
                const int w = m[u][1] ? 1 : 0;
                m[u][w] &= ~(1ull << (63 - __clzll(m[u][w])));
            }
            nbt[u] = (c[u] + 3) >> 2;
            s_mask[2 * lane + u][0] = m[u][0];
            s_mask[2 * lane + u][1] = m[u][1];
            s_first[2 * lane + u] = first[u];
        }
        // the candidate columns
        unsigned long long cm[2];
#pragma unroll
        for (int w = 0; w < 2; w++) {
            const unsigned long long x = m[0][w] | m[1][w];
            cm[w] = (unsigned long long)wave_or64((uint32_t)x) | (unsigned long long)wave_or64((uint32_t)(x >> 32)) << 32;
        }
        auto col_slot = [&](int a) {
            const unsigned long long below = (1ull << (a & 63)) - 1ull;
            return a < 64 ? __popcll(cm[0] & below) : __popcll(cm[0]) + __popcll(cm[1] & below);
        };
        const int ncol = __popcll(cm[0]) + __popcll(cm[1]);
        const unsigned long long r0 = __ballot(c[0] > 0), r1 = __ballot(c[1] > 0);
        const int nrow = __popcll(r0) + __popcll(r1);
        const int slot0 = lane_prefix(r0) + lane_prefix(r1);                   // row slot of row 2 lane
        const uint32_t far_y = 4u * kKeyStride * (uint32_t)((nrow + 7) & ~7);
        const uint32_t far_x = far_y + 4u * kKeyStride * (uint32_t)((ncol + 7) & ~7);
#pragma unroll
        for (int w = 0; w < 2; w++) {
            const int a = 64 * w + lane;
            if ((cm[w] >> lane) & 1ull) plan->colbin[col_slot(a)] = (uint8_t)a;
        }
        const int incl = wave_incl_sum(nbt[0] + nbt[1]);
        const int total = __builtin_amdgcn_readlane(incl, 63), padded = (total + kBatchPad - 1) & ~(kBatchPad - 1);
        u32x4_pk *bo = plan_offsets(plan);
        uint32_t *bh = plan_rows(plan, max_bat), *bk = plan_first(plan, max_bat);
        int at = incl - nbt[0] - nbt[1];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int slot = slot0 + (u && c[0] > 0 ? 1 : 0);
            if (c[u] > 0) plan->rowbin[slot] = (uint8_t)(2 * lane + u);
            for (int j = 0; j < nbt[u]; j++, at++) {
                u32x4_pk o;
#pragma unroll
                for (int s4 = 0; s4 < 4; s4++) {
                    o[s4] = far_x;
                    const int w = m[u][0] ? 0 : 1;
                    if (m[u][w]) {
                        o[s4] = 4u * kKeyStride * (uint32_t)col_slot(64 * w + __builtin_ctzll(m[u][w]));
                        m[u][w] &= m[u][w] - 1ull;
                    }
                }
                bo[at] = o;
                bh[at] = 4u * kKeyStride * (uint32_t)slot;
                bk[at] = (uint32_t)(first[u] + 4 * j);
            }
        }
        if (lane < padded - total) {
            bo[total + lane] = u32x4_pk{far_x, far_x, far_x, far_x};
            bh[total + lane] = far_y;
            bk[total + lane] = 0u;
        }
        if (lane == 0) {
            *num = K;
            plan->Kc = min(K, cap);
            plan->nbat = padded;
            plan->nbat_real = total;
            plan->ncol = ncol;
            plan->nrow = nrow;
        }
    }
    __syncthreads();
    for (int i = wv; i < words; i += 16) {
        int a, b;
        if (!bin(i, a, b)) continue;
        const long long v = s_h[(b + 1) * stride + a + 1];
        hlast[b * Bw + a] = (unsigned long long)v;
        const unsigned long long m = s_mask[b][i & csh];
        if ((m >> lane) & 1ull) {
            cpe_centroid rec;
            rec.bin_x = a;
            rec.bin_y = b;
            rec.x = cx[a];
            rec.y = cy[b];
            rec.score = (double)v * 0x1p-30;
            rec.npix = 0;
            rec.reserved = 0;
            cents[s_first[b] + __popcll(m & ((1ull << lane) - 1ull)) + (i & csh ? __popcll(s_mask[b][0]) : 0)] = rec;
        }
    }
}

}  // namespace

}  // namespace cpe
