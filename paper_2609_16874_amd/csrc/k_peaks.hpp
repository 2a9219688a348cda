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
//   peak_extract  any grid: the stand-alone kernel k_peaks between the
//                 generic vote and assignment kernels; it writes the records,
//                 K, the compact list and the summed histogram to memory.
//
// Candidate batches.  The first min(K, cap) candidates are grouped by row b
// into batches of 4 columns (a row's last batch is filled with the far row,
// which never attains a minimum).  Batch i is bo[i] = the byte offsets
// 128 j of its 4 column slots j in the assignment kernel's [slot][32 pixels]
// x array, bh[i] the byte offset of its row's slot in the y array, and bk[i]
// the index of its first candidate.  The list is padded to a multiple of 8
// batches of the far row.
#pragma once

#include "cpe_common.hpp"

namespace cpe {

typedef uint32_t u32x4_pk __attribute__((ext_vector_type(4)));

// Strict local maxima of a B_w x B_h grid are pairwise non-adjacent, so there
// are at most ceil(B_w / 2) * ceil(B_h / 2) of them.
__host__ __device__ constexpr int max_peaks(int Bw, int Bh) { return ((Bw + 1) / 2) * ((Bh + 1) / 2); }

// Strict 8-neighbour local maximum of s_h (LDS, row-major [Bh][Bw]) above
// `cut`; out-of-range neighbours are ignored.
__device__ __forceinline__ bool is_peak(const unsigned long long *s_h, int i, int Bw, int Bh, long long cut)
{
    const int a = i % Bw, b = i / Bw;
    const unsigned long long v = s_h[i];
    bool f = (long long)v > cut;
#pragma unroll
    for (int db = -1; db <= 1; db++)
#pragma unroll
        for (int da = -1; da <= 1; da++) {
            if (!da && !db) continue;
            const int nb_ = b + db, na = a + da;
            const bool in = nb_ >= 0 && nb_ < Bh && na >= 0 && na < Bw;
            const unsigned long long w = s_h[in ? nb_ * Bw + na : i];   // self when out of range
            f = f && (!in || v > w);
        }
    return f;
}

// Block-level scratch of the compaction (LDS).
struct CompactScratch {
    int wave[32];                 // per-wave counts of the two bins per thread
    int base;
};

// Mark and compact the candidates of s_h in ascending bin order into s_pk;
// returns K (every thread).  Two bins per thread and pass, bins
// c0 + u * blockDim + tid.  on_peak(i, pos) runs for every candidate bin i
// at list position pos.
template <typename OnPeak>
__device__ __forceinline__ int compact_peaks(const unsigned long long *s_h, int Bw, int Bh, long long cut, int *s_pk,
                                             CompactScratch &cs, OnPeak on_peak)
{
    const int tid = threadIdx.x, nb = Bw * Bh;
    const int lane = tid & 63, wid = tid >> 6, nwaves = blockDim.x >> 6;
    if (tid == 0) cs.base = 0;
    __syncthreads();
    for (int c0 = 0; c0 < nb; c0 += 2 * (int)blockDim.x) {
        bool flag[2];
        unsigned long long mask[2];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int i = c0 + u * (int)blockDim.x + tid;
            flag[u] = i < nb && is_peak(s_h, i, Bw, Bh, cut);
            mask[u] = __ballot(flag[u]);
        }
        if (lane == 0) {
            cs.wave[wid] = __popcll(mask[0]);
            cs.wave[nwaves + wid] = __popcll(mask[1]);
        }
        __syncthreads();
        // all counts of this pass: pass 0 of every wave, then pass 1
        int off0 = cs.base, off1 = cs.base, tot = 0;
#pragma unroll
        for (int w = 0; w < 16; w++) {          // nwaves <= 16; all reads independent
            const int n0 = w < nwaves ? cs.wave[w] : 0, n1 = w < nwaves ? cs.wave[nwaves + w] : 0;
            off0 += w < wid ? n0 : 0;
            off1 += n0 + (w < wid ? n1 : 0);
            tot += n0 + n1;
        }
#pragma unroll
        for (int u = 0; u < 2; u++) {
            if (flag[u]) {
                const int i = c0 + u * (int)blockDim.x + tid;
                const int pos = (u ? off1 : off0) + lane_prefix(mask[u]);   // < max_peaks(Bw, Bh)
                s_pk[pos] = i;
                on_peak(i, pos);
            }
        }
        __syncthreads();
        if (tid == 0) cs.base += tot;
        __syncthreads();
    }
    return cs.base;
}

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
// Any grid: the stand-alone peak kernel of the generic path
// ---------------------------------------------------------------------------
struct PeakOut {
    cpe_centroid *cents;          // caller's centroid records [cap]
    int32_t *num;                 // caller's K
    int32_t *peaks;               // [cap] a | b << 16
    int32_t *kinfo;               // [0] = min(K, cap), [1] = K
};

// The whole extraction; every thread of the block calls it.  s_h: LDS
// scratch of Bw * Bh u64; s_pk: LDS scratch of max_peaks(Bw, Bh) ints.
// Until the last barrier every result goes to LDS only, so that no barrier
// waits for global stores; the outputs are written at the end.
__device__ __forceinline__ void peak_extract(const unsigned long long *__restrict__ hrep,
                                             unsigned long long *__restrict__ hlast, int32_t Bw, int32_t Bh,
                                             long long cut, int32_t cap, const float *__restrict__ cx,
                                             const float *__restrict__ cy, const PeakOut &po,
                                             unsigned long long *s_h, int *s_pk, CompactScratch &cs)
{
    const int tid = threadIdx.x;
    const int nb = Bw * Bh;
    for (int i = tid; i < nb; i += blockDim.x) {
        unsigned long long v[kReplicas];
#pragma unroll
        for (int r = 0; r < kReplicas; r++) v[r] = hrep[(size_t)r * nb + i];
        unsigned long long sum = 0;
#pragma unroll
        for (int r = 0; r < kReplicas; r++) sum += v[r];
        s_h[i] = sum;
    }
    const int K = compact_peaks(s_h, Bw, Bh, cut, s_pk, cs, [](int, int) {});
    const int Kc = K < cap ? K : cap;

    // ---- outputs (global stores only from here on) ----
    for (int k = tid; k < Kc; k += blockDim.x) {
        const int i = s_pk[k], a = i % Bw, b = i / Bw;
        cpe_centroid rec;
        rec.bin_x = a;
        rec.bin_y = b;
        rec.x = cx[a];
        rec.y = cy[b];
        rec.score = (double)s_h[i] * 0x1p-30;
        rec.npix = 0;
        rec.reserved = 0;
        po.cents[k] = rec;
        po.peaks[k] = a | (b << 16);
    }
    for (int i = tid; i < nb; i += blockDim.x) hlast[i] = s_h[i];
    if (tid == 0) {
        *po.num = K;
        po.kinfo[0] = Kc;
        po.kinfo[1] = K;
    }
}

namespace {   // one private copy per translation unit that launches it

__global__ __launch_bounds__(1024) void k_peaks(const unsigned long long *__restrict__ hrep,
                                                unsigned long long *__restrict__ hlast, int32_t Bw, int32_t Bh,
                                                long long cut, int32_t cap, const float *__restrict__ cx,
                                                const float *__restrict__ cy, PeakOut po)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ CompactScratch cs;
    unsigned long long *s_h = reinterpret_cast<unsigned long long *>(smem);    // [Bw * Bh]
    int *s_pk = reinterpret_cast<int *>(s_h + Bw * Bh);                          // [max_peaks(Bw, Bh)]
    peak_extract(hrep, hlast, Bw, Bh, cut, cap, cx, cy, po, s_h, s_pk, cs);
}

}  // namespace

}  // namespace cpe
