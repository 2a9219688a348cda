// k_assign_big.hpp -- the assignment for bin grids above 32 x 32 (up to
// 128 x 128): the tiles, distances and search of k_mfma.hpp on a plan that the
// peak kernel (k_peaks.hpp) leaves in global memory.
//
// Only the columns and rows that hold candidates are numbered (slots), so
// the work follows the candidates and not the grid: a tile's distances take
// one set of matrix products per 32 slots of an axis.  The LDS is cut at run
// time, by the plan's counts: the slots' palette operands, the batches, then
// as many waves' distance arrays as fit (the other waves take no tiles).  The
// largest plan, 128 slots per axis and 2048 batches, leaves room for one wave;
// 80 slots in all, a usual count on a 64 x 64 grid, for 12.
//
// On a 704 x 704 fp32 frame with 4 harmonics the peak kernel and this one take
// 8.9 and 16.7 us at 64 x 64 bins, 20.7 and 19.3 us at 128 x 128; one thread per
// pixel with packed 16-bit dot products, every distance corrected and a scan
// over the candidates took 55.3 and 183 us, the peak kernel included.
#pragma once

#include "k_mfma.hpp"

namespace cpe {

constexpr int kBigWaves = 3;                       // per SIMD
constexpr int kBigWpb = 4 * kBigWaves;
constexpr int kBigLds = 160 * 1024;
constexpr int kBigFixed = (kCountCap * 4 + (kMaxSlices + 1) * 4 + 4 + 15) & ~15;   // counts, slice prefix, next tile

// LDS bytes of one wave's distance arrays and far row.
__host__ __device__ constexpr int big_wave_bytes(int ncol, int nrow)
{
    return 4 * kKeyStride * (((ncol + 7) & ~7) + ((nrow + 7) & ~7) + 1);
}
template <int F>
constexpr int big_shared_bytes(int ncol, int nrow, int nbat)
{
    return kBigFixed + ((ncol + 31) / 32 + (nrow + 31) / 32) * kAxisKinds<F> * 1024 + nbat * 24;
}

template <typename T, int F, bool FAST>
__global__ __launch_bounds__(kBigWpb * 64) __attribute__((amdgpu_waves_per_eu(kBigWaves))) void k_assign_big(
    const T *__restrict__ emb, int32_t dstride, int32_t yoff, const int32_t *__restrict__ list,
    const int32_t *__restrict__ counts, int32_t nslices, int32_t slice_px, int32_t npix, double tau32, Tables tb,
    const BigPlan *__restrict__ plan, int32_t max_bat, cpe_centroid *__restrict__ cents,
    int32_t *__restrict__ labels, float *__restrict__ score_map, int32_t force_exact)
{
    constexpr int kThreads = kBigWpb * 64, kKinds = kAxisKinds<F>;
    static_assert(big_shared_bytes<F>(kMaxBins, kMaxBins, max_batches(kMaxBins, kMaxBins)) +
                  big_wave_bytes(kMaxBins, kMaxBins) <= kBigLds, "the largest plan leaves one wave");
    __shared__ __align__(16) unsigned char smem[kBigLds];
    int32_t *s_cnt = reinterpret_cast<int32_t *>(smem);                    // [kCountCap]
    int *s_pref = s_cnt + kCountCap;                                       // [kMaxSlices + 1]
    int *s_next = s_pref + kMaxSlices + 1;                                 // next tile of the run

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int g = lane >> 5, ln = lane & 31;

    SliceLoad sl;
    if (list) slice_load(counts, nslices, sl);
    const int Kc = plan->Kc, ncol = plan->ncol, nrow = plan->nrow, nbat = plan->nbat, real = plan->nbat_real;
    const int ncb = (ncol + 31) >> 5, nrb = (nrow + 31) >> 5;              // blocks of 32 slots
    uint32_t *s_pop = reinterpret_cast<uint32_t *>(smem + kBigFixed);      // [block][kKinds][64][4 words]
    u32x4 *s_bo = reinterpret_cast<u32x4 *>(s_pop + (ncb + nrb) * kKinds * 256);
    uint32_t *s_bh = reinterpret_cast<uint32_t *>(s_bo + nbat);
    uint32_t *s_bk = s_bh + nbat;
    const int shared = big_shared_bytes<F>(ncol, nrow, nbat), per_wave = big_wave_bytes(ncol, nrow);
    const int waves = min(kBigWpb, (kBigLds - shared) / per_wave);         // at least 1
    uint32_t *kx = reinterpret_cast<uint32_t *>(smem + shared + (wv < waves ? wv : 0) * per_wave);
    uint32_t *ky = kx + ((ncol + 7) & ~7) * kKeyStride;

    // the first tile's list entries, then its rows, load while the tables are staged
    const int n = list ? slice_scan(sl, nslices, s_pref) : npix, ntiles = (n + 31) >> 5;
    int t0, tend;
    block_run(ntiles, blockIdx.x, gridDim.x, t0, tend);
    if (wv >= waves) tend = 0;
    int t = t0 + wv;
    ListCursor cur_list;
    cur_list.start(list, s_pref, nslices, slice_px, t < tend ? 32 * t : 0);
    auto pixel = [&](int tt) { return cur_list.pixel(32 * tt + ln < n ? 32 * tt + ln : 32 * tt); };
    int ip = t < tend ? pixel(t) : 0;
    for (int i = tid; i < kCountCap; i += kThreads) s_cnt[i] = 0;
    if (tid == 0) *s_next = 0;
    for (int i = tid; i < (ncb + nrb) * kKinds * 64; i += kThreads) {
        const int blk = i / (kKinds * 64), kind = (i >> 6) % kKinds, l = i & 63;
        const int ax = blk >= ncb ? 1 : 0, slot = 32 * (blk - (ax ? ncb : 0)) + (l & 31);
        const int bin = ax ? (slot < nrow ? plan->rowbin[slot] : 0) : (slot < ncol ? plan->colbin[slot] : 0);
        // kinds of S in Tables::pop: 0, 1, then the limbs from 3 on
        reinterpret_cast<u32x4 *>(s_pop)[i] = reinterpret_cast<const u32x4 *>(
            tb.pop)[((ax * kMaxBinBlocks + (bin >> 5)) * kPopKinds + (kind < 2 ? kind : kind + 1)) * 64 + (l & 32) +
                    (bin & 31)];
    }
    for (int i = tid; i < nbat; i += kThreads) {
        s_bo[i] = plan_offsets(plan)[i];
        s_bh[i] = plan_rows(plan, max_bat)[i];
        s_bk[i] = plan_first(plan, max_bat)[i];
    }
    if (wv < waves && lane < 32) ky[((nrow + 7) & ~7) * kKeyStride + lane] = kFarBits;
    RawSlices<T, F> raw;
    if (t < tend && Kc > 0) raw.load(emb + (size_t)ip * dstride, yoff, g);
    __syncthreads();

    if (Kc == 0) {              // no centroid: every participating pixel is unlabelled
        while (t < tend) {
            if (g == 0 && 32 * t + ln < n) {
                labels[ip] = 0;
                if (score_map) score_map[ip] = 0.0f;
            }
            t += waves;
            if (t < tend) ip = pixel(t);
        }
        return;
    }
    const int bits = step_bits(nbat);
    const Batches bt{s_bo, s_bh, s_bk, nbat, real};
    const Labeller<true> out{labels, score_map, tau32, s_cnt, cents};

    auto distances = [&](auto exact, auto next) {
        PixOps<T, F> X;
        X.from(raw, g);
        next();
#pragma unroll
        for (int ax = 0; ax < 2; ax++) {
            const int slots = ax ? nrow : ncol;
            const uint32_t *pop = s_pop + (ax ? ncb * kKinds * 256 : 0) + 4 * lane;
            uint32_t *dst = (ax ? ky : kx) + 4 * g * kKeyStride + ln;
            for (int s0 = 0; s0 < slots; s0 += 32, pop += kKinds * 256, dst += 32 * kKeyStride) {
                f16x8 P[kKinds];
#pragma unroll
                for (int k = 0; k < kKinds; k++) P[k] = *reinterpret_cast<const f16x8 *>(pop + k * 256);
                f32x16 A, R;
                axis_products<T, F, false>(X.ax[ax], X.e, P, A, R);
                store_distances<decltype(exact)::value>(A, R, slots - s0, dst);
            }
        }
    };

    int tn = tend, ipn = 0;                             // next tile; this lane's pixel in it
    if (t < tend) {
        tn = take_tile(s_next, lane, t0, waves);
        if (tn < tend) ipn = pixel(tn);
    }
    while (t < tend) {
        int tnn = tend, ipnn = 0;
        auto next = [&]() {
            if (tn < tend) {
                raw.load(emb + (size_t)ipn * dstride, yoff, g);
                tnn = take_tile(s_next, lane, t0, waves);
                if (tnn < tend) ipnn = pixel(tnn);
            }
        };
        const int nvalid = min(32, n - 32 * t);
        if constexpr (FAST) {
            distances(std::false_type{}, next);
            if (!search_tile<false>(bt, kx, ky, lane, ip, nvalid, bits, force_exact, out)) {
                raw.load(emb + (size_t)ip * dstride, yoff, g);          // this tile's rows again
                distances(std::true_type{}, []() {});
                if (tn < tend) raw.load(emb + (size_t)ipn * dstride, yoff, g);   // the next tile's rows again
                search_exact<4095>(bt, kx, ky, lane, ip, nvalid, out);
            }
        } else {
            distances(std::true_type{}, next);
            if (!search_tile<true>(bt, kx, ky, lane, ip, nvalid, bits, force_exact, out))
                search_exact<4095>(bt, kx, ky, lane, ip, nvalid, out);
        }
        t = tn;
        tn = tnn;
        ip = ipn;
        ipn = ipnn;
    }
    __syncthreads();
    for (int i = tid; i < Kc && i < kCountCap; i += kThreads)
        if (s_cnt[i]) atomicAdd(&cents[i].npix, s_cnt[i]);
}

}  // namespace cpe
