// Scatter of the binned backward pass in runs, for levels of 48 bins and more with more than one of either table.
//
// Written straight from the lanes that found them (bin_scatter_kernel), the 64 records of a store go to almost as many bins, and a
// cache line is requested for each: texture addressers at work 98.7 % of the time (2^20 points near a surface, 64 bins a level: 400 us).
// Here a workgroup ranks a round of 4096 references in their bins with LDS atomics, lays them out bin after bin and writes them in that
// order, a line or two per store of 64 records (237 us).  Ranks are taken per wavefront and the wavefronts' shares of a bin follow each
// other, so a bin keeps the order of the points, which the drain's gathers of points and gradients live on: its L2 requests fell from
// 259 to 243 M and its time from 1640 to 1557 us (the direct scatter lets four wavefronts share the cursors where there are that many
// bins).  With 24 bins and fewer the direct way, a wavefront per chunk, is the shorter one: 2^18 ray samples 60 us, in runs 78.
//
// What bounds it: LDS and vector ALU in turn (at work 40 and 58 % of the time), four barriers a round; four workgroups per CU.
// Whole records {rows, weight * dL/dy} in place of references, 12 bytes instead of 4, were tried: the drain then gathers no points
// (1557 -> 1362 us), but the scatter takes 643, and with 24 bins the drain is the slower one (337 -> 370 us).
#pragma once
#include "cngp_bwd_merge.h"

namespace cngp {

constexpr int      kScatBlock = 512;
constexpr uint32_t kScatWaves = kScatBlock / 64;
constexpr uint32_t kScatRefsPer = 8, kScatRefs = kScatBlock * kScatRefsPer;             // references of a lane and of a round
constexpr uint32_t kScatEntriesPer = 4, kScatEntries = kScatBlock * kScatEntriesPer;    // entries
constexpr uint32_t kScatSpan = 4;                   // chunks of a merged level that one workgroup takes
constexpr uint32_t kScatMaxBins = kScatBlock;       // for runs: a thread per bin
// Bins a workgroup sorts into, each table's rounded up to whole wavefronts.
__host__ __device__ __forceinline__ uint32_t scatter_bins(const uint32_t slices_f, const uint32_t slices_c) {
    return ((slices_f + 63u) & ~63u) + ((slices_c + 63u) & ~63u);
}
// LDS: a round of both tables' references, or of one table's whole entries; counts by wavefront and bin; what leads from slots to positions.
constexpr uint32_t kScatRoundBytes = kScatRefs * 8 > kScatEntries * 14 ? kScatRefs * 8 : kScatEntries * 14;
__host__ __forceinline__ size_t scatter_lds(const uint32_t bins) { return kScatRoundBytes + (size_t)bins * (kScatWaves + 1) * 4; }

// What a round leaves to the counters of thread t's bin: hist[wave][bin] becomes the wavefront's first slot, delta[bin] what leads from a
// slot to a position, made[table] the round's records.  The bins follow each other in any order.
__device__ __forceinline__ void scatter_places(uint32_t *hist, uint32_t *delta, uint32_t *made, const uint32_t bins, const uint32_t c_at, uint32_t &cursor) {
    const uint32_t t = threadIdx.x;
    if (t >= bins) return;                                          // (whole wavefronts)
    uint32_t share[kScatWaves], v = 0;
#pragma unroll
    for (uint32_t w = 0; w < kScatWaves; ++w) { share[w] = hist[w * bins + t]; v += share[w]; }
    const uint32_t incl = wave_inclusive_sum(v);
    uint32_t at = 0;
    if ((t & 63u) == 63u) at = atomicAdd(&made[t >= c_at ? 1 : 0], incl);
    at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + incl - v;
    delta[t] = cursor - at;
    cursor += v;
#pragma unroll
    for (uint32_t w = 0; w < kScatWaves; ++w) { hist[w * bins + t] = at; at += share[w]; }
}

// A chunk of a hashed level in runs.
template <int D>
__device__ __forceinline__ void scatter_refs_in_runs(
    const Params &p, const BinParams &bp, const float *__restrict__ x, const int64_t N, const uint32_t li, const uint32_t chunk,
    const uint32_t *__restrict__ cntF, const uint32_t *__restrict__ cntC, BinRecord *__restrict__ recF, BinRecord *__restrict__ recC,
    unsigned char *smem, uint32_t *made)
{
    constexpr uint32_t kCorners = D < 3 ? 1u << D : 8u, kPts = kScatRefsPer / kCorners;      // corners of a point that a lane takes; its points
    const uint32_t t = threadIdx.x, wave = t >> 6;
    const uint32_t sf = bp.slices_f, sc = bp.slices_c, c_at = (sf + 63u) & ~63u, bins = scatter_bins(sf, sc);
    uint32_t *first = reinterpret_cast<uint32_t *>(smem), *second = first + kScatRefs;      // reference of the round | bin << 16
    uint32_t *hist = reinterpret_cast<uint32_t *>(smem + kScatRoundBytes), *delta = hist + kScatWaves * bins, *mine = hist + wave * bins;
    const bool is_c = t >= c_at;
    uint32_t   cursor = 0;                                          // where the records of this thread's bin go on
    if ((is_c ? t - c_at : t) < (is_c ? sc : sf)) cursor = is_c ? cntC[((size_t)li * bp.chunks + chunk) * sc + (t - c_at)] : cntF[((size_t)li * bp.chunks + chunk) * sf + t];
    for (uint32_t i = t; i < kScatWaves * bins; i += kScatBlock) hist[i] = 0u;
    if (t < 2) made[t] = 0u;
    const int64_t  n0 = (int64_t)chunk * bp.chunk_pts;
    const uint32_t items = (uint32_t)((n0 + bp.chunk_pts < N ? bp.chunk_pts : N - n0) << D), N_l = p.N_l[(uint32_t)bp.level0 + li];
    float next[kPts][D];
    auto fetch = [&](const uint32_t r0) {
#pragma unroll
        for (uint32_t q = 0; q < kPts; ++q) {
            const uint32_t ref0 = r0 + (t * kPts + q) * kCorners;
            const int64_t  n = n0 + ((ref0 < items ? ref0 : 0u) >> D);
#pragma unroll
            for (int j = 0; j < D; ++j) next[q][j] = x[n * D + j];
        }
    };
    fetch(0);
    __syncthreads();
    for (uint32_t r0 = 0; r0 < items; r0 += kScatRefs) {
        uint32_t bf[kScatRefsPer], bc[kScatRefsPer];                // bin of a table | rank in the wavefront's share of it << 16
        uint32_t live = 0;
#pragma unroll
        for (uint32_t q = 0; q < kPts; ++q) {
            const uint32_t ref0 = r0 + (t * kPts + q) * kCorners;   // first of the lane's references to this point
            const bool     there = ref0 < items, half = D == 4 && (ref0 & 8u);               // d = 4: two lanes per point
            Cell<D> cell;
            cell.locate(next[q], N_l);
#pragma unroll
            for (uint32_t c = 0; c < kCorners; ++c) {
                constexpr int kLast = (1 << D) - 1;
                const uint32_t k = q * kCorners + c;
                uint32_t h1, h2;
                float    wt;
                if (half) { corner_rows<D>(cell, p, (int)(c | 8u) & kLast, h1, h2); wt = cell.weight((int)(c | 8u) & kLast); }
                else      { corner_rows<D>(cell, p, (int)c, h1, h2); wt = cell.weight((int)c); }
                bf[k] = h1;
                bc[k] = c_at + (h2 >> bp.rows_c_log2);
                live |= there && wt != 0.0f ? 1u << k : 0u;         // weight zero: adds nothing, and was not counted
            }
        }
        uint32_t edges = 0;                                         // records of the feature table: of an edge in its even corner's place, a second one in the odd one's
#pragma unroll
        for (uint32_t k = 0; k < kScatRefsPer; k += 2) {
            uint32_t first_bin, second_bin;
            const uint32_t n_f = edge_slices<D>(bf[k], bf[k + 1], live >> k & 1u, live >> k & 2u, bp.rows_f_log2, first_bin, second_bin);
            bf[k] = first_bin;
            bf[k + 1] = second_bin;
            edges |= (n_f > 1u ? 3u : n_f) << k;
        }
        if (r0 + kScatRefs < items) fetch(r0 + kScatRefs);
#pragma unroll
        for (uint32_t k = 0; k < kScatRefsPer; ++k) {
            if (sf && (edges >> k & 1u)) bf[k] |= atomicAdd(&mine[bf[k]], 1u) << 16;
            if (sc && (live >> k & 1u)) bc[k] |= atomicAdd(&mine[bc[k]], 1u) << 16;
        }
        __syncthreads();
        scatter_places(hist, delta, made, bins, c_at, cursor);
        __syncthreads();
#pragma unroll
        for (uint32_t k = 0; k < kScatRefsPer; ++k) {
            const uint32_t ref = t * kScatRefsPer + k;
            if (sf && (edges >> k & 1u)) first[mine[bf[k] & 0xFFFFu] + (bf[k] >> 16)] = (ref & ~1u) | bf[k] << 16;
            if (sc && (live >> k & 1u)) second[mine[bc[k] & 0xFFFFu] + (bc[k] >> 16)] = ref | bc[k] << 16;
        }
        __syncthreads();
        const uint32_t ref_at = ((uint32_t)n0 << D) + r0;
#pragma unroll
        for (int role = 0; role < 2; ++role) {
            BinRecord      *out = (role ? recC : recF) + (size_t)li * bp.cap;
            const uint32_t *from = role ? second : first, n = made[role];
            for (uint32_t i0 = t; i0 < n; i0 += 4 * kScatBlock) {
                uint32_t v[4], at[4];
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    const uint32_t i = i0 + k * kScatBlock < n ? i0 + k * kScatBlock : n - 1u;
                    v[k] = from[i];
                    at[k] = delta[v[k] >> 16] + i;
                }
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k)
                    if (i0 + k * kScatBlock < n) out[at[k]] = ref_at + (v[k] & 0xFFFFu);
            }
        }
        __syncthreads();
        if (t < 2) made[t] = 0u;                                    // (added to again behind the next round's first barrier)
        for (uint32_t i = t; i < kScatWaves * bins; i += kScatBlock) hist[i] = 0u;
        __syncthreads();
    }
}

// The entries of kScatSpan chunks of a merged level, in runs.  (Written directly, 12 bytes to a bin of their own each, the entries of 2^20
// points near a surface at 147 cells per axis, 2.3 M, took 50 us a level, in runs 30; those of 4096 .. 20000 vertices 7 and 1.)
template <int D>
__device__ __forceinline__ void scatter_entries(const BinParams &bp, const MergedBins &mb, const uint32_t lm, const uint32_t chunk,
                                                unsigned char *smem, uint32_t *made)
{
    __shared__ uint32_t upto[kScatSpan + 1];
    const uint32_t t = threadIdx.x, wave = t >> 6;
    const uint32_t sf = bp.slices_f, sc = bp.slices_c, c_at = (sf + 63u) & ~63u, bins = scatter_bins(sf, sc);
    float2   *sg = reinterpret_cast<float2 *>(smem);
    uint32_t *skey = reinterpret_cast<uint32_t *>(sg + kScatEntries);
    uint16_t *sbin = reinterpret_cast<uint16_t *>(skey + kScatEntries);
    uint32_t *hist = reinterpret_cast<uint32_t *>(smem + kScatRoundBytes), *delta = hist + kScatWaves * bins, *mine = hist + wave * bins;
    const bool is_c = t >= c_at;
    uint32_t   cursor = 0;
    if ((is_c ? t - c_at : t) < (is_c ? sc : sf)) cursor = is_c ? mb.cntC[((size_t)lm * mb.chunks + chunk) * sc + (t - c_at)] : mb.cntF[((size_t)lm * mb.chunks + chunk) * sf + t];
    for (uint32_t i = t; i < kScatWaves * bins; i += kScatBlock) hist[i] = 0u;
    if (t < 2) made[t] = 0u;
    if (t == 0) {
        uint32_t all = 0;
        upto[0] = 0u;
        for (uint32_t k = 0; k < kScatSpan; ++k) {
            all += chunk + k < mb.chunks ? mb.made[(size_t)lm * mb.chunks + chunk + k] : 0u;
            upto[k + 1] = all;
        }
    }
    __syncthreads();
    const uint32_t row_f_mask = (1u << bp.rows_f_log2) - 1u, row_c_mask = (1u << bp.rows_c_log2) - 1u, items = upto[kScatSpan];
    const uint4   *in = mb.entries + (size_t)lm * bp.cap;
    for (uint32_t r0 = 0; r0 < items; r0 += kScatEntries) {
        uint4    e[kScatEntriesPer];
        uint32_t bf[kScatEntriesPer], bc[kScatEntriesPer];
#pragma unroll
        for (uint32_t k = 0; k < kScatEntriesPer; ++k) {
            const uint32_t i = r0 + k * kScatBlock + t, at = i < items ? i : items - 1u;
            uint32_t c = 0;                                         // the chunk of the entry, and where it stands among the chunk's own
#pragma unroll
            for (uint32_t j = 1; j < kScatSpan; ++j) c += at >= upto[j] ? 1u : 0u;
            e[k] = in[((size_t)((chunk + c) * mb.chunk_pts) << D) + (at - upto[c])];
        }
#pragma unroll
        for (uint32_t k = 0; k < kScatEntriesPer; ++k) {
            bf[k] = e[k].x >> bp.rows_f_log2;
            bc[k] = c_at + (e[k].y >> bp.rows_c_log2);
            if (r0 + k * kScatBlock + t < items) {
                if (sf) bf[k] |= atomicAdd(&mine[bf[k]], 1u) << 16;
                if (sc) bc[k] |= atomicAdd(&mine[bc[k]], 1u) << 16;
            }
        }
        __syncthreads();
        scatter_places(hist, delta, made, bins, c_at, cursor);
        __syncthreads();
#pragma unroll
        for (int role = 0; role < 2; ++role) {
            if (role ? sc : sf) {
#pragma unroll
                for (uint32_t k = 0; k < kScatEntriesPer; ++k) {
                    if (r0 + k * kScatBlock + t < items) {
                        const uint32_t b = (role ? bc[k] : bf[k]) & 0xFFFFu, at = mine[b] + ((role ? bc[k] : bf[k]) >> 16);
                        skey[at] = role ? (e[k].y & row_c_mask) | e[k].x << bp.rows_c_log2 : (e[k].x & row_f_mask) | e[k].y << bp.rows_f_log2;
                        sg[at] = make_float2(__uint_as_float(e[k].z), __uint_as_float(e[k].w));
                        sbin[at] = (uint16_t)b;
                    }
                }
                __syncthreads();
                EntryRecord   *out = (role ? mb.recC : mb.recF) + (size_t)lm * bp.cap;
                const uint32_t n = made[role];
#pragma unroll
                for (uint32_t k = 0; k < kScatEntriesPer; ++k) {
                    const uint32_t i = k * kScatBlock + t;
                    if (i < n) out[delta[sbin[i]] + i] = {skey[i], sg[i].x, sg[i].y};
                }
                __syncthreads();
            }
        }
        if (t < 2) made[t] = 0u;
        for (uint32_t i = t; i < kScatWaves * bins; i += kScatBlock) hist[i] = 0u;
        __syncthreads();
    }
}

// Workgroups: kScatSpan chunks each of the merged levels, the one with the most entries first (they are the longest: after the others,
// 346 us instead of 237 for the points near a surface), then the chunks of the hashed levels, then those of the pre-reduced ones.
template <int D>
__global__ __launch_bounds__(kScatBlock) void bin_scatter_runs_kernel(
    const Params p, const BinParams bp, const DenseLevels dl, const float *__restrict__ x, const int64_t N,
    const uint32_t *__restrict__ cntF, const uint32_t *__restrict__ cntC, const uint32_t *__restrict__ cntG,
    BinRecord *__restrict__ recF, BinRecord *__restrict__ recC, BinRecord *__restrict__ recG, const MergedBins mb)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t made[2];
    const uint32_t spans = (mb.chunks + kScatSpan - 1) / kScatSpan, merged = mb.levels * spans;
    if (blockIdx.x < merged) {
        scatter_entries<D>(bp, mb, mb.levels - 1u - blockIdx.x / spans, blockIdx.x % spans * kScatSpan, smem, made);
        return;
    }
    const uint32_t block = blockIdx.x - merged, li = block / bp.chunks, chunk = block % bp.chunks;
    if (li < (uint32_t)bp.nlevels) scatter_refs_in_runs<D>(p, bp, x, N, li, chunk, cntF, cntC, recF, recC, smem, made);
    else scatter_grid_refs<D>(p, bp, dl, x, N, li - (uint32_t)bp.nlevels, chunk, cntG, recG, reinterpret_cast<uint32_t *>(smem));
}

}  // namespace cngp
