// Backward pass of the coarser levels with the corner references of neighbouring points MERGED per vertex first.
//
// The backward pass is linear in g = weight * dL/dy of a corner reference, and both hashes depend on the vertex only, so the
// references to one vertex may be summed before any table row is touched: two LDS atomics per reference instead of a
// 4-byte record in two bins, two random table rows and 3 N_p LDS atomics.  What stands in the way is finding the references of a
// vertex: points come in the caller's order.  So
//   1. cells    the points are counted and ordered by a coarse Morton cell (2^12 cells; three short kernels: a histogram per
//               tile that rides in the preparation launch, the prefix over the tiles, and the order itself: only indices move)
//   2. merge    a workgroup takes 4096 references of points that follow each other in that order and sums them per vertex in a
//               hash table in LDS (fp64); every vertex it saw leaves as ONE entry {two hashed rows, g}, and is counted by slice
//   3. the entries then go through the bins of cngp_bwd_binned.h in place of the references: offsets, scatter, drain.  A bin
//               holds the entries themselves, 12 bytes: naming their place instead cost the drain a 128-byte line from memory
//               per entry and table (nerf3d: drain 411 us so, 365 with whole entries; sdf3d 1676 and 1480)
// Nothing has to be complete: a vertex that two workgroups saw, or that found no room in a table, simply has two entries.
//
// Share of the references that is left (2^18 ray samples, the level's N_l: 42 0.11, 58 0.20, 80 0.33; 2^20 points near a surface:
// 48 0.04, 101 0.17, 147 0.27; 2^20 uniform points, d = 2: 445 0.08, 1024 0.29).
//
// What bounds the merge kernel: LDS (one compare-and-swap and two fp64 additions at random addresses per reference, 1.3 .. 1.5
// clocks of the CU, 38 .. 42 % of them bank conflicts: at work 67 % of the time a CU has waves with 2^18 ray samples, 74 % with
// 2^20 points near a surface) and, for a batch in no order, the lines of x and dL/dy (2^20 points, with a finer eighth level
// merged as well: 383 us with the levels one after the other, 276 with a chunk's levels side by side).  Features in planes instead
// of pairs, one lane per four corners instead of eight and a wavefront's points spread over the round took 78 us to 61 (2^18 ray
// samples, with a finer seventh level; the six levels now merged take 49, the seven of the surface's points 230).
#pragma once
#include "cngp_bwd_binned.h"

namespace cngp {

constexpr int      kMergeBlock = 1024;
constexpr uint32_t kMergeRefs  = 4096;              // references per round of a workgroup
// Slots of the table: with 20 bytes each, the lists and the counters, two workgroups fit the 160 KB of a CU, one inserting while
// the other loads or writes.  On average a merged level leaves a third of a round's 4096 references or less (list above); where
// the points are so sparse that more than 3520 are left, those that find no slot become entries of their own.
constexpr uint32_t kMergeSlots = 3520;
constexpr uint32_t kMergeProbes = 16;               // slots tried; a reference that finds none becomes an entry of its own
constexpr uint32_t kMergeEmpty = 0xFFFFFFFFu;
constexpr uint32_t kMergeMaxBins = 512;             // slices of both tables together whose counters fit beside the table
constexpr size_t   kMergeLdsBytes = kMergeSlots * 20 + kMergeMaxBins * 4 + kMergeRefs * 2;
static_assert(2 * (kMergeLdsBytes + 64) <= 160 * 1024, "two workgroups per CU");

// Bits a vertex coordinate has in a table key (d = 2 and 3 are merged).
template <int D> constexpr uint32_t kMergeKeyBits = D == 2 ? 16u : 10u;

// Coarse Morton cell of a point: 6 or 4 bits per axis.  Coordinates outside the cube fall into a border cell.
template <int D>
__device__ __forceinline__ uint32_t merge_cell(const float *xp) {
    constexpr uint32_t B = 12 / D;
    uint32_t cell = 0;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        uint32_t q = (uint32_t)(xp[j] * (float)(1u << B));          // saturates: negative and NaN give 0
        q = q < (1u << B) - 1u ? q : (1u << B) - 1u;
#pragma unroll
        for (uint32_t b = 0; b < B; ++b) cell |= ((q >> b) & 1u) << (b * D + (uint32_t)j);
    }
    return cell;
}

// Points of every cell in one tile; kMergeCells counters in LDS.
template <int D>
__device__ __forceinline__ void merge_hist_block(const MergeParams &mp, const float *__restrict__ x, const int64_t N,
                                                 uint32_t *__restrict__ cells, const uint32_t tile) {
    extern __shared__ uint32_t hist[];
    for (uint32_t i = threadIdx.x; i < kMergeCells; i += blockDim.x) hist[i] = 0u;
    __syncthreads();
    const int64_t n0 = (int64_t)tile * mp.tile_pts, n1 = n0 + mp.tile_pts < N ? n0 + mp.tile_pts : N;
    for (int64_t n = n0 + threadIdx.x; n < n1; n += blockDim.x) {
        float xp[D];
#pragma unroll
        for (int j = 0; j < D; ++j) xp[j] = x[n * D + j];
        atomicAdd(&hist[merge_cell<D>(xp)], 1u);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kMergeCells; i += blockDim.x) cells[(size_t)tile * kMergeCells + i] = hist[i];
}

// In place: cells[tile][cell] becomes the number of the cell's points in earlier tiles; total[cell] all of them.
// 64 cells per workgroup, its wavefronts a quarter of the tiles each.
constexpr int kMergeScanBlock = 256;
__global__ __launch_bounds__(kMergeScanBlock) void merge_scan_kernel(const MergeParams mp, uint32_t *__restrict__ cells,
                                                                     uint32_t *__restrict__ total) {
    constexpr uint32_t kSegs = kMergeScanBlock / 64;
    __shared__ uint32_t part[kSegs][64];
    const uint32_t lane = threadIdx.x & 63u, seg = threadIdx.x >> 6, cell = blockIdx.x * 64u + lane;
    const uint32_t per = (mp.tiles + kSegs - 1) / kSegs, t0 = seg * per, t1 = t0 + per < mp.tiles ? t0 + per : mp.tiles;
    uint32_t sum = 0;
#pragma unroll 8
    for (uint32_t t = t0; t < t1; ++t) sum += cells[(size_t)t * kMergeCells + cell];
    part[seg][lane] = sum;
    __syncthreads();
    uint32_t run = 0, all = 0;
    for (uint32_t g = 0; g < kSegs; ++g) {
        run += g < seg ? part[g][lane] : 0u;
        all += part[g][lane];
    }
#pragma unroll 8
    for (uint32_t t = t0; t < t1; ++t) {
        const uint32_t v = cells[(size_t)t * kMergeCells + cell];
        cells[(size_t)t * kMergeCells + cell] = run;
        run += v;
    }
    if (seg == 0) total[cell] = all;
}

// order[position] = point, by cell; inside a cell tile by tile.  Every workgroup sums the cells' totals up for itself.
template <int D>
__global__ __launch_bounds__(1024) void merge_order_kernel(const MergeParams mp, const float *__restrict__ x, const int64_t N,
                                                           const uint32_t *__restrict__ cells, const uint32_t *__restrict__ total,
                                                           uint32_t *__restrict__ order) {
    __shared__ uint32_t cursor[kMergeCells];
    __shared__ uint32_t part[16];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint4 t = reinterpret_cast<const uint4 *>(total)[threadIdx.x];
    const uint4 b = reinterpret_cast<const uint4 *>(cells + (size_t)blockIdx.x * kMergeCells)[threadIdx.x];
    uint32_t incl = t.x + t.y + t.z + t.w;
    const uint32_t own = incl;
#pragma unroll
    for (uint32_t o = 1; o < 64; o <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)incl, o, 64);
        incl += lane >= o ? v : 0u;
    }
    if (lane == 63) part[wave] = incl;
    __syncthreads();
    uint32_t run = incl - own;
    for (uint32_t w = 0; w < wave; ++w) run += part[w];
    reinterpret_cast<uint4 *>(cursor)[threadIdx.x] = make_uint4(run + b.x, run + t.x + b.y, run + t.x + t.y + b.z, run + t.x + t.y + t.z + b.w);
    __syncthreads();
    const int64_t n0 = (int64_t)blockIdx.x * mp.tile_pts, n1 = n0 + mp.tile_pts < N ? n0 + mp.tile_pts : N;
    for (int64_t n = n0 + threadIdx.x; n < n1; n += 1024) {
        float xp[D];
#pragma unroll
        for (int j = 0; j < D; ++j) xp[j] = x[n * D + j];
        order[atomicAdd(&cursor[merge_cell<D>(xp)], 1u)] = (uint32_t)n;
    }
}

// One workgroup per (level, chunk of the order).  The levels of a chunk run side by side on one XCD (workgroups are handed to
// the 8 XCDs in turn), so a point's coordinates and its row of dL/dy, which the order scatters over memory, come into one L2 once
// and serve all of them.
// The entries of (level, chunk) start at the chunk's first reference; count rows as the references' own (bin_count_block).
template <int D, typename IoT>
__global__ __launch_bounds__(kMergeBlock, 8) void bwd_merge_kernel(
    const Params p, const BinParams bp, const MergeParams mp, const float *__restrict__ x, const IoT *__restrict__ dy, const int64_t N,
    const uint32_t *__restrict__ order, const MergedBins mb)
{
    using Pair = typename std::conditional<sizeof(IoT) == 2, uint32_t, float2>::type;
    constexpr uint32_t kBits = kMergeKeyBits<D>, kLimit = (1u << kBits) - 1u;
    constexpr uint32_t kCorners = kMergeRefs / kMergeBlock;         // corners a lane takes of a point
    constexpr uint32_t kLanesPerPoint = (1u << D) / kCorners;
    constexpr uint32_t kPts = kMergeRefs >> D;                      // points per round
    extern __shared__ __align__(16) unsigned char smem[];
    double   *acc = reinterpret_cast<double *>(smem);               // [feature][slot]
    uint32_t *keys = reinterpret_cast<uint32_t *>(acc + 2 * kMergeSlots);
    uint32_t *count = keys + kMergeSlots;                           // [slices_f + slices_c]
    // the slots a wavefront was the first to use in a round: the entries are written from these lists, not by going
    // through the table (which took as long as the insertion: most slots of a coarse level are empty)
    uint16_t *list = reinterpret_cast<uint16_t *>(count + kMergeMaxBins) + (threadIdx.x >> 6) * 64u * kCorners;
    __shared__ uint32_t used;
    const uint32_t unit = blockIdx.x / kXcds, chunk = unit / mp.levels * kXcds + blockIdx.x % kXcds, l = mp.levels - 1u - unit % mp.levels;
    if (chunk >= mp.chunks) return;
    const uint32_t bins = bp.slices_f + bp.slices_c;
    const uint32_t n0 = chunk * mp.chunk_pts, n1 = (int64_t)n0 + mp.chunk_pts < N ? n0 + mp.chunk_pts : (uint32_t)N;
    const Pair *pairs = reinterpret_cast<const Pair *>(dy) + l;
    struct Item { float xp[D]; Pair y; };
    const uint32_t rounds = (n1 - n0 + kPts - 1) / kPts;            // n0 < n1: every chunk holds points
    // this lane's point of a round: a wavefront's points are spread over the round, because on a coarse level
    // points that follow each other lie in one cell and would add to the same few slots
    constexpr uint32_t kWavePts = 64 / kLanesPerPoint, kStep = kPts / kWavePts;
    const uint32_t turn_pt = threadIdx.x / kLanesPerPoint, mine = turn_pt % kWavePts * kStep + turn_pt / kWavePts;
    auto position = [&](const uint32_t round) {                     // ... in the order; beyond the chunk its last point
        const uint32_t at = n0 + (round < rounds ? round : 0u) * kPts + mine;
        return at < n1 ? at : n1 - 1u;
    };
    // the order two rounds ahead, the points and gradients it names one round ahead (three and two, waited for between the
    // insertion and the entries' stores, was slower: 50 and 55 us for 2^18 ray samples)
    auto fetch = [&](const uint32_t n, Item &it) {
#pragma unroll
        for (int j = 0; j < D; ++j) it.xp[j] = x[(size_t)n * D + j];
        it.y = pairs[(size_t)n * p.L];
    };
    uint32_t ahead = order[position(0)];
    Item     cur, next;
    fetch(ahead, cur);
    ahead = order[position(1)];
    for (uint32_t i = threadIdx.x; i < kMergeSlots; i += kMergeBlock) {
        keys[i] = kMergeEmpty;
        acc[i] = 0.0;
        acc[i + kMergeSlots] = 0.0;
    }
    for (uint32_t i = threadIdx.x; i < bins; i += kMergeBlock) count[i] = 0u;
    if (threadIdx.x == 0) used = 0u;
    __syncthreads();
    // The lane's corners: k = 0 .. kCorners - 1, offset (bit j of k) ^ (bit j of flip) along dimension j.  flip names the lane's
    // share of the point's corners in its upper bits and lets neighbouring points start at different corners.
    const uint32_t flip = (threadIdx.x % kLanesPerPoint) * kCorners + turn_pt % kCorners;
    {
        uint4 *out = mb.entries + (size_t)l * bp.cap + ((size_t)n0 << D);
        const float res = (float)p.N_l[l];
        auto entry = [&](const uint32_t at, const uint32_t (&v)[D], const float gx, const float gy) {
            uint32_t h1 = 0, h2 = 0;                                // Eq. 3
#pragma unroll
            for (int j = 0; j < D; ++j) {
                h1 ^= v[j] * kPi[j];
                h2 ^= v[j] * kPi2[j];
            }
            h1 &= p.row_mask;
            h2 &= p.c_mask;
            out[at] = make_uint4(h1, h2, __float_as_uint(gx), __float_as_uint(gy));
            if (bp.slices_f) atomicAdd(&count[h1 >> bp.rows_f_log2], 1u);
            if (bp.slices_c) atomicAdd(&count[bp.slices_f + (h2 >> bp.rows_c_log2)], 1u);
        };
        for (uint32_t r = 0; r < rounds; ++r) {
            uint32_t claims = 0;
            fetch(ahead, next);                                     // (past the last round: the first one's, unused)
            ahead = order[position(r + 2)];
            {
                const bool live = n0 + r * kPts + mine < n1;
                float    wa[D], wb[D];                              // weight along dimension j of the corners with bit j of k clear / set
                uint32_t va[D], vb[D];                              // ... their coordinate
                bool     fits = true;                               // coordinates a key can hold (points outside the cube may not)
                {
#pragma clang fp contract(off)
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        const float    pos = cur.xp[j] * res;       // one rounded fp32 multiply
                        const float    fl = floorf(pos), w = pos - fl;
                        const uint32_t v0 = (uint32_t)fl, up = (flip >> j) & 1u;
                        wa[j] = up ? w : 1.0f - w;
                        wb[j] = up ? 1.0f - w : w;
                        va[j] = v0 + up;
                        vb[j] = v0 + 1u - up;
                        fits = fits && v0 < kLimit - 1u;            // the upper vertex too, and never the empty key
                    }
                }
                const float2 g = pair_to_float2(cur.y);
                uint32_t slot[kCorners], key[kCorners], found[kCorners];
                float    wt[kCorners];
#pragma unroll
                for (uint32_t k = 0; k < kCorners; ++k) {
                    uint32_t q = 0;
#pragma unroll
                    for (int j = 0; j < D; ++j) q |= ((k >> j) & 1u ? vb[j] : va[j]) << (kBits * j);
                    // a corner of weight zero adds nothing and is left out; all of a lane's beyond the chunk are, whatever the point
                    // it repeats, so that a chunk makes at most 2^d entries per point of its own (the room it has)
                    wt[k] = corner_weight_if<D>(live, wa, wb, k);
                    key[k] = q;
                    slot[k] = __umulhi(q * 2654435769u, kMergeSlots);
                }
#pragma unroll
                for (uint32_t k = 0; k < kCorners; ++k)
                    if (wt[k] != 0.0f && fits) found[k] = atomicCAS(&keys[slot[k]], kMergeEmpty, key[k]);
#pragma unroll
                for (uint32_t k = 0; k < kCorners; ++k) {
                    bool claimed = false;
                    if (wt[k] != 0.0f) {
                        bool placed = false;
                        if (fits) {
                            uint32_t f = found[k];
                            for (uint32_t t = 1; ; ++t) {
                                claimed = f == kMergeEmpty;
                                placed = claimed || f == key[k];
                                if (placed || t == kMergeProbes) break;
                                slot[k] = slot[k] + 1u == kMergeSlots ? 0u : slot[k] + 1u;
                                f = atomicCAS(&keys[slot[k]], kMergeEmpty, key[k]);
                            }
                        }
                        if (placed) {
                            atomicAdd(&acc[slot[k]], (double)wt[k] * (double)g.x);
                            atomicAdd(&acc[slot[k] + kMergeSlots], (double)wt[k] * (double)g.y);
                        } else {
                            uint32_t v[D];
#pragma unroll
                            for (int j = 0; j < D; ++j) v[j] = (k >> j) & 1u ? vb[j] : va[j];
                            entry(atomicAdd(&used, 1u), v, wt[k] * g.x, wt[k] * g.y);
                        }
                    }
                    const uint64_t m = __ballot(claimed);
                    if (claimed) list[claims + lanes_below(m)] = (uint16_t)slot[k];
                    claims += (uint32_t)__popcll(m);
                }
            }
            __syncthreads();
            // the sums of the vertices this wavefront found first, and their slots empty again
            uint32_t first = 0;
            if (claims && (threadIdx.x & 63u) == 0) first = atomicAdd(&used, claims);
            first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
            for (uint32_t i = threadIdx.x & 63u; i < claims; i += 64u) {
                const uint32_t at = list[i], key = keys[at];
                uint32_t v[D];
#pragma unroll
                for (int j = 0; j < D; ++j) v[j] = (key >> (kBits * j)) & kLimit;
                entry(first + i, v, (float)acc[at], (float)acc[at + kMergeSlots]);
                keys[at] = kMergeEmpty;
                acc[at] = 0.0;
                acc[at + kMergeSlots] = 0.0;
            }
            __syncthreads();
            cur = next;
        }
        uint32_t *rowF = mb.cntF + ((size_t)l * mp.chunks + chunk) * bp.slices_f;
        uint32_t *rowC = mb.cntC + ((size_t)l * mp.chunks + chunk) * bp.slices_c;
        for (uint32_t s = threadIdx.x; s < bins; s += kMergeBlock) {
            if (s < bp.slices_f) rowF[s] = count[s];
            else rowC[s - bp.slices_f] = count[s];
        }
        if (threadIdx.x == 0) mb.made[(size_t)l * mp.chunks + chunk] = used;
    }
}

}  // namespace cngp
