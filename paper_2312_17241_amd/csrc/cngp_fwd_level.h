// Level-resident forward (Eq. 6 + interpolation) for large batches.
//
// The tile kernel takes 256 points through all levels; every one of its feature lookups is a divergent 4- or 8-byte
// load that the texture addresser and the L2 serve one cache line at a time, and that request rate is what bounds it.
// Here a workgroup belongs to ONE level for its whole life: it copies the level's index codebook and as much of the
// level's feature codebook as fits into LDS once, then streams its share of the points.  Lookups below `resident`
// are LDS reads; the rest still go to memory.  A workgroup produces one level's two columns only, so the encodings
// are written level-major (yT[l][n], coalesced) and a second kernel turns them into rows of y.
// A coarse level whose whole vertex grid fits in LDS is looked up once per VERTEX instead of 2^d times per point:
// its workgroups fill a dense table of the grid's (N_l + 2)^d resolved features and interpolate from that, with no
// hash, no index lookup and no memory access per point but the point itself.  Both kinds of workgroup measured, before
// the grids and with them (level kernel alone under rocprofv3, us, average): nerf3d's tables 2^24 uniform points 2734 ->
// 2103, 2^18 ray samples 50 -> 40; image2d's (2^20) 93 -> 66, sdf3d's (2^20) 451 -> 337.
// Per point and level the arithmetic is that of the tile kernel, in the same order: the results are bit-identical.
#pragma once
#include "cngp_kernels.h"

namespace cngp {

constexpr int kLevelBlock = 1024;        // 16 wavefronts: one workgroup per CU, the LDS is what limits residency
constexpr int kLevelUnroll = 2;          // points per lane in flight
constexpr int kMaxGridLevels = 16;       // levels that can be interpolated from a resolved grid
constexpr uint32_t kFwdXcds = 8;           // workgroups are handed to the XCDs in turn

// Which workgroup does what.  The levels [0, dense) interpolate from a resolved vertex grid, the others look up; the dense
// ones come last in the grid.  Looked-up units are numbered part by part, so that the levels read the same points at about
// the same time; `by_xcd` (the parts of the tables that are not in LDS do not fit one XCD's L2 together): instead each
// XCD (workgroup index mod 8) takes a run of them numbered level by level, so that a level's table is held by one or two L2s
// (the plan prefers numbers of levels that eight runs cut evenly: one table too many per L2 costs more than a grid saves).
struct LevelSplit {
    uint32_t dense, by_xcd;
    uint32_t hash_parts, hash_units;         // parts per looked-up level; workgroups for them (a multiple of 8 if by_xcd)
    int64_t  hash_per;                       // points per part
    uint32_t grid_first[kMaxGridLevels + 1]; // first workgroup of a dense level, behind hash_units; [dense] = end
    int64_t  grid_per[kMaxGridLevels];
};

// Features of every vertex of a level's grid (`side` vertices per axis, dimension 0 fastest), eight per lane in flight.
template <int D, typename FeatT, int FMT>
__device__ __forceinline__ void resolve_grid(FeatT *__restrict__ grid, const Params &p, const uint8_t *__restrict__ C_l,
                                             const FeatT *__restrict__ F_l, const uint32_t side, const uint32_t verts)
{
    using Raw = typename std::conditional<sizeof(FeatT) == 2, uint32_t, float2>::type;
    // quotient by multiplication: exact for (v + 1/2) / side, v < 2^16 (the error is below 2^-6 / side, the distance
    // to the next whole number at least 1 / (2 side))
    const float    inv = 1.0f / (float)side;
    constexpr int  kAhead = 8;
    const Raw     *F = reinterpret_cast<const Raw *>(F_l);
    Raw           *G = reinterpret_cast<Raw *>(grid);
    for (uint32_t v0 = 0; v0 < verts; v0 += kLevelBlock * kAhead) {
        uint32_t at[kAhead], idx[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t v = v0 + u * kLevelBlock + threadIdx.x;
            at[u] = v < verts ? v : verts - 1u;              // beyond the grid: its last vertex again
            uint32_t rest = at[u], h1 = 0, h2 = 0;
#pragma unroll
            for (int i = 0; i < D; ++i) {
                const uint32_t q = i == D - 1 ? 0u : (uint32_t)(((float)rest + 0.5f) * inv);
                const uint32_t vi = rest - q * side;
                h1 ^= vi * kPi[i];
                h2 ^= vi * kPi2[i];
                rest = q;
            }
            idx[u] = probe_base(h1, p) + read_probe<FMT>(C_l, h2 & p.c_mask, p.log2_Np);
        }
        Raw f[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) f[u] = F[idx[u]];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) G[at[u]] = f[u];
    }
}

template <int D, typename FeatT, typename IoT, int FMT>
__global__ __launch_bounds__(kLevelBlock) void encode_fwd_level_kernel(
    const Params p, const float *__restrict__ x, const FeatT *__restrict__ D_f, const uint8_t *__restrict__ D_c,
    IoT *__restrict__ yT, const int64_t N, const uint32_t c_stride, const int vec, const uint32_t resident,
    const LevelSplit ls)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int      t = threadIdx.x;
    const bool     on_grid = blockIdx.x >= ls.hash_units;                    // the same for the whole workgroup
    int            l;
    int64_t        n_begin, n_end;
    if (!on_grid) {
        const uint32_t levels = (uint32_t)p.L_loaded - ls.dense;
        uint32_t part;
        if (ls.by_xcd) {
            const uint32_t unit = blockIdx.x % kFwdXcds * (ls.hash_units / kFwdXcds) + blockIdx.x / kFwdXcds;
            // levels in the order 0, h, 1, h + 1, ... (h = half of them): an XCD gets a coarse and a fine one
            const uint32_t q = unit / ls.hash_parts;
            l = (int)(ls.dense + q / 2u + (q & 1u) * ((levels + 1u) / 2u));
            part = unit % ls.hash_parts;
            if (q >= levels) return;
        } else {
            l = (int)(ls.dense + blockIdx.x % levels);
            part = blockIdx.x / levels;
            if (part >= ls.hash_parts) return;
        }
        n_begin = (int64_t)part * ls.hash_per;
        n_end = n_begin + ls.hash_per;
    } else {
        const uint32_t unit = blockIdx.x - ls.hash_units;
        l = 0;
        while (l + 1 < (int)ls.dense && unit >= ls.grid_first[l + 1]) ++l;
        n_begin = (int64_t)(unit - ls.grid_first[l]) * ls.grid_per[l];
        n_end = n_begin + ls.grid_per[l];
    }
    if (n_end > N) n_end = N;
    const uint8_t *C_l = D_c + (size_t)l * c_stride;
    const FeatT   *F_l = D_f + (size_t)l * p.N_f * 2;
    IoT           *out = yT + (size_t)l * (size_t)N * 2;
    const uint32_t N_l = p.N_l[l];

    // The coordinates of the next step's points are loaded while this step's lookups are under way.  A wavefront takes runs of
    // 128 points and leaves when the part is done; a lane beyond the part
    // repeats its last point and stores the same values again: with a branch around the stores the wait for the
    // coordinates would be a wait for every store before them as well.
    constexpr int64_t kStep = (int64_t)kLevelUnroll * kLevelBlock;
    auto point = [&](const int64_t first, const int u) {
        const int64_t n = first + u * 64 + (t & 63);
        return n < n_end ? n : n_end - 1;
    };
    auto fetch = [&](const int64_t first, float (&xp)[kLevelUnroll][D]) {
#pragma unroll
        for (int u = 0; u < kLevelUnroll; ++u) {
            const int64_t n = point(first, u);
#pragma unroll
            for (int j = 0; j < D; ++j) xp[u][j] = x[n * D + j];
        }
    };
    auto interpolate = [&](const int64_t n, const float (&wt)[1 << D], const float2 (&feat)[1 << D]) {
        float y0 = 0.0f, y1 = 0.0f;
#pragma unroll
        for (int c = 0; c < (1 << D); ++c) {
            y0 = fmaf(wt[c], feat[c].x, y0);
            y1 = fmaf(wt[c], feat[c].y, y1);
        }
        store_pair(out, (size_t)n, y0, y1);
    };
    auto stream = [&](auto step) {
        float xa[kLevelUnroll][D], xb[kLevelUnroll][D];
        const int64_t first = n_begin + (int64_t)(t >> 6) * (64 * kLevelUnroll);
        fetch(first, xa);
        // (two buffers and a way out after each step: merging both steps into one block, or one buffer that is copied, was
        // 2 % and 10 % slower on 2^24 points)
        for (int64_t n0 = first; n0 < n_end;) {
            fetch(n0 + kStep, xb);
            step(n0, xa);
            if ((n0 += kStep) >= n_end) break;
            fetch(n0 + kStep, xa);
            step(n0, xb);
            n0 += kStep;
        }
    };

    if (on_grid) {
        // Bound by the LDS (8 reads per point and level at d = 3), the vector ALU and, when nothing else runs beside it, by
        // reading the points: 54 us for a level of 2^24 points against 160 where the features are looked up, which is the
        // rate at which a CU can ask the L2 for cache lines.
        FeatT         *grid = reinterpret_cast<FeatT *>(smem);
        const uint32_t side = N_l + 2u;
        uint32_t verts = 1, stride[D];
#pragma unroll
        for (int i = 0; i < D; ++i) { stride[i] = verts; verts *= side; }
        resolve_grid<D, FeatT, FMT>(grid, p, C_l, F_l, side, verts);
        __syncthreads();
        // the cell's lower vertex along an axis: the one rounded fp32 multiply of Cell<D>; beyond N_l for a coordinate beyond 1
        auto lower = [&](const float v) {
#pragma clang fp contract(off)
            return (uint32_t)floorf(v * (float)N_l);
        };
        int beyond = 0;
        stream([&](const int64_t n0, const float (&xp)[kLevelUnroll][D]) {
            float  wt[kLevelUnroll][1 << D];
            float2 feat[kLevelUnroll][1 << D];
#pragma unroll
            for (int u = 0; u < kLevelUnroll; ++u) {
                uint32_t v = 0;
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    const uint32_t at = lower(xp[u][i]);
                    beyond |= at > N_l ? 1 : 0;
                    v += (at < N_l ? at : N_l) * stride[i];
                }
                Cell<D> cell;
                cell.locate(xp[u], N_l);
#pragma unroll
                for (int c = 0; c < (1 << D); ++c) {
                    uint32_t at = v;
#pragma unroll
                    for (int i = 0; i < D; ++i) at += ((c >> i) & 1) ? stride[i] : 0u;
                    feat[u][c] = load_pair(grid, at);
                    wt[u][c] = cell.weight(c);
                }
            }
#pragma unroll
            for (int u = 0; u < kLevelUnroll; ++u) interpolate(point(n0, u), wt[u], feat[u]);
        });
        if (__syncthreads_or(beyond)) {                      // points with a coordinate beyond 1: looked up as on every other level
            for (int64_t n = n_begin + t; n < n_end; n += kLevelBlock) {
                float xp[D];
                bool  in = true;
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    xp[j] = x[n * D + j];
                    in = in && lower(xp[j]) <= N_l;
                }
                if (in) continue;
                Cell<D> cell;
                cell.locate(xp, N_l);
                float  wt[1 << D];
                float2 feat[1 << D];
#pragma unroll
                for (int c = 0; c < (1 << D); ++c) {
                    wt[c] = cell.weight(c);
                    feat[c] = load_pair(F_l, probe_base(cell.hash1(c), p) + read_probe<FMT>(C_l, cell.hash2(c) & p.c_mask, p.log2_Np));
                }
                interpolate(n, wt, feat);
            }
        }
        return;
    }

    uint8_t       *probes = smem;                                            // D_c of this level: 4-bit packed, or its bit string
    const uint32_t lds_c = (p.N_c + 1u) / 2u;
    FeatT         *feats = reinterpret_cast<FeatT *>(smem + ((lds_c + 15u) & ~15u));   // entries [0, resident) of this level
    stage_probes<FMT, kLevelBlock>(probes, C_l, c_stride, lds_c, vec, t);
    {
        const uint32_t bytes = resident * (uint32_t)(2 * sizeof(FeatT));     // a multiple of 16 (host)
        for (uint32_t i = (uint32_t)t * 16u; i < bytes; i += kLevelBlock * 16u)
            *reinterpret_cast<uint4 *>(reinterpret_cast<unsigned char *>(feats) + i) =
                *reinterpret_cast<const uint4 *>(reinterpret_cast<const unsigned char *>(F_l) + i);
    }
    __syncthreads();

    // WHOLE: every entry is in LDS, so no lookup needs a branch (compressed model, 2^18 points: 29 -> 25 us)
    auto look_up = [&](auto whole) {
        constexpr bool WHOLE = decltype(whole)::value;
        stream([&](const int64_t n0, const float (&xp)[kLevelUnroll][D]) {
            uint32_t idx[kLevelUnroll][1 << D];
            float    wt[kLevelUnroll][1 << D];
#pragma unroll
            for (int u = 0; u < kLevelUnroll; ++u) {
                Cell<D> cell;
                cell.locate(xp[u], N_l);
#pragma unroll
                for (int c = 0; c < (1 << D); ++c) {
                    idx[u][c] = probe_base(cell.hash1(c), p) +
                                (FMT == kFmtBits ? read_probe_bits_lds(probes, cell.hash2(c) & p.c_mask, p.log2_Np)
                                                 : read_probe<kFmtPacked4>(probes, cell.hash2(c) & p.c_mask, p.log2_Np));
                    wt[u][c] = cell.weight(c);
                }
            }
            float2 feat[kLevelUnroll][1 << D];
#pragma unroll
            for (int u = 0; u < kLevelUnroll; ++u)
#pragma unroll
                for (int c = 0; c < (1 << D); ++c) {
                    if (WHOLE || idx[u][c] < resident) feat[u][c] = load_pair(feats, idx[u][c]);
                    else feat[u][c] = load_pair(F_l, idx[u][c]);
                }
#pragma unroll
            for (int u = 0; u < kLevelUnroll; ++u) interpolate(point(n0, u), wt[u], feat[u]);
        });
    };
    if (resident >= p.N_f) look_up(std::true_type{});
    else look_up(std::false_type{});
}

// Levels whose tables fit in LDS side by side, four or a multiple of four of them (compressed models: the paper's Table 3 row takes 25 KB a
// level).  A workgroup then has a point's encodings of that many neighbouring levels together and writes them to the rows of y itself, 16 or
// 32 bytes at a time: no level-major copy, no second pass.  The compressed model, 2^22 points: level kernel
// and rows 417 us, so 340.
// The workgroups of a part's groups of levels run on one XCD at the same time, so that its L2 puts the pieces of a row together before
// they leave for memory.  What bounds it is what bounds the level kernel with all lookups in LDS: LDS, at work 86 % of the time, and vector ALU, 81 %.
struct GroupSplit {
    uint32_t levels = 0, groups = 0, parts = 0;              // levels per workgroup (0: not taken); groups of them; parts of the batch
    int64_t  per = 0;                                        // points per part
    uint32_t probes = 0, stride = 0;                         // LDS bytes of a level's index codebook, and of a level
};
constexpr uint32_t kQuad = 4;            // levels that leave together

template <int D, typename FeatT, typename IoT, int FMT>
__global__ __launch_bounds__(kLevelBlock) void encode_fwd_group_kernel(
    const Params p, const float *__restrict__ x, const FeatT *__restrict__ D_f, const uint8_t *__restrict__ D_c,
    IoT *__restrict__ y, const int64_t N, const uint32_t c_stride, const int vec, const GroupSplit gs)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int      t = threadIdx.x;
    const uint32_t j = blockIdx.x / kFwdXcds, part = j / gs.groups * kFwdXcds + blockIdx.x % kFwdXcds, l0 = j % gs.groups * gs.levels;
    if (part >= gs.parts) return;
    const int64_t n_begin = (int64_t)part * gs.per, n_end = n_begin + gs.per < N ? n_begin + gs.per : N;
    if (n_begin >= n_end) return;
    const uint32_t lds_c = (p.N_c + 1u) / 2u, feat_bytes = p.N_f * (uint32_t)(2 * sizeof(FeatT));      // (a multiple of 16: host)
    for (uint32_t g = 0; g < gs.levels; ++g) {
        unsigned char *tables = smem + g * gs.stride;
        const unsigned char *F_l = reinterpret_cast<const unsigned char *>(D_f + (size_t)(l0 + g) * p.N_f * 2);
        stage_probes<FMT, kLevelBlock>(tables, D_c + (size_t)(l0 + g) * c_stride, c_stride, lds_c, vec, t);
        for (uint32_t i = (uint32_t)t * 16u; i < feat_bytes; i += kLevelBlock * 16u)
            *reinterpret_cast<uint4 *>(tables + gs.probes + i) = *reinterpret_cast<const uint4 *>(F_l + i);
    }
    __syncthreads();
    // (a wavefront takes runs of 128 points; a lane beyond the part repeats its last point, as in the level kernel)
    constexpr int64_t kStep = (int64_t)kLevelUnroll * kLevelBlock;
    auto point = [&](const int64_t first, const int u) {
        const int64_t n = first + u * 64 + (t & 63);
        return n < n_end ? n : n_end - 1;
    };
    auto fetch = [&](const int64_t first, float (&xp)[kLevelUnroll][D]) {
#pragma unroll
        for (int u = 0; u < kLevelUnroll; ++u) {
            const int64_t n = point(first, u);
#pragma unroll
            for (int i = 0; i < D; ++i) xp[u][i] = x[n * D + i];
        }
    };
    struct alignas(2 * sizeof(IoT)) Piece { IoT v[2]; };     // a level's two features
    const size_t row = (size_t)p.L * 2;
    float xp[kLevelUnroll][D], next[kLevelUnroll][D];
    const int64_t first = n_begin + (int64_t)(t >> 6) * (64 * kLevelUnroll);
    fetch(first, xp);
    for (int64_t n0 = first; n0 < n_end; n0 += kStep) {
        fetch(n0 + kStep, next);
        Piece out[kLevelUnroll][kQuad];
#pragma unroll 1                                             // (four levels at once, mixed by the compiler, take 128 registers and spill)
        for (uint32_t g = 0; g < gs.levels; ++g) {
            const uint8_t *probes = smem + g * gs.stride;
            const FeatT   *feats = reinterpret_cast<const FeatT *>(probes + gs.probes);
            uint32_t idx[kLevelUnroll][1 << D];
            float    wt[kLevelUnroll][1 << D];
#pragma unroll
            for (int u = 0; u < kLevelUnroll; ++u) {
                Cell<D> cell;
                cell.locate(xp[u], p.N_l[l0 + g]);
#pragma unroll
                for (int c = 0; c < (1 << D); ++c) {
                    idx[u][c] = probe_base(cell.hash1(c), p) +
                                (FMT == kFmtBits ? read_probe_bits_lds(probes, cell.hash2(c) & p.c_mask, p.log2_Np)
                                                 : read_probe<kFmtPacked4>(probes, cell.hash2(c) & p.c_mask, p.log2_Np));
                    wt[u][c] = cell.weight(c);
                }
            }
            float2 feat[kLevelUnroll][1 << D];
#pragma unroll
            for (int u = 0; u < kLevelUnroll; ++u)
#pragma unroll
                for (int c = 0; c < (1 << D); ++c) feat[u][c] = load_pair(feats, idx[u][c]);
#pragma unroll
            for (int u = 0; u < kLevelUnroll; ++u) {
                float y0 = 0.0f, y1 = 0.0f;
#pragma unroll
                for (int c = 0; c < (1 << D); ++c) {
                    y0 = fmaf(wt[u][c], feat[u][c].x, y0);
                    y1 = fmaf(wt[u][c], feat[u][c].y, y1);
                }
#pragma unroll
                for (uint32_t i = 0; i + 1 < kQuad; ++i) out[u][i] = out[u][i + 1];
                store_pair(out[u][kQuad - 1].v, 0, y0, y1);
            }
            if (g % kQuad == kQuad - 1u) {
#pragma unroll
                for (int u = 0; u < kLevelUnroll; ++u) {
                    uint4 piece[sizeof(out[0]) / 16];
                    __builtin_memcpy(piece, out[u], sizeof(piece));
                    uint4 *dst = reinterpret_cast<uint4 *>(y + (size_t)point(n0, u) * row + (size_t)(l0 + g - (kQuad - 1u)) * 2);
#pragma unroll
                    for (int i = 0; i < (int)(sizeof(out[0]) / 16); ++i) dst[i] = piece[i];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kLevelUnroll; ++u)
#pragma unroll
            for (int i = 0; i < D; ++i) xp[u][i] = next[u][i];
    }
}

// yT[l][n] (pairs) -> y[row(n)][l], row(n) = perm ? perm[n] : n; levels from L_loaded on are written as zeros.
// One workgroup per 256 points: coalesced reads per level into a padded LDS tile, then the tile's rows leave as one
// contiguous block (whole rows, piece by piece, under a permutation).
constexpr int kRowsTile = 256;
template <typename IoT>
__global__ __launch_bounds__(kRowsTile) void level_major_to_rows_kernel(
    const IoT *__restrict__ yT, IoT *__restrict__ y, const int64_t N, const int L, const int L_loaded,
    const int32_t *__restrict__ perm)
{
    using Pair = typename std::conditional<sizeof(IoT) == 2, uint32_t, uint2>::type;
    extern __shared__ __align__(16) unsigned char smem[];
    Pair         *tile = reinterpret_cast<Pair *>(smem);                     // [kRowsTile][L + 1]
    const int     t = threadIdx.x;
    const int64_t n0 = (int64_t)blockIdx.x * kRowsTile;
    const int64_t rows = (N - n0 < kRowsTile) ? N - n0 : kRowsTile;
    const Pair   *src = reinterpret_cast<const Pair *>(yT);
    Pair          zero;
    __builtin_memset(&zero, 0, sizeof(zero));
    for (int l0 = 0; l0 < L; l0 += 8) {                     // eight levels' loads in flight, then their LDS writes
        Pair v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            v[j] = (l0 + j < L_loaded && t < rows) ? src[(size_t)(l0 + j) * (size_t)N + (size_t)(n0 + t)] : zero;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (l0 + j < L) tile[t * (L + 1) + l0 + j] = v[j];
    }
    __syncthreads();
    Pair *dst = reinterpret_cast<Pair *>(y);
    for (int i = t; i < (int)rows * L; i += kRowsTile) {
        const int r = i / L, c = i - r * L;
        const size_t row = perm ? (size_t)perm[n0 + r] : (size_t)(n0 + r);
        dst[row * (size_t)L + c] = tile[r * (L + 1) + c];
    }
}

}  // namespace cngp
