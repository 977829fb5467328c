// C ABI of the Compact NGP encoding library: argument checks, level table, kernel
// selection and launches.  See include/cngp.h for the contract of every entry point.
#include "../../include/cngp.h"
#include "cngp_kernels.h"
#include "cngp_fwd_level.h"
#include "cngp_bwd_sliced.h"
#include "cngp_bwd_binned.h"
#include "cngp_bwd_runs.h"
#include "cngp_rates.h"
#include "cngp_optim.h"
#include "cngp_mlp.h"

#include <cmath>
#include <cstdio>
#include <cstring>
#include <numeric>
#include <type_traits>
#include <string>
#include <vector>
#include <algorithm>
#include <utility>

namespace {

using namespace cngp;

thread_local std::string g_hip_error;

bool is_pow2(uint32_t v) { return v != 0 && (v & (v - 1)) == 0; }
uint32_t ilog2(uint32_t v) { uint32_t r = 0; while (v > 1) { v >>= 1; ++r; } return r; }

int hip_fail(hipError_t e, const char *what) {
    g_hip_error = std::string(what) + ": " + hipGetErrorString(e);
    return CNGP_ERR_HIP;
}
}  // namespace

// for the other translation unit of the library (cngp_sort.hip): same record as cngp_last_hip_error() reads
namespace cngp { int record_hip_failure(hipError_t e, const char *what) { return hip_fail(e, what); } }

namespace {
#define CNGP_HIP(call) do { hipError_t e_ = (call); if (e_ != hipSuccess) return hip_fail(e_, #call); } while (0)

// ---------------------------------------------------------------- static scratch of the allocation-free entry point
// cngp_encode_bwd_static works in this array instead of a caller's workspace.  Every GPU the library runs on
// holds its own copy, at its own address, until the process ends.  In host code the array's NAME is only a
// handle: the device address comes from hipGetSymbolAddress, once per device, and is what every launch gets.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
constexpr int    kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
void *g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void **out) {
    int dev = -1;
    CNGP_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return CNGP_ERR_UNSUPPORTED;
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        CNGP_HIP(hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return CNGP_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return CNGP_OK;
}

// ---------------------------------------------------------------- validation (host only)
int validate(const cngp_config *c) {
    if (!c) return CNGP_ERR_NULL;
    if (c->d < 2 || c->d > 4) return CNGP_ERR_INVALID;
    if (c->L < 1 || c->L > kMaxLevels) return CNGP_ERR_INVALID;
    if (c->F < 1) return CNGP_ERR_INVALID;
    if (!is_pow2(c->N_f) || !is_pow2(c->N_c) || !is_pow2(c->N_p)) return CNGP_ERR_INVALID;
    if (c->N_p > 16 || c->N_p > c->N_f) return CNGP_ERR_INVALID;
    if (c->N_f > (1u << 30) || c->N_c > (1u << 30)) return CNGP_ERR_INVALID;
    if (c->N_min < 1) return CNGP_ERR_INVALID;
    if (c->L > 1 && (c->N_max < c->N_min || c->N_max > (1u << 24))) return CNGP_ERR_INVALID;
    if (c->N_min > (1u << 24)) return CNGP_ERR_INVALID;
    if (c->feat_dtype != CNGP_F32 && c->feat_dtype != CNGP_F16) return CNGP_ERR_INVALID;
    if (c->io_dtype != CNGP_F32 && c->io_dtype != CNGP_F16) return CNGP_ERR_INVALID;
    if (c->index_format != CNGP_IDX_U8 && c->index_format != CNGP_IDX_PACKED4 && c->index_format != CNGP_IDX_BITS) return CNGP_ERR_INVALID;
    if (c->index_format == CNGP_IDX_PACKED4 && c->N_c < 2) return CNGP_ERR_INVALID;
    if (c->flags & ~(uint32_t)(CNGP_ZERO_GRADS | CNGP_BWD_DIRECT | CNGP_BWD_SLICED | CNGP_BWD_NO_PREREDUCE | CNGP_FWD_SIMPLE | CNGP_BWD_BINNED | CNGP_FWD_LEVEL | CNGP_FWD_TILE)) return CNGP_ERR_INVALID;
    if ((c->flags & CNGP_BWD_DIRECT) && (c->flags & (CNGP_BWD_SLICED | CNGP_BWD_BINNED))) return CNGP_ERR_INVALID;
    if ((c->flags & CNGP_FWD_LEVEL) && (c->flags & (CNGP_FWD_SIMPLE | CNGP_FWD_TILE))) return CNGP_ERR_INVALID;
    if (c->top_k > c->N_p || c->reserved != 0) return CNGP_ERR_INVALID;
    if (c->F != 1 && c->F != 2 && c->F != 4 && c->F != 8) return CNGP_ERR_UNSUPPORTED;
    return CNGP_OK;
}

// Table 1 (N_min, N_max, L): geometric growth, floor with a 1e-6 guard so that exact powers
// (in particular N_{L-1} = N_max) survive the rounding of exp / pow.
// (The last table is kept, per thread: sixteen powers are half a microsecond of a call.)
void level_table(const cngp_config *c, uint32_t *out) {
    if (c->L == 1) { out[0] = c->N_min; return; }
    thread_local uint32_t kept[kMaxLevels], kept_min = 0, kept_max = 0;
    thread_local int32_t  kept_L = 0;
    if (c->L != kept_L || c->N_min != kept_min || c->N_max != kept_max) {
        const double b = std::exp(std::log((double)c->N_max / (double)c->N_min) / (double)(c->L - 1));
        for (int l = 0; l < c->L; ++l)
            kept[l] = (uint32_t)std::floor((double)c->N_min * std::pow(b, (double)l) + 1e-6);
        kept_L = c->L;
        kept_min = c->N_min;
        kept_max = c->N_max;
    }
    std::memcpy(out, kept, sizeof(uint32_t) * (size_t)c->L);
}

Params make_params(const cngp_config *c) {
    Params p;
    std::memset(&p, 0, sizeof(p));
    level_table(c, p.N_l);
    p.L = c->L;
    p.L_loaded = c->L;
    p.N_f = c->N_f;
    p.N_c = c->N_c;
    p.row_mask = c->N_f / c->N_p - 1;
    p.c_mask = c->N_c - 1;
    p.log2_Np = ilog2(c->N_p);
    p.top_k = (c->top_k && c->top_k < c->N_p) ? c->top_k : 0;
    return p;
}

// Bytes between the index codebooks of consecutive levels.
size_t index_level_bytes(const cngp_config *c) {
    if (c->index_format == CNGP_IDX_PACKED4) return c->N_c / 2;
    if (c->index_format == CNGP_IDX_BITS) return 4 * (((size_t)c->N_c * ilog2(c->N_p) + 31) / 32);
    return c->N_c;
}
// The exact-width format of a codebook with N_p = 1 has no bytes at all: its pointer may be NULL.
bool index_codebook_is_empty(const cngp_config *c) { return c->index_format == CNGP_IDX_BITS && c->N_p == 1; }

int check_blocks(int64_t blocks) { return (blocks > 0x7fffffffLL) ? CNGP_ERR_INVALID : CNGP_OK; }

// ---------------------------------------------------------------- per-kernel timing
enum KernelId { K_FWD = 0, K_BWD_DIRECT, K_BWD_PREP, K_BWD_SLICED, K_BWD_SLICED_V, K_BWD_GRID_DRAIN,
                K_BAKE, K_ZERO, K_DEBUG, K_ADAM, K_MLP_FWD, K_MLP_BWD,
                K_BWD_BIN_OFFSETS, K_BWD_BIN_SCATTER, K_BWD_BIN_DRAIN, K_BWD_INPUT, K_FUSED_FWD, K_PLANES, K_FWD_ROWS, K_BWD_SMALL, K_BWD_CELLS, K_BWD_MERGE, K_BWD_PARTIAL, K_COUNT };
const char *const kKernelNames[K_COUNT] = {"encode_fwd", "encode_bwd_direct", "encode_bwd_prepare",
                                           "encode_bwd_sliced_points_and_grid", "encode_bwd_sliced_vertices",
                                           "encode_bwd_bin_grid_sums", "bake_probes", "zero", "debug_indices",
                                           "adam_step_bake", "mlp_fwd", "mlp_bwd",
                                           "encode_bwd_bin_offsets", "encode_bwd_bin_scatter",
                                           "encode_bwd_bin_drain", "encode_bwd_input", "encode_mlp_fwd", "feature_planes",
                                           "encode_fwd_rows", "encode_bwd_small", "encode_bwd_cells", "encode_bwd_merge",
                                           "encode_bwd_partial_sums"};

struct TimedLaunch { int id; hipEvent_t t0, t1; };
bool g_profile = false;
std::vector<TimedLaunch> g_timed;

struct LaunchTimer {
    hipStream_t s; int id; hipEvent_t t0 = nullptr, t1 = nullptr; bool on;
    LaunchTimer(hipStream_t s_, int id_) : s(s_), id(id_), on(g_profile) {
        if (on && (hipEventCreate(&t0) != hipSuccess || hipEventCreate(&t1) != hipSuccess)) on = false;
        if (on) (void)hipEventRecord(t0, s);
    }
    ~LaunchTimer() {
        if (on) { (void)hipEventRecord(t1, s); g_timed.push_back({id, t0, t1}); }
    }
};

int launch_status(const char *what) {
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? CNGP_OK : hip_fail(e, what);
}

// ---------------------------------------------------------------- launches
// Collects the arrays one call has to clear and clears them with a single launch.
struct ZeroList {
    ZeroSegments seg;
    int          n = 0;
    int64_t      largest = 0;
    void add(float *ptr, int64_t count) {
        if (count <= 0 || n >= kZeroSegments) return;
        seg.ptr[n] = ptr;
        seg.count[n] = count;
        if (count > largest) largest = count;
        ++n;
    }
    int launch(hipStream_t s) {
        if (n == 0) return CNGP_OK;
        int64_t blocks = (largest / 4 + kBlock - 1) / kBlock;
        if (blocks > 2048) blocks = 2048;
        if (blocks < 1) blocks = 1;
        LaunchTimer t(s, K_ZERO);
        zero_kernel<<<dim3((unsigned)blocks, (unsigned)n), kBlock, 0, s>>>(seg);
        n = 0;
        largest = 0;
        return launch_status("zero_kernel");
    }
};

template <typename K>
int allow_big_lds(K kernel, size_t bytes) {
    if (bytes <= 64 * 1024) return CNGP_OK;
    hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    return e == hipSuccess ? CNGP_OK : hip_fail(e, "hipFuncSetAttribute(MaxDynamicSharedMemorySize)");
}

// Level-resident forward (cngp_fwd_level.h): which calls take it, and its launch shape.  Host arithmetic only.
struct FwdLevelPlan {
    bool     use = false;
    uint32_t resident = 0;       // entries of a level's feature codebook that sit in LDS
    size_t   lds = 0;            // dynamic LDS of the kernel
    LevelSplit split = {};       // levels that interpolate from a resolved grid; points per workgroup of either kind
    size_t   yT_bytes = 0;       // the level-major copy of the encodings: the workspace this variant needs
    GroupSplit group = {};       // levels whose tables all fit in LDS, several to a workgroup: rows of y are written directly
};
constexpr int64_t kCus = 256;
// Corner lookups (N * L * 2^d) up to which encode_fwd_kernel, one launch with every lookup in flight at once, is the
// fastest forward.  Measured, GPU and call together, us: nerf3d's tables, 8192 points (2^20 lookups): 11.5 against 12.9 for
// the level-resident pair of launches and 57 for the tile kernel, 16384 points: 19 / 13 / 52; fp32 tables of 2^18 entries
// (sdf3d) 18.8 / 29 / 120 at 8192, 33 / 28 / 119 at 16384; d = 2, 16384 points: 10.5 / 13.0 / 28; d = 4, 4096: 10.3 / 15.3 / 81.
constexpr int64_t kSmallFwdRefs = 1 << 20;
// The same against the tile kernel alone, for a caller without a workspace.  That kernel takes the levels one after the other,
// so with few of them it is the faster one sooner.  One launch / tiles, us, at 2^21.5 .. 2^22 lookups: L = 2 11.2 / 6.8 and
// 11.8 / 10.0, L = 4 11.7 / 7.9, L = 6 23 / 16, L = 8 9.4 / 18, L = 16 (nerf3d) 34 / 46, the compressed model 23 / 31, L = 24
// 24 / 49; at 2^21 lookups L = 4 9.8 / 20, L = 6 21.6 / 22; at 2^25 nerf3d 217 / 99.
constexpr int64_t kSmallFwdRefsNoRoom = 1 << 22, kSmallFwdRefsNoRoomFewLevels = 1 << 21;
constexpr int     kFewLevels = 8;
constexpr size_t  kLevelLdsBudget = 156 * 1024;
constexpr int64_t kLevelPartPoints = 65536;              // points per workgroup when the batch is large
constexpr uint64_t kFwdL2Bytes = 3u << 20;               // of an XCD's 4 MB, what tables can count on
constexpr int64_t kGroupPartPoints = 65536;              // points per workgroup of several levels

FwdLevelPlan fwd_level_plan_uncached(const cngp_config *c, int levels_loaded, int64_t N) {
    FwdLevelPlan f;
    if (c->F != 2 || levels_loaded < 1 || N <= 0 || (c->flags & (CNGP_FWD_SIMPLE | CNGP_FWD_TILE))) return f;
    const size_t entry = 2 * (c->feat_dtype == CNGP_F16 ? 2 : 4), io = c->io_dtype == CNGP_F16 ? 2 : 4;
    const size_t probes = (((size_t)c->N_c + 1) / 2 + 15) & ~(size_t)15;
    if (((size_t)c->N_f * entry) % 16 != 0 || probes > 64 * 1024) return f;
    size_t resident = (kLevelLdsBudget - probes) / entry;
    if (resident > c->N_f) resident = c->N_f;
    resident &= ~(size_t)3;                                              // whole 16-byte pieces
    // Measured on nerf3d's, image2d's and the compressed model's tables from 2^12 to 2^24 points: never slower than the
    // tile variant (1.2x - 3x faster), also when only a seventh of a level's feature codebook fits (sdf3d, 1.15x).  So it
    // can be taken whenever it can run -- except for a few thousand points, where its second launch costs more than it
    // saves (that line is encode_mlp_fwd's; the encode_fwd calls have a shorter way up to kSmallFwdRefs).
    if (!(c->flags & CNGP_FWD_LEVEL) && N * levels_loaded < ((int64_t)1 << 15)) return f;
    f.use = true;
    f.resident = (uint32_t)resident;
    f.lds = probes + resident * entry + 16;
    // Levels whose whole vertex grid fits the same LDS can interpolate from it (not where all of D_f is in LDS anyway:
    // the compressed model got 9 % slower, filling the grids costs what the shorter lookups save).
    uint32_t res[kMaxLevels];
    level_table(c, res);
    int      most_grids = 0;
    uint64_t verts[kMaxGridLevels];
    while (resident < c->N_f && most_grids < levels_loaded && most_grids < kMaxGridLevels && res[most_grids] < 4096) {
        uint64_t v = 1;
        for (int i = 0; i < c->d; ++i) v *= (uint64_t)res[most_grids] + 2;
        if (v * entry > kLevelLdsBudget) break;
        verts[most_grids++] = v;
    }
    // Clocks of a CU, fitted to measurements of single levels (fp16, nerf3d's and image2d's tables, 2^18 .. 2^24 points): a
    // point that is looked up, by the share of lookups that leave the CU; a point on a grid; a vertex to fill in.  Checked on
    // 260 drawn configurations (d = 2 .. 4, fp16 and fp32, N_f 2^12 .. 2^18, 2^16 .. 2^21 points) with every number of grids timed.
    const double miss = 1.0 - (double)resident / c->N_f, lookup = (double)(1 << c->d) * (0.21 + 1.66 * miss);
    const double on_grid = c->d == 2 ? 1.8 : c->d == 3 ? 2.4 : 4.0, fill = 3.3;
    const int64_t step = (int64_t)kLevelBlock * kLevelUnroll;
    auto parts_of = [&](double per) {                        // parts of at most `per` points, whole steps of a workgroup at least
        const int64_t least = per < (double)step ? step : (int64_t)per;
        return (N + least - 1) / least;
    };
    auto grid_points = [&](int l, double per) { return (per * lookup - (double)verts[l] * fill) / on_grid; };
    // The launch in whole rounds of one workgroup per CU, all of about the same length: one round while the batch is small,
    // more for a large one (the levels differ in cost).  The longest parts of looked-up levels that need no more workgroups
    // than that, for every number of levels on grids; the shortest of these wins.
    // (the looked-up levels in eight runs of equal length if they are kept apart by XCD)
    auto by_xcd = [&](int64_t levels) { return (uint64_t)(c->N_f - resident) * entry * levels > kFwdL2Bytes; };
    auto looked_up_units = [&](int64_t levels, int64_t parts) {
        return by_xcd(levels) ? (levels * parts + kFwdXcds - 1) / kFwdXcds * kFwdXcds : levels * parts;
    };
    auto units_of = [&](int grids, double per) {
        int64_t u = looked_up_units(levels_loaded - grids, parts_of(per));
        for (int l = 0; l < grids; ++l) {
            const double n = grid_points(l, per);
            if (n < 64.0) return (int64_t)1 << 40;
            u += parts_of(n);
        }
        return u;
    };
    // The tables (their parts outside LDS) that an XCD's L2 gets to see.  Every one of them is fetched into it once, at about
    // 700 bytes a clock; and where the tables do not fit one L2 together, a run of units that begins and ends inside a level
    // holds one more than it has to (14 levels in eight runs touch three each, 16 levels two), which costs 6 % per MB of a
    // table (260 drawn configurations: 1.2x for 1.86 MB tables (fp32, 2^18 entries), 1.1x for 0.87 MB, 1.04x for 0.36 MB).
    const double table = (double)((uint64_t)(c->N_f - resident) * entry);
    auto tables_per_xcd = [&](int64_t levels, int64_t parts) {
        if (levels < 1) return (int64_t)0;
        if (!by_xcd(levels)) return levels / std::gcd(levels, (int64_t)kFwdXcds);
        const int64_t run = looked_up_units(levels, parts) / kFwdXcds;
        int64_t most = 0;
        for (int64_t x = 0; x < (int64_t)kFwdXcds; ++x) {
            const int64_t first = x * run / parts;
            int64_t       last = ((x + 1) * run - 1) / parts;
            if (last > levels - 1) last = levels - 1;
            if (last - first + 1 > most) most = last - first + 1;
        }
        return most;
    };
    auto cost_of = [&](int64_t levels, double per, int64_t rounds) {
        const int64_t tables = tables_per_xcd(levels, parts_of(per)), least = (levels + kFwdXcds - 1) / kFwdXcds;
        const int64_t too_many = by_xcd(levels) && tables > least ? tables - least : 0;
        return per * (double)rounds * (1.0 + 0.06 * table / (1 << 20) * (double)too_many) + (double)tables * table / (700.0 * lookup);
    };
    int    grids = 0;
    double best = 0.0, best_per = 0.0;
    for (int g = 0; g <= most_grids; ++g) {
        const double load = (double)N * ((levels_loaded - g) + g * on_grid / lookup) / kCus;      // in looked-up points per CU
        int64_t rounds = (int64_t)(load / kLevelPartPoints + 0.5);
        if (rounds < 1) rounds = 1;
        double lo = 0.0, hi = 2.0 * (double)N * levels_loaded + 1e6;
        for (int i = 0; i < 48 && hi - lo > 64.0; ++i) {
            const double mid = 0.5 * (lo + hi);
            if (units_of(g, mid) <= kCus * rounds) hi = mid;
            else lo = mid;
        }
        const double cost = cost_of(levels_loaded - g, hi, rounds);
        if (g == 0 || cost < 0.97 * best) { best = cost; best_per = hi; grids = g; }
    }
    auto cut = [&](double per, int64_t &size) {
        const int64_t parts = parts_of(per);
        size = ((N + parts - 1) / parts + 63) / 64 * 64;
        return (uint32_t)((N + size - 1) / size);
    };
    LevelSplit &ls = f.split;
    const int64_t hashed = levels_loaded - grids;
    ls.dense = (uint32_t)grids;
    ls.by_xcd = by_xcd(hashed) ? 1u : 0u;
    ls.hash_parts = cut(best_per, ls.hash_per);
    ls.hash_units = (uint32_t)looked_up_units(hashed, ls.hash_parts);
    for (int l = 0; l < grids; ++l) {
        ls.grid_first[l + 1] = ls.grid_first[l] + cut(grid_points(l, best_per), ls.grid_per[l]);
        if (verts[l] * entry > f.lds) f.lds = verts[l] * entry;
    }
    f.yT_bytes = (size_t)N * c->L * 2 * io;
    // Several levels to a workgroup (encode_fwd_group_kernel), where all their tables fit: as many fours as do and as make whole groups of
    // the levels, but no more than leave a workgroup of one round a whole step of points.  Level kernel and rows / groups, us: the compressed model
    // (four levels to a workgroup) 2^13 points 11 / 10, 2^16 16 / 13, 2^18 36 / 29, 2^20 114 / 91, 2^22 417 / 340; with fp32 encodings 523 / 356;
    // N_f = 2^12, N_c = 2^14 2^13 11 / 8, 2^18 31 / 23, 2^22 345 / 256; d = 2, L = 12, N_f = 2^10 2^22 191 / 106.  N_f = 2^8, N_c = 2^12, of
    // which sixteen levels fit: 2^22 points 341 / 263, but 2^16 14 / 22, where four take 10.
    const size_t bits = c->index_format == CNGP_IDX_BITS ? (index_level_bytes(c) + 4 + 15) & ~(size_t)15 : probes, of_level = bits + (size_t)c->N_f * entry;
    int group = (int)(kLevelLdsBudget / of_level) / (int)kQuad * (int)kQuad;
    if (group > c->L) group = c->L / (int)kQuad * (int)kQuad;
    auto at_once = [&](int levels) {                         // parts of the batch that run side by side, a whole number of them on every XCD
        const int64_t per_xcd = kCus / kFwdXcds / (c->L / levels);
        return (per_xcd > 1 ? per_xcd : 1) * (int64_t)kFwdXcds;
    };
    while (group > 0 && (c->L % group || (group > (int)kQuad && N < at_once(group) * step))) group -= (int)kQuad;
    if (resident >= c->N_f && group > 0 && levels_loaded == c->L) {
        GroupSplit &gs = f.group;
        gs.levels = (uint32_t)group;
        gs.groups = (uint32_t)(c->L / group);
        gs.probes = (uint32_t)bits;
        gs.stride = (uint32_t)of_level;
        const int64_t parts = at_once(group), rounds = (N + parts * kGroupPartPoints - 1) / (parts * kGroupPartPoints);
        gs.per = ((N + parts * rounds - 1) / (parts * rounds) + 63) / 64 * 64;
        gs.parts = (uint32_t)((N + gs.per - 1) / gs.per);
    }
    return f;
}

// The plan depends on (configuration, levels, N) only; the last one is kept (host memory, per thread).
FwdLevelPlan fwd_level_plan(const cngp_config *c, int levels_loaded, int64_t N) {
    thread_local cngp_config  last_cfg;
    thread_local int          last_levels = -1;
    thread_local int64_t      last_N = -1;
    thread_local FwdLevelPlan last_plan;
    if (last_N == N && last_levels == levels_loaded && std::memcmp(&last_cfg, c, sizeof(*c)) == 0) return last_plan;
    last_plan = fwd_level_plan_uncached(c, levels_loaded, N);
    last_cfg = *c;
    last_levels = levels_loaded;
    last_N = N;
    return last_plan;
}

template <int D, typename FeatT, typename IoT>
int launch_fwd_level(const cngp_config *c, const FwdLevelPlan &f, const Params &p, const float *x, int64_t N, const void *D_f,
                     const void *D_c, void *y, void *yT, hipStream_t s, const int32_t *perm, bool rows = true) {
    const size_t  c_stride = index_level_bytes(c);
    const int vec = (c_stride % 16 == 0 && ((uintptr_t)D_c & 15u) == 0) ? 1 : 0;
    if (f.group.levels && rows && !perm && ((uintptr_t)y & 15u) == 0) {          // (rows of a multiple of four levels: whole pieces of 16 bytes)
        const int64_t blocks = ((int64_t)f.group.parts + kFwdXcds - 1) / kFwdXcds * kFwdXcds * f.group.groups;
        if (int rc = check_blocks(blocks)) return rc;
        const size_t lds = (size_t)f.group.levels * f.group.stride;
#define CNGP_FWD_GROUP_LAUNCH(FMT)                                                                          \
    do {                                                                                                    \
        auto kernel = encode_fwd_group_kernel<D, FeatT, IoT, FMT>;                                          \
        if (int rc = allow_big_lds(kernel, lds)) return rc;                                                 \
        LaunchTimer t(s, K_FWD);                                                                            \
        kernel<<<(unsigned)blocks, kLevelBlock, lds, s>>>(p, x, (const FeatT *)D_f, (const uint8_t *)D_c,   \
                                                          (IoT *)y, N, (uint32_t)c_stride, vec, f.group);   \
    } while (0)
        if (c->index_format == CNGP_IDX_PACKED4) CNGP_FWD_GROUP_LAUNCH(kFmtPacked4);
        else if (c->index_format == CNGP_IDX_BITS) CNGP_FWD_GROUP_LAUNCH(kFmtBits);
        else CNGP_FWD_GROUP_LAUNCH(kFmtU8);
#undef CNGP_FWD_GROUP_LAUNCH
        return launch_status("encode_fwd_group_kernel");
    }
    const int64_t blocks = (int64_t)f.split.hash_units + f.split.grid_first[f.split.dense];
    if (int rc = check_blocks(blocks)) return rc;
#define CNGP_FWD_LEVEL_LAUNCH(FMT)                                                                          \
    do {                                                                                                    \
        auto kernel = encode_fwd_level_kernel<D, FeatT, IoT, FMT>;                                          \
        if (int rc = allow_big_lds(kernel, f.lds)) return rc;                                               \
        LaunchTimer t(s, K_FWD);                                                                            \
        kernel<<<(unsigned)blocks, kLevelBlock, f.lds, s>>>(p, x, (const FeatT *)D_f, (const uint8_t *)D_c, \
                                                            (IoT *)yT, N, (uint32_t)c_stride, vec, f.resident, f.split); \
    } while (0)
    if (c->index_format == CNGP_IDX_PACKED4) CNGP_FWD_LEVEL_LAUNCH(kFmtPacked4);
    else if (c->index_format == CNGP_IDX_BITS) CNGP_FWD_LEVEL_LAUNCH(kFmtBits);
    else CNGP_FWD_LEVEL_LAUNCH(kFmtU8);
#undef CNGP_FWD_LEVEL_LAUNCH
    if (int rc = launch_status("encode_fwd_level_kernel")) return rc;
    if (!rows) return CNGP_OK;                               // the caller reads the level-major array itself
    const int64_t tiles = (N + kRowsTile - 1) / kRowsTile;
    if (int rc = check_blocks(tiles)) return rc;
    const size_t lds = (size_t)kRowsTile * (c->L + 1) * 2 * sizeof(IoT);
    {
        LaunchTimer t(s, K_FWD_ROWS);
        level_major_to_rows_kernel<IoT><<<(unsigned)tiles, kRowsTile, lds, s>>>((const IoT *)yT, (IoT *)y, N, c->L, p.L_loaded, perm);
    }
    return launch_status("level_major_to_rows_kernel");
}

// Which kernel encodes a batch, given `room` usable bytes of workspace: one of CNGP_FWD_ROUTE_*, or the error of a forced
// variant that cannot run.  `plan` is filled in for the level-resident one.
int fwd_route(const cngp_config *c, int levels_loaded, int64_t N, size_t room, FwdLevelPlan *plan) {
    const int64_t refs = (N * c->L) << c->d;
    if (refs > kSmallFwdRefs || (c->flags & (CNGP_FWD_LEVEL | CNGP_FWD_TILE))) {
        *plan = fwd_level_plan(c, levels_loaded, N);
        if (plan->use && room >= plan->yT_bytes) return CNGP_FWD_ROUTE_LEVEL;
        if (c->flags & CNGP_FWD_LEVEL) return plan->use ? CNGP_ERR_WORKSPACE : CNGP_ERR_UNSUPPORTED;
    }
    // tile variant: one level's index codebook and the tile's outputs fit in LDS
    const size_t lds = (((size_t)c->N_c + 1) / 2 + 15) / 16 * 16 + (size_t)kFwdTile * c->L * 2 * (c->io_dtype == CNGP_F16 ? 2 : 4);
    const bool   small = refs <= (c->L < kFewLevels ? kSmallFwdRefsNoRoomFewLevels : kSmallFwdRefsNoRoom) && !(c->flags & CNGP_FWD_TILE);
    return lds <= 64 * 1024 && N >= kFwdTile && !small && !(c->flags & CNGP_FWD_SIMPLE) ? CNGP_FWD_ROUTE_TILE : CNGP_FWD_ROUTE_LANES;
}

template <int D, typename FeatT, typename IoT>
int launch_fwd(const cngp_config *c, const Params &p, const float *x, int64_t N, const void *D_f,
               const void *D_c, void *y, hipStream_t s, const int32_t *perm = nullptr,
               void *workspace = nullptr, size_t workspace_bytes = 0) {
    // (level-resident: when the caller lent the room for the level-major copy)
    const bool   usable = workspace && ((uintptr_t)workspace & 255u) == 0 && ((uintptr_t)D_f & 15u) == 0;
    FwdLevelPlan f;
    const int    route = fwd_route(c, p.L_loaded, N, usable ? workspace_bytes : 0, &f);
    if (route < 0) return route;
    if (route == CNGP_FWD_ROUTE_LEVEL) return launch_fwd_level<D, FeatT, IoT>(c, f, p, x, N, D_f, D_c, y, workspace, s, perm);
    const size_t c_stride = index_level_bytes(c);
    const int    fmt = c->index_format;
    const size_t lds_probes = (((size_t)c->N_c + 1) / 2 + 15) & ~(size_t)15;
    const size_t lds = lds_probes + (size_t)kFwdTile * c->L * 2 * sizeof(IoT);
    const size_t lds_large = lds_probes + (size_t)kFwdTileLarge * c->L * 2 * sizeof(IoT);
    if (route == CNGP_FWD_ROUTE_TILE) {
        // Staging a level's codebook costs c_stride bytes per workgroup; a tile looks up TILE * 2^d entries.
        // When the staging outweighs the lookups of a small tile and there are points enough to keep every
        // CU busy with large ones, take the large tile.
        const bool large = c_stride >= 8192 && lds_large <= 128 * 1024 && N >= (int64_t)kFwdTileLarge * 1024;
        const int  tile = large ? kFwdTileLarge : kFwdTile;
        // a small feature codebook (the paper's compressed models) goes to LDS with the index codebook
        const size_t   feat_bytes = (size_t)c->N_f * 2 * sizeof(FeatT);
        // (measured: a third faster at N_f = 2^10, even at 2^12, slower from 2^13: the copy then costs more than the gathers it saves)
        const uint32_t feat_lds = (c->N_f <= 4096 && (large ? lds_large : lds) + feat_bytes <= 150 * 1024) ? (uint32_t)feat_bytes : 0u;
        const int64_t blocks = (N + tile - 1) / tile;
        if (int rc = check_blocks(blocks)) return rc;
        const int vec = (c_stride % 16 == 0 && ((uintptr_t)D_c & 15u) == 0) ? 1 : 0;
#define CNGP_FWD_TILE(FMT, TILE, LDS)                                                                   \
        do {                                                                                            \
            auto kernel = encode_fwd_tile_kernel<D, FeatT, IoT, FMT, TILE>;                             \
            if (int rc = allow_big_lds(kernel, LDS + feat_lds)) return rc;                              \
            LaunchTimer t(s, K_FWD);                                                                    \
            kernel<<<(unsigned)blocks, TILE, LDS + feat_lds, s>>>(                                      \
                p, x, (const FeatT *)D_f, (const uint8_t *)D_c, (IoT *)y, N, (uint32_t)c_stride, vec, perm, feat_lds); \
        } while (0)
#define CNGP_FWD_TILE_FMT(FMT)                                                                          \
        if (large) CNGP_FWD_TILE(FMT, kFwdTileLarge, lds_large); else CNGP_FWD_TILE(FMT, kFwdTile, lds)
        if (fmt == CNGP_IDX_PACKED4) { CNGP_FWD_TILE_FMT(kFmtPacked4); }
        else if (fmt == CNGP_IDX_BITS) { CNGP_FWD_TILE_FMT(kFmtBits); }
        else { CNGP_FWD_TILE_FMT(kFmtU8); }
#undef CNGP_FWD_TILE_FMT
#undef CNGP_FWD_TILE
        return launch_status("encode_fwd_tile_kernel");
    }
    // one wavefront per workgroup spreads a small batch over more CUs
    const unsigned block = N * c->L <= 64 * 4 * kCus ? 64u : (unsigned)kBlock;
    const uint32_t points = block / (uint32_t)c->L, level_magic = (65536u + (uint32_t)c->L - 1u) / (uint32_t)c->L;
    const int64_t  blocks = (N + points - 1) / points;
    if (int rc = check_blocks(blocks)) return rc;
    LaunchTimer t(s, K_FWD);
#define CNGP_FWD_SIMPLE_LAUNCH(FMT)                                                                     \
    encode_fwd_kernel<D, FeatT, IoT, FMT><<<(unsigned)blocks, block, 0, s>>>(                           \
        p, x, (const FeatT *)D_f, (const uint8_t *)D_c, (IoT *)y, N, points, level_magic, (uint32_t)c_stride, perm)
    if (fmt == CNGP_IDX_PACKED4) CNGP_FWD_SIMPLE_LAUNCH(kFmtPacked4);
    else if (fmt == CNGP_IDX_BITS) CNGP_FWD_SIMPLE_LAUNCH(kFmtBits);
    else CNGP_FWD_SIMPLE_LAUNCH(kFmtU8);
#undef CNGP_FWD_SIMPLE_LAUNCH
    return launch_status("encode_fwd_kernel");
}

// Workgroups of the input gradient.  256 lanes, a point each, stage the level's codebook once per 256 points; 1024 lanes stage
// it a quarter as often and keep the chip's lookups closer together, but fill fewer wavefronts while the batch is small, and
// hold each other up at the barriers.  Where the large ones pay was measured on d = 2 .. 4, fp16 and fp32, all three formats,
// N_f 2^8 .. 2^18, N_c 2^14 .. 2^17 and 60000 to 1600000 points (time with them by time without):
//  * from 160 Ki points where only two 256-lane workgroups fit a CU (N_c = 2^17: 0.24 .. 0.9), and where what is staged is
//    at least 32 KB in memory (with 8-byte entries of a table below 1 MB 64 KB: two points a lane leave it fewer wavefronts)
//    and d <= 3 (bytes, N_c = 2^16: 0.65 .. 0.9; at d = 4 the lookups are what takes the time: 0.9 .. 1.2); 200 Ki with
//    8-byte tables of 2 MB (0.72 .. 0.95);
//  * from 2^18 points, which is all that 256-lane workgroups hold at once beside N_c = 2^16, with tables of 1 MB or more
//    (0.5 .. 0.95), with bytes or d <= 3 there (0.45 .. 0.95) and with bytes and d <= 3 at N_c = 2^15 (0.7 .. 0.95); else it
//    is 0.9 .. 1.2, at d = 4 up to 1.6;
//  * from 2^20 points for any codebook of 8 KB or more.
// 8-byte entries: one workgroup per CU with two points per lane (fp32, N_f = 2^18, 300007 points: 0.6, with one point 0.65);
// from 2^20 points only where that still gains: a table of 2 MB (0.57 against 0.65), at d = 2 of 128 KB; smaller ones take
// up to 1.15 times as long.  (The d = 4 instance with packed bytes spills 8 registers: 0.57 .. 0.7, as with one point.)
// Below 2^20 points all are of the same size, in whole rounds (nothing but the last round's lanes is idle); above, full ones
// with one point per lane (1300000 points: 5 .. 9 % faster, the rounds no longer run in step).
struct BwdInputShape { bool large; int pts; int64_t per; };
BwdInputShape bwd_input_shape(const cngp_config *c, int64_t N) {
    const size_t stride = index_level_bytes(c), lds = (((size_t)c->N_c + 1) / 2 + 15) & ~(size_t)15;
    const bool   wide = c->feat_dtype == CNGP_F32, huge = N >= (int64_t)kFwdTileLarge * 1024, bytes = c->index_format == CNGP_IDX_U8;
    const size_t table = (size_t)c->N_f * (wide ? 8 : 4);
    BwdInputShape b = {false, 1, kFwdTile};
    if (lds > 64 * 1024 || N < kFwdTile) return b;
    const bool codebook = lds >= 16 * 1024;
    if (codebook && N >= 160 * 1024)
        b.large = lds >= 64 * 1024 || (c->d <= 3 && stride >= (size_t)(wide && table < (1u << 20) ? 64 : 32) * 1024) ||
                  (wide && table >= (2u << 20) && N >= 200 * 1024);
    if (codebook && N > 256 * 1024)
        b.large = b.large || table >= (1u << 20) || (c->d <= 3 && (lds >= 32 * 1024 || bytes)) || (lds >= 32 * 1024 && bytes);
    if (huge && stride >= 8192) b.large = true;
    if (!b.large) return b;
    if (wide && codebook && (!huge || table >= (c->d == 2 ? 128u << 10 : 2u << 20))) b.pts = 2;
    const int64_t most = (int64_t)b.pts * kFwdTileLarge, slots = b.pts == 2 ? kCus : 2 * kCus;
    b.per = most;
    if (!huge || b.pts == 2) {
        const int64_t wgs = (N + slots * most - 1) / (slots * most) * slots;
        b.per = ((N + wgs - 1) / wgs + 63) / 64 * 64;
    }
    return b;
}
template <int D, typename FeatT, typename IoT>
int launch_bwd_input(const cngp_config *c, const Params &p, const float *x, int64_t N, const void *D_f,
                     const void *D_c, const void *dy, float *grad_x, hipStream_t s) {
    const size_t c_stride = index_level_bytes(c);
    const int    fmt = c->index_format;
    const size_t lds = (((size_t)c->N_c + 1) / 2 + 15) & ~(size_t)15;
    const bool   staged = lds <= 64 * 1024 && N >= kFwdTile;
    constexpr bool wide = sizeof(FeatT) == 4;
    const BwdInputShape shape = bwd_input_shape(c, N);
    const int64_t per = shape.per;
    const int64_t blocks = (N + per - 1) / per;
    if (int rc = check_blocks(blocks)) return rc;
    const int vec = (c_stride % 16 == 0 && ((uintptr_t)D_c & 15u) == 0) ? 1 : 0;
    LaunchTimer t(s, K_BWD_INPUT);
#define CNGP_BWD_INPUT(FMT, TILE, STAGED, PTS)                                                              \
    encode_bwd_input_kernel<D, FeatT, IoT, FMT, TILE, STAGED, PTS><<<(unsigned)blocks, TILE, STAGED ? lds : 0, s>>>( \
        p, x, (const FeatT *)D_f, (const uint8_t *)D_c, (const IoT *)dy, grad_x, N, (uint32_t)c_stride, vec, (uint32_t)per)
#define CNGP_BWD_INPUT_FMT(FMT)                                                                             \
    if (!staged) CNGP_BWD_INPUT(FMT, kFwdTile, false, 1);                                                   \
    else if (shape.large && shape.pts == 2) CNGP_BWD_INPUT(FMT, kFwdTileLarge, true, (wide ? 2 : 1));        \
    else if (shape.large) CNGP_BWD_INPUT(FMT, kFwdTileLarge, true, 1);                                       \
    else CNGP_BWD_INPUT(FMT, kFwdTile, true, 1)
    if (fmt == CNGP_IDX_PACKED4) { CNGP_BWD_INPUT_FMT(kFmtPacked4); }
    else if (fmt == CNGP_IDX_BITS) { CNGP_BWD_INPUT_FMT(kFmtBits); }
    else { CNGP_BWD_INPUT_FMT(kFmtU8); }
#undef CNGP_BWD_INPUT_FMT
#undef CNGP_BWD_INPUT
    return launch_status("encode_bwd_input_kernel");
}

template <int D, int NP, typename FeatT, typename IoT>
int launch_bwd_direct(const cngp_config *c, const Params &p, int level0, int nlevels, const float *x,
                      int64_t N, const void *D_f, const float *Dhat_c, const void *dy, float *gD_f,
                      float *gDhat_c, hipStream_t s) {
    (void)c;
    if (nlevels <= 0) return CNGP_OK;
    constexpr int PTS = kBlock / NP;
    const int64_t blocks = (N + PTS - 1) / PTS;
    if (int rc = check_blocks(blocks)) return rc;
    LaunchTimer t(s, K_BWD_DIRECT);
    encode_bwd_direct_kernel<D, NP, FeatT, IoT><<<dim3((unsigned)blocks, (unsigned)nlevels), kBlock, 0, s>>>(
        p, level0, x, (const FeatT *)D_f, Dhat_c, (const IoT *)dy, gD_f, gDhat_c, N);
    return launch_status("encode_bwd_direct_kernel");
}


// ---------------------------------------------------------------- backward plan
size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// How one sliced kernel launch splits its items (points or grid vertices) into chunks.
struct Geom { uint32_t chunks, chunk_items; };

struct BwdPlan {
    bool     sliced;
    uint32_t rows_f_log2, slices_f;     // feature-gradient slices per level
    uint32_t rows_c_log2, slices_c;     // logit-gradient slices per level (0 when N_p == 1)
    Geom     feat_pts, logit_pts;       // hashed levels: chunks of points
    Geom     feat_vtx, logit_vtx;       // dense levels: chunks of grid vertices
    Geom     grid;                      // vertex-grid accumulation: chunks of points
    size_t   lds_f, lds_c;              // dynamic LDS bytes of the two kernels
    bool     split;                     // replicated scan in many chunks whose sums meet in the workspace (bwd_partial_sums_kernel)
    size_t   sigma_off, dyT_off, G_off, partF_off, partC_off, ws_bytes;
    bool     binned;                    // hashed levels: references binned by slice first (cngp_bwd_binned.h)
    bool     sum_f, sum_c, sum_wide;    // ... and a table's sums of a bin's drain workgroups meet in the workspace, where the merged entries were; in 64 bits
    bool     scarce;                    // ... of tables whose slices alone would be scanned: because levels are merged, or plain hashing of few slices
    bool     fused;                     // ... by slice of the confidence table only: a level's whole feature gradient sits in LDS beside it
    uint32_t bin_chunks, bin_chunk_pts; // point chunks of the count / scatter kernels
    bool     lone;                      // one drain workgroup per bin (kMostSoonRefsPerBin)
    uint32_t subs_f, subs_c;            // drain workgroups per bin
    size_t   cntF_off, cntC_off, baseF_off, baseC_off, recF_off, recC_off;
    size_t   cntG_off, baseG_off, recG_off;          // pre-reduced levels binned by slice of their vertex grid; merged ones by slice of the tables
    bool     merged;                    // the first levels' references are merged per vertex and binned as entries (cngp_bwd_merge.h); dense.count of them
    MergeParams merge;
    uint64_t G_bytes, cntG_bytes, baseG_bytes, recG_bytes;
    GridDrainPlan grid_drain;
    DenseLevels dense;                  // levels pre-reduced per grid vertex (a prefix of the levels); merged: only their number
    uint32_t dense_slices, dense_verts, dense_max_verts;
};

constexpr uint64_t kMaxAutoBinBytes = 8ull << 30;   // workspace the library asks for on its own initiative
constexpr uint32_t kMaxFusedNf = 4096;          // largest feature table per level whose gradient is kept whole in LDS
constexpr size_t   kFusedLdsBytes = 152 * 1024; // LDS of the workgroups that accumulate both gradients
constexpr uint32_t kMinBinnedSlicesPerLevel = 24; // from here on binning the references beats the replicated scan
// Plain hashing (N_p = 1), whose scans cost as much as any and whose references cost the least, is binned from fewer slices on: slices, and
// slices times references per level.  Backward, scanned / binned, us: N_f = 2^17 (16 slices) d = 3, L = 8, 2^20 points 1030 / 379,
// 2^18 278 / 149, L = 16 100000 217 / 131, 30000 97 / 107; d = 2 300000 244 / 142; d = 4 100000 300 / 144; N_f = 2^16 (8) d = 3, 2^18
// 195 / 135, 100000 138 / 139, d = 4 2^18 473 / 308; d = 2, N_max = 512, 439631 points, four levels to scan (kMinMergedScans) 174 / 191.
constexpr uint32_t kMinBinnedPlainSlices = 8;
constexpr int64_t  kMinBinnedPlainScans = 12 << 20;
// One drain workgroup per bin then, where no levels are merged (fp64 sums, rounded once), and stretches of kPlainGridRecords of the grid sums'
// records each: with 32768, and two to five workgroups per bin, more fp32 sums met in an entry than the scan's chunks add (error against 64
// bits, 2-norm, scanned / so / now: N_f = 2^17, L = 8, 2^18 points 6.7e-8 / 7.6e-8 / 5.7e-8, 700009 points 9.0e-8 / 10.5e-8 / 6.6e-8).
// Fewer bins than kMinBinnedPlainGroups would leave CUs idle (L = 8, 8 slices, 520823 points: 335 us, so 401).
constexpr int64_t  kMinBinnedPlainGroups = 96, kPlainGridRecords = 131072;
constexpr uint32_t kMaxSlicesPerLevel = 128;   // beyond this the replicated scan costs more than global atomics
// Both gradient tables of a level (fp64) that a small batch accumulates in LDS.  420 drawn tables up to that size, 30 points to
// 2^19 references, kernel alone against the direct one: 2.4x faster on average (up to 48 KB 2.6x, 96 .. 128 KB 1.6x), up to 145x
// where a coarse level's few vertices collide; the slowest 0.95x (12.2 us against 11.5).
constexpr size_t   kSmallBwdLds = 128 * 1024;
constexpr int64_t  kMinBinnedRefs = 1 << 21;    // corner references from which any table that can be binned with a gain is (measured: 2^14 points of the headline shape)
// Tables with several slices of both kinds are binned sooner: from kMinBinnedSoonRefs, and with many candidates, whose scans and atomics
// cost the most, from kMinBinnedCandidateRefs.  us, before (scan, below 2^19 references atomics) / binned: 8 + 16 slices, N_p = 16 2^18.5 126 / 73,
// 2^19.5 96 / 76, 2^20.3 133 / 88, 2^21 185 / 118; 32 + 32, N_p = 8 2^20.3 148 / 107, 2^21 197 / 124, but 2^18.6 75 / 92, 2^19.1 97 / 91; 16 + 8,
// N_p = 4 2^19.1 56 / 63; d = 2 16 + 16, N_p = 16 2^19.9 78 / 80.  With one slice of either table the drain has few, long workgroups: 1 + 32, N_p = 8
// 2^20.7 118 / 170, 32 + 2, N_p = 16 2^20.8 170 / 198.
constexpr int64_t  kMinBinnedSoonRefs = 1 << 20, kMinBinnedCandidateRefs = 1 << 18;
// 90 drawn batches that this and the next rules bin (d = 2 .. 4, 1 .. 16 levels): 68 with atomics before 1.08 .. 17.9x, 3.4x on average, 22 scanned before
// 1.08 .. 2.8x, 1.8x; left out: d = 4 (16 + 8, N_p = 16 2^19.1 48 / 53), 96 slices (2^18.2 104 / 106), a small feature table with 256
// slices of the other (2^18.3 101 / 163), or with 64 and fewer candidates (N_p = 8 2^18.1 60 / 69).
constexpr uint32_t kMinBinnedSoonSlices = 8, kManyCandidates = 16, kMostCandidateSlices = 64;
// A small feature table is binned from here on (kMinSlicedRefs: above it the scan's sums meet in 64 bits); us, atomics / binned: N_f = 2^8, N_c = 2^14, N_p = 16
// 3608 points 250 / 47; N_f = 2^12, N_c = 2^15, N_p = 8 3504 points 76 / 55, 4756 points, L = 8 57 / 40.
constexpr int64_t  kMinBinnedFusedRefs = 1 << 18;
// Where such a batch was scanned (kMinSlicedRefs), its bins have one drain workgroup each: a scan rounds the fp64 sum of an entry once, while two
// workgroups and more round theirs to fp32 before they meet.  Few levels then leave few, long bins: with more than kMostSoonRefsPerBin references times levels
// in a bin of the table with fewer slices the batch is scanned (never from eight levels on).  us, scanned / binned (in brackets with the
// workgroups that fill the chip), and the errors of both gradients against 64 bits, 2-norm, 1e-8: 8 + 16 slices, N_p = 16, L = 8, 17559 points 85 / 69 (57),
// 8.00 8.22 / 7.76 7.97 (8.19 7.97), 30573 115 / 95 (80), 8.08 8.30 / 7.76 7.99 (8.50 8.44); L = 6, 23413 91 / 78 (56), 40765 96 / 113 (84); L = 4, 18821 67 / 65
// (48), 35119 80 / 99 (54), 8.11 8.32 / 7.77 7.96 (8.72 8.42); L = 1, 140479 49 / 305 (62).  32 + 32, N_p = 8, L = 4, 61147 122 / 69 (80); L = 2, 70239 69 / 65
// (53), 122295 92 / 95 (72).  Points anything but evenly spread, 8 + 16, L = 8, 30573: all equal 239 / 189, on a plane 112 / 95, in a cube of side
// 0.02 237 / 333; L = 16, 15287: 357 / 192, 207 / 73, 357 / 192; 32 + 32, L = 8, 30573: 273 / 205, 153 / 72, 292 / 127.
constexpr int64_t  kMostSoonRefsPerBin = 4096;
// Workgroups of the scatter, one per level and chunk, up to which each has four wavefronts: so few leave most SIMDs without one, and the walk of 1024 points by a
// single wavefront is a chain of memory latencies (scatter, us, one wavefront / four: 320 workgroups 25 / 13, 640 27 / 17, 1264 29 / 23; but the
// drain of 1570 loses 3 % of 270, more than that gains).  Whole backward, one / four, 25 batches up to the line, a table with a single bin or several: 1.00 .. 1.28x; 1 + 32
// slices, N_p = 8, 16411 points 149 / 137, 63001 173 / 171; 32 + 1, N_p = 4, 63001 117 / 112; 8 + 16, N_p = 16, 2048 60 / 47, 63001 169 / 162.
constexpr int64_t  kFewBinChunks = 1024;
// References per level (N * 2^d) from which the binned variant, where it does not merge, always pre-reduces coarse levels; below,
// binned_bwd_us decides.
// Backward, us, with / without, beyond it: nerf3d's tables 163840 points 384 / 403, 2^18 539 / 569; sdf3d's 2^20 2786 / 3294;
// d = 2 600000 1001 / 1175.
constexpr int64_t  kMinBinnedPrereduceRefs = 1 << 20;
// Merging (cngp_bwd_merge.h): references per level from which the three launches more are worth it, and references per vertex of
// a level's grid, in hundredths, from which the level is merged (points are never spread more evenly than over the whole grid).
// Backward, us, without / with merging, at 2^19, 2^20, 3 * 2^19 and 2^21 references per level: nerf3d's tables 244 / 238, 334 / 306,
// 434 / 403, 541 / 489; sdf3d's 351 / 236, 507 / 407, 669 / 576, 831 / 739; d = 2 (N_f = 2^18, N_c = 2^16, N_p = 8) 343 / 208,
// 661 / 325, 800 / 463, 926 / 596; N_f = 2^18, N_c = 2^14, N_p = 4 197 / 175, 270 / 231, 343 / 314, 429 / 371; plain hashing
// (N_f = 2^19) 95 / 98, 296 / 147, 342 / 183, 400 / 226; 2^19 .. 2^20 0.86 .. 1.1x.
// Up to kMinMergedRefs only with kMinMergeLevels levels, two of them merged, or plain hashing: of 218 drawn batches there of tables that are binned
// either way these are 130, 1.31x, two of them below 0.97x; the others are 0.99 .. 1.02x on average and 37 of 88 below 0.97x (d = 2, five levels, 64 + 8 slices,
// 347924 points: 157 us, merged 207).  The line itself is on the safe side, an eighth above kMinBinnedPrereduceRefs: from 2^20 on the tables above gain
// too, and the plans of the batches in between are as they were.
// Points anything but evenly spread, without / with: all equal 1719 / 1279 (nerf3d's tables, 2^18 points), in a cube of side 0.02
// 1233 / 812, on a line 1145 / 951, on a plane 544 / 519; sdf3d's 2^20 points 6127 / 3684, 3693 / 2137, 3548 / 2329, 2780 / 2139.
// Sum of the kernels of a step, us, lines at 20 / 80 / 150 / 300 / 1500: nerf3d 728 / 611 / 594 / 587 / 601 (649 with grid sums),
// sdf3d, whose points are anything but evenly spread, 2750 / 2704 / 2786 / 2815 / 2977 (3184), compact3d 504 / 465 / 448 / 453 / 478 (469).
// Backward without / with merging, mean (slowest) of 40 drawn batches of 2^18 .. 2^20 points, lines at 60 / 90 / 150 / 250: 1.25 (0.91), 1.25 (0.91), 1.26
// (0.94), 1.27 (0.97).
// Backward without / with merging over 110 drawn configurations from that batch size on: d = 3 1.19x faster on average (slowest 0.95x),
// d = 2 1.28x; d = 4, where two or three levels have that many references per vertex, 0.99x (0.78 .. 1.21), and small feature
// tables with d = 2 and N_p = 2, whose references cost the least, 0.90x: neither is merged.
constexpr int64_t  kMinMergeRefs = 9 << 17;
constexpr int      kMinMergeLevels = 8;
constexpr uint64_t kMinMergePerVertexPct = 240;
// Bins of a level from which the scatter writes in runs (cngp_bwd_runs.h).  Backward, direct / in runs, us, with a record per corner in both tables' bins: sdf3d's tables (32 + 32
// bins) 30000 points 150 / 140, 100000 345 / 309, 2^18 uniform 723 / 656, 2^20 near a surface 2407 / 2170; 32 + 16 bins 681 / 632,
// 8 + 64 797 / 746, 64 + 128 1078 / 997, d = 2, 32 + 32 999 / 922.  Below the line the scatter gains as well, but the drain loses as
// much: 32 + 8 bins 579 / 579, 16 + 16 624 / 621, 16 + 8 566 / 576, nerf3d's 8 + 16 533 / 542, 32 + 2 564 / 594.  A table with a single
// bin has nothing to gain, and its drain lives on the order that a lone wavefront keeps: 72 drawn batches of such tables 0.99x,
// 27 of them below 0.97x (128 + 1 bins, d = 3, 358780 points: 288 us, in runs 328), while those of two bins and more in both tables, or of plain
// hashing, gain 1.02 .. 1.19x.
constexpr uint32_t kMinRunBins = 48;
// Tables of fewer slices than kMinBinnedSlicesPerLevel are binned all the same where levels are merged (kMinMergeRefs and what stands
// there) and few_slices_pay says so: references per level from which (59 drawn batches of 2^20 .. 3 * 2^19 scanned / binned: 0.54 .. 1.76x),
// slices per level from which, slices times levels that a scan would not pre-reduce, and what the scan has to do per reference that is
// binned.  image2d's tables (8 + 2 slices): backward 958 us scanned, 783 binned.  1742 drawn batches of these tables (d = 2 and 3, 2 .. 16
// levels, every N_p from 2 on, 3 * 2^19 .. 2^23 references a level, uniform points, rays and a shell), scanned / binned: all of them 1.24x,
// but the slowest 0.19x (every level pre-reduced: 79.6 us, 411), and 300 below 0.97x; the 912 from a gain of 2.8 on 1.47x, 14 below 0.97x.  Of 208
// others from 2.8 on 1.42x, nine below 0.97x, the slowest 0.78x (d = 3, L = 6, 4 + 4 slices, 548667 points: 388 us, 496), every one below 0.9x with a gain
// under 3.0; from there on the slowest 0.95x (d = 2, where the merged levels leave fewer of their references, 2.8 .. 3: 1.14 .. 1.6x).  With six slices 1.1x at most on average, down to 0.81x.
// They ask for up to 65 times the workspace of the scan, 28 times on the median (image2d's 66 -> 1994 MB; 2^21 points 4238, 3 * 2^20 6354), and
// from where that passes kMaxAutoBinBytes, at 2^22 points there, the batch is scanned; so is one in a smaller workspace.
constexpr int64_t  kMinMergedRefs = 3 << 19;
constexpr uint32_t kMinMergedSlices = 8;
constexpr int64_t  kMinMergedScans = 48;
constexpr double   kMinMergedGain = 3.0, kMinMergedGainFlat = 2.8;      // (d = 3, d = 2)
constexpr int64_t  kMinSlicedRefs = 1 << 19;    // corner references (N * L * 2^d) below which launch overheads win
constexpr uint64_t kMaxDenseVerts = 32ull * kDenseSliceVerts;   // largest vertex grid that is pre-reduced
constexpr int64_t  kMinRefsPerVertex = 4;      // below this reuse the vertex pass saves nothing

// Drain workgroups per bin of a table with `slices` slices per level: about 2^16 corners each (a record, or half of one in the feature table's
// bins), and enough workgroups to fill the chip twice, but never less than 8192 each.  `refs` references per level, `levels` hashed levels.
// `longer`: of the long bins of a few slices, 1.5 times the records each, whose sums are fewer to add up.  `alone`: of plain hashing with few slices, whose
// one table has few bins, enough to fill it once (N_f = 2^17, L = 16, 100000 points: 131 us, so 83).
uint32_t drain_subs(double refs, uint32_t slices, int levels, uint32_t slices_per_level, bool longer = false, bool alone = false) {
    if (!slices) return 1;
    double want = refs / slices / (longer ? 98304.0 : 65536.0);
    const double fill = (alone ? 256.0 : 512.0) / ((double)levels * slices_per_level), by_size = refs / slices / 8192.0;
    if (want < fill) want = fill;
    if (want > by_size) want = by_size;
    const uint32_t r = (uint32_t)(want + 0.5);
    return r < 1 ? 1 : (r > 64 ? 64 : r);
}

// Chunk count that minimises (rounds of workgroups over the CUs) x (items per chunk + fixed cost per
// workgroup, in items: clearing and flushing its LDS slice).  `groups` workgroups exist per chunk.
Geom pick_chunks(int64_t items, int64_t groups, int64_t fixed, int64_t min_chunk) {
    Geom best = {1, (uint32_t)((items + 63) / 64 * 64)};
    int64_t best_cost = -1;
    for (int64_t c = 1; c <= 64; ++c) {
        int64_t chunk = ((items + c - 1) / c + 63) / 64 * 64;
        if (chunk < 64) chunk = 64;
        if (c > 1 && chunk < min_chunk) break;
        const int64_t real = (items + chunk - 1) / chunk;                 // chunks that hold items
        const int64_t rounds = (groups * real + kCus - 1) / kCus;
        const int64_t cost = rounds * (chunk + fixed);
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = {(uint32_t)real, (uint32_t)chunk}; }
    }
    if (best.chunks < 1) best.chunks = 1;
    return best;
}

// Chunk counts of the four roles of the sliced kernel, by simulating its launch: workgroups are
// handed out in grid order to the first free of 256 CUs; a workgroup costs a fixed part (clearing and
// flushing its LDS slice, about 12000 scanned points' worth) plus its items times a per-item cost that
// grows with the share of corners it keeps.  Measured on MI355X: fewer, longer workgroups win unless a
// finer split fills the last round.
// (CUs that become free at the same time are taken together: a few dozen steps where there are thousands of workgroups.)
double simulate_makespan(const std::pair<int64_t, double> *batches /* count, duration */, int n) {
    struct Free { double at; int64_t cus; };
    Free   f[kCus];
    int    groups = 1;
    double end = 0.0;
    f[0] = {0.0, kCus};
    for (int b = 0; b < n; ++b)
        for (int64_t left = batches[b].first; left > 0; ) {
            int first = 0, same = -1;
            for (int g = 1; g < groups; ++g) if (f[g].at < f[first].at) first = g;
            const int64_t took = left < f[first].cus ? left : f[first].cus;
            const double  at = f[first].at + batches[b].second;
            for (int g = 0; g < groups; ++g) if (f[g].at == at) same = g;
            left -= took;
            f[first].cus -= took;
            if (same >= 0) f[same].cus += took;
            else if (f[first].cus == 0) { f[first] = {at, took}; }
            else f[groups++] = {at, took};
            if (f[first].cus == 0) f[first] = f[--groups];
            if (at > end) end = at;
        }
    return end;
}

Geom chunks_of(int64_t items, int64_t c) {
    int64_t chunk = ((items + c - 1) / c + 63) / 64 * 64;
    if (chunk < 64) chunk = 64;
    return {(uint32_t)((items + chunk - 1) / chunk), (uint32_t)chunk};
}

constexpr int64_t kFilledWorkgroups = 224, kMostPartials = 768;     // (256 CUs)
void choose_geometry(const cngp_config *c, int64_t N, BwdPlan &b, const bool split) {
    const int    Ld = b.dense.count, Lh = c->L - Ld;
    const double corners = (double)(1 << c->d);
    // fixed cost per workgroup ~ clearing and flushing its slice: 12000 points' worth for a full 128 KB slice
    const double fixed_f = 1500.0 + 10500.0 * (double)(((size_t)1 << b.rows_f_log2) * c->N_p * 16) / kSliceBytes;
    const double fixed_c = 1500.0 + 10500.0 * (double)(((size_t)1 << b.rows_c_log2) * c->N_p * 8) / kSliceBytes;
    const double item_f = 1.0 + 2.0 * corners / b.slices_f;                      // per point, feature role
    const double item_c = b.slices_c ? 1.0 + 1.5 * corners / b.slices_c : 0.0;   // per point, logit role
    const double vtx_f = 0.6 + 2.0 / b.slices_f, vtx_c = b.slices_c ? 0.6 + 1.5 / b.slices_c : 0.0;
    b.feat_vtx = b.logit_vtx = chunks_of(b.dense_max_verts ? b.dense_max_verts : 64, 1);
    if (Ld > 0) {
        b.grid = pick_chunks(N, b.dense_slices, 4096, 8192);
        const int64_t cv = (b.dense_max_verts + 16383) / 16384;                  // vertex chunks of <= 16384
        b.feat_vtx = b.logit_vtx = chunks_of(b.dense_max_verts, cv > 0 ? cv : 1);
    }
    if (b.binned) {                         // the point roles of the hashed levels are not launched
        b.logit_pts = b.feat_pts = chunks_of(N, 1);
        return;
    }
    // small slices are cheap to clear and flush: allow finer chunks there
    const bool    small = fixed_f + fixed_c < 8000.0;
    const int64_t min_chunk = small ? 8192 : 16384, cap = small ? 32 : 12;
    const int64_t cmax = N / min_chunk > 1 ? (N / min_chunk < cap ? N / min_chunk : cap) : 1;
    auto workgroups = [&](const Geom &gc, const Geom &gf) { return (int64_t)Lh * ((int64_t)b.slices_c * gc.chunks + (int64_t)b.slices_f * gf.chunks); };
    double best = -1.0;
    for (int64_t cc = 1; cc <= (b.slices_c ? cmax : 1); ++cc)
        for (int64_t cf = 1; cf <= cmax; ++cf) {
            const Geom gc = chunks_of(N, cc), gf = chunks_of(N, cf);
            std::pair<int64_t, double> batches[4];
            int n = 0;
            if (Lh > 0 && b.slices_c) batches[n++] = {(int64_t)Lh * b.slices_c * gc.chunks, fixed_c + gc.chunk_items * item_c};
            if (Lh > 0) batches[n++] = {(int64_t)Lh * b.slices_f * gf.chunks, fixed_f + gf.chunk_items * item_f};
            if (Ld > 0 && b.slices_c) batches[n++] = {(int64_t)Ld * b.slices_c * b.logit_vtx.chunks, fixed_c + b.logit_vtx.chunk_items * vtx_c};
            if (Ld > 0) batches[n++] = {(int64_t)Ld * b.slices_f * b.feat_vtx.chunks, fixed_f + b.feat_vtx.chunk_items * vtx_f};
            const double t = simulate_makespan(batches, n);
            if (best < 0.0 || t < best) { best = t; b.logit_pts = gc; b.feat_pts = gf; }
        }
    if (!split || workgroups(b.logit_pts, b.feat_pts) >= kFilledWorkgroups) return;
    // A batch that leaves CUs without a workgroup is cut finer, to chunks of 512 points: costs that follow N_p, the grid sums that share
    // the launch, and the partial sums of slices with several chunks (per 64 bytes of gradient, as much as an atomic would take); of the choices within 5 % of
    // the shortest the one with the fewest workgroups.  Of 70 drawn configurations (d = 2 .. 4, 1 .. 23 slices, every N_p, 2^16 .. 2^22
    // references a level), each timed with up to 24 pairs of chunk counts, the choice is 1.04x slower than the best pair on average.
    // Backward over 240 drawn configurations: 1.6x faster on average than with chunks of 8192 points at least, 10x at most (d = 3,
    // N_f = 2^13, N_c = 2^11, N_p = 16, L = 8, 25752 points: 539 us, now 92).
    const double kept = corners * (0.3 + 0.06 * c->N_p), scan_f = 1.0 + 2.0 * kept / b.slices_f, scan_c = b.slices_c ? 1.0 + 1.5 * kept / b.slices_c : 0.0;
    static const int64_t kTry[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 16, 24, 32, 48, 64};
    const double segs_c = (double)(((size_t)1 << b.rows_c_log2) * c->N_p * 4) / 64, segs_f = (double)(((size_t)1 << b.rows_f_log2) * c->N_p * 8) / 64;
    auto cost = [&](const Geom &gc, const Geom &gf) {
        std::pair<int64_t, double> batches[3];
        int n = 0;
        double segments = 0.0;
        if (b.slices_c) {
            batches[n++] = {(int64_t)Lh * b.slices_c * gc.chunks, fixed_c + gc.chunk_items * scan_c};
            if (gc.chunks > 1) segments += (double)Lh * b.slices_c * gc.chunks * segs_c;
        }
        batches[n++] = {(int64_t)Lh * b.slices_f * gf.chunks, fixed_f + gf.chunk_items * scan_f};
        if (gf.chunks > 1) segments += (double)Lh * b.slices_f * gf.chunks * segs_f;
        if (Ld > 0) batches[n++] = {(int64_t)b.dense_slices * b.grid.chunks, 12000.0 + 1.5 * b.grid.chunk_items};
        return simulate_makespan(batches, n) + segments * 0.095;
    };
    struct Tried { double t; int64_t groups; Geom gc, gf; };
    std::vector<Tried> tried;
    // a gain that the costs cannot tell from none is left; of plain hashing, whose scans they overrate, a gain of less than three times
    // (d = 3, N_f = 2^8, L = 16, 31452 ray samples, 45 workgroups made 120: 83 us, 90)
    best = cost(b.logit_pts, b.feat_pts) * (c->N_p > 1 ? 0.89 : 0.35);
    for (const int64_t cc : kTry)
        for (const int64_t cf : kTry) {
            if ((cc > 1 && (cc * 512 > N || !b.slices_c)) || (cf > 1 && cf * 512 > N)) continue;
            const Geom gc = chunks_of(N, cc), gf = chunks_of(N, cf);
            const int64_t groups = workgroups(gc, gf);
            if (groups > kMostPartials) continue;
            const double t = cost(gc, gf);
            tried.push_back({t, groups, gc, gf});
            if (t < best) best = t;
        }
    int64_t fewest = -1;
    for (const Tried &g : tried)
        if (g.t <= best * 1.05 && (fewest < 0 || g.groups < fewest)) { fewest = g.groups; b.logit_pts = g.gc; b.feat_pts = g.gf; b.split = true; }
    if (b.logit_pts.chunks == 1 && b.feat_pts.chunks == 1) b.split = false;
}


// Time of a binned backward with its first Ld levels pre-reduced, us.  The drain takes the longer of its work spread over the
// CUs and its longest workgroup: a coarse level has few vertices, all of a vertex's references fall into one bin, and the
// bins of such a level are far from equal (d = 2, N_min = 16: 324 vertices for all the references of the coarsest level).
// Pre-reducing takes that away and makes its workgroups scan the whole vertex grid per slice, besides one launch more.
// (Fitted with a record per corner in either table's bins; the feature table's hold half as many now, so that what is binned costs less than this says.)
// Fitted to 560 drawn configurations (d = 2 .. 4, 2 .. 24 levels, N_f 2^12 .. 2^19, N_c to 2^17, uniform points, rays and a
// shell), each timed both ways: 12 % off on average, and 13 % on the ratio of the two ways.  Always pre-reducing was 1.19x slower than
// the better of the two on average, never pre-reducing 1.08x (up to 4.6x); this choice 1.009x.  With / without, us: nerf3d's
// tables 20011 points 152 / 119, 100003 290 / 235; d = 2, L = 12, the same tables to N_max = 512, 262143 points: 259 / 384.
double binned_bwd_us(const cngp_config *c, int64_t N, const BwdPlan &b, int Ld) {
    uint32_t res[kMaxLevels];
    level_table(c, res);
    const uint32_t tables[2] = {b.slices_f, b.slices_c}, slices = b.slices_f + b.slices_c;
    const double   refs = (double)((uint64_t)N << c->d), flush = 5.8, record = 1.37e-3 + 4.3e-5 * c->N_p, vertex = 1.15e-3;
    double work = 0.0, longest = 0.0, records = 0.0, most_verts = 0.0;
    for (int l = 0; l < c->L; ++l) {
        const double verts = std::pow((double)res[l] + 2.0, c->d);
        if (l < Ld) {
            work += slices * verts * vertex;
            if (verts > most_verts) most_verts = verts;
            continue;
        }
        const double seen = verts < refs ? verts : refs;
        for (const uint32_t s : tables) {
            if (!s) continue;
            const uint32_t subs = b.lone ? 1u : drain_subs(refs, s, c->L - Ld, slices);
            const double   mean = seen / s;
            double fullest = mean + std::sqrt(2.0 * mean * std::log(s > 2 ? (double)s : 2.0)) + (mean < 3.0 ? 1.0 : 0.0);    // vertices of the fullest bin
            if (fullest > seen) fullest = seen;
            work += (double)s * subs * flush + refs * record;
            records += refs;
            const double t = refs / seen * fullest / subs * record + flush;
            if (t > longest) longest = t;
        }
    }
    work = (work + (double)Ld * slices * std::ceil(most_verts / 16384.0) * flush) / (double)kCus;
    return 18.0 + 6.6e-6 * c->L * (double)c->N_c * c->N_p + std::sqrt(std::sqrt(work * work * work * work + longest * longest * longest * longest)) +
           3.1e-6 * records + (Ld > 0 ? 23.0 + 6.4e-6 * Ld * refs : 0.0);
}

// Which levels a binned batch merges or pre-reduces: merged where that pays, else those whose grid sums pay, those that pay in a
// large batch, or every one that can be (its set does not depend on N, so what the last layout needs only grows with N).
enum Layout { LAYOUT_MERGED = 0, LAYOUT_FAST, LAYOUT_REDUCED, LAYOUT_LEAST, LAYOUT_COUNT };

// The arrays of the merged levels inside the workspace regions of the pre-reduced ones.
struct MergedSpace { size_t entries, order, cells, total, G_bytes, cntF, cntC, made, cntG_bytes, baseF, baseC, baseG_bytes, recF, recC, recG_bytes; };
MergedSpace merged_space(const BwdPlan &b, int64_t N, int d) {
    const size_t M = (size_t)b.dense.count, cap = (size_t)N << d, sf = b.fused ? 0 : b.slices_f, sc = b.slices_c;
    MergedSpace m;
    m.entries = 0;
    m.order = align256(M * cap * sizeof(uint4));
    m.cells = m.order + align256((size_t)N * 4);
    m.total = m.cells + (size_t)b.merge.tiles * kMergeCells * 4;
    m.G_bytes = m.total + kMergeCells * 4;
    m.cntF = 0;
    m.cntC = align256(M * b.merge.chunks * sf * 4);
    m.made = m.cntC + align256(M * b.merge.chunks * sc * 4);
    m.cntG_bytes = m.made + M * b.merge.chunks * 4;
    m.baseF = 0;
    m.baseC = align256(M * (sf + 1) * 4);
    m.baseG_bytes = m.baseC + M * (sc + 1) * 4;
    m.recF = 0;
    m.recC = sf ? align256(M * cap * sizeof(EntryRecord)) : 0;
    m.recG_bytes = m.recC + (sc ? M * cap * sizeof(EntryRecord) : 0);
    return m;
}
struct MergeArrays { MergedBins bins; uint32_t *order, *cells, *total; };
MergeArrays merge_arrays(const BwdPlan &b, int64_t N, int d, void *workspace) {
    const MergedSpace m = merged_space(b, N, d);
    char *G = (char *)workspace + b.G_off, *cnt = (char *)workspace + b.cntG_off, *base = (char *)workspace + b.baseG_off, *rec = (char *)workspace + b.recG_off;
    MergeArrays a;
    a.bins = {(uint32_t *)(cnt + m.cntF), (uint32_t *)(cnt + m.cntC), (uint32_t *)(cnt + m.made),
              (uint32_t *)(base + m.baseF), (uint32_t *)(base + m.baseC), (EntryRecord *)(rec + m.recF), (EntryRecord *)(rec + m.recC),
              b.merge.levels, b.merge.chunks, b.merge.chunk_pts, (uint4 *)(G + m.entries)};
    a.order = (uint32_t *)(G + m.order);
    a.cells = (uint32_t *)(G + m.cells);
    a.total = (uint32_t *)(G + m.total);
    return a;
}

// Levels (a prefix) whose references a batch of N points merges.
int merge_levels(const cngp_config *c, int64_t N) {
    uint32_t res[kMaxLevels];
    level_table(c, res);
    const uint64_t limit = (c->d == 2 ? 1u << 16 : 1u << 10) - 2u;                              // coordinates a table key holds
    int M = 0;
    while (M < c->L - 1 && M < kMaxDense && (uint64_t)res[M] + 1 < limit) {
        uint64_t verts = 1;
        for (int i = 0; i < c->d; ++i) verts *= (uint64_t)res[M] + 2;
        if (((uint64_t)N << c->d) * 100 < verts * kMinMergePerVertexPct) break;
        ++M;
    }
    return M;
}

// Whether a level with `verts` vertices is pre-reduced: its dense vertex grid is small, much smaller than the number of references, and takes
// clearly fewer slice scans than the level's hashed tables.
bool pre_reduces(uint64_t verts, int64_t refs, uint32_t per_level) {
    const uint64_t slices = (verts + kDenseSliceVerts - 1) / kDenseSliceVerts;
    return verts <= kMaxDenseVerts && refs >= kMinRefsPerVertex * (int64_t)verts && (slices * 2 <= per_level || slices <= 1);
}

// Levels that a replicated scan over `per_level` slices pre-reduces.
int scan_dense_levels(const cngp_config *c, int64_t N, uint32_t per_level) {
    uint32_t res[kMaxLevels];
    level_table(c, res);
    int l = 0;
    for (; l < c->L && l < kMaxDense; ++l) {
        uint64_t verts = 1;
        for (int i = 0; i < c->d; ++i) verts *= (uint64_t)res[l] + 2;
        if (!pre_reduces(verts, N << c->d, per_level)) break;
    }
    return l;
}

// Whether binning pays for tables of few slices where levels are merged (kMinMergedRefs).  A scan reads every point once per slice of the
// levels it does not pre-reduce, with less to do in a slice of logits, and adds up every reference; a merged level leaves less than half
// of its references to the bins.  (`refs`: a record per corner and table, as measured then; the feature table's bins hold half as many now, so the
// line is on the safe side.)
bool few_slices_pay(const cngp_config *c, int64_t N, uint32_t slices_f, uint32_t slices_c) {
    const int    D = scan_dense_levels(c, N, slices_f + slices_c), U = c->L - D, M = merge_levels(c, N);
    const double corners = 1 << c->d, refs = 2.0 * corners;
    const double scan = U * (slices_f + 0.5 * slices_c + 2.0 * refs) + 0.8 * D * corners, binned = (c->L - M + 0.45 * M) * refs;
    return M >= 1 && slices_f + slices_c >= kMinMergedSlices && U * (int64_t)(slices_f + slices_c) >= kMinMergedScans && scan >= (c->d == 2 ? kMinMergedGainFlat : kMinMergedGain) * binned;
}

// Sums that `writers` workgroups per slice of a table leave in the workspace on `levels` levels.
size_t partial_bytes(const cngp_config *c, const BwdPlan &b, bool logit, uint32_t writers, int levels, size_t sum_bytes) {
    const size_t slice = ((size_t)c->N_p << (logit ? b.rows_c_log2 : b.rows_f_log2)) * (logit ? 1 : 2) * sum_bytes;
    return writers > 1 ? (size_t)levels * writers * (logit ? b.slices_c : b.slices_f) * slice : 0;
}
size_t partial_bytes(const cngp_config *c, const BwdPlan &b, bool logit) {
    return b.split ? partial_bytes(c, b, logit, (logit ? b.logit_pts : b.feat_pts).chunks, c->L - b.dense.count, sizeof(double)) : 0;
}
// Where a binned batch's drain leaves them, from the start of the merged entries on, which nothing reads any more: roles as in PartialRoles.
struct DrainPartials { uint32_t writers[4]; size_t off[4], bytes; };
DrainPartials drain_partials(const cngp_config *c, const BwdPlan &b) {
    const uint32_t writers[4] = {b.subs_f, b.subs_c, b.feat_vtx.chunks, b.logit_vtx.chunks};
    DrainPartials d;
    d.bytes = 0;
    for (int r = 0; r < 4; ++r) {
        d.writers[r] = (r & 1 ? b.sum_c : b.sum_f) ? writers[r] : 0;
        d.off[r] = d.bytes;
        d.bytes += align256(partial_bytes(c, b, r & 1, d.writers[r], r < 2 ? c->L - b.dense.count : b.dense.count, b.sum_wide ? sizeof(double) : sizeof(float)));
    }
    return d;
}

// Whether merging `levels` levels of a batch from kMinMergeRefs on is worth its launches.
bool merging_pays(const cngp_config *c, int64_t N, int levels) {
    return levels > 0 && ((N << c->d) >= kMinMergedRefs || c->N_p == 1 || (c->L >= kMinMergeLevels && levels >= 2));
}

BwdPlan make_bwd_plan_uncached(const cngp_config *c, int64_t N, Layout layout = LAYOUT_MERGED) {
    BwdPlan b;
    std::memset(&b, 0, sizeof(b));
    const uint32_t groups = c->N_f / c->N_p;                               // hashed rows of D_f
    const uint32_t max_rows_f = (uint32_t)kSliceBytes / (c->N_p * 2 * 8);
    const uint32_t rows_f = groups < max_rows_f ? groups : max_rows_f;
    b.rows_f_log2 = ilog2(rows_f);
    b.slices_f = groups / rows_f;
    if (c->N_p > 1) {
        const uint32_t max_rows_c = (uint32_t)kSliceBytes / (c->N_p * 8);
        const uint32_t rows_c = c->N_c < max_rows_c ? c->N_c : max_rows_c;
        b.rows_c_log2 = ilog2(rows_c);
        b.slices_c = c->N_c / rows_c;
    }
    // A small feature table (the paper's N_f = 2^6 .. 2^12): a level's whole feature gradient (fp64) and a copy of
    // its codebook fit in LDS beside a slice of the confidence table, and one pass over that table's bins gives
    // both gradients.  The confidence slice shrinks until everything fits in kFusedLdsBytes.
    const size_t feat_lds = (size_t)c->N_f * (2 * sizeof(double) + (c->feat_dtype == CNGP_F16 ? 4 : 8));
    bool fused_ok = c->N_p > 1 && c->N_f <= kMaxFusedNf;
    uint32_t fused_rows_c_log2 = b.rows_c_log2;
    while (fused_ok && (((size_t)1 << fused_rows_c_log2) * c->N_p * 8 + feat_lds > kFusedLdsBytes)) {
        if (fused_rows_c_log2 == 0) fused_ok = false;
        else --fused_rows_c_log2;
    }
    if (fused_ok && (c->N_c >> fused_rows_c_log2) > 8192) fused_ok = false;
    const uint32_t per_level = b.slices_f + b.slices_c;
    // a queued reference packs (row inside the slice, row of the other table) into 32 bits
    const bool keys_fit = b.rows_f_log2 + ilog2(c->N_c) <= 32 && b.rows_c_log2 + ilog2(groups) <= 32;
    const bool enough = (N << c->d) * c->L >= kMinSlicedRefs;
    b.sliced = per_level <= kMaxSlicesPerLevel && enough;
    // Binning the references of the hashed levels first (cngp_bwd_binned.h): possible whenever record
    // positions and byte offsets into a level fit 32 bits and a level's bins can be counted in LDS.  It pays
    // from about two dozen slices per level (measured: 24 slices 1.15x, 64 slices 1.6x over the replicated
    // scan; 10 slices 0.75x) and is the only LDS variant for tables of hundreds of slices.
    const bool bin_ok = keys_fit && N > 0 && ((uint64_t)N << c->d) < (1ull << 31) &&
                        b.slices_f <= 8192 && b.slices_c <= 8192 &&
                        (uint64_t)c->N_c * c->N_p <= (1ull << 29) && c->N_f <= (1u << 28);
    // (the bins take 4 bytes per reference, level and table: not chosen unasked beyond kMaxAutoBinBytes)
    const uint64_t bin_bytes = ((uint64_t)N << c->d) * kRecordBytes * (uint64_t)c->L * (c->N_p > 1 ? 2u : 1u);
    const uint64_t bin_bytes_max = c->bin_bytes_max ? c->bin_bytes_max : kMaxAutoBinBytes;
    // (with both gradients in one pass binning pays from four slices per level: below that the replicated scan is as fast)
    const bool plenty = (N << c->d) * c->L >= kMinBinnedRefs;           // below, the three extra launches cost more than they save
    // (these and the tables of a few slices below are scanned in a workspace that holds no bins, and under a bound on them)
    const bool plain = c->N_p == 1 && layout != LAYOUT_LEAST && !c->bin_bytes_max &&
                       per_level >= kMinBinnedPlainSlices && (N << c->d) * (int64_t)per_level >= kMinBinnedPlainScans &&
                       (c->L - scan_dense_levels(c, N, per_level)) * (int64_t)per_level >=
                           (c->d <= 3 && layout == LAYOUT_MERGED && (N << c->d) >= kMinMergeRefs && merge_levels(c, N) >= 4 ? kMinMergedScans : kMinBinnedPlainGroups);
    const bool both = b.slices_f >= kMinBinnedSoonSlices && b.slices_c >= kMinBinnedSoonSlices && per_level >= kMinBinnedSlicesPerLevel;
    const int64_t refs = (N << c->d) * c->L;
    const int64_t per_bin = (N << c->d) / (b.slices_f < b.slices_c ? b.slices_f : b.slices_c ? b.slices_c : 1u);      // references of the longer bins
    const bool few_bins = enough && per_bin > kMostSoonRefsPerBin * c->L;
    const bool soon = layout != LAYOUT_LEAST && !c->bin_bytes_max && !plenty &&
                      ((both && !few_bins && refs >= kMinBinnedSoonRefs) ||
                       (both && !few_bins && c->d == 3 && c->N_p >= kManyCandidates && per_level <= kMostCandidateSlices && refs >= kMinBinnedCandidateRefs) ||
                       (fused_ok && per_level >= 4 && (c->N_c >> fused_rows_c_log2) <= (c->N_p >= kManyCandidates ? kMostCandidateSlices : kMostCandidateSlices / 2) && refs >= kMinBinnedFusedRefs && !enough));
    b.lone = soon && enough && !(c->flags & CNGP_BWD_BINNED);
    b.binned = bin_ok && (plenty || soon) && (per_level >= kMinBinnedSlicesPerLevel || (fused_ok && per_level >= 4) || plain) && bin_bytes <= bin_bytes_max;
    if (c->flags & CNGP_BWD_BINNED) b.binned = bin_ok;
    if (c->flags & (CNGP_BWD_DIRECT | CNGP_BWD_SLICED)) b.binned = false;
    // tables of a few slices, where enough of the levels are merged
    const bool few = !b.binned && bin_ok && plenty && bin_bytes <= bin_bytes_max && layout == LAYOUT_MERGED && c->d <= 3 && c->N_p > 1 &&
            !(c->flags & (CNGP_BWD_DIRECT | CNGP_BWD_SLICED | CNGP_BWD_NO_PREREDUCE)) && !c->bin_bytes_max && (N << c->d) >= kMinMergedRefs &&
            few_slices_pay(c, N, b.slices_f, b.slices_c);
    b.binned = b.binned || few;
    b.scarce = b.binned && per_level < kMinBinnedSlicesPerLevel && !fused_ok;
    b.fused = b.binned && fused_ok;
    if (b.fused) {
        b.rows_c_log2 = fused_rows_c_log2;
        b.slices_c = c->N_c >> fused_rows_c_log2;
    }
    if (b.binned) b.sliced = true;
    if (c->flags & CNGP_BWD_DIRECT) b.sliced = false;
    if ((c->flags & CNGP_BWD_SLICED) && (uint64_t)per_level * 32u * 64u < 0x7fffffffull) b.sliced = true;
    if (!keys_fit) b.sliced = false;
    b.merged = b.binned && layout == LAYOUT_MERGED && !(c->flags & CNGP_BWD_NO_PREREDUCE) && !c->bin_bytes_max &&
               c->d <= 3 && !(b.fused && c->d == 2 && c->N_p == 2) && (N << c->d) >= kMinMergeRefs && (b.fused ? 0 : b.slices_f) + b.slices_c <= kMergeMaxBins;
    if (b.merged) {
        b.dense.count = merge_levels(c, N);
        const uint32_t per_level_now = b.slices_f + b.slices_c;
        // (a small feature table's gradient is added up by every drain workgroup of its level, in fp32: merging must not make
        // them more for the levels that are left, and with as few as before their last round is mostly empty -- N_f = 2^8,
        // N_c = 2^16, N_p = 8, 250007 points: 456 us, merged with two workgroups per bin 436 and an error of 1.5e-7 instead of
        // 1.3e-7, with one 468)
        b.merged = merging_pays(c, N, b.dense.count) && !(b.fused && drain_subs((double)((uint64_t)N << c->d), b.slices_c, c->L - b.dense.count, per_level_now) !=
                                                         drain_subs((double)((uint64_t)N << c->d), b.slices_c, c->L, per_level_now));
        // (plain hashing has one table and the cheapest references: three merged levels do not pay for the order of the points.
        // 32 drawn batches, d = 2 and 3, L = 8 .. 16, N_f = 2^18 .. 2^20, without / with merging: three levels 0.965 .. 0.984 (three
        // batches; d = 3, L = 8, N_max = 8192, 385625 points: 227 us, merged 235), four and more 1.07 .. 2.5)
        if (c->N_p == 1 && b.dense.count < 4) b.merged = false;
        if (!b.merged) b.dense.count = 0;
    }
    // coarse levels whose dense vertex grid is small, much smaller than the number of references, and
    // takes clearly fewer slice scans than the level's hashed tables.  With binning a hashed level costs
    // no replicated scan, and pre-reduction only pays for grids of a few slices.
    if (b.sliced && !b.merged && !(c->flags & CNGP_BWD_NO_PREREDUCE)) {
        uint32_t res[kMaxLevels];
        level_table(c, res);
        for (int l = 0; l < c->L && l < kMaxDense; ++l) {
            uint64_t verts = 1;
            for (int i = 0; i < c->d; ++i) verts *= (uint64_t)res[l] + 2;
            const uint64_t slices = (verts + kDenseSliceVerts - 1) / kDenseSliceVerts;
            if (!pre_reduces(verts, b.binned && layout == LAYOUT_LEAST ? INT64_MAX : N << c->d, per_level)) break;
            if (b.fused) break;      // both gradients from one pass over the bins: cheaper than the grid sums and vertex scans (measured)
            if (b.binned && l == c->L - 1) break;                        // (at least one level stays hashed)
            b.dense.side[l] = res[l] + 2;
            b.dense.verts[l] = (uint32_t)verts;
            b.dense.slices[l] = (uint32_t)slices;
            b.dense.g_off[l] = b.dense_verts;
            b.dense_verts += (uint32_t)verts;
            b.dense_slices += (uint32_t)slices;
            if (verts > b.dense_max_verts) b.dense_max_verts = (uint32_t)verts;
            b.dense.count = l + 1;
        }
        // (a caller who bounds the bins gets the smaller workspace: a pre-reduced level has records once instead of twice)
        if (b.binned && b.dense.count > 0 && (N << c->d) < kMinBinnedPrereduceRefs && !(c->flags & CNGP_BWD_BINNED) &&
            !c->bin_bytes_max && layout <= LAYOUT_FAST &&
            binned_bwd_us(c, N, b, b.dense.count) > 0.96 * binned_bwd_us(c, N, b, 0)) {
            std::memset(&b.dense, 0, sizeof(b.dense));
            b.dense_verts = b.dense_slices = b.dense_max_verts = 0;
        }
    }
    const bool plain_bins = b.scarce && c->N_p == 1 && !b.merged && !(c->flags & CNGP_BWD_BINNED);     // (kMinBinnedPlainGroups)
    const int Lh = c->L - b.dense.count;
    if (b.sliced) choose_geometry(c, N, b, layout == LAYOUT_MERGED && !c->bin_bytes_max);
    if (b.binned) {
        // chunks of at least 1024 points, at most 256 of them
        int64_t cp = ((N + 255) / 256 + 63) / 64 * 64;
        if (cp < 1024) cp = 1024;
        b.bin_chunk_pts = (uint32_t)cp;
        b.bin_chunks = (uint32_t)((N + cp - 1) / cp);
        const double refs = (double)((uint64_t)N << c->d);
        b.subs_f = drain_subs(refs, b.slices_f, b.merged ? c->L : Lh, b.slices_f + b.slices_c, b.scarce, b.scarce && c->N_p == 1);
        b.subs_c = drain_subs(refs, b.slices_c, b.merged ? c->L : Lh, b.slices_f + b.slices_c, b.scarce, b.scarce && c->N_p == 1);
        if (plain_bins) b.subs_f = 1;
        if (b.lone) b.subs_f = b.subs_c = 1;
        if (b.fused) b.subs_f = 2;              // never one writer per entry: the feature gradient is cleared first and added to
        if (b.merged) {
            // half as many drain workgroups per bin: at most about half of a merged level's references are left
            b.feat_vtx = Geom{b.fused ? 2u : (b.subs_f + 1) / 2, 0};
            b.logit_vtx = Geom{(b.subs_c + 1) / 2, 0};
            // Of tables of few slices a bin has up to 64 workgroups, and a scan at most a dozen chunks per slice: a table whose bins have more
            // of them than that leaves their sums, rounded to 32 bits, in the workspace, where they are added up in 64 (as they are where a
            // scan rounds only once).  Error against 64 bits, 2-norm, 1e-7, scanned / added with atomics / so: logit gradient d = 3, L = 10, 8 + 1
            // slices, N_p = 4, 800000 points 1.06 / 1.60 / 0.86, image2d's tables 1.03 / 0.97 / 0.79; 41 drawn tables, either gradient: 0.5 ..
            // 1.0, none above the scan's.  In 64 bits throughout, of both tables: image2d's step 888 us, so 855, as with atomics alone.
            if (b.scarce) {
                const BwdPlan scan = make_bwd_plan_uncached(c, N, LAYOUT_LEAST);
                const auto least = [&](const Geom &pts, const Geom &vtx) { return scan.dense.count > 0 && vtx.chunks < pts.chunks ? vtx.chunks : pts.chunks; };
                const uint32_t least_f = least(scan.feat_pts, scan.feat_vtx), least_c = least(scan.logit_pts, scan.logit_vtx);
                b.sum_f = b.subs_f > scan.feat_pts.chunks || b.feat_vtx.chunks > least_f;
                b.sum_c = b.slices_c && (b.subs_c > scan.logit_pts.chunks || b.logit_vtx.chunks > least_c);
                b.sum_wide = (b.sum_f && least_f == 1) || (b.sum_c && least_c == 1);
            }
            b.merge.levels = (uint32_t)b.dense.count;
            // chunks of at least two rounds, at most 512 of them: sparse parts of space leave several times the entries of
            // dense ones, and the many short workgroups even that out.  With 128 slices of a table or more at most as many as the
            // references' own: beyond, the counts leave the LDS of bin_offsets_kernel, or make its scans through memory longer
            // (N_f = 2^20, N_c = 2^18, N_p = 4, 2^19 points: offsets 100 us with 512 chunks, 31 with 256; merge 112 and 109)
            const int64_t round = kMergeRefs >> c->d, most = (b.fused || b.slices_c > b.slices_f ? b.slices_c : b.slices_f) >= 128 ? 256 : 512;
            int64_t mp = ((N + most - 1) / most + round - 1) / round * round;
            if (mp < 2 * round) mp = 2 * round;
            b.merge.chunk_pts = (uint32_t)mp;
            b.merge.chunks = (uint32_t)((N + mp - 1) / mp);
            // tiles of at least 4096 points, at most 256 of them
            int64_t tp = ((N + 255) / 256 + 1023) / 1024 * 1024;
            if (tp < 4096) tp = 4096;
            b.merge.tile_pts = (uint32_t)tp;
            b.merge.tiles = (uint32_t)((N + tp - 1) / tp);
        }
    }
    const size_t queues = (size_t)kSlicedWaves * kRingBytes;
    b.lds_f = ((size_t)1 << b.rows_f_log2) * c->N_p * 2 * 8 + queues;
    b.lds_c = ((size_t)1 << b.rows_c_log2) * c->N_p * 8 + queues;
    if (b.sliced) {
        const size_t io = c->io_dtype == CNGP_F16 ? 2 : 4;
        b.sigma_off = 0;
        b.dyT_off = align256((size_t)c->L * c->N_c * c->N_p * sizeof(float));
        b.G_off = b.dyT_off + align256((size_t)N * c->L * c->F * io);
        b.G_bytes = (size_t)b.dense_verts * 2 * sizeof(float);
        MergedSpace m;
        if (b.merged) {
            m = merged_space(b, N, c->d);
            const size_t sums = drain_partials(c, b).bytes;
            b.G_bytes = m.G_bytes > sums ? m.G_bytes : sums;
        }
        b.ws_bytes = b.G_off + align256(b.G_bytes);
        if (b.split) {
            b.partF_off = b.ws_bytes;
            b.partC_off = b.partF_off + align256(partial_bytes(c, b, false));
            b.ws_bytes = b.partC_off + align256(partial_bytes(c, b, true));
        }
        if (b.binned) {
            const size_t cap = (size_t)N << c->d;
            // (room for as many chunks as any shorter batch has: 2^18 points are counted in 256, one more in 241)
            const size_t rows = layout == LAYOUT_LEAST ? b.bin_chunks : (size_t)(N >= 256 * 1024 ? 256 : (N + 1023) / 1024);
            b.cntF_off = b.ws_bytes;
            b.cntC_off = b.cntF_off + align256((size_t)Lh * rows * b.slices_f * 4);
            b.baseF_off = b.cntC_off + align256((size_t)Lh * rows * b.slices_c * 4);
            b.baseC_off = b.baseF_off + align256((size_t)Lh * (b.slices_f + 1) * 4);
            b.recF_off = b.baseC_off + align256((size_t)Lh * (b.slices_c + 1) * 4);
            b.recC_off = b.recF_off + (b.fused ? 0 : align256((size_t)Lh * cap * kRecordBytes));
            b.cntG_off = b.recC_off + (b.slices_c ? align256((size_t)Lh * cap * kRecordBytes) : 0);
            const size_t Ld = (size_t)b.dense.count;
            b.baseG_off = b.cntG_off + align256(b.merged ? m.cntG_bytes : Ld * rows * kGridBins * 4);
            b.recG_off = b.baseG_off + align256(b.merged ? m.baseG_bytes : Ld * (kGridBins + 1) * 4);
            b.ws_bytes = b.recG_off + align256(b.merged ? m.recG_bytes : Ld * cap * kRecordBytes);
            b.cntG_bytes = b.merged ? m.cntG_bytes : Ld * b.bin_chunks * kGridBins * 4;
            b.baseG_bytes = b.merged ? m.baseG_bytes : Ld * (kGridBins + 1) * 4;
            b.recG_bytes = b.merged ? m.recG_bytes : Ld * cap * kRecordBytes;
            // (an entry takes 16 bytes and there may be as many as references: not asked for beyond what the bins may take)
            if (b.merged && b.ws_bytes > kMaxAutoBinBytes) return make_bwd_plan_uncached(c, N, LAYOUT_FAST);
            // workgroups per slice of a level's grid: about 2^15 references each
            uint32_t next = 0;
            for (int l = 0; l < b.dense.count && !b.merged; ++l) {
                const uint64_t each = plain_bins ? kPlainGridRecords : 32768;
                uint64_t subs = (cap / b.dense.slices[l] + each - 1) / each;
                if (subs < 1) subs = 1;
                if (subs > 256) subs = 256;
                b.grid_drain.first[l] = next;
                b.grid_drain.subs[l] = (uint32_t)subs;
                next += b.dense.slices[l] * (uint32_t)subs;
            }
            b.grid_drain.first[b.dense.count] = next;
        }
    }
    return b;
}

// The plan depends on (configuration, N) only; the last one of each layout is kept (host memory, per thread).
const BwdPlan &make_bwd_plan(const cngp_config *c, int64_t N, Layout layout = LAYOUT_MERGED) {
    struct Kept { cngp_config cfg; int64_t N = -1; BwdPlan plan; };
    thread_local Kept kept[LAYOUT_COUNT];
    Kept &k = kept[layout];
    if (k.N == N && std::memcmp(&k.cfg, c, sizeof(*c)) == 0) return k.plan;
    k.plan = make_bwd_plan_uncached(c, N, layout);
    k.cfg = *c;
    k.N = N;
    return k.plan;
}

// The plan of a call that has `room` bytes: the first layout that fits.  What the fastest one needs does not only grow with N (a
// level that is not pre-reduced has records in two tables instead of one: nerf3d's tables take 144 MB at 2^17 points, 160 at one
// less), so that a workspace sized for the largest batch of a training run serves the shorter ones too.
const BwdPlan &bwd_plan_for(const cngp_config *c, int64_t N, size_t room) {
    const BwdPlan &b = make_bwd_plan(c, N);
    if (!(b.binned || b.split) || b.ws_bytes <= room) return b;
    if (b.split) return make_bwd_plan(c, N, LAYOUT_LEAST);
    const BwdPlan &fast = make_bwd_plan(c, N, LAYOUT_FAST);
    if (fast.ws_bytes <= room) return fast;
    const BwdPlan &reduced = make_bwd_plan(c, N, LAYOUT_REDUCED);
    return reduced.ws_bytes <= room ? reduced : make_bwd_plan(c, N, LAYOUT_LEAST);
}

// Points per pass of cngp_encode_bwd.  A batch whose bins would pass the configured limit (or whose references
// would not fit the 31-bit record positions) is taken in equal passes, each a complete backward over a run
// of points that accumulates onto the one before, when a pass of that size is binned; otherwise N.
int64_t most_pass_points(const cngp_config *c) {
    int64_t most = (((int64_t)1 << 31) - 1) >> c->d;
    if (!(c->flags & CNGP_BWD_BINNED) || c->bin_bytes_max) {
        const int64_t per_point = ((int64_t)kRecordBytes << c->d) * c->L * (c->N_p > 1 ? 2 : 1);
        const int64_t by_bytes = (int64_t)((c->bin_bytes_max ? c->bin_bytes_max : kMaxAutoBinBytes) / (uint64_t)per_point);
        if (by_bytes < most) most = by_bytes;
    }
    return most >= 65536 ? most / 65536 * 65536 : most / 1024 * 1024;
}
int64_t bwd_pass_points(const cngp_config *c, int64_t N) {
    if (N <= 0 || (c->flags & (CNGP_BWD_DIRECT | CNGP_BWD_SLICED))) return N;
    const int64_t most = most_pass_points(c);
    if (N <= most || most <= 0) return N;
    const int64_t passes = (N + most - 1) / most;
    const int64_t per = ((N + passes - 1) / passes + 63) / 64 * 64;
    return make_bwd_plan_uncached(c, per).binned ? per : N;
}
// Whether passes of `per` points are scanned where the room for their bins is missing.
bool scanned_in_least_room(const cngp_config *c, int64_t per) { return !make_bwd_plan_uncached(c, per, LAYOUT_LEAST).binned; }
// Points per pass in a workspace that does not hold passes of bwd_pass_points: at most half the longest, which the workspace of every
// longer batch in passes holds, as its own passes are no shorter (one more point than fits one pass is taken in two halves); 0 where the
// batch is no longer than that, or not binned.
int64_t short_pass_points(const cngp_config *c, int64_t N) {
    const int64_t half = most_pass_points(c) / 2;
    if (N <= half || half < 64 || (c->flags & (CNGP_BWD_DIRECT | CNGP_BWD_SLICED))) return 0;
    const int64_t passes = (N + half - 1) / half, per = ((N + passes - 1) / passes + 63) / 64 * 64;
    return scanned_in_least_room(c, per) ? 0 : per;
}

template <int NP>
BinParams make_bin_params(const cngp_config *c, const BwdPlan &b, int64_t N) {
    BinParams bp;
    std::memset(&bp, 0, sizeof(bp));
    bp.level0 = b.dense.count;
    bp.nlevels = c->L - b.dense.count;
    bp.rows_f_log2 = b.rows_f_log2; bp.slices_f = b.fused ? 0 : b.slices_f;
    bp.rows_c_log2 = b.rows_c_log2; bp.slices_c = NP > 1 ? b.slices_c : 0;
    bp.chunks = b.bin_chunks; bp.chunk_pts = b.bin_chunk_pts;
    bp.cap = (uint32_t)((uint64_t)N << c->d);
    bp.merged = b.merged ? 1 : 0;
    return bp;
}
// Bins of the level with the most of them, and the copies of the histogram the count keeps in LDS.
uint32_t most_bins_of(const BinParams &bp) { return bp.slices_f + bp.slices_c > kGridBins ? bp.slices_f + bp.slices_c : kGridBins; }
uint32_t hist_replicas_of(uint32_t most_bins) { return most_bins <= 64 ? 16u : most_bins <= 512 ? 4u : 1u; }

// What the workgroups of a slice left, added up; nothing where no role has any.
template <int NP, typename Sum>
int launch_partial_sums(const Params &p, PartialRoles &roles, const float *sigma, bool zero_first, float *gD_f, float *gDhat_c, hipStream_t s) {
    roles.first[0] = 0;
    for (int r = 0; r < 4; ++r) {
        const SliceParams &sp = roles.sp[r];
        roles.first[r + 1] = roles.first[r] + (sp.partial ? (uint32_t)sp.nlevels * sp.slices * ((((uint32_t)NP << sp.rows_log2) + kBlock - 1) / kBlock) : 0u);
    }
    if (roles.first[4] == 0) return CNGP_OK;
    LaunchTimer t(s, K_BWD_PARTIAL);
    bwd_partial_sums_kernel<NP, Sum><<<roles.first[4], kBlock, 0, s>>>(p, roles, sigma, zero_first ? 1 : 0, gD_f, gDhat_c);
    return launch_status("bwd_partial_sums_kernel");
}

// Binned variant: (the count has run with the preparation launch) merge of the merged levels, offsets, scatter (+ vertex-grid accumulation of the dense levels), drain
// (+ the two roles of the dense levels, which scan the finished vertex grids).
template <int D, int NP, typename FeatT, typename IoT>
int launch_bwd_binned(const cngp_config *c, const Params &p, const BwdPlan &b, const float *x, int64_t N,
                      const void *D_f, const float *sigma, const IoT *dy, const IoT *dyT, float *G, float *gD_f, float *gDhat_c,
                      void *workspace, hipStream_t s) {
    const int Ld = b.dense.count, Lh = c->L - Ld;
    char *ws = (char *)workspace;
    uint32_t *cntF = (uint32_t *)(ws + b.cntF_off), *cntC = (uint32_t *)(ws + b.cntC_off);
    uint32_t *baseF = (uint32_t *)(ws + b.baseF_off), *baseC = (uint32_t *)(ws + b.baseC_off);
    BinRecord *recF = (BinRecord *)(ws + b.recF_off), *recC = (BinRecord *)(ws + b.recC_off);
    uint32_t *cntG = (uint32_t *)(ws + b.cntG_off), *baseG = (uint32_t *)(ws + b.baseG_off);
    MergeArrays ma;
    std::memset(&ma, 0, sizeof(ma));
    if (b.merged) ma = merge_arrays(b, N, D, workspace);
    const MergedBins &mb = ma.bins;
    BinRecord *recG = (BinRecord *)(ws + b.recG_off);
    const bool zero_first = (c->flags & CNGP_ZERO_GRADS) != 0;
    const BinParams bp = make_bin_params<NP>(c, b, N);
    const int64_t blocks = (int64_t)(b.merged ? Lh : Lh + Ld) * bp.chunks + (int64_t)mb.levels * mb.chunks;
    if (int rc = check_blocks(blocks)) return rc;
    const size_t lds_bins = (size_t)most_bins_of(bp) * sizeof(uint32_t);
    if constexpr (D <= 3) if (b.merged) {      // the points in the order of their cells (the histogram ran with the preparation), then the entries
        {
            LaunchTimer t(s, K_BWD_CELLS);
            merge_scan_kernel<<<kMergeCells / 64, kMergeScanBlock, 0, s>>>(b.merge, ma.cells, ma.total);
            if (int rc = launch_status("merge_scan_kernel")) return rc;
            merge_order_kernel<D><<<b.merge.tiles, 1024, 0, s>>>(b.merge, x, N, ma.cells, ma.total, ma.order);
            if (int rc = launch_status("merge_order_kernel")) return rc;
        }
        auto kernel = bwd_merge_kernel<D, IoT>;
        if (int rc = allow_big_lds(kernel, kMergeLdsBytes)) return rc;
        LaunchTimer t(s, K_BWD_MERGE);
        kernel<<<(b.merge.chunks + kXcds - 1) / kXcds * kXcds * b.merge.levels, kMergeBlock, kMergeLdsBytes, s>>>(p, bp, b.merge, x, dy, N, ma.order, mb);
        if (int rc = launch_status("bwd_merge_kernel")) return rc;
    }
    // Direct scatter: one wavefront per chunk keeps a bin's records in the order of the points, which the drain's gathers
    // like (measured: drain 7 % faster).  Four wavefronts share the cursors with kMinRunBins bins and more, where the scatter in runs is not taken
    // (a lone one fills its cache lines too slowly for the memory system to merge the 4-byte writes), and where the chunks are few (kFewBinChunks).
    const unsigned bin_block = bp.slices_f + bp.slices_c >= kMinRunBins || blocks <= kFewBinChunks ? 256u : (unsigned)kBinBlock;
    {
        LaunchTimer t(s, K_BWD_BIN_OFFSETS);
        uint32_t big = bp.slices_f > bp.slices_c ? bp.slices_f : bp.slices_c;
        if (Ld > 0 && !b.merged && big < kGridBins) big = kGridBins;
        const uint32_t most = mb.chunks > bp.chunks ? mb.chunks : bp.chunks;
        const uint32_t words = (uint64_t)most * big <= 36864 ? most * big : 0u;    // up to 144 KB of LDS
        if (int rc = allow_big_lds(bin_offsets_kernel, (size_t)words * 4)) return rc;
        bin_offsets_kernel<<<(unsigned)(2 * Lh + (b.merged ? 2 * Ld : Ld)), kOffsetsBlock, (size_t)words * 4, s>>>(
            bp, cntF, cntC, cntG, baseF, baseC, baseG, mb, words);
        if (int rc = launch_status("bin_offsets_kernel")) return rc;
    }
    {
        LaunchTimer t(s, K_BWD_BIN_SCATTER);
        const uint32_t bins = scatter_bins(bp.slices_f, bp.slices_c);
        if (bp.slices_f + bp.slices_c >= kMinRunBins && bins <= kScatMaxBins && bp.slices_f != 1 && bp.slices_c != 1) {
            const int64_t runs = (int64_t)(b.merged ? Lh : Lh + Ld) * bp.chunks + (int64_t)mb.levels * ((mb.chunks + kScatSpan - 1) / kScatSpan);
            if (int rc = allow_big_lds(bin_scatter_runs_kernel<D>, scatter_lds(bins))) return rc;
            bin_scatter_runs_kernel<D><<<(unsigned)runs, kScatBlock, scatter_lds(bins), s>>>(p, bp, b.dense, x, N, cntF, cntC, cntG, recF, recC, recG, mb);
        } else {
            bin_scatter_kernel<D><<<(unsigned)blocks, bin_block, lds_bins, s>>>(p, bp, b.dense, x, N, cntF, cntC, cntG, recF, recC, recG, mb);
        }
        if (int rc = launch_status("bin_scatter_kernel")) return rc;
    }
    if (Ld > 0 && !b.merged) {   // vertex-grid sums of the pre-reduced levels from their bins
        auto kernel = bin_grid_drain_kernel<D, IoT>;
        const size_t lds_grid = (size_t)kDenseSliceVerts * 2 * sizeof(double);
        if (int rc = allow_big_lds(kernel, lds_grid)) return rc;
        LaunchTimer t(s, K_BWD_GRID_DRAIN);
        kernel<<<b.grid_drain.first[Ld], kSlicedBlock, lds_grid, s>>>(p, b.dense, b.grid_drain, x, dyT, N, recG, baseG, bp.cap, G);
        if (int rc = launch_status("bin_grid_drain_kernel")) return rc;
    }
    auto role = [&](uint32_t rows_log2, uint32_t slices, const Geom &g, int level0, int nlevels, uint32_t &wgs) {
        SliceParams sp;
        std::memset(&sp, 0, sizeof(sp));
        sp.rows_log2 = rows_log2;
        sp.slices = slices ? slices : 1;
        sp.chunks = g.chunks ? g.chunks : 1;
        sp.chunk_pts = g.chunk_items;
        sp.store_direct = (sp.chunks == 1 && zero_first) ? 1 : 0;       // matches the clearing in cngp_encode_bwd
        sp.level0 = level0;
        sp.nlevels = slices ? nlevels : 0;
        wgs = (slices && nlevels > 0) ? (uint32_t)kXcds * (((uint32_t)nlevels * sp.slices * sp.chunks + kXcds - 1) / kXcds) : 0u;
        return sp;
    };
    const DrainPartials left = drain_partials(c, b);
    uint32_t wgs_c = 0, wgs_f = 0, wgs_cv = 0, wgs_fv = 0;
    const uint32_t slices_c = NP > 1 ? b.slices_c : 0;
    SliceParams sp_c = role(b.rows_c_log2, slices_c, Geom{b.subs_c, 0}, Ld, Lh, wgs_c);
    SliceParams sp_f = role(b.rows_f_log2, b.fused ? 0u : b.slices_f, Geom{b.subs_f, 0}, Ld, Lh, wgs_f);
    BwdRoles vtx;
    std::memset(&vtx, 0, sizeof(vtx));
    vtx.sp[ROLE_LOGIT_VTX] = role(b.rows_c_log2, slices_c, b.logit_vtx, 0, Ld, wgs_cv);
    vtx.sp[ROLE_FEAT_VTX] = role(b.rows_f_log2, b.merged && b.fused ? 0u : b.slices_f, b.feat_vtx, 0, Ld, wgs_fv);
    vtx.first[ROLE_LOGIT_VTX] = 0;
    vtx.first[ROLE_FEAT_VTX] = wgs_cv;
    PartialRoles sums;
    SliceParams *const drained[4] = {&sp_f, &sp_c, &vtx.sp[ROLE_FEAT_VTX], &vtx.sp[ROLE_LOGIT_VTX]};
    for (int r = 0; r < 4; ++r) {
        if (left.writers[r] > 1) drained[r]->partial = (char *)G + left.off[r];
        drained[r]->wide = b.sum_wide ? 1 : 0;
        sums.sp[r] = *drained[r];
    }
    auto kernel = bin_drain_kernel<D, NP, FeatT, IoT>;
    size_t lds = b.lds_f > b.lds_c ? b.lds_f : b.lds_c;                 // slice + the vertex roles' ring buffers
    if (b.fused) {
        const size_t both = ((size_t)1 << b.rows_c_log2) * NP * 8 + (size_t)c->N_f * (2 * sizeof(double) + sizeof(typename RawPair<FeatT>::type));
        if (both > lds) lds = both;
    }
    if (int rc = allow_big_lds(kernel, lds)) return rc;
    const uint32_t total = wgs_c + wgs_f + wgs_cv + wgs_fv;
    if (total == 0) return CNGP_OK;
    // A corner costs a feature slice 2.2 ns and a logit slice 1.95 (N_p = 16, both roles in flight), the fixed part of a workgroup is alike.  Backward, us,
    // logits / features first: workgroups of features twice as long, 8 + 16 slices, N_p = 16, 20011 points 92 / 76, 60007 198 / 169, 131101 (two per bin) 328 / 315; four or eight times,
    // 4 + 32, N_p = 8, 20011 127 / 107, 60007 202 / 179; half as long or less, 32 + 4, N_p = 4, 90 / 103, 32 + 2, N_p = 8, 60007 131 / 166.  Alike, where it matters
    // little, features first take 0.98 .. 1.05 of the time (4 + 32 with eight per bin and one, 262144 points 468 / 488; 16 + 16, L = 8 272 / 279; 32 + 32, N_p = 8, 500009 903 / 890).
    const bool feat_first = wgs_f > 0 && (wgs_c == 0 || 2.2 * b.slices_c * b.subs_c > 1.95 * b.slices_f * b.subs_f);
    {
        LaunchTimer t(s, K_BWD_BIN_DRAIN);
        kernel<<<total, kSlicedBlock, lds, s>>>(p, sp_c, sp_f, feat_first ? wgs_f : wgs_c, wgs_c + wgs_f, feat_first ? 1 : 0, x, dyT, N, (const FeatT *)D_f, sigma, recF, recC,
                                                baseF, baseC, bp.cap, vtx, b.dense, G, b.merged ? 1 : 0, mb, gD_f, gDhat_c);
        if (int rc = launch_status("bin_drain_kernel")) return rc;
    }
    return b.sum_wide ? launch_partial_sums<NP, double>(p, sums, sigma, zero_first, gD_f, gDhat_c, s)
                      : launch_partial_sums<NP, float>(p, sums, sigma, zero_first, gD_f, gDhat_c, s);
}

template <int D, int NP, typename FeatT, typename IoT>
int launch_bwd_sliced(const cngp_config *c, const Params &p, const BwdPlan &b, const float *x, int64_t N,
                      const void *D_f, const float *Dhat_c, const void *dy, float *gD_f, float *gDhat_c,
                      void *workspace, ZeroList &zero, hipStream_t s) {
    float *sigma = reinterpret_cast<float *>((char *)workspace + b.sigma_off);
    IoT   *dyT = reinterpret_cast<IoT *>((char *)workspace + b.dyT_off);
    // per-vertex sums of weight * dL/dy on the dense levels
    float *G = reinterpret_cast<float *>((char *)workspace + b.G_off);
    const int Ld = b.dense.count, Lh = c->L - Ld;
    bool grid_direct = b.grid.chunks == 1;
    if (b.binned) {
        grid_direct = true;
        for (int l = 0; l < Ld; ++l) grid_direct = grid_direct && b.grid_drain.subs[l] == 1;
    }
    if (Ld > 0 && !b.merged && !grid_direct) zero.add(G, (int64_t)b.dense_verts * 2);
    {   // one launch: clear what is accumulated with atomics, softmax table, level-major dL/dy
        using PairT = typename std::conditional<sizeof(IoT) == 2, uint32_t, float2>::type;
        const int64_t elems = NP > 1 ? (int64_t)c->L * c->N_c * NP : 0;
        const int64_t softmax_blocks = (elems + kBlock - 1) / kBlock;
        const int64_t transpose_blocks = (N + kBlock - 1) / kBlock;
        int64_t zero_blocks = (zero.largest / 4 + kBlock - 1) / kBlock;
        if (zero_blocks > 1024) zero_blocks = 1024;
        if (zero_blocks < 1) zero_blocks = 1;
        const int64_t blocks = (int64_t)zero.n * zero_blocks + softmax_blocks + transpose_blocks;
        if (int rc = check_blocks(blocks)) return rc;
        PrepArgs a;
        a.seg = zero.seg; a.seg_count = (uint32_t)zero.n; a.zero_blocks = (uint32_t)zero_blocks;
        a.Dhat_c = Dhat_c; a.sigma = sigma; a.elems = elems; a.softmax_blocks = (uint32_t)softmax_blocks;
        a.dy = dy; a.dyT = dyT; a.N = N; a.L = c->L; a.level0 = b.merged ? Ld : 0; a.top_k = p.top_k;
        LaunchTimer t(s, K_BWD_PREP);
        if (b.binned) {          // the count of the binned variant rides along: it needs nothing this launch writes
            const BinParams bp = make_bin_params<NP>(c, b, N);
            const int64_t   count_blocks = (int64_t)(b.merged ? Lh : c->L) * bp.chunks;
            if (int rc = check_blocks(blocks + count_blocks + b.merge.tiles)) return rc;
            const uint32_t most = most_bins_of(bp), reps = hist_replicas_of(most);
            char *ws = (char *)workspace;
            size_t lds = (size_t)most * reps * sizeof(uint32_t);
            if (b.merged && lds < kMergeCells * sizeof(uint32_t)) lds = kMergeCells * sizeof(uint32_t);
            uint32_t *cells = b.merged ? merge_arrays(b, N, D, workspace).cells : nullptr;
            bwd_prep_count_kernel<D, NP, PairT><<<(unsigned)(blocks + count_blocks + b.merge.tiles), kBlock, lds, s>>>(
                a, p, bp, b.dense, x, (uint32_t *)(ws + b.cntF_off), (uint32_t *)(ws + b.cntC_off), (uint32_t *)(ws + b.cntG_off),
                reps, (uint32_t)count_blocks, b.merge, cells);
        } else {
            bwd_prep_kernel<NP, PairT><<<(unsigned)blocks, kBlock, 0, s>>>(a);
        }
        zero.n = 0;
        zero.largest = 0;
        if (int rc = launch_status("bwd_prep_kernel")) return rc;
    }

    if (b.binned)
        return launch_bwd_binned<D, NP, FeatT, IoT>(c, p, b, x, N, D_f, sigma, (const IoT *)dy, dyT, G, gD_f, gDhat_c, workspace, s);

    // Launch 1: feature and logit gradients of the hashed levels (scan the points) together with the
    // vertex-grid accumulation of the dense levels.  Launch 2: the two gradients of the dense levels
    // (scan the vertex grids, which launch 1 has completed).
    const bool zero_first = (c->flags & CNGP_ZERO_GRADS) != 0;
    auto kernel = bwd_sliced_kernel<D, NP, FeatT, IoT>;
    size_t lds = b.lds_f > b.lds_c ? b.lds_f : b.lds_c;
    const size_t lds_grid = (size_t)kDenseSliceVerts * 2 * sizeof(double);
    if (Ld > 0 && lds_grid > lds) lds = lds_grid;
    if (int rc = allow_big_lds(kernel, lds)) return rc;
    PartialRoles sums;                         // what the chunks of the point roles leave
    std::memset(&sums, 0, sizeof(sums));
    for (int launch = 0; launch < 2; ++launch) {
        BwdRoles roles;
        std::memset(&roles, 0, sizeof(roles));
        uint32_t next = 0;
        auto add_role = [&](int role, bool present, const Geom &g, uint32_t rows_log2, uint32_t slices, int level0,
                            int nlevels) {
            SliceParams &sp = roles.sp[role];
            sp.rows_log2 = rows_log2;
            sp.slices = slices ? slices : 1;
            sp.chunks = g.chunks ? g.chunks : 1;
            sp.chunk_pts = g.chunk_items;
            sp.store_direct = (g.chunks == 1 && zero_first) ? 1 : 0;     // matches the clearing in cngp_encode_bwd
            sp.level0 = level0;
            sp.nlevels = present ? nlevels : 0;
            if (b.split && g.chunks > 1 && role == ROLE_LOGIT_PTS) sp.partial = (char *)workspace + b.partC_off;
            if (b.split && g.chunks > 1 && role == ROLE_FEAT_PTS) sp.partial = (char *)workspace + b.partF_off;
            roles.first[role] = next;
            if (present && nlevels > 0)      // 8 equal runs of (level, slice, chunk) units, one per XCD
                next += (uint32_t)kXcds * (((uint32_t)nlevels * sp.slices * sp.chunks + kXcds - 1) / kXcds);
        };
        const bool pts = launch == 0, vtx = launch == 1;
        add_role(ROLE_LOGIT_PTS, pts && NP > 1, b.logit_pts, b.rows_c_log2, b.slices_c, Ld, Lh);
        add_role(ROLE_FEAT_PTS, pts, b.feat_pts, b.rows_f_log2, b.slices_f, Ld, Lh);
        add_role(ROLE_LOGIT_VTX, vtx && NP > 1, b.logit_vtx, b.rows_c_log2, b.slices_c, 0, Ld);
        add_role(ROLE_FEAT_VTX, vtx, b.feat_vtx, b.rows_f_log2, b.slices_f, 0, Ld);
        roles.first[ROLE_GRID] = next;
        roles.sp[ROLE_GRID].chunks = b.grid.chunks ? b.grid.chunks : 1;
        roles.sp[ROLE_GRID].chunk_pts = b.grid.chunk_items;
        roles.sp[ROLE_GRID].store_direct = grid_direct;
        if (pts && Ld > 0) next += b.dense_slices * roles.sp[ROLE_GRID].chunks;
        roles.first[ROLE_COUNT] = next;
        if (next == 0) continue;
        LaunchTimer t(s, pts ? K_BWD_SLICED : K_BWD_SLICED_V);
        kernel<<<next, kSlicedBlock, lds, s>>>(p, roles, b.dense, x, (const FeatT *)D_f, sigma, dyT, G, gD_f, gDhat_c, N);
        if (int rc = launch_status("bwd_sliced_kernel")) return rc;
        if (pts) { sums.sp[0] = roles.sp[ROLE_FEAT_PTS]; sums.sp[1] = roles.sp[ROLE_LOGIT_PTS]; }
    }
    return launch_partial_sums<NP, double>(p, sums, sigma, zero_first, gD_f, gDhat_c, s);
}

// LDS of encode_bwd_small_kernel, 0 where it is not taken.
size_t small_bwd_lds(const cngp_config *c) {
    const size_t lds = ((size_t)c->N_f * 2 + (c->N_p > 1 ? (size_t)c->N_c * c->N_p : 0)) * sizeof(double);
    return lds <= kSmallBwdLds && !(c->flags & CNGP_BWD_DIRECT) ? lds : 0;
}

template <int D, int NP, typename FeatT, typename IoT>
int launch_bwd_small(const cngp_config *c, const Params &p, const float *x, int64_t N, const void *D_f, const float *Dhat_c,
                     const void *dy, float *gD_f, float *gDhat_c, hipStream_t s) {
    constexpr int64_t PTS = kSmallBwdBlock / NP, WAVE = 64 / NP;
    // One point per lane group while the chip has room for that many workgroups.  A batch that fills only a few of them is cut
    // finer, into whole wavefronts: all the corners of a point follow each other in its lanes, so 16 wavefronts on one CU
    // take their time in turn (kernel alone, us, direct / uncut / cut: d = 4, 12 levels, N_p = 16, 100 points 17 / 22 / 13;
    // d = 3, L = 2, N_p = 16, 315 points 10.8 / 13.2 / 10.0; d = 3, L = 1, N_p = 2, 513 points 10.9 / 13.3 / 8.5).  Fewer pieces
    // where a lane group is short and holds more of the batch: every piece adds what it touched to memory (N_p = 1, 128 KB of
    // tables, 4095 points on 16 levels: a call 11.7 in 4 pieces, 14.4 in 16; N_p = 2, 65 KB 14.8 in 8, 16.6 in 16).
    constexpr int64_t kLeastChunks = NP >= 4 ? 16 : NP == 2 ? 8 : 4;
    int64_t chunks = (N + PTS - 1) / PTS, unit = PTS;
    if (chunks < kLeastChunks) { chunks = kLeastChunks; unit = WAVE; }
    if (chunks > kCus / c->L) chunks = kCus / c->L;
    if (chunks < 1) chunks = 1;
    const int64_t chunk = ((N + chunks - 1) / chunks + unit - 1) / unit * unit;
    chunks = (N + chunk - 1) / chunk;
    auto kernel = encode_bwd_small_kernel<D, NP, FeatT, IoT>;
    const size_t lds = small_bwd_lds(c);
    if (int rc = allow_big_lds(kernel, lds)) return rc;
    LaunchTimer t(s, K_BWD_SMALL);
    kernel<<<dim3((unsigned)chunks, (unsigned)c->L), kSmallBwdBlock, lds, s>>>(p, x, (const FeatT *)D_f, Dhat_c, (const IoT *)dy,
                                                                              gD_f, gDhat_c, N, chunk);
    return launch_status("encode_bwd_small_kernel");
}

template <int D, typename FeatT, typename IoT>
int dispatch_bwd_np(const cngp_config *c, const Params &p, const BwdPlan &b, const float *x, int64_t N,
                    const void *D_f, const float *Dhat_c, const void *dy, float *gD_f, float *gDhat_c,
                    void *workspace, ZeroList &zero, hipStream_t s) {
#define CNGP_BWD_CASE(NP)                                                                                        \
    if (b.sliced) return launch_bwd_sliced<D, NP, FeatT, IoT>(c, p, b, x, N, D_f, Dhat_c, dy, gD_f, gDhat_c, workspace, zero, s); \
    if (int rc = zero.launch(s)) return rc;                                                                         \
    if (small_bwd_lds(c)) return launch_bwd_small<D, NP, FeatT, IoT>(c, p, x, N, D_f, Dhat_c, dy, gD_f, gDhat_c, s); \
    return launch_bwd_direct<D, NP, FeatT, IoT>(c, p, 0, c->L, x, N, D_f, Dhat_c, dy, gD_f, gDhat_c, s)
    switch (c->N_p) {
    case 1:  CNGP_BWD_CASE(1);
    case 2:  CNGP_BWD_CASE(2);
    case 4:  CNGP_BWD_CASE(4);
    case 8:  CNGP_BWD_CASE(8);
    default: CNGP_BWD_CASE(16);
    }
#undef CNGP_BWD_CASE
}

// d x feat_dtype x io_dtype -> template instance
#define CNGP_DISPATCH_TYPES(FN, ...)                                                             \
    do {                                                                                         \
        const bool f16 = cfg->feat_dtype == CNGP_F16, io16 = cfg->io_dtype == CNGP_F16;          \
        if (cfg->d == 2) {                                                                       \
            if (f16) return io16 ? FN<2, __half, __half>(__VA_ARGS__) : FN<2, __half, float>(__VA_ARGS__); \
            return io16 ? FN<2, float, __half>(__VA_ARGS__) : FN<2, float, float>(__VA_ARGS__);  \
        }                                                                                        \
        if (cfg->d == 3) {                                                                       \
            if (f16) return io16 ? FN<3, __half, __half>(__VA_ARGS__) : FN<3, __half, float>(__VA_ARGS__); \
            return io16 ? FN<3, float, __half>(__VA_ARGS__) : FN<3, float, float>(__VA_ARGS__);  \
        }                                                                                        \
        if (f16) return io16 ? FN<4, __half, __half>(__VA_ARGS__) : FN<4, __half, float>(__VA_ARGS__);     \
        return io16 ? FN<4, float, __half>(__VA_ARGS__) : FN<4, float, float>(__VA_ARGS__);      \
    } while (0)

}  // namespace

// ==================================================================== exported C ABI
namespace {
template <int D, typename FeatT, typename IoT>
int launch_fused_fwd(const cngp_config *c, const Params &p, const MlpDims &d, const float *x, int64_t N, const void *D_f,
                     const void *D_c, const void *W, float *out, hipStream_t s) {
    const size_t c_stride = index_level_bytes(c);
    size_t rest = (((size_t)c->N_c + 1) / 2 + 15) & ~(size_t)15;
    if (rest < kMlpRawBytes) rest = kMlpRawBytes;
    const size_t lds = kMlpFwdOps + (size_t)kFusedTile * kFusedStride * sizeof(_Float16) + rest;
    if (lds > 128 * 1024) return CNGP_ERR_UNSUPPORTED;
    const int64_t tiles = (N + kFusedTile - 1) / kFusedTile;
    int64_t per_cu = (int64_t)(160 * 1024 / lds);            // workgroups that fit a CU at once: LDS, and three
    if (per_cu > 3) per_cu = 3;                              // wavefronts per SIMD by registers
    if (per_cu < 1) per_cu = 1;
    const int64_t blocks = tiles < 256 * per_cu ? tiles : 256 * per_cu;
    const int vec = (c_stride % 16 == 0 && ((uintptr_t)D_c & 15u) == 0) ? 1 : 0;
#define CNGP_FUSED(FMT)                                                                                   \
    do {                                                                                                  \
        auto kernel = encode_mlp_fwd_kernel<D, FeatT, FMT>;                                               \
        if (int rc = allow_big_lds(kernel, lds)) return rc;                                               \
        LaunchTimer t(s, K_FUSED_FWD);                                                                    \
        kernel<<<(unsigned)blocks, kFusedTile, lds, s>>>(p, d, x, (const FeatT *)D_f, (const uint8_t *)D_c, \
                                                         (const __half *)W, out, N, tiles, (uint32_t)c_stride, vec); \
    } while (0)
    if (c->index_format == CNGP_IDX_PACKED4) CNGP_FUSED(kFmtPacked4);
    else if (c->index_format == CNGP_IDX_BITS) CNGP_FUSED(kFmtBits);
    else CNGP_FUSED(kFmtU8);
#undef CNGP_FUSED
    return launch_status("encode_mlp_fwd_kernel");
}
}  // namespace

namespace {
// Workspace of the entry points for entries of two features (every kernel's native width).
size_t workspace_bytes_passes(const cngp_config *cfg, int64_t N, int64_t per, Layout layout) {
    const size_t most = make_bwd_plan_uncached(cfg, per, layout).ws_bytes;   // the last pass is the shorter one
    const size_t last = make_bwd_plan_uncached(cfg, N - (N - 1) / per * per, layout).ws_bytes;
    return most > last ? most : last;
}
size_t workspace_bytes_pairs(const cngp_config *cfg, int64_t N) {
    const int64_t per = bwd_pass_points(cfg, N);
    return per >= N ? make_bwd_plan(cfg, N).ws_bytes : workspace_bytes_passes(cfg, N, per, LAYOUT_MERGED);
}
// The smallest workspace with which cngp_encode_bwd runs (in passes: without merging, which may take three times as much and is
// left out by bwd_plan_for where it does not fit; tables that are scanned without room for the bins: without those).
size_t least_workspace_pairs(const cngp_config *cfg, int64_t N) {
    const size_t  bytes = workspace_bytes_pairs(cfg, N);
    const int64_t per = bwd_pass_points(cfg, N);
    const size_t  least = per < N ? workspace_bytes_passes(cfg, N, per, scanned_in_least_room(cfg, per) ? LAYOUT_LEAST : LAYOUT_FAST)
                                  : make_bwd_plan(cfg, N, LAYOUT_LEAST).ws_bytes;
    return least < bytes ? least : bytes;
}

// What passes of short_pass_points take at least; 0 where the batch is not taken in those.
size_t short_passes_workspace_pairs(const cngp_config *cfg, int64_t N) {
    const int64_t per = short_pass_points(cfg, N);
    return per > 0 ? workspace_bytes_passes(cfg, N, per, LAYOUT_LEAST) : 0;
}

// ---------------------------------------------------------------- feature widths other than two
// F = 1, 4, 8 run as ceil(F / 2) passes over pair planes (cngp_kernels.h, plane_take_kernel): behind the workspace
// of the two-feature problem sit one plane of D_f, one plane of y or dL/dy, and one plane of grad D_f.
struct PlaneSpace { size_t pairs, D_off, io_off, g_off, total; };
cngp_config as_pairs(const cngp_config *c) { cngp_config p = *c; p.F = 2; return p; }
PlaneSpace plane_space(const cngp_config *c, int64_t N, bool least = false, size_t short_passes = 0) {
    const cngp_config c2 = as_pairs(c);
    PlaneSpace ps;
    const size_t bwd = short_passes ? short_passes : least ? least_workspace_pairs(&c2, N) : workspace_bytes_pairs(&c2, N), fwd = fwd_level_plan(&c2, c2.L, N).yT_bytes;
    ps.pairs = align256(bwd > fwd ? bwd : fwd);
    ps.D_off = ps.pairs;
    ps.io_off = ps.D_off + align256((size_t)c->L * c->N_f * 2 * (c->feat_dtype == CNGP_F16 ? 2 : 4));
    ps.g_off = ps.io_off + align256((size_t)N * c->L * 2 * (c->io_dtype == CNGP_F16 ? 2 : 4));
    ps.total = ps.g_off + align256((size_t)c->L * c->N_f * 2 * sizeof(float));
    return ps;
}

template <typename T>
int take_plane(const void *src, void *dst, int64_t rows, int F, int plane, hipStream_t s) {
    if (rows <= 0) return CNGP_OK;
    const int64_t blocks = (rows + kBlock - 1) / kBlock;
    if (int rc = check_blocks(blocks)) return rc;
    LaunchTimer t(s, K_PLANES);
    plane_take_kernel<T><<<(unsigned)blocks, kBlock, 0, s>>>((const T *)src, (T *)dst, rows, F, plane);
    return launch_status("plane_take_kernel");
}
template <typename T>
int put_plane(const void *src, void *dst, int64_t rows, int F, int plane, bool accumulate, hipStream_t s) {
    if (rows <= 0) return CNGP_OK;
    const int64_t blocks = (rows + kBlock - 1) / kBlock;
    if (int rc = check_blocks(blocks)) return rc;
    LaunchTimer t(s, K_PLANES);
    plane_put_kernel<T><<<(unsigned)blocks, kBlock, 0, s>>>((const T *)src, (T *)dst, rows, F, plane, accumulate ? 1 : 0);
    return launch_status("plane_put_kernel");
}
int take_plane_dt(int dtype, const void *src, void *dst, int64_t rows, int F, int plane, hipStream_t s) {
    return dtype == CNGP_F16 ? take_plane<__half>(src, dst, rows, F, plane, s) : take_plane<float>(src, dst, rows, F, plane, s);
}
int put_plane_dt(int dtype, const void *src, void *dst, int64_t rows, int F, int plane, bool acc, hipStream_t s) {
    return dtype == CNGP_F16 ? put_plane<__half>(src, dst, rows, F, plane, acc, s) : put_plane<float>(src, dst, rows, F, plane, acc, s);
}
PlaneSpace plane_space_for(const cngp_config *c, int64_t N, size_t room) {
    const PlaneSpace ps = plane_space(c, N);
    if (ps.total <= room) return ps;
    const PlaneSpace least = plane_space(c, N, true);
    const cngp_config c2 = as_pairs(c);
    const size_t passes = least.total <= room ? 0 : short_passes_workspace_pairs(&c2, N);
    return passes ? plane_space(c, N, true, passes) : least;
}
bool plane_workspace_ok(const void *ws, size_t bytes, const PlaneSpace &ps) {
    return ws && ((uintptr_t)ws & 255u) == 0 && bytes >= ps.total;
}

int fwd_planes(const cngp_config *cfg, int32_t levels_loaded, const float *x, int64_t N, const void *D_f, const void *D_c,
               void *y, void *workspace, size_t workspace_bytes, void *stream) {
    const PlaneSpace ps = plane_space_for(cfg, N, workspace_bytes);
    if (!plane_workspace_ok(workspace, workspace_bytes, ps)) return CNGP_ERR_WORKSPACE;
    const cngp_config c2 = as_pairs(cfg);
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    for (int p = 0; p < (cfg->F + 1) / 2; ++p) {
        if (int rc = take_plane_dt(cfg->feat_dtype, D_f, ws + ps.D_off, (int64_t)levels_loaded * cfg->N_f, cfg->F, p, s)) return rc;
        if (int rc = cngp_encode_fwd_partial(&c2, levels_loaded, x, N, ws + ps.D_off, D_c, ws + ps.io_off, workspace, ps.pairs, stream)) return rc;
        if (int rc = put_plane_dt(cfg->io_dtype, ws + ps.io_off, y, N * cfg->L, cfg->F, p, false, s)) return rc;
    }
    return CNGP_OK;
}

int bwd_planes(const cngp_config *cfg, const float *x, int64_t N, const void *D_f, const float *Dhat_c, const void *dy,
               float *grad_D_f, float *grad_Dhat_c, void *workspace, size_t workspace_bytes, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    const bool zero_first = (cfg->flags & CNGP_ZERO_GRADS) != 0;
    if (N == 0) {                                   // nothing to add; clear if asked
        ZeroList z;
        if (zero_first) { z.add(grad_D_f, (int64_t)cfg->L * cfg->N_f * cfg->F); z.add(grad_Dhat_c, (int64_t)cfg->L * cfg->N_c * cfg->N_p); }
        return z.launch(s);
    }
    const PlaneSpace ps = plane_space_for(cfg, N, workspace_bytes);
    if (!plane_workspace_ok(workspace, workspace_bytes, ps)) return CNGP_ERR_WORKSPACE;
    cngp_config c2 = as_pairs(cfg);
    c2.flags &= ~(uint32_t)CNGP_ZERO_GRADS;         // the plane of grad D_f is cleared here, grad D^_c once if asked
    char  *ws = (char *)workspace;
    float *gp = (float *)(ws + ps.g_off);
    for (int p = 0; p < (cfg->F + 1) / 2; ++p) {
        ZeroList z;
        z.add(gp, (int64_t)cfg->L * cfg->N_f * 2);
        if (p == 0 && zero_first) z.add(grad_Dhat_c, (int64_t)cfg->L * cfg->N_c * cfg->N_p);
        if (int rc = z.launch(s)) return rc;
        if (int rc = take_plane_dt(cfg->feat_dtype, D_f, ws + ps.D_off, (int64_t)cfg->L * cfg->N_f, cfg->F, p, s)) return rc;
        if (int rc = take_plane_dt(cfg->io_dtype, dy, ws + ps.io_off, N * cfg->L, cfg->F, p, s)) return rc;
        if (int rc = cngp_encode_bwd(&c2, x, N, ws + ps.D_off, Dhat_c, ws + ps.io_off, gp, grad_Dhat_c, workspace, ps.pairs, stream)) return rc;
        if (int rc = put_plane<float>(gp, grad_D_f, (int64_t)cfg->L * cfg->N_f, cfg->F, p, !zero_first, s)) return rc;
    }
    return CNGP_OK;
}

int adam_coefficients(const cngp_adam *o, AdamCoef *a) {
    if (!(o->lr >= 0.0f) || !std::isfinite(o->lr)) return CNGP_ERR_INVALID;
    if (!(o->beta1 >= 0.0f && o->beta1 < 1.0f) || !(o->beta2 >= 0.0f && o->beta2 < 1.0f)) return CNGP_ERR_INVALID;
    if (!(o->eps > 0.0f) || !std::isfinite(o->eps) || !std::isfinite(o->grad_scale) || o->step < 1) return CNGP_ERR_INVALID;
    const double c1 = 1.0 - std::pow((double)o->beta1, (double)o->step);
    const double c2 = 1.0 - std::pow((double)o->beta2, (double)o->step);
    a->b1 = o->beta1;  a->one_minus_b1 = (float)(1.0 - (double)o->beta1);
    a->b2 = o->beta2;  a->one_minus_b2 = (float)(1.0 - (double)o->beta2);
    a->step = (float)((double)o->lr / c1);
    a->rsqrt_c2 = (float)(1.0 / std::sqrt(c2));
    a->eps = o->eps;
    a->grad_scale = o->grad_scale;
    return CNGP_OK;
}
bool aligned(const void *p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) == 0; }
}  // namespace

extern "C" {

int cngp_version(void) { return 100; }

const char *cngp_error_string(int status) {
    switch (status) {
    case CNGP_OK:              return "success";
    case CNGP_ERR_NULL:        return "a required pointer is NULL";
    case CNGP_ERR_INVALID:     return "invalid argument (size out of range or not a power of two)";
    case CNGP_ERR_UNSUPPORTED: return "valid in the paper's terms, not supported by this entry point (F other than 1, 2, 4, 8; F != 2 where no workspace can hold the pair planes)";
    case CNGP_ERR_WORKSPACE:   return "workspace missing, misaligned or too small";
    case CNGP_ERR_HIP:         return "a HIP call failed (see cngp_last_hip_error)";
    default:                   return "unknown status";
    }
}

const char *cngp_last_hip_error(void) { return g_hip_error.c_str(); }

int cngp_level_resolutions(const cngp_config *cfg, uint32_t *out_N_l) {
    if (!cfg || !out_N_l) return CNGP_ERR_NULL;
    int rc = validate(cfg);
    if (rc != CNGP_OK && rc != CNGP_ERR_UNSUPPORTED) return rc;
    level_table(cfg, out_N_l);
    return CNGP_OK;
}

size_t cngp_workspace_bytes(const cngp_config *cfg, int64_t N) {
    if (validate(cfg) != CNGP_OK || N <= 0) return 0;
    if (cfg->F != 2) return plane_space(cfg, N).total;
    const size_t bwd = workspace_bytes_pairs(cfg, N), fwd = fwd_level_plan(cfg, cfg->L, N).yT_bytes;
    return bwd > fwd ? bwd : fwd;
}

int cngp_fwd_plan_info(const cngp_config *cfg, int64_t N, int32_t *info) {
    if (!info) return CNGP_ERR_NULL;
    if (int rc = validate(cfg)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    const cngp_config pairs = as_pairs(cfg);
    const FwdLevelPlan f = fwd_level_plan(&pairs, cfg->L, N);
    info[0] = f.use ? 1 : 0;
    info[1] = (int32_t)f.resident;
    info[2] = (int32_t)(f.group.levels ? f.group.parts : f.split.hash_parts);
    info[3] = (int32_t)(f.group.levels ? (size_t)f.group.levels * f.group.stride : f.lds);
    return CNGP_OK;
}

int cngp_fwd_group_levels(const cngp_config *cfg, int64_t N) {
    if (int rc = validate(cfg)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    const cngp_config pairs = as_pairs(cfg);
    return (int)fwd_level_plan(&pairs, cfg->L, N).group.levels;
}

int cngp_fwd_route(const cngp_config *cfg, int32_t levels_loaded, int64_t N, size_t workspace_bytes, int32_t *grids) {
    if (int rc = validate(cfg)) return rc;
    if (N < 0 || levels_loaded < 0 || levels_loaded > cfg->L) return CNGP_ERR_INVALID;
    cngp_config pairs = as_pairs(cfg);
    if (cfg->F != 2) {                                       // passes over pairs of features, in their part of the workspace
        const PlaneSpace ps = plane_space_for(cfg, N, workspace_bytes);
        if (workspace_bytes < ps.total) return CNGP_ERR_WORKSPACE;
        workspace_bytes = ps.pairs;
    }
    FwdLevelPlan f;
    const int route = fwd_route(&pairs, levels_loaded, N, workspace_bytes, &f);
    if (grids) *grids = route == CNGP_FWD_ROUTE_LEVEL ? (int32_t)f.split.dense : 0;
    return route;
}

size_t cngp_fwd_workspace_bytes(const cngp_config *cfg, int64_t N) {
    if (validate(cfg) != CNGP_OK || N <= 0) return 0;
    if (cfg->F != 2) return plane_space(cfg, N).total;
    return fwd_level_plan(cfg, cfg->L, N).yT_bytes;
}

int cngp_bwd_plan_info(const cngp_config *cfg, int64_t N, int32_t *info) {
    if (!info) return CNGP_ERR_NULL;
    if (int rc = validate(cfg)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    const cngp_config pairs = as_pairs(cfg);                // other widths run as passes over pairs of features
    cfg = &pairs;
    const int64_t per = bwd_pass_points(cfg, N);
    const BwdPlan b = make_bwd_plan(cfg, per < N ? per : N);
    const int32_t v[CNGP_PLAN_INFO_COUNT] = {
        b.sliced ? 1 : 0, b.merged ? 0 : b.dense.count, (int32_t)(b.fused ? 0 : b.slices_f), (int32_t)b.slices_c,
        (int32_t)b.feat_pts.chunks, (int32_t)b.logit_pts.chunks, b.merged ? 1 : (int32_t)b.feat_vtx.chunks,
        b.merged ? 1 : (int32_t)b.logit_vtx.chunks, b.merged ? 0 : (int32_t)b.grid.chunks, (int32_t)b.dense_slices,
        b.binned ? 1 : 0, (int32_t)b.subs_f, (int32_t)b.subs_c, (int32_t)b.bin_chunks,
        (int32_t)(N > 0 ? (N + per - 1) / per : 1)};
    for (int i = 0; i < CNGP_PLAN_INFO_COUNT; ++i) info[i] = v[i];
    return CNGP_OK;
}

int cngp_bwd_merge_info(const cngp_config *cfg, int64_t N, int32_t *info) {
    if (!info) return CNGP_ERR_NULL;
    if (int rc = validate(cfg)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    const cngp_config pairs = as_pairs(cfg);
    cfg = &pairs;
    const int64_t per = bwd_pass_points(cfg, N);
    const BwdPlan b = make_bwd_plan(cfg, per < N ? per : N);
    const int32_t v[CNGP_MERGE_INFO_COUNT] = {b.dense.count, (int32_t)b.merge.chunks, (int32_t)b.merge.chunk_pts, (int32_t)b.merge.tiles,
                                              (int32_t)b.feat_vtx.chunks, (int32_t)b.logit_vtx.chunks};
    for (int i = 0; i < CNGP_MERGE_INFO_COUNT; ++i) info[i] = b.merged ? v[i] : 0;
    return CNGP_OK;
}

int cngp_bwd_plan_layout(const cngp_config *cfg, int64_t N, uint64_t *regions) {
    if (!regions) return CNGP_ERR_NULL;
    if (int rc = validate(cfg)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    const cngp_config pairs = as_pairs(cfg);
    cfg = &pairs;
    const int64_t per = bwd_pass_points(cfg, N);
    const int64_t n = per < N ? per : N;
    const BwdPlan b = make_bwd_plan(cfg, n);
    if (!b.sliced || n == 0) return 0;
    // what the kernels index, region by region (not the differences of the offsets: those would prove nothing)
    const uint64_t io = cfg->io_dtype == CNGP_F16 ? 2 : 4;
    const uint64_t Ld = (uint64_t)b.dense.count, Lh = (uint64_t)cfg->L - Ld, cap = (uint64_t)n << cfg->d;
    int k = 0;
    auto add = [&](size_t off, uint64_t bytes) { regions[2 * k] = off; regions[2 * k + 1] = bytes; ++k; };
    add(b.sigma_off, (uint64_t)cfg->L * cfg->N_c * cfg->N_p * 4);
    add(b.dyT_off, (uint64_t)n * cfg->L * cfg->F * io);
    add(b.G_off, b.G_bytes);
    if (b.split) {
        add(b.partF_off, partial_bytes(cfg, b, false));
        add(b.partC_off, partial_bytes(cfg, b, true));
    }
    if (b.binned) {
        const uint64_t sf = b.fused ? 0 : b.slices_f, sc = cfg->N_p > 1 ? b.slices_c : 0;
        add(b.cntF_off, Lh * b.bin_chunks * sf * 4);
        add(b.cntC_off, Lh * b.bin_chunks * sc * 4);
        add(b.baseF_off, sf ? Lh * (sf + 1) * 4 : 0);
        add(b.baseC_off, sc ? Lh * (sc + 1) * 4 : 0);
        add(b.recF_off, sf ? Lh * cap * kRecordBytes : 0);
        add(b.recC_off, sc ? Lh * cap * kRecordBytes : 0);
        add(b.cntG_off, b.cntG_bytes);
        add(b.baseG_off, b.baseG_bytes);
        add(b.recG_off, b.recG_bytes);
    }
    return k;
}

int cngp_bwd_merge_layout(const cngp_config *cfg, int64_t N, uint64_t *regions) {
    if (!regions) return CNGP_ERR_NULL;
    if (int rc = validate(cfg)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    const cngp_config pairs = as_pairs(cfg);
    cfg = &pairs;
    const int64_t per = bwd_pass_points(cfg, N);
    const int64_t n = per < N ? per : N;
    const BwdPlan b = make_bwd_plan(cfg, n);
    if (!b.merged) return 0;
    // the pointers a launch is given, as if the workspace began at an address of that alignment, and what the kernels index from them
    char *const       ws = (char *)(uintptr_t)(1u << 20);
    const MergeArrays a = merge_arrays(b, n, cfg->d, ws);
    const uint64_t    M = a.bins.levels, chunks = a.bins.chunks, cap = (uint64_t)n << cfg->d, sf = b.fused ? 0 : b.slices_f, sc = cfg->N_p > 1 ? b.slices_c : 0;
    int k = 0;
    auto add = [&](const void *p, uint64_t bytes) { regions[2 * k] = (uint64_t)((const char *)p - ws); regions[2 * k + 1] = bytes; ++k; };
    add(a.bins.entries, M * cap * sizeof(uint4));
    add(a.order, (uint64_t)n * 4);
    add(a.cells, (uint64_t)b.merge.tiles * kMergeCells * 4);
    add(a.total, kMergeCells * 4);
    add(a.bins.cntF, M * chunks * sf * 4);
    add(a.bins.cntC, M * chunks * sc * 4);
    add(a.bins.made, M * chunks * 4);
    add(a.bins.baseF, sf ? M * (sf + 1) * 4 : 0);
    add(a.bins.baseC, sc ? M * (sc + 1) * 4 : 0);
    add(a.bins.recF, sf ? M * cap * sizeof(EntryRecord) : 0);
    add(a.bins.recC, sc ? M * cap * sizeof(EntryRecord) : 0);
    return k;
}

int cngp_encode_fwd(const cngp_config *cfg, const float *x, int64_t N, const void *D_f, const void *D_c,
                    void *y, void *workspace, size_t workspace_bytes, void *stream) {
    if (int rc = validate(cfg)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    if (N == 0) return CNGP_OK;
    if (!x || !D_f || !y || (!D_c && !index_codebook_is_empty(cfg))) return CNGP_ERR_NULL;
    if (cfg->index_format == CNGP_IDX_BITS && ((uintptr_t)D_c & 3u)) return CNGP_ERR_INVALID;
    if (cfg->F != 2) return fwd_planes(cfg, cfg->L, x, N, D_f, D_c, y, workspace, workspace_bytes, stream);
    const Params p = make_params(cfg);
    hipStream_t s = (hipStream_t)stream;
    CNGP_DISPATCH_TYPES(launch_fwd, cfg, p, x, N, D_f, D_c, y, s, nullptr, workspace, workspace_bytes);
}

int cngp_encode_fwd_partial(const cngp_config *cfg, int32_t levels_loaded, const float *x, int64_t N, const void *D_f,
                            const void *D_c, void *y, void *workspace, size_t workspace_bytes, void *stream) {
    if (int rc = validate(cfg)) return rc;
    if (N < 0 || levels_loaded < 0 || levels_loaded > cfg->L) return CNGP_ERR_INVALID;
    if (N == 0) return CNGP_OK;
    if (!x || !y) return CNGP_ERR_NULL;
    if (levels_loaded > 0 && (!D_f || (!D_c && !index_codebook_is_empty(cfg)))) return CNGP_ERR_NULL;
    if (cfg->index_format == CNGP_IDX_BITS && ((uintptr_t)D_c & 3u)) return CNGP_ERR_INVALID;
    if (cfg->F != 2) return fwd_planes(cfg, levels_loaded, x, N, D_f, D_c, y, workspace, workspace_bytes, stream);
    Params p = make_params(cfg);
    p.L_loaded = levels_loaded;
    hipStream_t s = (hipStream_t)stream;
    CNGP_DISPATCH_TYPES(launch_fwd, cfg, p, x, N, D_f, D_c, y, s, nullptr, workspace, workspace_bytes);
}

int cngp_encode_fwd_permuted(const cngp_config *cfg, const float *x_sorted, const int32_t *perm, int64_t N, const void *D_f,
                             const void *D_c, void *y, void *workspace, size_t workspace_bytes, void *stream) {
    if (int rc = validate(cfg)) return rc;
    if (N < 0 || N > 0x7fffffffLL) return CNGP_ERR_INVALID;
    if (cfg->F != 2) return CNGP_ERR_UNSUPPORTED;
    if (N == 0) return CNGP_OK;
    if (!x_sorted || !perm || !D_f || !y || (!D_c && !index_codebook_is_empty(cfg))) return CNGP_ERR_NULL;
    if (cfg->index_format == CNGP_IDX_BITS && ((uintptr_t)D_c & 3u)) return CNGP_ERR_INVALID;
    const Params p = make_params(cfg);
    hipStream_t s = (hipStream_t)stream;
    CNGP_DISPATCH_TYPES(launch_fwd, cfg, p, x_sorted, N, D_f, D_c, y, s, perm, workspace, workspace_bytes);
}

int cngp_encode_bwd(const cngp_config *cfg, const float *x, int64_t N, const void *D_f,
                    const float *Dhat_c, const void *dy, float *grad_D_f, float *grad_Dhat_c,
                    void *workspace, size_t workspace_bytes, void *stream) {
    if (int rc = validate(cfg)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    if (!grad_D_f || !grad_Dhat_c) return CNGP_ERR_NULL;
    if (N > 0 && (!x || !D_f || !Dhat_c || !dy)) return CNGP_ERR_NULL;
    if (cfg->F != 2) return bwd_planes(cfg, x, N, D_f, Dhat_c, dy, grad_D_f, grad_Dhat_c, workspace, workspace_bytes, stream);
    hipStream_t s = (hipStream_t)stream;
    int64_t per = bwd_pass_points(cfg, N);
    // (passes whose bins do not fit, of tables that are scanned then: one scan where that fits, which adds fewer fp32 sums to an entry than scans in passes)
    if (per < N && !bwd_plan_for(cfg, per, workspace_bytes).binned && make_bwd_plan(cfg, N, LAYOUT_LEAST).ws_bytes <= workspace_bytes) per = N;
    size_t least = per < N ? least_workspace_pairs(cfg, N) : 0;
    if (N > 0 && workspace_bytes < (per < N ? least : bwd_plan_for(cfg, N, workspace_bytes).ws_bytes)) {
        const size_t passes = short_passes_workspace_pairs(cfg, N);
        if (passes && passes <= workspace_bytes) { per = short_pass_points(cfg, N); least = passes; }
    }
    if (per < N) {      // several passes over runs of points; the first one clears if asked, the rest accumulate
        if (!workspace || ((uintptr_t)workspace & 255u) || workspace_bytes < least) return CNGP_ERR_WORKSPACE;
        cngp_config   pass = *cfg;
        const size_t  io = cfg->io_dtype == CNGP_F16 ? 2 : 4;
        for (int64_t first = 0; first < N; first += per) {
            const int64_t n = N - first < per ? N - first : per;
            const int rc = cngp_encode_bwd(&pass, x + first * cfg->d, n, D_f, Dhat_c,
                                           (const char *)dy + (size_t)first * cfg->L * cfg->F * io, grad_D_f, grad_Dhat_c,
                                           workspace, workspace_bytes, stream);
            if (rc) return rc;
            pass.flags &= ~(uint32_t)CNGP_ZERO_GRADS;
        }
        return CNGP_OK;
    }
    const BwdPlan b = bwd_plan_for(cfg, N, workspace_bytes);
    if (N > 0 && b.sliced) {
        if (!workspace || ((uintptr_t)workspace & 255u) || workspace_bytes < b.ws_bytes) return CNGP_ERR_WORKSPACE;
    }
    // A sliced launch with a single chunk writes every gradient entry of its levels itself; the other
    // level ranges (dense levels 0 .. Ld-1, hashed levels Ld .. L-1) are cleared here.
    ZeroList z;
    if (cfg->flags & CNGP_ZERO_GRADS) {
        const int64_t per_f = (int64_t)cfg->N_f * cfg->F, per_c = (int64_t)cfg->N_c * cfg->N_p;
        const bool    sl = N > 0 && b.sliced;
        const int     Ld = sl ? b.dense.count : 0, Lh = cfg->L - Ld;
        const bool    once_f = b.split || b.sum_f, once_c = b.split || b.sum_c;      // partial sums: an entry is written once
        if (!(sl && (b.feat_vtx.chunks == 1 || b.sum_f)) && Ld > 0) z.add(grad_D_f, per_f * Ld);
        const uint32_t wg_f = once_f ? 1u : b.binned ? b.subs_f : b.feat_pts.chunks, wg_c = once_c ? 1u : b.binned ? b.subs_c : b.logit_pts.chunks;
        if (!(sl && wg_f == 1) && Lh > 0) z.add(grad_D_f + per_f * Ld, per_f * Lh);
        const bool logit = sl && cfg->N_p > 1;
        if (!(logit && (b.logit_vtx.chunks == 1 || b.sum_c)) && Ld > 0) z.add(grad_Dhat_c, per_c * Ld);
        if (!(logit && wg_c == 1) && Lh > 0) z.add(grad_Dhat_c + per_c * Ld, per_c * Lh);
    }
    if (N == 0) return z.launch(s);
    const Params p = make_params(cfg);
    // the LDS variants clear these ranges in their preparation launch, the direct one with a launch of its own
    CNGP_DISPATCH_TYPES(dispatch_bwd_np, cfg, p, b, x, N, D_f, Dhat_c, dy, grad_D_f, grad_Dhat_c, workspace, z, s);
}

size_t cngp_static_scratch_bytes(void) { return kStaticScratchBytes; }

int cngp_encode_bwd_static(const cngp_config *cfg, const float *x, int64_t N, const void *D_f,
                           const float *Dhat_c, const void *dy, float *grad_D_f, float *grad_Dhat_c, void *stream) {
    if (int rc = validate(cfg)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    if (!grad_D_f || !grad_Dhat_c) return CNGP_ERR_NULL;
    if (N > 0 && (!x || !D_f || !Dhat_c || !dy)) return CNGP_ERR_NULL;
    // The variant is the one cngp_encode_bwd would pick for (cfg, N) in a workspace of this size: in one pass where its
    // smallest layout fits (without merged levels or partial sums, and tables of few slices scanned, where there is no room for those).
    // Else the bins are bounded until everything fits (the batch is then taken in several passes inside the one call, like any
    // batch beyond cfg->bin_bytes_max), as long as a pass is still binned: tables that are binned whatever the room are not scanned here.
    cngp_config c = *cfg;
    size_t need = cngp_workspace_bytes(&c, N);
    if (need > kStaticScratchBytes && N > 0) {      // in one pass all the same, if the smallest layout fits
        const cngp_config pairs = as_pairs(cfg);
        const size_t least = cfg->F != 2 ? plane_space(cfg, N, true).total : least_workspace_pairs(&pairs, N);
        if (least <= kStaticScratchBytes) need = least;
    }
    if (need > kStaticScratchBytes && N > 0) {
        const int64_t per0 = bwd_pass_points(cfg, N);
        const bool    binned = make_bwd_plan_uncached(cfg, per0 < N ? per0 : N).binned;
        for (uint64_t bins = kStaticScratchBytes / 2; binned && bins >= ((uint64_t)1 << 20); bins /= 2) {
            if (cfg->bin_bytes_max && cfg->bin_bytes_max < bins) continue;      // never beyond the caller's own bound
            cngp_config t = *cfg;
            t.bin_bytes_max = bins;
            const int64_t per = bwd_pass_points(&t, N);
            if (!make_bwd_plan_uncached(&t, per < N ? per : N).binned) break;   // passes too small to bin
            const size_t  n = cngp_workspace_bytes(&t, N);
            if (n <= kStaticScratchBytes) { c = t; need = n; break; }
        }
    }
    if (need > kStaticScratchBytes) {
        g_hip_error = "cngp_encode_bwd_static: this configuration and N need " + std::to_string(need) +
                      " bytes of scratch, the static array holds " + std::to_string(kStaticScratchBytes) +
                      "; use cngp_encode_bwd with a workspace";
        return CNGP_ERR_WORKSPACE;
    }
    void *ws = nullptr;
    if (int rc = static_scratch(&ws)) return rc;
    return cngp_encode_bwd(&c, x, N, D_f, Dhat_c, dy, grad_D_f, grad_Dhat_c, ws, kStaticScratchBytes, stream);
}

int cngp_encode_bwd_input(const cngp_config *cfg, const float *x, int64_t N, const void *D_f, const void *D_c,
                          const void *dy, float *grad_x, void *stream) {
    if (int rc = validate(cfg)) return rc;
    if (cfg->F != 2) return CNGP_ERR_UNSUPPORTED;           // (no workspace argument to hold the pair planes)
    if (N < 0) return CNGP_ERR_INVALID;
    if (N == 0) return CNGP_OK;
    if (!x || !D_f || !dy || !grad_x || (!D_c && !index_codebook_is_empty(cfg))) return CNGP_ERR_NULL;
    if (cfg->index_format == CNGP_IDX_BITS && ((uintptr_t)D_c & 3u)) return CNGP_ERR_INVALID;
    const Params p = make_params(cfg);
    hipStream_t s = (hipStream_t)stream;
    CNGP_DISPATCH_TYPES(launch_bwd_input, cfg, p, x, N, D_f, D_c, dy, grad_x, s);
}

int cngp_storage_bytes(const cngp_config *cfg, size_t *D_f_bytes, size_t *D_c_level_bytes, size_t *D_c_bytes) {
    if (int rc = validate(cfg)) return rc;
    const size_t level = index_level_bytes(cfg);
    if (D_f_bytes) *D_f_bytes = (size_t)cfg->L * cfg->N_f * cfg->F * (cfg->feat_dtype == CNGP_F16 ? 2 : 4);
    if (D_c_level_bytes) *D_c_level_bytes = level;
    if (D_c_bytes) *D_c_bytes = level * cfg->L;
    return CNGP_OK;
}

int cngp_bake_probes(const cngp_config *cfg, const float *Dhat_c, void *D_c, void *stream) {
    if (int rc = validate(cfg)) return rc;
    if (index_codebook_is_empty(cfg)) return Dhat_c ? CNGP_OK : CNGP_ERR_NULL;       // nothing to write
    if (!Dhat_c || !D_c) return CNGP_ERR_NULL;
    hipStream_t s = (hipStream_t)stream;
    if (cfg->index_format == CNGP_IDX_BITS) {
        if ((uintptr_t)D_c & 3u) return CNGP_ERR_INVALID;
        const uint32_t wpl = (uint32_t)(index_level_bytes(cfg) / 4);
        const int64_t  words = (int64_t)cfg->L * wpl;
        const int64_t  blocks = (words + kBlock - 1) / kBlock;
        if (int rc = check_blocks(blocks)) return rc;
        LaunchTimer t(s, K_BAKE);
#define CNGP_BAKE_BITS(NP) bake_probes_bits_kernel<NP><<<(unsigned)blocks, kBlock, 0, s>>>(Dhat_c, (uint32_t *)D_c, cfg->N_c, wpl, words)
        switch (cfg->N_p) {
        case 2:  CNGP_BAKE_BITS(2); break;
        case 4:  CNGP_BAKE_BITS(4); break;
        case 8:  CNGP_BAKE_BITS(8); break;
        default: CNGP_BAKE_BITS(16); break;
        }
#undef CNGP_BAKE_BITS
        return launch_status("bake_probes_bits_kernel");
    }
    const bool packed = cfg->index_format == CNGP_IDX_PACKED4;
    const int64_t rows = (int64_t)cfg->L * cfg->N_c;
    const int64_t bytes_out = packed ? rows / 2 : rows;
    const int64_t blocks = (bytes_out + kBlock - 1) / kBlock;
    if (int rc = check_blocks(blocks)) return rc;
    LaunchTimer t(s, K_BAKE);
#define CNGP_BAKE(NP)                                                                                  \
    if (packed) bake_probes_kernel<NP, true><<<(unsigned)blocks, kBlock, 0, s>>>(Dhat_c, (uint8_t *)D_c, bytes_out); \
    else        bake_probes_kernel<NP, false><<<(unsigned)blocks, kBlock, 0, s>>>(Dhat_c, (uint8_t *)D_c, bytes_out)
    switch (cfg->N_p) {
    case 1:  CNGP_BAKE(1); break;
    case 2:  CNGP_BAKE(2); break;
    case 4:  CNGP_BAKE(4); break;
    case 8:  CNGP_BAKE(8); break;
    default: CNGP_BAKE(16); break;
    }
#undef CNGP_BAKE
    return launch_status("bake_probes_kernel");
}

int cngp_adam_step_bake(const cngp_config *cfg, const cngp_adam *opt_f, const cngp_adam *opt_c,
                        float *D_f_master, void *D_f, float *m_f, float *v_f, float *grad_D_f,
                        float *Dhat_c, float *m_c, float *v_c, float *grad_Dhat_c, void *D_c, void *stream) {
    if (int rc = validate(cfg)) return rc;
    if (cfg->index_format == CNGP_IDX_BITS) return CNGP_ERR_UNSUPPORTED;   // training keeps whole-byte or 4-bit entries
    AdamTable f, c;
    std::memset(&f, 0, sizeof(f));
    std::memset(&c, 0, sizeof(c));
    __half *D_f_half = nullptr;
    if (opt_f) {
        if (!D_f_master || !m_f || !v_f || !grad_D_f) return CNGP_ERR_NULL;
        if (int rc = adam_coefficients(opt_f, &f.a)) return rc;
        if (cfg->feat_dtype == CNGP_F16) {
            if (!D_f) return CNGP_ERR_NULL;
            if (!aligned(D_f, 8)) return CNGP_ERR_INVALID;
            D_f_half = (__half *)D_f;
        } else if (D_f && D_f != (void *)D_f_master) {
            return CNGP_ERR_INVALID;
        }
        if (!aligned(D_f_master, 16) || !aligned(m_f, 16) || !aligned(v_f, 16) || !aligned(grad_D_f, 16)) return CNGP_ERR_INVALID;
        f.theta = D_f_master; f.m = m_f; f.v = v_f; f.grad = grad_D_f;
        f.n = (int64_t)cfg->L * cfg->N_f * cfg->F;
    }
    if (opt_c) {
        if (!Dhat_c || !m_c || !v_c || !grad_Dhat_c || !D_c) return CNGP_ERR_NULL;
        if (int rc = adam_coefficients(opt_c, &c.a)) return rc;
        if (!aligned(Dhat_c, 16) || !aligned(m_c, 16) || !aligned(v_c, 16) || !aligned(grad_Dhat_c, 16)) return CNGP_ERR_INVALID;
        c.theta = Dhat_c; c.m = m_c; c.v = v_c; c.grad = grad_Dhat_c;
        c.n = (int64_t)cfg->L * cfg->N_c * cfg->N_p;
    }
    const int64_t per_block = (int64_t)kOptBlock * 4;
    const int64_t blocks_f = (f.n + per_block - 1) / per_block;
    const int64_t blocks_c = (c.n + per_block - 1) / per_block;
    if (blocks_f + blocks_c == 0) return CNGP_OK;
    if (int rc = check_blocks(blocks_f + blocks_c)) return rc;
    const bool packed = cfg->index_format == CNGP_IDX_PACKED4;
    const int  clear = (cfg->flags & CNGP_ZERO_GRADS) ? 1 : 0;
    hipStream_t s = (hipStream_t)stream;
    LaunchTimer t(s, K_ADAM);
#define CNGP_ADAM(NP)                                                                                   \
    if (packed) adam_step_bake_kernel<NP, true><<<(unsigned)(blocks_f + blocks_c), kOptBlock, 0, s>>>(  \
                    f, c, D_f_half, (uint8_t *)D_c, (uint32_t)blocks_f, clear);                         \
    else        adam_step_bake_kernel<NP, false><<<(unsigned)(blocks_f + blocks_c), kOptBlock, 0, s>>>( \
                    f, c, D_f_half, (uint8_t *)D_c, (uint32_t)blocks_f, clear)
    switch (cfg->N_p) {
    case 1:  CNGP_ADAM(1); break;
    case 2:  CNGP_ADAM(2); break;
    case 4:  CNGP_ADAM(4); break;
    case 8:  CNGP_ADAM(8); break;
    default: CNGP_ADAM(16); break;
    }
#undef CNGP_ADAM
    return launch_status("adam_step_bake_kernel");
}

int cngp_adam_step(const cngp_adam *opt, int64_t n, float *master, void *half_copy, float *m, float *v,
                   float *grad, int clear_grad, void *stream) {
    if (!opt || !master || !m || !v || !grad) return CNGP_ERR_NULL;
    if (n < 0) return CNGP_ERR_INVALID;
    AdamTable f, c;
    std::memset(&f, 0, sizeof(f));
    std::memset(&c, 0, sizeof(c));
    if (int rc = adam_coefficients(opt, &f.a)) return rc;
    if (!aligned(master, 16) || !aligned(m, 16) || !aligned(v, 16) || !aligned(grad, 16) || !aligned(half_copy, 8)) return CNGP_ERR_INVALID;
    if (n == 0) return CNGP_OK;
    f.theta = master; f.m = m; f.v = v; f.grad = grad; f.n = n;
    const int64_t per_block = (int64_t)kOptBlock * 4;
    const int64_t blocks = (n + per_block - 1) / per_block;
    if (int rc = check_blocks(blocks)) return rc;
    hipStream_t s = (hipStream_t)stream;
    LaunchTimer t(s, K_ADAM);
    adam_step_bake_kernel<1, false><<<(unsigned)blocks, kOptBlock, 0, s>>>(f, c, (__half *)half_copy, nullptr,
                                                                           (uint32_t)blocks, clear_grad ? 1 : 0);
    return launch_status("adam_step_bake_kernel");
}

namespace {
int mlp_dims(const cngp_mlp_config *cfg, MlpDims *d) {
    if (!cfg) return CNGP_ERR_NULL;
    if (cfg->n_in < 1 || cfg->n_in > kMlpMaxIn || cfg->n_out < 1 || cfg->n_out > kMlpMaxOut) return CNGP_ERR_INVALID;
    if (cfg->io_dtype != CNGP_F32 && cfg->io_dtype != CNGP_F16) return CNGP_ERR_INVALID;
    if (cfg->flags & ~(uint32_t)CNGP_ZERO_GRADS) return CNGP_ERR_INVALID;
    d->n_in = cfg->n_in; d->n_out = cfg->n_out;
    d->ks1 = (cfg->n_in + 7) / 8; d->ks3 = (cfg->n_out + 7) / 8;
    d->vec_in = d->vec_out = 0;            // set by the caller once the pointers are known
    return CNGP_OK;
}
// A persistent grid: every wavefront walks over tiles of 32 points.  At most `per_cu` workgroups per CU
// (what fits at once), and no more than gives each wavefront `min_tiles` tiles, so that the staging of the
// weights, which every workgroup repeats, stays a small part of its work.
unsigned mlp_blocks(int64_t tiles, int per_cu, int min_tiles, int block = kMlpBlock) {
    const int64_t per_block = (int64_t)(block / 64) * min_tiles;
    const int64_t want = (tiles + per_block - 1) / per_block;
    const int64_t cap = 256 * (int64_t)per_cu;
    return (unsigned)(want < cap ? want : cap);
}
}  // namespace

size_t cngp_mlp_weight_count(const cngp_mlp_config *cfg) {
    MlpDims d;
    if (mlp_dims(cfg, &d)) return 0;
    return (size_t)kMlpHidden * d.n_in + (size_t)kMlpHidden * kMlpHidden + (size_t)kMlpHidden * d.n_out;
}

int cngp_mlp_fwd(const cngp_mlp_config *cfg, const void *y, int64_t N, const void *W, float *out, void *stream) {
    MlpDims d;
    if (int rc = mlp_dims(cfg, &d)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    if (N == 0) return CNGP_OK;
    if (!y || !W || !out) return CNGP_ERR_NULL;
    const int64_t tiles = (N + 31) / 32;
    hipStream_t s = (hipStream_t)stream;
    d.vec_in = (cfg->n_in % 4 == 0 && aligned(y, 16)) ? 1 : 0;
    d.vec_out = (cfg->n_out % 4 == 0 && aligned(out, 16)) ? 1 : 0;
    LaunchTimer t(s, K_MLP_FWD);
    if (cfg->io_dtype == CNGP_F16)
        mlp_fwd_kernel<__half><<<mlp_blocks(tiles, 3, 4), kMlpBlock, kMlpFwdLds, s>>>(d, (const __half *)y, N, (const __half *)W, out, tiles);
    else
        mlp_fwd_kernel<float><<<mlp_blocks(tiles, 3, 4), kMlpBlock, kMlpFwdLds, s>>>(d, (const float *)y, N, (const __half *)W, out, tiles);
    return launch_status("mlp_fwd_kernel");
}

int cngp_encode_mlp_fwd(const cngp_config *cfg, const cngp_mlp_config *mlp, const float *x, int64_t N,
                        const void *D_f, const void *D_c, const void *W, float *out,
                        void *workspace, size_t workspace_bytes, void *stream) {
    if (int rc = validate(cfg)) return rc;
    MlpDims d;
    if (int rc = mlp_dims(mlp, &d)) return rc;
    if (cfg->F != 2) return CNGP_ERR_UNSUPPORTED;
    if (d.n_in != cfg->L * cfg->F) return CNGP_ERR_INVALID;
    if (N < 0) return CNGP_ERR_INVALID;
    if (N == 0) return CNGP_OK;
    if (!x || !D_f || !W || !out || (!D_c && !index_codebook_is_empty(cfg))) return CNGP_ERR_NULL;
    if (cfg->index_format == CNGP_IDX_BITS && ((uintptr_t)D_c & 3u)) return CNGP_ERR_INVALID;
    const Params p = make_params(cfg);
    hipStream_t s = (hipStream_t)stream;
    // With room for the level-major fp16 encodings: the level-resident forward without its rows kernel, and the
    // decoder reading the planes as they are.
    {
        cngp_config c16 = *cfg;
        c16.io_dtype = CNGP_F16;
        const FwdLevelPlan f = fwd_level_plan(&c16, cfg->L, N);
        if (f.use && workspace && workspace_bytes >= f.yT_bytes && ((uintptr_t)workspace & 255u) == 0 && ((uintptr_t)D_f & 15u) == 0) {
            int rc;
            const bool f16 = cfg->feat_dtype == CNGP_F16;
            if (cfg->d == 2) rc = f16 ? launch_fwd_level<2, __half, __half>(&c16, f, p, x, N, D_f, D_c, nullptr, workspace, s, nullptr, false)
                                      : launch_fwd_level<2, float, __half>(&c16, f, p, x, N, D_f, D_c, nullptr, workspace, s, nullptr, false);
            else if (cfg->d == 3) rc = f16 ? launch_fwd_level<3, __half, __half>(&c16, f, p, x, N, D_f, D_c, nullptr, workspace, s, nullptr, false)
                                           : launch_fwd_level<3, float, __half>(&c16, f, p, x, N, D_f, D_c, nullptr, workspace, s, nullptr, false);
            else rc = f16 ? launch_fwd_level<4, __half, __half>(&c16, f, p, x, N, D_f, D_c, nullptr, workspace, s, nullptr, false)
                          : launch_fwd_level<4, float, __half>(&c16, f, p, x, N, D_f, D_c, nullptr, workspace, s, nullptr, false);
            if (rc) return rc;
            const int64_t tiles = (N + 31) / 32;
            d.vec_out = (d.n_out % 4 == 0 && aligned(out, 16)) ? 1 : 0;
            LaunchTimer t(s, K_MLP_FWD);
            mlp_fwd_kernel<__half, true><<<mlp_blocks(tiles, 3, 4), kMlpBlock, kMlpFwdLds, s>>>(d, (const __half *)workspace, N, (const __half *)W, out, tiles);
            return launch_status("mlp_fwd_kernel");
        }
    }
    CNGP_DISPATCH_TYPES(launch_fused_fwd, cfg, p, d, x, N, D_f, D_c, W, out, s);
}

int cngp_mlp_bwd(const cngp_mlp_config *cfg, const void *y, int64_t N, const void *W, const float *dout,
                 void *dy, float *grad_W, void *stream) {
    MlpDims d;
    if (int rc = mlp_dims(cfg, &d)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    if (!grad_W) return CNGP_ERR_NULL;
    if (N > 0 && (!y || !W || !dout || !dy)) return CNGP_ERR_NULL;
    hipStream_t s = (hipStream_t)stream;
    if (cfg->flags & CNGP_ZERO_GRADS) {
        ZeroList z;
        z.add(grad_W, (int64_t)cngp_mlp_weight_count(cfg));
        if (int rc = z.launch(s)) return rc;
    }
    if (N == 0) return CNGP_OK;
    const int64_t tiles = (N + 31) / 32;
    d.vec_in = (cfg->n_in % 4 == 0 && aligned(y, 16) && aligned(dy, 16)) ? 1 : 0;
    d.vec_out = (cfg->n_out % 4 == 0 && aligned(dout, 16)) ? 1 : 0;
    if (cfg->io_dtype == CNGP_F16) {
        auto kernel = mlp_bwd_kernel<__half>;
        if (int rc = allow_big_lds(kernel, kMlpBwdLds)) return rc;
        LaunchTimer t(s, K_MLP_BWD);
        kernel<<<mlp_blocks(tiles, 1, 2, kMlpBwdBlock), kMlpBwdBlock, kMlpBwdLds, s>>>(d, (const __half *)y, N, (const __half *)W, dout, (__half *)dy, grad_W, tiles);
    } else {
        auto kernel = mlp_bwd_kernel<float>;
        if (int rc = allow_big_lds(kernel, kMlpBwdLds)) return rc;
        LaunchTimer t(s, K_MLP_BWD);
        kernel<<<mlp_blocks(tiles, 1, 2, kMlpBwdBlock), kMlpBwdBlock, kMlpBwdLds, s>>>(d, (const float *)y, N, (const __half *)W, dout, (float *)dy, grad_W, tiles);
    }
    return launch_status("mlp_bwd_kernel");
}

int cngp_debug_indices(const cngp_config *cfg, const float *x, int64_t N, const void *D_c, uint32_t *base,
                       uint32_t *h2, uint8_t *probe, uint32_t *feat_idx, void *stream) {
    if (int rc = validate(cfg)) return rc;
    if (N < 0) return CNGP_ERR_INVALID;
    if (N == 0) return CNGP_OK;
    if (!x) return CNGP_ERR_NULL;
    if (!D_c && (probe || feat_idx) && !index_codebook_is_empty(cfg)) return CNGP_ERR_NULL;
    const Params p = make_params(cfg);
    const int64_t pairs = N * cfg->L;
    const int64_t blocks = (pairs + kBlock - 1) / kBlock;
    if (int rc = check_blocks(blocks)) return rc;
    hipStream_t s = (hipStream_t)stream;
    if (cfg->index_format == CNGP_IDX_BITS && ((uintptr_t)D_c & 3u)) return CNGP_ERR_INVALID;
    const uint32_t c_stride = (uint32_t)index_level_bytes(cfg);
    LaunchTimer t(s, K_DEBUG);
#define CNGP_DBG(D, FMT) debug_indices_kernel<D, FMT><<<(unsigned)blocks, kBlock, 0, s>>>(p, x, (const uint8_t *)D_c, base, h2, probe, feat_idx, pairs, c_stride)
#define CNGP_DBG_FMT(D)                                                     \
    if (cfg->index_format == CNGP_IDX_PACKED4) CNGP_DBG(D, kFmtPacked4);   \
    else if (cfg->index_format == CNGP_IDX_BITS) CNGP_DBG(D, kFmtBits);    \
    else CNGP_DBG(D, kFmtU8)
    if (cfg->d == 2) { CNGP_DBG_FMT(2); } else if (cfg->d == 3) { CNGP_DBG_FMT(3); } else { CNGP_DBG_FMT(4); }
#undef CNGP_DBG_FMT
#undef CNGP_DBG
    return launch_status("debug_indices_kernel");
}

int cngp_measure_rates(cngp_rates *out, void *scratch, size_t scratch_bytes, void *stream) {
    if (!out || !scratch) return CNGP_ERR_NULL;
    const size_t need = (size_t)64 << 20;
    if (scratch_bytes < need || ((uintptr_t)scratch & 255u)) return CNGP_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    hipEvent_t  t0, t1;
    CNGP_HIP(hipEventCreate(&t0));
    CNGP_HIP(hipEventCreate(&t1));
    int rc = CNGP_OK;
    auto timed = [&](auto launch, int reps, double &ms_out) {       // one untimed run, then `reps` timed ones
        launch();
        if (hipEventRecord(t0, s) != hipSuccess) rc = CNGP_ERR_HIP;
        for (int i = 0; i < reps; ++i) launch();
        if (hipEventRecord(t1, s) != hipSuccess || hipEventSynchronize(t1) != hipSuccess) rc = CNGP_ERR_HIP;
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, t0, t1) != hipSuccess) rc = CNGP_ERR_HIP;
        ms_out = (double)ms / reps;
    };
    float *tab = (float *)scratch;
    float *sink = tab + (need / 4 - 64);                            // last 256 bytes: never inside a table
    double ms = 0.0;
    const size_t half = need / 2 - 256;
    timed([&] { rate_copy_kernel<<<8192, kBlock, 0, s>>>((const float4 *)scratch, (float4 *)((char *)scratch + need / 2), half / 16); }, 3, ms);
    out->copy_GBps = 2.0 * (double)(half / 16 * 16) / ms / 1e6;
    const int      blocks = 256 * 32, iters = 16;
    const double   lane_ops = (double)blocks * kBlock * iters * 8;
    const uint32_t table_floats = (4u << 20) / 4;                   // 4 MB table: L2 resident
    timed([&] { rate_rows_kernel<1, false><<<blocks, kBlock, 0, s>>>(tab, table_floats - 1, iters, sink); }, 3, ms);
    out->gather4_Gps = lane_ops / ms / 1e6;
    timed([&] { rate_rows_kernel<16, false><<<blocks, kBlock, 0, s>>>(tab, table_floats / 16 - 1, iters, sink); }, 3, ms);
    out->row_gather_Gps = lane_ops / 16 / ms / 1e6;
    timed([&] { rate_rows_kernel<16, true><<<blocks, kBlock, 0, s>>>(tab, table_floats / 16 - 1, iters, sink); }, 3, ms);
    out->global_atomic_Gseg = lane_ops / 16 / ms / 1e6;
    const uint32_t far_floats = (32u << 20) / 4;                    // 32 MB table: beyond every L2, in the memory-side cache
    timed([&] { rate_rows_kernel<16, false><<<blocks, kBlock, 0, s>>>(tab, far_floats / 16 - 1, iters, sink); }, 3, ms);
    out->row_gather_far_Gps = lane_ops / 16 / ms / 1e6;
    timed([&] { rate_rows_kernel<1, false><<<blocks, kBlock, 0, s>>>(tab, far_floats - 1, iters, sink); }, 3, ms);
    out->gather4_far_Gps = lane_ops / ms / 1e6;
    auto lds_rate = [&](auto kernel, size_t lds, double &gps) {
        if (int r2 = allow_big_lds(kernel, lds)) rc = r2;
        const int lblocks = 1024, liters = 64;
        timed([&] { kernel<<<lblocks, 1024, lds, s>>>(liters, sink); }, 3, ms);
        gps = (double)lblocks * 1024 * liters * 8 / ms / 1e6;
    };
    lds_rate(rate_lds_atomic_kernel<double>, 16384 * sizeof(double), out->lds_atomic_f64_Gps);
    lds_rate(rate_lds_atomic_kernel<float>, 16384 * sizeof(float), out->lds_atomic_f32_Gps);
    lds_rate(rate_lds_atomic_kernel<uint32_t>, 16384 * sizeof(uint32_t), out->lds_atomic_u32_Gps);
    lds_rate(rate_lds_gather_kernel, 32768 * sizeof(uint32_t), out->lds_gather4_Gps);
    (void)hipEventDestroy(t0);
    (void)hipEventDestroy(t1);
    if (rc == CNGP_OK) rc = launch_status("cngp_measure_rates");
    return rc;
}

int cngp_profile_enable(int on) {
    const int was = g_profile ? 1 : 0;
    g_profile = on != 0;
    return was;
}

const char *cngp_profile_kernel_name(int i) { return (i >= 0 && i < K_COUNT) ? kKernelNames[i] : ""; }

int cngp_profile_read(double *ms_sum, int64_t *launches, int max_kernels) {
    for (auto &t : g_timed) {
        float ms = 0.0f;
        if (hipEventSynchronize(t.t1) == hipSuccess && hipEventElapsedTime(&ms, t.t0, t.t1) == hipSuccess &&
            t.id < max_kernels) {
            if (ms_sum) ms_sum[t.id] += (double)ms;
            if (launches) launches[t.id] += 1;
        }
        (void)hipEventDestroy(t.t0);
        (void)hipEventDestroy(t.t1);
    }
    g_timed.clear();
    return K_COUNT;
}

}  // extern "C"
