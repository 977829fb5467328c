// Decoder after the encoding (Fig. 3: the interpolated features are fed into an MLP; Table 1: 64 hidden
// neurons).  Assumed, because the paper does not say: two hidden layers, ReLU, linear output, no biases.
//
//     h1 = relu(W1 y)   h2 = relu(W2 h1)   out = W3 h2        W1 [64, n_in], W2 [64, 64], W3 [n_out, 64]
//
// The only dense contraction of the method, hence the only user of the matrix cores here.  Everything is
// computed transposed, points along the columns: one wavefront owns 32 points and every layer is
//     (weights as the A operand, 32 x 16 per instruction) x (activations^T as the B operand, 16 x 32)
// with v_mfma_f32_32x32x16_f16.  The accumulator layout (lane = column, four consecutive rows per register
// group, the two halves of the wavefront four rows apart) feeds the next layer straight from registers:
// after ReLU and rounding to fp16, accumulator registers 4j .. 4j+3 of row tile t hold rows
// 32t + 8j + 4h .. + 3 (h = lane / 32), a "quarter step"; two quarter steps 2s', 2s'+1 side by side are
// this lane's eight B values of K-step s'.  That is not the instruction's natural K order (rows
// 16s' + 8h .. + 7) but a permutation of it inside the step, and a contraction does not care about the
// order of its terms as long as both operands use the same one: the weights are staged in LDS in that
// order.  Only the weight gradients, which contract over the points, need a transpose; it goes through a
// per-wavefront tile in LDS, by the transposing LDS read.
#pragma once
#include "cngp_bwd_sliced.h"   // wave_lds_fence

namespace cngp {

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float    acc16_t __attribute__((ext_vector_type(16)));

constexpr int kMlpHidden = 64;
constexpr int kMlpBlock = 256;                 // 4 wavefronts
constexpr int kMlpMaxIn = 32, kMlpMaxOut = 16;

struct MlpDims {
    int n_in, n_out;
    int ks1;                                   // quarter steps (8 rows) of layer 1: ceil(n_in / 8)
    int ks3;                                   // quarter steps of the transposed output layer: ceil(n_out / 8)
    int vec_in, vec_out;                       // rows of y (and dL/dy) / of dL/dout can be read four values at a time
};

// Slots of the weight operands in LDS, counted in quarter steps (one half4 per lane: rows 8s + 4h .. + 3 of the
// contraction).  Slots 2p and 2p + 1 lie side by side per lane, so that operand p of an instruction is one
// 16-byte read: half8 number p * 64 + lane.
enum : int { kOpW1 = 0, kOpW2 = 8, kOpW3 = 24, kOpW3T = 32, kOpW2T = 36, kOpW1T = 52, kOpFwdSlots = 32, kOpAllSlots = 60 };

__device__ __forceinline__ half8_t cat(const half4_t lo, const half4_t hi) {
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ acc16_t mfma(const half8_t a, const half8_t b, const acc16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ acc16_t acc_zero() {
    acc16_t z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.0f;
    return z;
}

// `SLOTS` operand slots from `slot0` on, of a matrix stored row-major [rows, cols] (TR: of its transpose), `STEPS` quarter steps to a
// row tile; the slots are dealt to the wavefronts.  Four neighbouring columns are one read where rows start at multiples of four.
template <int BLOCK, bool TR, int SLOTS, int STEPS>
__device__ __forceinline__ void fill_operands(half4_t *ops, const int slot0, const __half *M, const int rows, const int cols) {
    constexpr int kWaves = BLOCK / 64, kMine = (SLOTS + kWaves - 1) / kWaves;
    const int  lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool quads = !TR && cols % 4 == 0;
    half4_t v[kMine];
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        const int at = i * kWaves + wave;                    // a slot beyond the last is read as the last, and not written
        const int slot = at < SLOTS ? at : SLOTS - 1;
        const int out = 32 * (slot / STEPS) + (lane & 31), k = 8 * (slot % STEPS) + 4 * (lane >> 5);
        if (quads) {
            const bool in = out < rows && k < cols;
            const half4_t w = *reinterpret_cast<const half4_t *>(M + (in ? out * cols + k : 0));
#pragma unroll
            for (int j = 0; j < 4; ++j) v[i][j] = in ? w[j] : (_Float16)0.0f;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int  r = TR ? k + j : out, c = TR ? out : k + j;
                const bool in = r < rows && c < cols;
                const _Float16 w = (_Float16)__half2float(M[in ? r * cols + c : 0]);
                v[i][j] = in ? w : (_Float16)0.0f;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        const int slot = slot0 + i * kWaves + wave;
        if (i * kWaves + wave < SLOTS) ops[(((slot >> 1) * 64 + lane) << 1) + (slot & 1)] = v[i];
    }
}

// Fills the operand slots (BWD: all of them, else the forward pass's), the work spread over the workgroup.  The weights first come into LDS as
// they are, with wide coalesced loads, all under way at once (`raw`: room for weight_count halves, 16-byte aligned, may be reused
// after the barrier at the end); building the operand layout from global memory element by element is a
// chain of dependent cache round trips that costs more than the whole forward pass of a small batch.
template <int BLOCK, bool BWD>
__device__ __forceinline__ void stage_operands(half8_t *ops8, __half *raw, const __half *W, const MlpDims d) {
    half4_t *ops = reinterpret_cast<half4_t *>(ops8);
    const int count = kMlpHidden * d.n_in + kMlpHidden * kMlpHidden + kMlpHidden * d.n_out;     // a multiple of 64
    if ((reinterpret_cast<uintptr_t>(W) & 15u) == 0) {
        constexpr int kLoads = (kMlpHidden * (kMlpMaxIn + kMlpHidden + kMlpMaxOut) / 8 + BLOCK - 1) / BLOCK;
        uint4 v[kLoads];
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int at = (i * BLOCK + (int)threadIdx.x) * 8;
            v[i] = *reinterpret_cast<const uint4 *>(W + (at < count ? at : count - 8));
        }
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int at = (i * BLOCK + (int)threadIdx.x) * 8;
            if (at < count) *reinterpret_cast<uint4 *>(raw + at) = v[i];
        }
    } else {
        for (int i = threadIdx.x; i < count; i += BLOCK) raw[i] = W[i];
    }
    __syncthreads();
    const __half *W1 = raw, *W2 = raw + kMlpHidden * d.n_in, *W3 = W2 + kMlpHidden * kMlpHidden;
    fill_operands<BLOCK, false, kOpW2 - kOpW1, 4>(ops, kOpW1, W1, kMlpHidden, d.n_in);
    fill_operands<BLOCK, false, kOpW3 - kOpW2, 8>(ops, kOpW2, W2, kMlpHidden, kMlpHidden);
    fill_operands<BLOCK, false, kOpW3T - kOpW3, 8>(ops, kOpW3, W3, d.n_out, kMlpHidden);
    if constexpr (BWD) {
        fill_operands<BLOCK, true, kOpW2T - kOpW3T, 2>(ops, kOpW3T, W3, d.n_out, kMlpHidden);
        fill_operands<BLOCK, true, kOpW1T - kOpW2T, 8>(ops, kOpW2T, W2, kMlpHidden, kMlpHidden);
        fill_operands<BLOCK, true, kOpAllSlots - kOpW1T, 8>(ops, kOpW1T, W1, kMlpHidden, d.n_in);
    }
    __syncthreads();
}

template <typename T> __device__ __forceinline__ float to_float(T v);
template <> __device__ __forceinline__ float to_float<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_float<__half>(__half v) { return __half2float(v); }
template <typename T> __device__ __forceinline__ T from_float(float v);
template <> __device__ __forceinline__ float from_float<float>(float v) { return v; }
template <> __device__ __forceinline__ __half from_float<__half>(float v) { return __float2half_rn(v); }

// The 32 points of a tile in a row-major array of `cols` columns: the tile's first row (the same for a wavefront, so that a lane's address is a
// 32-bit offset) and how many of its rows there are.  A tile beyond the last is the last.
template <typename T>
struct TileRows { T *base; int rows; };
template <typename T>
__device__ __forceinline__ TileRows<T> tile_rows(T *a, const int64_t tile, const int64_t tiles, const int64_t N, const int cols) {
    const int64_t at = tile < tiles ? tile : tiles - 1, left = N - at * 32;
    return {a + at * 32 * cols, left < 32 ? (int)left : 32};
}

// Four columns k0 .. k0 + 3 of this lane's point, as stored: the B operand of a quarter step once keep_columns / keep_rows have been over it.  Nothing is
// computed from a value here, because the wait for it would come with that: the loads are a tile ahead.  No branch either: a row
// or column that is not there is read as one that is.
// `vec`: cols is a multiple of four and the array 16-byte aligned, so the four values are one load.
__device__ __forceinline__ float4  quad_of(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ __forceinline__ half4_t quad_of(const __half *p) { return *reinterpret_cast<const half4_t *>(p); }
__device__ __forceinline__ float4  quad_of(const float a, const float b, const float c, const float e) { return make_float4(a, b, c, e); }
__device__ __forceinline__ half4_t quad_of(const __half a, const __half b, const __half c, const __half e) {
    half4_t v;
    v[0] = *reinterpret_cast<const _Float16 *>(&a); v[1] = *reinterpret_cast<const _Float16 *>(&b);
    v[2] = *reinterpret_cast<const _Float16 *>(&c); v[3] = *reinterpret_cast<const _Float16 *>(&e);
    return v;
}
__device__ __forceinline__ half4_t to_half4(const half4_t v) { return v; }
__device__ __forceinline__ half4_t to_half4(const float4 f) {
    half4_t v;
    v[0] = (_Float16)f.x; v[1] = (_Float16)f.y; v[2] = (_Float16)f.z; v[3] = (_Float16)f.w;
    return v;
}
template <typename T> using QuadOf = typename std::conditional<sizeof(T) == 2, half4_t, float4>::type;

// Quarter steps 0 .. STEPS - 1, or only the first `steps` of them.
template <typename T, int STEPS>
__device__ __forceinline__ void load_quads(const TileRows<const T> a, const int lane, const int cols, const bool vec, QuadOf<T> (&b)[STEPS],
                                           const int steps = STEPS) {
    const int row = lane & 31, k4 = 4 * (lane >> 5), off = (row < a.rows ? row : a.rows - 1) * cols;
    if (vec) {
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
            if (s < steps) b[s] = quad_of(a.base + off + (8 * s + k4 < cols ? 8 * s + k4 : 0));
    } else {
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
            if (s < steps) {
                T e[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) e[j] = a.base[off + (8 * s + k4 + j < cols ? 8 * s + k4 + j : 0)];
                b[s] = quad_of(e[0], e[1], e[2], e[3]);
            }
    }
}

// Columns from `cols` on become zero (the weights there are zero too, but zero times a value that is not finite is not zero) ...
template <int STEPS>
__device__ __forceinline__ void keep_columns(half4_t (&b)[STEPS], const int cols, const int lane) {
    if (cols == 8 * STEPS) return;
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) b[s][j] = 8 * s + 4 * (lane >> 5) + j < cols ? b[s][j] : (_Float16)0.0f;
}
// ... and points from `rows` on: none of them adds to the weight gradients.
template <int STEPS>
__device__ __forceinline__ void keep_rows(half4_t (&b)[STEPS], const int rows, const int lane) {
    if (rows == 32) return;
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) b[s][j] = (lane & 31) < rows ? b[s][j] : (_Float16)0.0f;
}

__device__ __forceinline__ void store4(float *p, float a, float b, float c, float e) {
    *reinterpret_cast<float4 *>(p) = make_float4(a, b, c, e);
}
__device__ __forceinline__ void store4(__half *p, float a, float b, float c, float e) {
    half4_t v;
    v[0] = (_Float16)a; v[1] = (_Float16)b; v[2] = (_Float16)c; v[3] = (_Float16)e;
    *reinterpret_cast<half4_t *>(p) = v;
}

// ReLU, rounding to fp16, and the re-use of an accumulator tile as B operands of the next layer.
__device__ __forceinline__ void relu_to_b(const acc16_t a, half4_t (&b)[8], const int t) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        half4_t v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = (_Float16)fmaxf(a[4 * j + q], 0.0f);
        b[4 * t + j] = v;
    }
}

// Same for a gradient tile: entries whose forward pre-activation was not positive are dropped.
__device__ __forceinline__ void mask_to_b(const acc16_t g, const uint32_t mask, half4_t (&b)[8], const int t) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        half4_t v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = ((mask >> (4 * j + q)) & 1u) ? (_Float16)g[4 * j + q] : (_Float16)0.0f;
        b[4 * t + j] = v;
    }
}

__device__ __forceinline__ uint32_t positive_mask(const acc16_t a) {
    uint32_t m = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) m |= (a[r] > 0.0f ? 1u : 0u) << r;
    return m;
}

// Layers 1 and 2 for this wavefront's 32 points.
struct Hidden {
    half4_t  yb[4], h1[8], h2[8];
    uint32_t m1[2], m2[2];
};

// This lane's part of the inputs of one tile of 32 points (the B operands of layer 1, once keep_columns has been over them).
template <typename IoT>
__device__ __forceinline__ void load_inputs(const MlpDims d, const IoT *__restrict__ y, const int64_t tile, const int64_t tiles,
                                            const int64_t N, const int lane, QuadOf<IoT> (&yb)[4]) {
    load_quads(tile_rows(y, tile, tiles, N, d.n_in), lane, d.n_in, d.vec_in != 0, yb);
}

// The same from a level-major array yT[n_in / 2][N] of fp16 pairs (what the level-resident forward of the encoding
// writes before its rows kernel): four halves of a row are two neighbouring planes' pairs, and the 32 lanes of a
// tile read 128 contiguous bytes of each plane.
__device__ __forceinline__ void load_inputs_planes(const MlpDims d, const uint32_t *__restrict__ yT, const int64_t tile, const int64_t tiles,
                                                   const int64_t N, const int lane, half4_t (&yb)[4]) {
    const int     k2 = 2 * (lane >> 5), planes = d.n_in / 2;
    const int64_t at = (tile < tiles ? tile : tiles - 1) * 32 + (lane & 31), pt = at < N ? at : N - 1;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int l0 = 4 * s + k2;
        const uint2 v = make_uint2(yT[(size_t)(l0 < planes ? l0 : 0) * (size_t)N + (size_t)pt], yT[(size_t)(l0 + 1 < planes ? l0 + 1 : 0) * (size_t)N + (size_t)pt]);
        yb[s] = *reinterpret_cast<const half4_t *>(&v);
    }
}

// The same value, which the compiler takes for another one: what is computed from it in a loop is computed there, and not before it and kept
// in registers (forty offsets and conditions of loads and stores).
__device__ __forceinline__ int anew(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Nothing is moved across: the scheduler hoists operand reads into earlier stages until the registers spill.
__device__ __forceinline__ void apart() { __builtin_amdgcn_sched_barrier(0); }

// H.yb holds the inputs on entry; op(i): operand i.  TIGHT: one tile of neurons after the other, with fewer registers at a time.
template <bool TIGHT = false, typename Op>
__device__ __forceinline__ void hidden_layers(Op op, const MlpDims d, Hidden &H) {
    // (the mask as a value of its own: else a itself is kept to the end, and compared there)
    auto mask = [](const acc16_t &a) { return TIGHT ? (uint32_t)anew((int)positive_mask(a)) : positive_mask(a); };
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        acc16_t a = mfma(op(kOpW1 / 2 + 2 * t), cat(H.yb[0], H.yb[1]), acc_zero());
        if (d.ks1 > 2) a = mfma(op(kOpW1 / 2 + 2 * t + 1), cat(H.yb[2], H.yb[3]), a);
        H.m1[t] = mask(a);
        relu_to_b(a, H.h1, t);
        if (TIGHT) apart();
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        acc16_t a = acc_zero();
#pragma unroll
        for (int s = 0; s < 4; ++s) a = mfma(op(kOpW2 / 2 + 4 * t + s), cat(H.h1[2 * s], H.h1[2 * s + 1]), a);
        H.m2[t] = mask(a);
        relu_to_b(a, H.h2, t);
        if (TIGHT) apart();
    }
}

// Transpose tile of a wavefront of the backward pass: one array [32 points][neurons, input dimensions or output channels] per operand of the products over
// the points, its rows padded by four halves (the 8-byte writes of 32 points then fall into different banks).  The three products use the tile
// one after the other, the first and the last the same part: h2 and dL/dout, then h1 and dL/dh2, then dL/dh1 and y.
constexpr int kMlpBwdBlock = 512;              // 8 wavefronts, two per SIMD
constexpr int kTile64 = 64 + 4, kTile32 = 32 + 4;                                  // halves per point
enum : int { kAtH2 = 0, kAtDo = 32 * kTile64, kAtD1 = 0, kAtY = 32 * kTile64,
             kAtH1 = 32 * (kTile64 + kTile32), kAtD2 = kAtH1 + 32 * kTile64, kTileHalves = kAtD2 + 32 * kTile64 };
constexpr size_t kMlpBwdOps = (size_t)kOpAllSlots * 64 * sizeof(half4_t);
constexpr size_t kMlpBwdLds = kMlpBwdOps + (size_t)(kMlpBwdBlock / 64) * kTileHalves * sizeof(_Float16);
constexpr size_t kMlpRawBytes = ((size_t)kMlpHidden * (kMlpMaxIn + kMlpHidden + kMlpMaxOut) * 2 + 15) & ~(size_t)15;
constexpr size_t kMlpFwdOps = (size_t)kOpFwdSlots * 64 * sizeof(half4_t);
constexpr size_t kMlpFwdLds = kMlpFwdOps + kMlpRawBytes;
constexpr int    kMlpAccs = 8;                 // weight-gradient tiles of 32 x 32
constexpr size_t kMlpAccBytes = (size_t)kMlpAccs * 16 * 64 * sizeof(float);        // one wavefront's
static_assert(kMlpBwdLds <= 160 * 1024, "LDS of a CU");
static_assert(kMlpRawBytes <= kMlpBwdLds - kMlpBwdOps, "raw weights share the tile region");
static_assert(kMlpBwdBlock / 64 / 2 * kMlpAccBytes <= kMlpBwdLds, "the reduction takes all of the LDS");

// ------------------------------------------------------------------ forward
// PLANES: y is the level-major array of fp16 pairs described at load_inputs_planes (IoT = __half, n_in even).
// Large batches are bound by memory (32 fp16 inputs, 3 or 4 outputs: 2^21 points 45 us for 160 MB), small ones by the launch and the
// staging of the weights.  The operands stay in registers and the next tile's inputs are used by nothing before the next tile (a selection or a
// conversion right behind the load waits for it); the bound of three wavefronts per SIMD also keeps the accumulators out of the
// accumulation registers, which the vector ALU cannot read.  us, before / now: 2^12 points 10.0 / 6.6, 2^18 14.5 / 10.0, 2^21 55 / 45; fp32
// inputs and 16 outputs 15 / 13, 29 / 26, 170 / 149.
template <typename IoT, bool PLANES = false>
__global__ __launch_bounds__(kMlpBlock, 3) void mlp_fwd_kernel(
    const MlpDims d, const IoT *__restrict__ y, const int64_t N, const __half *__restrict__ W,
    float *__restrict__ out, const int64_t tiles)
{
    auto fetch = [&](const int64_t tile, const int lane, QuadOf<IoT> (&yb)[4]) {
        if constexpr (PLANES) load_inputs_planes(d, reinterpret_cast<const uint32_t *>(y), tile, tiles, N, lane, yb);
        else load_inputs(d, y, tile, tiles, N, lane, yb);
    };
    extern __shared__ __align__(16) unsigned char smem[];
    half8_t *ops = reinterpret_cast<half8_t *>(smem);
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (kMlpBlock / 64);
    int64_t tile = (int64_t)blockIdx.x * (kMlpBlock / 64) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    QuadOf<IoT> next[4];
    fetch(tile, lane, next);                                    // on its way while the weights are staged
    stage_operands<kMlpBlock, false>(ops, reinterpret_cast<__half *>(smem + kMlpFwdOps), W, d);
    half8_t w[kOpFwdSlots / 2];                                 // the operands stay in registers: 64 of the 168 that three wavefronts per SIMD leave
#pragma unroll
    for (int i = 0; i < kOpFwdSlots / 2; ++i) w[i] = ops[i * 64 + lane];
    for (; tile < tiles; tile += waves) {
        Hidden H;
#pragma unroll
        for (int s = 0; s < 4; ++s) H.yb[s] = to_half4(next[s]);
        keep_columns(H.yb, d.n_in, lane);
        fetch(tile + waves, lane, next);                        // next tile, in flight during this one
        hidden_layers([&](const int i) { return w[i]; }, d, H);
        acc16_t o = acc_zero();
#pragma unroll
        for (int s = 0; s < 4; ++s) o = mfma(w[kOpW3 / 2 + s], cat(H.h2[2 * s], H.h2[2 * s + 1]), o);
        const TileRows<float> to = tile_rows(out, tile, tiles, N, d.n_out);
        float *row = to.base + (lane & 31) * d.n_out;
        if ((lane & 31) < to.rows) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {                       // rows 0 .. 15 of the tile are the outputs
                const int ch = 8 * q + 4 * (lane >> 5);
                if (d.vec_out) {
                    if (ch < d.n_out) store4(row + ch, o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]);
                } else if (8 * q < d.n_out) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (ch + j < d.n_out) row[ch + j] = o[4 * q + j];
                }
            }
        }
    }
}

// ------------------------------------------------------------------ encoding + decoder in one kernel (inference)
// The forward tile kernel of the encoding (cngp_kernels.h: 256 points per workgroup through all levels,
// the level's index codebook staged in LDS) with the decoder applied to the tile while it is still in LDS:
// the encoded features never go to memory.  y is kept as fp16, the value the decoder's matrix
// instructions would read from a stored y of either type, so the result equals the two separate calls.
// Row stride of the tile: 36 halves (the operand reads of 32 lanes then fall into different banks);
// columns from 2 L on are zero, which is what the K-steps beyond n_in need.
constexpr int kFusedTile = 256;
constexpr int kFusedStride = 36;

template <int D, typename FeatT, int FMT>
__global__ __launch_bounds__(kFusedTile) void encode_mlp_fwd_kernel(
    const Params p, const MlpDims d, const float *__restrict__ x, const FeatT *__restrict__ D_f,
    const uint8_t *__restrict__ D_c, const __half *__restrict__ W, float *__restrict__ out, const int64_t N,
    const int64_t tiles, const uint32_t c_stride, const int vec)
{
    extern __shared__ __align__(16) unsigned char smem[];
    half8_t  *ops = reinterpret_cast<half8_t *>(smem);
    _Float16 *ytile = reinterpret_cast<_Float16 *>(smem + kMlpFwdOps);                      // [kFusedTile][kFusedStride]
    unsigned char *rest = smem + kMlpFwdOps + (size_t)kFusedTile * kFusedStride * sizeof(_Float16);
    uint8_t  *probes = rest;                                 // the raw weights first, then each level's index codebook
    const uint32_t lds_c = (p.N_c + 1u) / 2u;
    stage_operands<kFusedTile, false>(ops, reinterpret_cast<__half *>(rest), W, d);
    const int t = threadIdx.x;
    for (int i = t; i < kFusedTile * kFusedStride; i += kFusedTile) ytile[i] = (_Float16)0.0f;
    const int lane = t & 63, k4 = 4 * (lane >> 5);

    // persistent: a workgroup stages the decoder's weights once and then walks over tiles of points
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t n0 = tile * kFusedTile;
        const int64_t n = n0 + t;
        const bool    valid = n < N;
        float xp[D];
#pragma unroll
        for (int j = 0; j < D; ++j) xp[j] = valid ? x[n * D + j] : 0.0f;

        for (int l = 0; l < p.L; ++l) {
            const uint8_t *C_l = D_c + (size_t)l * c_stride;
            __syncthreads();                                 // previous lookups, previous tile's decoder reads, the clearing above
            stage_probes<FMT, kFusedTile>(probes, C_l, c_stride, lds_c, vec, t);
            __syncthreads();
            Cell<D> cell;
            cell.locate(xp, p.N_l[l]);
            const FeatT *F_l = D_f + (size_t)l * p.N_f * 2;
            uint32_t idx[1 << D];
#pragma unroll
            for (int c = 0; c < (1 << D); ++c)
                idx[c] = probe_base(cell.hash1(c), p) +
                         (FMT == kFmtBits ? read_probe_bits_lds(probes, cell.hash2(c) & p.c_mask, p.log2_Np)
                                          : read_probe<kFmtPacked4>(probes, cell.hash2(c) & p.c_mask, p.log2_Np));
            float2 feat[1 << D];
#pragma unroll
            for (int c = 0; c < (1 << D); ++c) feat[c] = load_pair(F_l, idx[c]);
            float y0 = 0.0f, y1 = 0.0f;
#pragma unroll
            for (int c = 0; c < (1 << D); ++c) {
                const float wt = cell.weight(c);
                y0 = fmaf(wt, feat[c].x, y0);
                y1 = fmaf(wt, feat[c].y, y1);
            }
            ytile[t * kFusedStride + 2 * l] = (_Float16)y0;
            ytile[t * kFusedStride + 2 * l + 1] = (_Float16)y1;
        }
        wave_lds_fence();                                    // a wavefront decodes the rows it wrote itself

        // decoder: every wavefront takes its own 64 points as two tiles of 32
#pragma unroll 1
        for (int half = 0; half < 2; ++half) {
            const int row = (t & ~63) + 32 * half + (lane & 31);
            Hidden H;
#pragma unroll
            for (int s = 0; s < 4; ++s)
                H.yb[s] = *reinterpret_cast<const half4_t *>(ytile + row * kFusedStride + 8 * s + k4);
            hidden_layers([&](const int i) { return ops[i * 64 + lane]; }, d, H);
            acc16_t o = acc_zero();
#pragma unroll
            for (int s = 0; s < 4; ++s) o = mfma(ops[(kOpW3 / 2 + s) * 64 + lane], cat(H.h2[2 * s], H.h2[2 * s + 1]), o);
            const int64_t pt = n0 + row;
            if (pt < N) {
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const int ch = 8 * (r >> 2) + k4 + (r & 3);
                    if (ch < d.n_out) out[pt * d.n_out + ch] = o[r];
                }
            }
        }
    }
}

// ------------------------------------------------------------------ backward
// B-layout registers (lane = point, K-step s holds rows 8s + 4h .. + 3) written to the point's row of an array.
template <int STRIDE, int STEPS>
__device__ __forceinline__ void put_rows(_Float16 *to, const half4_t (&b)[STEPS], const int lane) {
    _Float16 *row = to + (lane & 31) * STRIDE + 4 * (lane >> 5);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) *reinterpret_cast<half4_t *>(row + 8 * s) = b[s];
}

// Operand whose K index runs over the 32 points: column 32u + lane % 32 of an array, points 16s + 8h .. + 7 (both operands of
// these products come from the tile, so the instruction's natural K order serves).  The transposing LDS read gives lane i of a group of 16
// column i of the 4 x 16 block whose row q the lanes 4q .. 4q + 3 name, four columns each: two of them are an operand, where an array kept by column
// took four 2-byte writes for each 8-byte one.
__device__ __forceinline__ half4_t read_transposed(const _Float16 *from) {
    typedef short short4_t __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) short4_t LdsShort4;
    return __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsShort4 *)from));
}
template <int STRIDE>
__device__ __forceinline__ half8_t get_op(const _Float16 *from, const int u, const int s, const int lane) {
    const int i = lane & 15;
    const _Float16 *q = from + (16 * s + 8 * (lane >> 5) + (i >> 2)) * STRIDE + 32 * u + (lane & 16) + 4 * (i & 3);
    return cat(read_transposed(q), read_transposed(q + 4 * STRIDE));
}

// One product over the 32 points of the tile: acc[t][u] += (columns 32 t .. of a) x (columns 32 u .. of b)^T.
template <int SA, int SB, int TA, int TB>
__device__ __forceinline__ void add_outer(const _Float16 *a_, const _Float16 *b_, const int lane, acc16_t (&acc)[TA][TB]) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        half8_t a[TA], b[TB];
#pragma unroll
        for (int t = 0; t < TA; ++t) a[t] = get_op<SA>(a_, t, s, lane);
#pragma unroll
        for (int u = 0; u < TB; ++u) b[u] = get_op<SB>(b_, u, s, lane);
#pragma unroll
        for (int t = 0; t < TA; ++t)
#pragma unroll
            for (int u = 0; u < TB; ++u) acc[t][u] = mfma(a[t], b[u], acc[t][u]);
    }
}

// Two wavefronts to a SIMD: one alone left every dependency stall exposed.  A wavefront's 128 registers of weight-gradient sums and
// what a tile needs fit the 256 that each then has, because a product is formed as soon as its operands are there and the masks are
// bits.  What bounds it: a tile's chain of matrix instructions, conversions and LDS transposes (2^21 points 190 us for 300 MB);
// below 2^16 points the launch, the staging of the weights and the sum over the wavefronts (19 us with the clearing of the gradient; that sum,
// one wavefront after the other, and a staging without loads in flight took 41).  us, before / now: n_in = 32, n_out = 3, fp16 2^12 points 41 / 19,
// 2^18 69 / 40, 2^21 340 / 190; operands kept by column and written two bytes at a time 44 at 2^18, 228 at 2^21.
template <typename IoT>
__global__ __launch_bounds__(kMlpBwdBlock) void mlp_bwd_kernel(
    const MlpDims d, const IoT *__restrict__ y, const int64_t N, const __half *__restrict__ W,
    const float *__restrict__ dout, IoT *__restrict__ dy, float *__restrict__ gW, const int64_t tiles)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int kWaves = kMlpBwdBlock / 64;
    half8_t  *ops = reinterpret_cast<half8_t *>(smem);
    _Float16 *tile = reinterpret_cast<_Float16 *>(smem + kMlpBwdOps) + (size_t)(threadIdx.x >> 6) * kTileHalves;
    const int lane = threadIdx.x & 63, k4 = 4 * (lane >> 5), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t waves = (int64_t)gridDim.x * kWaves;
    int64_t tl = (int64_t)blockIdx.x * kWaves + wave;
    QuadOf<IoT> next[4];
    float4    next_db[2];
    auto fetch = [&](const int64_t at, const int ln) {
        load_inputs(d, y, at, tiles, N, ln, next);
        load_quads(tile_rows(dout, at, tiles, N, d.n_out), ln, d.n_out, d.vec_out != 0, next_db, d.ks3);
    };
    next_db[1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    fetch(tl, lane);                                            // on its way while the weights are staged
    stage_operands<kMlpBwdBlock, true>(ops, reinterpret_cast<__half *>(smem + kMlpBwdOps), W, d);

    acc16_t gW1[2][1], gW2[2][2], gW3[1][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        gW1[t][0] = acc_zero(); gW3[0][t] = acc_zero();
        gW2[t][0] = acc_zero(); gW2[t][1] = acc_zero();
    }
    for (; tl < tiles; tl += waves) {
        Hidden H;
        half4_t db[2], dh2[8], dh1[8];
#pragma unroll
        for (int s = 0; s < 4; ++s) H.yb[s] = to_half4(next[s]);
#pragma unroll
        for (int s = 0; s < 2; ++s) db[s] = to_half4(next_db[s]);
        {
            const int ln = anew(lane), rows = tile_rows(dout, tl, tiles, N, d.n_out).rows;
            keep_columns(H.yb, d.n_in, ln);
            keep_columns(db, d.n_out, ln);
            keep_rows(H.yb, rows, ln);
            keep_rows(db, rows, ln);
        }
        hidden_layers<true>([&](const int i) { return ops[i * 64 + lane]; }, d, H);

        // The weight gradients contract over the points: their operands are transposed through the tile.  Each product follows as soon
        // as its operands are there, so that they need not be kept (two wavefronts to a SIMD leave 256 registers, half of them for the sums).
        apart();
        wave_lds_fence();                                       // the previous tile's operand reads are done
        put_rows<kTile64>(tile + kAtH2, H.h2, lane);
        put_rows<kTile32>(tile + kAtDo, db, lane);                    // (channels 16 .. 31: whatever is there; rows of gW3 that nobody reads)
#pragma unroll
        for (int t = 0; t < 2; ++t) {                           // dL/dh2 = W3^T dout, where h2 was active
            acc16_t g = acc_zero();
            g = mfma(ops[(kOpW3T / 2 + t) * 64 + lane], cat(db[0], db[1]), g);   // rows beyond n_out are zero in both operands
            mask_to_b(g, H.m2[t], dh2, t);
            apart();
        }
        put_rows<kTile64>(tile + kAtH1, H.h1, lane);
        put_rows<kTile64>(tile + kAtD2, dh2, lane);
        apart();
        wave_lds_fence();
        add_outer<kTile32, kTile64>(tile + kAtDo, tile + kAtH2, lane, gW3);       // [channel, hidden 32u..]
        apart();
        fetch(tl + waves, anew(lane));                          // next tile, in flight during the rest of this one
#pragma unroll
        for (int t = 0; t < 2; ++t) {                           // dL/dh1 = W2^T dL/dh2, where h1 was active
            acc16_t g = acc_zero();
#pragma unroll
            for (int s = 0; s < 4; ++s) g = mfma(ops[(kOpW2T / 2 + 4 * t + s) * 64 + lane], cat(dh2[2 * s], dh2[2 * s + 1]), g);
            mask_to_b(g, H.m1[t], dh1, t);
            apart();
        }
        wave_lds_fence();                                       // the reads of the first rows are done
        put_rows<kTile64>(tile + kAtD1, dh1, lane);
        put_rows<kTile32>(tile + kAtY, H.yb, lane);
        add_outer<kTile64, kTile64>(tile + kAtD2, tile + kAtH1, lane, gW2);       // [hidden 32t.., hidden 32u..]
        apart();
        {                                                       // dL/dy = W1^T dL/dh1
            acc16_t g = acc_zero();
#pragma unroll
            for (int s = 0; s < 4; ++s) g = mfma(ops[(kOpW1T / 2 + s) * 64 + lane], cat(dh1[2 * s], dh1[2 * s + 1]), g);
            const TileRows<IoT> to = tile_rows(dy, tl, tiles, N, d.n_in);
            const int ls = anew(lane), at = (ls & 31) * d.n_in;
            if ((ls & 31) < to.rows) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {                   // register group q: input dimensions 8q + 4h .. + 3
                    const int i = 8 * q + 4 * (ls >> 5);
                    if (d.vec_in && i < d.n_in) {
                        store4(to.base + at + i, g[4 * q], g[4 * q + 1], g[4 * q + 2], g[4 * q + 3]);
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (i + j < d.n_in) to.base[at + i + j] = from_float<IoT>(g[4 * q + j]);
                    }
                }
            }
        }
        apart();
        wave_lds_fence();
        add_outer<kTile64, kTile32>(tile + kAtD1, tile + kAtY, lane, gW1);        // [hidden 32t.., input dim]
        apart();
    }

    // Sum over the workgroup's wavefronts in LDS, of which nothing else is left: the upper half leaves its sums, the lower half adds its own,
    // then every lane adds the four up for a few entries, and one set of global atomics leaves.  Four
    // registers (q) of accumulator a, lane l: red[wave][(a * 4 + q) * 64 + l].
    float4 *red = reinterpret_cast<float4 *>(smem);
    constexpr int kAcc4 = kMlpAccs * 4 * 64;
    float4 *own = red + (size_t)(wave % (kWaves / 2)) * kAcc4 + lane;
    auto each = [&](auto put) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            put(t, gW1[t][0]);
            put(2 + t, gW3[0][t]);
            put(4 + 2 * t, gW2[t][0]);
            put(5 + 2 * t, gW2[t][1]);
        }
    };
    __syncthreads();
    if (wave >= kWaves / 2)
        each([&](const int a, const acc16_t &v) {
#pragma unroll
            for (int q = 0; q < 4; ++q) own[(a * 4 + q) * 64] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        });
    __syncthreads();
    if (wave < kWaves / 2)
        each([&](const int a, const acc16_t &v) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 o = own[(a * 4 + q) * 64];
                own[(a * 4 + q) * 64] = make_float4(o.x + v[4 * q], o.y + v[4 * q + 1], o.z + v[4 * q + 2], o.w + v[4 * q + 3]);
            }
        });
    __syncthreads();
    // lane = column, registers = rows 8 q + 4 h + 0 .. 3
    float *g1 = gW, *g2 = gW + kMlpHidden * d.n_in, *g3 = g2 + kMlpHidden * kMlpHidden;
    const int col = lane & 31;
#pragma unroll
    for (int i = 0; i < kAcc4 / kMlpBwdBlock; ++i) {
        const int group = i * kWaves + wave, a = group >> 2, row0 = 8 * (group & 3) + k4;       // the same a for a wavefront
        float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < kWaves / 2; ++w) {
            const float4 v = red[(size_t)w * kAcc4 + group * 64 + lane];
            sum[0] += v.x; sum[1] += v.y; sum[2] += v.z; sum[3] += v.w;
        }
        float *g;                                               // of row0
        int    stride;
        bool   in = true;
        if (a < 2) { g = g1 + (32 * a + row0) * d.n_in + col; stride = d.n_in; in = col < d.n_in; }
        else if (a < 4) { g = g3 + row0 * kMlpHidden + 32 * (a - 2) + col; stride = kMlpHidden; }
        else { g = g2 + (32 * ((a - 4) >> 1) + row0) * kMlpHidden + 32 * (a & 1) + col; stride = kMlpHidden; }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool here = in && (a < 2 || a >= 4 || row0 + j < d.n_out);
            if (here && sum[j] != 0.0f) atomic_add(g + j * stride, sum[j]);
        }
    }
}

}  // namespace cngp
