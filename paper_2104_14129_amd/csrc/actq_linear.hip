// Gradients of a linear layer from its output's gradient, its weight and its (dequantized) input, in one launch: the
// backward pass of a small activation-compressed layer (ActNN, Sec. 3.2, Eq. (4)).
//
//   grad_x [rows, inputs]    = grad_y [rows, outputs] . weight [outputs, inputs]
//   grad_w [outputs, inputs] = grad_y^T . x [rows, inputs]
//   grad_b [outputs]         = sum of grad_y over the rows
//
// What bounds it: a layer of this size is bound by the host, which spends 18 us on each product of the library and 5 on
// the sum, and the three kernels leave the chip partly idle one behind the other.  Here the tiles of both products are
// the workgroups of one grid, and the workgroups that own the first columns of grad_w add up grad_b from what they have loaded anyway.
// QLinear, 128 x 2048 -> 1000, forward and backward: 154 -> 109 us (binary32; host); the three kernels alone 26 -> 19 us there and
// 27 -> 8 in binary16.  A compute unit takes in some 25 GB/s of lines that are not in its cache, whatever the wavefronts that ask: few
// tiles with long sums are bound by that (grad_x of [16, 1024, 1024]: 16 workgroups, 12 us).
//
// A workgroup owns a tile of 32 x 64 and its four wavefronts split the sum over k, so that a product with few outputs
// still fills the chip and every wavefront has a short chain.  A lane loads its own operands from memory in the matrix
// instructions' layout, without the LDS: the right operands (weight, x) are [k, n] with n contiguous, and a lane that
// loads four neighbouring columns of a row serves four 16-column tiles whose columns are dealt modulo four (a lane's four
// results are then neighbours of an output row again).  The order of k inside a chunk is free as long as both
// operands have the same: lane group q takes rows q S .. q S + S - 1 of a chunk of 4 S (S = 4 in binary32, 8 in binary16).
// Tiles that reach past the last column are moved back to end with it and store what is theirs alone.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "actq_internal.h"

namespace actq {
namespace {

constexpr int kWave = 64;
constexpr int kLinWaves = 4;                      // share the sum over k of a tile [8, 16: alike or slower]
constexpr int kLinBlock = kLinWaves * kWave;
constexpr int kTileM = 32, kTileN = 64;           // of a workgroup
constexpr int kSubM = kTileM / 16, kSubN = kTileN / 16;

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Operand types: kSlots consecutive rows of k per lane, kStages chunks in flight.
template <typename T>
struct Operand;

template <>
struct Operand<float> {
    typedef f32x2 two;
    typedef f32x4 four;
    typedef f32x4 slots;
    static constexpr int kSlots = 4;
    static constexpr uint32_t kStages = 3;
};

template <>
struct Operand<_Float16> {
    typedef f16x2 two;
    typedef f16x4 four;
    typedef f16x8 slots;
    static constexpr int kSlots = 8;
    static constexpr uint32_t kStages = 4;
};

// The same vectors at the alignment of an element: global accesses of any width may start at any byte.
template <typename V, typename T>
__device__ __forceinline__ V load_unaligned(const T* p)
{
    typedef V __attribute__((aligned(sizeof(T)))) V_unaligned;
    return *reinterpret_cast<const V_unaligned*>(p);
}

// What a lane holds of a chunk, as loaded: its S values of k for each 16-row tile of the left operand (LEFT_K) or its S pairs of
// columns of it, and its S rows of the right one.
template <typename T, bool LEFT_K>
struct Fragment {
    typedef Operand<T> O;
    typename std::conditional<LEFT_K, typename O::slots, typename O::two>::type left[LEFT_K ? kSubM : O::kSlots];
    typename O::four right[O::kSlots];

    __device__ __forceinline__ typename O::slots a(int i) const
    {
        if constexpr (LEFT_K) {
            return left[i];
        } else {
            typename O::slots v;
#pragma unroll
            for (int s = 0; s < O::kSlots; ++s) v[s] = left[s][i];
            return v;
        }
    }
};

__device__ __forceinline__ void multiply(const f32x4 (&a)[kSubM], const f32x4 (&right)[4], f32x4 (&acc)[kSubM][kSubN])
{
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < kSubM; ++i)
#pragma unroll
            for (int j = 0; j < kSubN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][s], right[s][j], acc[i][j], 0, 0, 0);
}

__device__ __forceinline__ void multiply(const f16x8 (&a)[kSubM], const f16x4 (&right)[8], f32x4 (&acc)[kSubM][kSubN])
{
#pragma unroll
    for (int j = 0; j < kSubN; ++j) {
        f16x8 b;
#pragma unroll
        for (int s = 0; s < 8; ++s) b[s] = right[s][j];
#pragma unroll
        for (int i = 0; i < kSubM; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[i], b, acc[i][j], 0, 0, 0);
    }
}

struct TileLds {
    float plane[kLinWaves][kSubM][4][kSubN][kWave];
    double bias[kLinWaves][kTileM];
};

// One product [M, N] = left . right [K, N].  LEFT_K: the left operand is [M, K] (grad_y), otherwise [K, M] (grad_y as its transpose).
template <typename T>
struct Product {
    const T* left;
    const T* right;
    T* out;
    uint32_t M, N, K, lda;
};

// Tile (m0, n0); own_n: the first column that this tile stores (one that was moved back shares some with the tile before).
// bias: the sums of the left operand over k, or null.
template <typename T, bool LEFT_K>
__device__ __forceinline__ void product_tile(const Product<T>& p, uint32_t m0, uint32_t n0, uint32_t own_n, T* bias, TileLds& lds)
{
    constexpr int S = Operand<T>::kSlots;
    constexpr uint32_t kStages = Operand<T>::kStages;
    constexpr uint32_t kChunk = 4 * S;
    typedef typename Operand<T>::two two;
    typedef typename Operand<T>::four four;
    typedef typename Operand<T>::slots slots;
    typedef Fragment<T, LEFT_K> Piece;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));
    const uint32_t c = lane & 15, q = lane >> 4;

    // Where the lane reads, in bytes: of the left operand from the chunk's first column in the tile's first row (LEFT_K), or from
    // the chunk's first row; of the right one from the chunk's first row.  What it reads for rows past M it does not store.
    uint32_t left_at[kSubM], right_at;
    const uint32_t pair = m0 + kSubM * c;   // !LEFT_K: the lane's two columns, the last two if there are fewer
    const bool second = !LEFT_K && pair + 1 == p.M;   // of those, the second is the lane's first
#pragma unroll
    for (int i = 0; i < kSubM; ++i) {
        if (LEFT_K) {
            const uint32_t m = m0 + 16u * i + c;
            left_at[i] = ((m < p.M ? m : p.M - 1) - m0) * p.lda + q * S;
        } else {
            left_at[i] = q * S * p.lda + (pair + 1 < p.M ? pair : p.M - 2);
        }
        left_at[i] *= static_cast<uint32_t>(sizeof(T));
    }
    right_at = (q * S * p.N + n0 + 4 * c) * static_cast<uint32_t>(sizeof(T));
    const auto at_byte = [](const T* base, uint32_t bytes) { return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + bytes); };
    const auto load = [&](Piece& f, uint32_t k0) {   // a whole chunk
        if constexpr (LEFT_K) {
            const T* const base = p.left + static_cast<uint64_t>(m0) * p.lda + k0;
#pragma unroll
            for (int i = 0; i < kSubM; ++i) f.left[i] = load_unaligned<slots>(at_byte(base, left_at[i]));
        } else {
#pragma unroll
            for (int s = 0; s < S; ++s) f.left[s] = load_unaligned<two>(at_byte(p.left + static_cast<uint64_t>(k0 + s) * p.lda, left_at[0]));
        }
#pragma unroll
        for (int s = 0; s < S; ++s) f.right[s] = load_unaligned<four>(at_byte(p.right + static_cast<uint64_t>(k0 + s) * p.N, right_at));
    };
    const auto load_rest = [&](Piece& f, uint32_t k0) {   // the last, partial chunk: what lies past K counts as zero on both sides
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const uint32_t k = k0 + q * S + s, at = k < p.K ? k : p.K - 1;
            const bool live = k < p.K;
            if constexpr (LEFT_K) {
#pragma unroll
                for (int i = 0; i < kSubM; ++i) {
                    const T v = *at_byte(p.left + static_cast<uint64_t>(m0) * p.lda, left_at[i] + (at - q * S) * static_cast<uint32_t>(sizeof(T)));
                    f.left[i][s] = live ? v : T(0);
                }
            } else {
                const two v = load_unaligned<two>(at_byte(p.left, left_at[0] + (at - q * S) * p.lda * static_cast<uint32_t>(sizeof(T))));
                f.left[s] = live ? v : two{T(0), T(0)};
            }
            const four v = load_unaligned<four>(at_byte(p.right, right_at + (at - q * S) * p.N * static_cast<uint32_t>(sizeof(T))));
            f.right[s] = live ? v : four{T(0), T(0), T(0), T(0)};
        }
    };

    f32x4 acc[kSubM][kSubN];
    double sum[kSubM] = {0.0, 0.0};   // grad_b: in binary64 its error is that of the last rounding
#pragma unroll
    for (int i = 0; i < kSubM; ++i)
#pragma unroll
        for (int j = 0; j < kSubN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const auto use = [&](const Piece& f) {
        slots of[kSubM];
#pragma unroll
        for (int i = 0; i < kSubM; ++i) of[i] = f.a(i);
        if (!LEFT_K) {
            if (second) of[0] = of[1];
            if (bias != nullptr) {
#pragma unroll
                for (int i = 0; i < kSubM; ++i) {
#pragma unroll
                    for (int s = 0; s < S; ++s) sum[i] += static_cast<double>(of[i][s]);
                }
            }
        }
        multiply(of, f.right, acc);
    };

    // whole chunks wave, wave + 4, ..: kStages of them in flight
    const uint32_t whole = p.K / kChunk;
    const uint32_t mine = whole > wave ? (whole - wave + kLinWaves - 1) / kLinWaves : 0;
    const auto start_of = [&](uint32_t t) { return (wave + kLinWaves * t) * kChunk; };
    Piece ring[kStages];
    uint32_t t = 0;
#pragma unroll
    for (uint32_t s = 0; s < kStages; ++s)
        if (s < mine) load(ring[s], start_of(s));
    for (; t + 2 * kStages <= mine; t += kStages) {
#pragma unroll
        for (uint32_t s = 0; s < kStages; ++s) {
            use(ring[s]);
            load(ring[s], start_of(t + s + kStages));
        }
    }
#pragma unroll
    for (uint32_t s = 0; s < kStages; ++s) {
        if (t + s < mine) use(ring[s]);
        if (t + s + kStages < mine) load(ring[s], start_of(t + s + kStages));
    }
#pragma unroll
    for (uint32_t s = 0; s < kStages; ++s)
        if (t + s + kStages < mine) use(ring[s]);
    if (whole * kChunk != p.K && whole % kLinWaves == wave) {
        Piece f;
        load_rest(f, whole * kChunk);
        use(f);
    }

    // the wavefronts' sums meet in the LDS, a plane of 64 lanes per result; then a wavefront adds up one row of a lane's results at a time
#pragma unroll
    for (int i = 0; i < kSubM; ++i)
#pragma unroll
        for (int j = 0; j < kSubN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) lds.plane[wave][i][e][j][lane] = acc[i][j][e];
    if (!LEFT_K && bias != nullptr) {
#pragma unroll
        for (int i = 0; i < kSubM; ++i) {
            sum[i] += __shfl_xor(sum[i], 16);
            sum[i] += __shfl_xor(sum[i], 32);
            if (q == 0) lds.bias[wave][kSubM * c + i] = sum[i];
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t task = wave; task < 4 * kSubM; task += kLinWaves) {
        const uint32_t i = task >> 2, e = task & 3;
        const uint32_t in_tile = 4 * q + e;
        const uint32_t m = LEFT_K ? m0 + 16u * i + in_tile : m0 + kSubM * in_tile + i;
        float r[kSubN];
#pragma unroll
        for (int j = 0; j < kSubN; ++j) {
            float v[kLinWaves];
#pragma unroll
            for (int k = 0; k < kLinWaves; ++k) v[k] = lds.plane[k][i][e][j][lane];
#pragma unroll
            for (int step = 1; step < kLinWaves; step *= 2)
#pragma unroll
                for (int k = 0; k < kLinWaves; k += 2 * step) v[k] += v[k + step];
            r[j] = v[0];
        }
        if (m >= p.M) continue;
        T* const to = p.out + static_cast<uint64_t>(m) * p.N;
        const uint32_t n = n0 + 4 * c;
        if (n >= own_n) {
            four v;
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = static_cast<T>(r[j]);
            typedef four __attribute__((aligned(sizeof(T)))) four_unaligned;
            *reinterpret_cast<four_unaligned*>(to + n) = v;
        } else {
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j)
                if (n + j >= own_n) to[n + j] = static_cast<T>(r[j]);
        }
    }
    if (!LEFT_K && bias != nullptr && threadIdx.x < kTileM) {
        const uint32_t m = m0 + threadIdx.x;
        double total = 0.0;
#pragma unroll
        for (int k = 0; k < kLinWaves; ++k) total += lds.bias[k][threadIdx.x];
        if (m < p.M) bias[m] = static_cast<T>(total);   // by way of binary32, binary16 would be rounded twice
    }
}

struct LinearArgs {
    const void* grad_y;
    const void* weight;
    const void* x;
    void* grad_x;
    void* grad_w;
    void* grad_b;
    uint32_t rows, inputs, outputs;
    uint32_t blocks_x;              // the workgroups of grad_x come first, a multiple of eight
    uint32_t per_xcd_x, per_xcd_w;  // tiles of an XCD, grad_x and grad_w
    uint32_t tiles_x, tiles_w;
    FastDiv by_m_x, by_m_w;         // division by the tiles along the rows of the result
    uint32_t m_x, m_w;
};

// The tiles, column by column of tiles, are cut into eight ranges, one per XCD (workgroups go to the XCDs in turn), so that the
// tiles that share columns of the right operand share an L2.
template <typename T>
__global__ __launch_bounds__(kLinBlock) void linear_backward_kernel(LinearArgs a)
{
    __shared__ TileLds lds;
    const bool of_x = blockIdx.x < a.blocks_x;
    const uint32_t b = of_x ? blockIdx.x : blockIdx.x - a.blocks_x;
    const uint32_t tile = (b & 7u) * (of_x ? a.per_xcd_x : a.per_xcd_w) + (b >> 3);
    if (tile >= (of_x ? a.tiles_x : a.tiles_w)) return;
    const FastDiv by = of_x ? a.by_m_x : a.by_m_w;
    const uint32_t nt = (__umulhi(tile, by.m) + tile) >> by.s, mt = tile - nt * (of_x ? a.m_x : a.m_w);
    const uint32_t own_m = mt * kTileM, own_n = nt * kTileN;
    const uint32_t N = a.inputs;   // a tile at least
    const uint32_t n0 = own_n + kTileN > N ? N - kTileN : own_n;
    if (of_x) {
        const Product<T> p = {static_cast<const T*>(a.grad_y), static_cast<const T*>(a.weight), static_cast<T*>(a.grad_x), a.rows, N, a.outputs, a.outputs};
        product_tile<T, true>(p, own_m, n0, own_n, nullptr, lds);
    } else {
        const Product<T> p = {static_cast<const T*>(a.grad_y), static_cast<const T*>(a.x), static_cast<T*>(a.grad_w), a.outputs, N, a.rows, a.outputs};
        product_tile<T, false>(p, own_m, n0, own_n, nt == 0 ? static_cast<T*>(a.grad_b) : nullptr, lds);
    }
}

}  // namespace

int launch_linear_backward(const void* grad_y, const void* weight, const void* x, int dtype, int64_t rows, int64_t inputs, int64_t outputs,
                           void* grad_x, void* grad_w, void* grad_b, void* stream)
{
    LinearArgs a = {};
    a.grad_y = grad_y;
    a.weight = weight;
    a.x = x;
    a.grad_x = grad_x;
    a.grad_w = grad_w;
    a.grad_b = grad_b;
    a.rows = static_cast<uint32_t>(rows);
    a.inputs = static_cast<uint32_t>(inputs);
    a.outputs = static_cast<uint32_t>(outputs);
    const auto tiles = [](uint32_t extent, int tile) { return (extent + tile - 1) / tile; };
    const uint32_t n = tiles(a.inputs, kTileN);
    a.m_x = tiles(a.rows, kTileM);
    a.m_w = tiles(a.outputs, kTileM);
    a.by_m_x = make_fastdiv(a.m_x);
    a.by_m_w = make_fastdiv(a.m_w);
    a.tiles_x = grad_x ? a.m_x * n : 0;
    a.tiles_w = grad_w ? a.m_w * n : 0;
    a.per_xcd_x = (a.tiles_x + 7) / 8;
    a.per_xcd_w = (a.tiles_w + 7) / 8;
    a.blocks_x = 8 * a.per_xcd_x;
    const unsigned blocks = a.blocks_x + 8 * a.per_xcd_w;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (dtype == ACTQ_F32) launch(linear_backward_kernel<float>, blocks, kLinBlock, s, a);
    else launch(linear_backward_kernel<_Float16>, blocks, kLinBlock, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(ACTQ_EHIP, "actq_linear_backward: launch failed: %s", hipGetErrorString(e));
    return ACTQ_OK;
}

}  // namespace actq
