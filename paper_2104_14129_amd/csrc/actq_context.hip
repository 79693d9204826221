// HIP kernels of libactq for gfx950 (MI355X): the exact layer contexts of ActNN's appendix.
//
//   * ReLU ("Activation Layers"): the context is one bit per element, f'(x) = [x > 0].
//     Forward writes y = max(x, 0) and the bit stream; backward multiplies the incoming
//     gradient by the stored bit (as a selection, so a cleared bit always gives +0).
//   * Max pooling ("Pooling Layers"): the context is, per output location, the 8-bit
//     position of the maximum inside its window.  Backward gathers, for every input
//     location, the output gradients whose stored position points at it.
//
// Both are pure streaming kernels bound by HBM.  In ReLU the comparison masks
// come out of v_cmp as 64-bit wavefront masks, and a few lanes interleave them into the
// LSB-first stream, so the bits leave as one coalesced store per wavefront without LDS.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "actq_internal.h"

namespace actq {
namespace {

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;
constexpr int kBlock = kWave * kWavesPerBlock;

int launched(const char* who)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(ACTQ_EHIP, "%s: launch failed: %s", who, hipGetErrorString(e));
    return ACTQ_OK;
}

// ------------------------------------------------------------------------------------
// ReLU.  A lane owns E consecutive elements (E = 4 binary32 or 8 binary16 values: 128 bits); a wavefront
// covers 64*E elements = 2*E words of the bit stream, with one load and one store per lane.  What bounds it
// is the mixed stream of reads and writes (6.4 TB/s of the stem's 1.67 GB); short wavefronts and a bit stream
// that is written and read through the L2 serve it best: with four loads per lane and a non-temporal bit stream
// ReLU and 3x3 pooling, forward and backward, took 145 instead of 139 us on binary16 [64, 64, 113, 113]
// and 908 instead of 892 us on binary32 [256, 64, 112, 112] (one load 141 / 896, two 143 / 914).
template <typename T>
struct Lanes;

template <>
struct Lanes<float> {
    static constexpr int E = 4;
    typedef float vec __attribute__((ext_vector_type(4)));
};

template <>
struct Lanes<_Float16> {
    static constexpr int E = 8;
    typedef _Float16 vec __attribute__((ext_vector_type(8)));
};

// Moves bit t of `piece` (32 / E bits wide) to bit E * t.
template <int E>
__device__ __forceinline__ uint32_t spread(uint32_t piece)
{
    if (E == 4) {  // 8 bits -> every 4th bit
        uint32_t x = piece & 0xffu;
        x = (x | (x << 12)) & 0x000f000fu;
        x = (x | (x << 6)) & 0x03030303u;
        x = (x | (x << 3)) & 0x11111111u;
        return x;
    } else {  // 4 bits -> every 8th bit
        uint32_t x = piece & 0xfu;
        x = (x | (x << 14)) & 0x00030003u;
        x = (x | (x << 7)) & 0x01010101u;
        return x;
    }
}

// NT: non-temporal stores of y.
template <typename T, bool NT>
__global__ __launch_bounds__(kBlock) void relu_forward_kernel(const T* x, int64_t n, int64_t mask_words,
                                                              T* y, uint32_t* __restrict__ mask)
{
    constexpr int E = Lanes<T>::E;
    typedef typename Lanes<T>::vec vec;
    constexpr int kWords = 2 * E;                  // 64 * E bits
    constexpr int kLanesPerWord = 32 / E;          // lanes whose bits share one word
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t tile = (static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x) * kWavesPerBlock + (threadIdx.x >> 6);
    const int64_t first = tile * (kWave * E), mine = first + lane * E;
    if (first >= n) return;
    const bool full = first + kWave * E <= n;

    vec v;
    if (full) {
        v = __builtin_nontemporal_load(reinterpret_cast<const vec*>(x + mine));
    } else {
#pragma unroll
        for (int k = 0; k < E; ++k) v[k] = mine + k < n ? x[mine + k] : static_cast<T>(0.0f);  // past the end: bit 0, nothing stored
    }
    uint64_t m[E];   // lane l's bit says whether element k of lane l is positive
    vec out;
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const bool positive = static_cast<float>(v[k]) > 0.0f;
        m[k] = __ballot(positive);
        out[k] = positive ? v[k] : static_cast<T>(0.0f);
    }
    if (full) {
        if (NT) __builtin_nontemporal_store(out, reinterpret_cast<vec*>(y + mine));
        else *reinterpret_cast<vec*>(y + mine) = out;
    } else {
#pragma unroll
        for (int k = 0; k < E; ++k)
            if (mine + k < n) y[mine + k] = out[k];
    }

    // Word j of the tile's stream (j = lane) holds the bits of kLanesPerWord lanes: stream bit E*l + k is bit l of m[k].
    uint32_t word = 0;
#pragma unroll
    for (int k = 0; k < E; ++k) word |= spread<E>(static_cast<uint32_t>(m[k] >> (lane % kWords * kLanesPerWord))) << k;
    const int64_t w = tile * kWords + lane;
    if (lane < kWords && w < mask_words) mask[w] = word;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void relu_backward_kernel(const uint32_t* __restrict__ mask, int64_t mask_words,
                                                               const T* grad_y, int64_t n, T* grad_x)
{
    constexpr int E = Lanes<T>::E;
    typedef typename Lanes<T>::vec vec;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t tile = (static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x) * kWavesPerBlock + (threadIdx.x >> 6);
    const int64_t first = tile * (kWave * E), mine = first + lane * E;
    if (first >= n) return;
    const bool full = first + kWave * E <= n;

    // the lane's E bits start at bit E*lane of the tile's 64*E-bit stretch
    const int64_t w = tile * (2 * E) + (lane * E >> 5);
    const uint32_t word = mask[w < mask_words ? w : mask_words - 1];  // past the end: any word, its elements are not stored
    vec g;
    if (full) {
        g = __builtin_nontemporal_load(reinterpret_cast<const vec*>(grad_y + mine));
    } else {
#pragma unroll
        for (int k = 0; k < E; ++k) g[k] = mine + k < n ? grad_y[mine + k] : static_cast<T>(0.0f);
    }
    const uint32_t bits = word >> ((lane * E) & 31);
    vec out;
#pragma unroll
    for (int k = 0; k < E; ++k) out[k] = (bits >> k) & 1u ? g[k] : static_cast<T>(0.0f);
    if (full) {
        __builtin_nontemporal_store(out, reinterpret_cast<vec*>(grad_x + mine));
    } else {
#pragma unroll
        for (int k = 0; k < E; ++k)
            if (mine + k < n) grad_x[mine + k] = out[k];
    }
}

// ------------------------------------------------------------------------------------
// Max pooling.

// n / d with the host-computed constants of FastDiv (see actq_internal.h)
__device__ __forceinline__ uint32_t fastdiv(uint32_t n, FastDiv f) { return (__umulhi(n, f.m) + n) >> f.s; }

struct Pool {
    int32_t H, W, OH, OW;
    int32_t kh, kw, sh, sw, ph, pw, dh, dw;
    FastDiv by_OW, by_W, by_sh, by_sw, by_dh, by_dw;
    uint32_t grid_y;  // planes are spread over blockIdx.y and blockIdx.z
};

// One thread per output location; blockIdx.x runs over the locations of one plane, so
// consecutive lanes walk along the rows of the output.  The window is scanned row by row and
// only a strictly larger value replaces the running maximum, so among equal values the first
// position wins; padded positions are skipped.  KH = KW = 0 takes the window size at run time.
template <typename T, int KH, int KW>
__global__ __launch_bounds__(kBlock) void maxpool2d_forward_kernel(const T* __restrict__ x, int64_t planes, Pool g,
                                                                   T* __restrict__ y, uint8_t* __restrict__ argmax)
{
    const int64_t plane = static_cast<int64_t>(blockIdx.z) * g.grid_y + blockIdx.y;
    const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
    if (plane >= planes || idx >= static_cast<uint32_t>(g.OH * g.OW)) return;
    const int32_t i = static_cast<int32_t>(fastdiv(idx, g.by_OW));
    const int32_t j = static_cast<int32_t>(idx) - i * g.OW;
    const T* xp = x + plane * g.H * g.W;
    const int32_t r0 = g.sh * i - g.ph, c0 = g.sw * j - g.pw;
    const int32_t kh = KH ? KH : g.kh, kw = KW ? KW : g.kw;
    bool have = false;
    float best = 0.0f;
    int32_t best_k = 0;
    if (KH) {
        // fixed window: every load is issued up front from a clamped address, then the scan
        float v[KH ? KH : 1][KW ? KW : 1];
        bool ok[KH ? KH : 1][KW ? KW : 1];
#pragma unroll
        for (int32_t a = 0; a < KH; ++a)
#pragma unroll
            for (int32_t b = 0; b < KW; ++b) {
                const int32_t r = r0 + g.dh * a, c = c0 + g.dw * b;
                ok[a][b] = r >= 0 && r < g.H && c >= 0 && c < g.W;
                const int32_t rc = min(max(r, 0), g.H - 1), cc = min(max(c, 0), g.W - 1);
                v[a][b] = static_cast<float>(xp[rc * g.W + cc]);
            }
#pragma unroll
        for (int32_t a = 0; a < KH; ++a)
#pragma unroll
            for (int32_t b = 0; b < KW; ++b) {
                const bool take = ok[a][b] && (!have || v[a][b] > best);
                best = take ? v[a][b] : best;
                best_k = take ? a * KW + b : best_k;
                have = have || ok[a][b];
            }
    } else {
        for (int32_t a = 0; a < kh; ++a) {
            const int32_t r = r0 + g.dh * a;
            if (r < 0 || r >= g.H) continue;
            for (int32_t b = 0; b < kw; ++b) {
                const int32_t c = c0 + g.dw * b;
                if (c < 0 || c >= g.W) continue;
                const float v = static_cast<float>(xp[r * g.W + c]);
                if (!have || v > best) {
                    have = true;
                    best = v;
                    best_k = a * kw + b;
                }
            }
        }
    }
    const int64_t o = plane * g.OH * g.OW + idx;
    y[o] = static_cast<T>(best);  // exact: `best` is one of the inputs
    argmax[o] = static_cast<uint8_t>(best_k);
}

// One thread per input location.  The outputs whose window contains it are visited row by row
// (ascending output row, then column) and those whose stored position points here are added
// in binary32, the order in which a scatter over the outputs would have added them.
// MC > 0: at most MC output rows (and MC output columns) have a window that contains a given
// input location, i.e. ceil((d*(k-1)+1) / s) <= MC in both directions; the candidates are then
// enumerated directly and all their loads are issued up front from clamped addresses.
// MC = 0: any geometry, window positions scanned one by one.
template <typename T, int MC>
__global__ __launch_bounds__(kBlock) void maxpool2d_backward_kernel(const uint8_t* __restrict__ argmax,
                                                                    const T* __restrict__ grad_y, int64_t planes,
                                                                    Pool g, T* __restrict__ grad_x)
{
    const int64_t plane = static_cast<int64_t>(blockIdx.z) * g.grid_y + blockIdx.y;
    const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
    if (plane >= planes || idx >= static_cast<uint32_t>(g.H * g.W)) return;
    const int32_t r = static_cast<int32_t>(fastdiv(idx, g.by_W));
    const int32_t c = static_cast<int32_t>(idx) - r * g.W;
    const uint8_t* ap = argmax + plane * g.OH * g.OW;
    const T* gp = grad_y + plane * g.OH * g.OW;
    float acc = 0.0f;
    if (MC) {
        // output rows i with 0 <= r + ph - sh*i <= dh*(kh-1), the offset a multiple of dh
        const int32_t i_hi = static_cast<int32_t>(fastdiv(static_cast<uint32_t>(r + g.ph), g.by_sh));
        const int32_t j_hi = static_cast<int32_t>(fastdiv(static_cast<uint32_t>(c + g.pw), g.by_sw));
        uint32_t code[MC ? MC : 1][MC ? MC : 1];
        float gy[MC ? MC : 1][MC ? MC : 1];
        int32_t want[MC ? MC : 1][MC ? MC : 1];
#pragma unroll
        for (int32_t u = MC - 1; u >= 0; --u)
#pragma unroll
            for (int32_t v = MC - 1; v >= 0; --v) {
                const int32_t i = i_hi - u, j = j_hi - v;
                const int32_t off_r = r + g.ph - g.sh * i, off_c = c + g.pw - g.sw * j;  // >= 0
                const int32_t a = static_cast<int32_t>(fastdiv(static_cast<uint32_t>(off_r), g.by_dh));
                const int32_t b = static_cast<int32_t>(fastdiv(static_cast<uint32_t>(off_c), g.by_dw));
                const bool ok = i >= 0 && j >= 0 && i < g.OH && j < g.OW && a < g.kh && b < g.kw &&
                                a * g.dh == off_r && b * g.dw == off_c;
                const int32_t ic = min(max(i, 0), g.OH - 1), jc = min(max(j, 0), g.OW - 1);
                code[u][v] = ap[ic * g.OW + jc];
                gy[u][v] = static_cast<float>(gp[ic * g.OW + jc]);
                want[u][v] = ok ? a * g.kw + b : -1;
            }
        // ascending output row, then column
#pragma unroll
        for (int32_t u = MC - 1; u >= 0; --u)
#pragma unroll
            for (int32_t v = MC - 1; v >= 0; --v)
                acc += static_cast<int32_t>(code[u][v]) == want[u][v] ? gy[u][v] : 0.0f;  // + 0 changes nothing
    } else {
        for (int32_t a = g.kh - 1; a >= 0; --a) {  // descending window row = ascending output row
            const int32_t tr = r + g.ph - g.dh * a;
            if (tr < 0) continue;
            const int32_t i = static_cast<int32_t>(fastdiv(static_cast<uint32_t>(tr), g.by_sh));
            if (i * g.sh != tr || i >= g.OH) continue;
            for (int32_t b = g.kw - 1; b >= 0; --b) {
                const int32_t tc = c + g.pw - g.dw * b;
                if (tc < 0) continue;
                const int32_t j = static_cast<int32_t>(fastdiv(static_cast<uint32_t>(tc), g.by_sw));
                if (j * g.sw != tc || j >= g.OW) continue;
                if (ap[i * g.OW + j] == static_cast<uint8_t>(a * g.kw + b)) acc += static_cast<float>(gp[i * g.OW + j]);
            }
        }
    }
    grad_x[plane * g.H * g.W + idx] = static_cast<T>(acc);
}

// ------------------------------------------------------------------------------------
// Backward path for square windows K in {2, 3}, stride S in {1, 2}, dilation 1 with the paddings that the row kernels
// further down do not serve (2x2 / 1, 2x2 / 2 with padding, 3x3 / 1 without, padding along one axis).  With one element per lane the kernel above is bound by
// instruction issue, not by HBM (a wavefront that produces 256 bytes can afford only about two
// dozen vector instructions), so here a lane produces four consecutive elements of a row: the
// index arithmetic, the row checks and the loads of the neighbouring outputs are shared, and
// the result leaves as one 128-bit (binary16: 64-bit) store.  The arithmetic and its order are
// those of the kernel above.

template <typename T>
struct Quad;
template <>
struct Quad<float> {
    typedef float vec __attribute__((ext_vector_type(4)));
};
template <>
struct Quad<_Float16> {
    typedef _Float16 vec __attribute__((ext_vector_type(4)));
};

struct QuadGeometry {
    int32_t quads_per_row;  // ceil(row length / 4) of the tensor the kernel produces
    FastDiv by_quads;
    uint32_t vector_ok;     // rows are a multiple of 4 long and the outputs are aligned for vector stores
};

template <typename T, int K, int S>
__global__ __launch_bounds__(kBlock) void maxpool2d_backward_quad_kernel(const uint8_t* __restrict__ argmax,
                                                                         const T* __restrict__ grad_y, int64_t planes,
                                                                         Pool g, QuadGeometry q, T* __restrict__ grad_x)
{
    constexpr int LOG_S = S == 2 ? 1 : 0;
    constexpr int MR = (K - 1) / S + 1;      // output rows whose window can contain one input row
    constexpr int NJ = (S + K + 1) / S + 1;  // output columns whose window can contain one of four input columns
    const int64_t plane = static_cast<int64_t>(blockIdx.z) * g.grid_y + blockIdx.y;
    const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
    if (plane >= planes || idx >= static_cast<uint32_t>(g.H * q.quads_per_row)) return;
    const int32_t r = static_cast<int32_t>(fastdiv(idx, q.by_quads));
    const int32_t c0 = (static_cast<int32_t>(idx) - r * q.quads_per_row) * 4;
    const uint8_t* ap = argmax + plane * g.OH * g.OW;
    const T* gp = grad_y + plane * g.OH * g.OW;
    // c0 is a multiple of 4 and S divides 4, so the position of column c0 + e inside the window
    // of output column j_lo + t is the same for every lane: b = spare + (K - 1) + e - S*t
    const int32_t spare = S == 2 ? ((g.pw - (K - 1)) & 1) : 0;  // (c0 + pw - (K-1)) mod S
    const int32_t j_lo = (c0 + g.pw - (K - 1) - spare) >> LOG_S;  // exact; arithmetic shift for negative values
    const int32_t i_hi = (r + g.ph) >> LOG_S;
    uint32_t code[MR][NJ];
    float gy[MR][NJ];
    int32_t row_code[MR];                    // a * K for the row, or a value no stored position can match
#pragma unroll
    for (int u = 0; u < MR; ++u) {
        const int32_t i = i_hi - u;
        const int32_t a = r + g.ph - S * i;  // >= 0
        const bool row_ok = i >= 0 && i < g.OH && a < K;
        row_code[u] = row_ok ? a * K : -1000;
        const int32_t ic = min(max(i, 0), g.OH - 1);
#pragma unroll
        for (int t = 0; t < NJ; ++t) {
            const int32_t j = j_lo + t;
            const int32_t jc = min(max(j, 0), g.OW - 1);
            const bool ok = j >= 0 && j < g.OW;
            code[u][t] = ok ? static_cast<uint32_t>(ap[ic * g.OW + jc]) : 0xffffu;
            gy[u][t] = static_cast<float>(gp[ic * g.OW + jc]);
        }
    }
    typename Quad<T>::vec out;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float acc = 0.0f;
#pragma unroll
        for (int u = MR - 1; u >= 0; --u)    // ascending output row
#pragma unroll
            for (int t = 0; t < NJ; ++t) {   // ascending output column
                const int32_t b = spare + (K - 1) + e - S * t;  // the same in every lane
                if (b < 0 || b >= K) continue;
                acc += static_cast<int32_t>(code[u][t]) == row_code[u] + b ? gy[u][t] : 0.0f;  // + 0 changes nothing
            }
        out[e] = static_cast<T>(acc);
    }
    const int64_t o = plane * g.H * g.W + r * g.W + c0;
    if (q.vector_ok) {
        __builtin_nontemporal_store(out, reinterpret_cast<typename Quad<T>::vec*>(grad_x + o));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c0 + e < g.W) grad_x[o + e] = out[e];
    }
}

// ------------------------------------------------------------------------------------
// Pools of any extent with the windows networks use: stride 2 with K = 3 (padding 0 or 1) or K = 2
// (padding 0), and stride 1 with K = 3 and padding 1; dilation 1, rows of any length and alignment.
// What bounds these kernels is memory (input once, output and positions once); one element per lane
// costs three to five times that in address cycles (the texture addresser takes a wavefront's 64
// addresses in 16 clocks whatever the width of the load).  So a lane owns 16 bytes of an input row (E
// columns, from column E c; at the alignment of an element, rows of odd length start anywhere) and the
// NO = E / S output columns that lie over them.  The lanes run over (plane, row, c) flattened, so the
// neighbouring lanes hold the columns to the left and right, and the one column that a window needs
// from there comes by a wavefront shift; the wavefront's edge lane takes it through the scalar data path.
// Columns past the end of a row are read (they belong to the next row) and ignored; the wavefront that
// would read past the tensor's end goes element by element.
// Against one output (forward) and four inputs (backward) per lane, over a few tensors in turn: 3x3 / 2 / 1 on binary16
// [4096, 113, 113] 74 -> 29 us forward and 122 -> 31 us backward, binary32 87 -> 47 and 150 -> 49 us.
struct RowPool {
    uint32_t chunks;              // lanes per row
    FastDiv by_chunks, by_rows;   // by_rows: division by the rows (forward: output rows; backward: stretches of S input rows) of a plane
    uint32_t rows;
    uint32_t total;               // lanes in all
    int64_t elems;                // elements of the tensor that is read
};

// Where a lane of a row kernel is, for its BRIEF form: the workgroup's first lane is located by the scalar unit, and a lane counts rows and
// elements from there in 32 bits (a plane has fewer than 2^31 elements, and a workgroup reaches little further than one).  64-bit element
// numbers of its own cost every lane two dozen multiplications, which the vector ALU takes four times as long for as for additions.
struct RowLane {
    uint32_t plane0, strip0, row0;   // of the workgroup's first lane: its plane, its row over all planes and inside its plane (scalars)
    uint32_t at, c;                  // lanes from the start of row strip0; the lane's stretch of its row
    uint32_t down, planes;           // rows and planes below those of the workgroup's first lane
    int32_t row;                     // inside the lane's plane
    bool live;
};

__device__ __forceinline__ RowLane row_lane(uint32_t total, uint32_t chunks, FastDiv by_chunks, uint32_t rows, FastDiv by_rows)
{
    RowLane l;
    const uint32_t first = blockIdx.x * kBlock;
    l.strip0 = fastdiv(first, by_chunks);
    const uint32_t c0 = first - l.strip0 * chunks;
    l.plane0 = fastdiv(l.strip0, by_rows);
    l.row0 = l.strip0 - l.plane0 * rows;
    const uint32_t last = total - 1 - first;   // every lane takes part in the shifts: those past the end as the last one
    l.live = threadIdx.x <= last;
    l.at = c0 + (l.live ? threadIdx.x : last);
    l.down = fastdiv(l.at, by_chunks);
    l.c = l.at - __umul24(l.down, chunks);     // at most 256 rows; W is below 2^22
    const uint32_t below = l.row0 + l.down;
    l.planes = fastdiv(below, by_rows);
    l.row = static_cast<int32_t>(below - l.planes * rows);
    return l;
}

// Row `row` of the lane's plane as a row of the planes from plane0 on, where a plane has `height` rows for `rows` rows times `scale` of
// the lanes' (the difference is a few rows either way, so that 24 bits hold it).
__device__ __forceinline__ uint32_t row_from_plane0(const RowLane& l, uint32_t scale, int32_t height, uint32_t rows)
{
    return scale * (l.row0 + l.down) + static_cast<uint32_t>(__mul24(static_cast<int>(l.planes), height - static_cast<int32_t>(scale * rows)));
}

__device__ __forceinline__ uint32_t elements_up_to_32_bits(int64_t elems) { return elems > 0xffffffffll ? 0xffffffffu : static_cast<uint32_t>(elems); }

// Stretches of E elements and of NO elements and positions.
template <typename T, int S>
struct RowVec;
template <>
struct RowVec<float, 1> {
    typedef float in __attribute__((ext_vector_type(4), aligned(4)));
    typedef in out;
    typedef uint32_t codes __attribute__((aligned(1)));
};
template <>
struct RowVec<float, 2> {
    typedef float in __attribute__((ext_vector_type(4), aligned(4)));
    typedef float out __attribute__((ext_vector_type(2), aligned(4)));
    typedef uint16_t codes __attribute__((aligned(1)));
};
template <>
struct RowVec<_Float16, 1> {
    typedef _Float16 in __attribute__((ext_vector_type(8), aligned(2)));
    typedef in out;
    typedef uint64_t codes __attribute__((aligned(1)));
};
template <>
struct RowVec<_Float16, 2> {
    typedef _Float16 in __attribute__((ext_vector_type(8), aligned(2)));
    typedef _Float16 out __attribute__((ext_vector_type(4), aligned(2)));
    typedef uint32_t codes __attribute__((aligned(1)));
};

template <typename V>
__device__ __forceinline__ V load_uniform(const V* p)
{
    typedef const V __attribute__((address_space(4))) * constant_ptr;
    return *(constant_ptr)(reinterpret_cast<uintptr_t>(p));
}

// One element at a wavefront-uniform address, as (part of) the aligned 32-bit word around it.
template <typename V>
__device__ __forceinline__ V load_uniform_element(const V* p)
{
    const uintptr_t at = reinterpret_cast<uintptr_t>(p);
    const uint32_t word = load_uniform(reinterpret_cast<const uint32_t*>(at & ~uintptr_t(3))) >> (8 * static_cast<uint32_t>(at & 3u));
    V v;
    __builtin_memcpy(&v, &word, sizeof(V));
    return v;
}

// A word from the lane to the left / right; the wavefront's edge lane keeps garbage.
__device__ __forceinline__ uint32_t from_lane(uint32_t w, bool left)
{
    constexpr int kWaveShiftRight1 = 0x138, kWaveShiftLeft1 = 0x130;
    return static_cast<uint32_t>(left ? __builtin_amdgcn_update_dpp(0, static_cast<int>(w), kWaveShiftRight1, 0xf, 0xf, false)
                                      : __builtin_amdgcn_update_dpp(0, static_cast<int>(w), kWaveShiftLeft1, 0xf, 0xf, false));
}

__device__ __forceinline__ int64_t read_lane_i64(int64_t v, int lane)
{
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint64_t>(v) & 0xffffffffu), lane));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint64_t>(v) >> 32), lane));
    return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
}

// What a word of memory becomes in the kernels: positions are words as they are, gradients binary32 patterns.
struct PositionWord {
    typedef uint8_t memory;
    static __device__ __forceinline__ uint32_t of(uint8_t v) { return v; }
};
template <typename T>
struct GradientWord {
    typedef T memory;
    static __device__ __forceinline__ uint32_t of(T v) { return __float_as_uint(static_cast<float>(v)); }
};

// The aligned 32-bit word around an element that the wavefront's edge lane needs of its neighbour, and where the element is in it.
struct Edge {
    uint32_t word, shift;
};

// Of element `at` of p (a scalar) if the edge lane (LEFT: the first) has a neighbour to that side (`inside`), of element 0 otherwise.
template <bool LEFT, typename M>
__device__ __forceinline__ Edge edge_element(const M* p, uint32_t at, bool inside)
{
    constexpr int kEdge = LEFT ? 0 : kWave - 1;
    const uint32_t edge_at = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(at), kEdge));
    const uintptr_t address = reinterpret_cast<uintptr_t>(p + (__builtin_amdgcn_readlane(static_cast<int>(inside), kEdge) != 0 ? edge_at : 0u));
    return {load_uniform(reinterpret_cast<const uint32_t*>(address & ~uintptr_t(3))), 8 * static_cast<uint32_t>(address & 3u)};
}

// The word `own` of the lane to the left (LEFT) or right; the edge lane's is made of `edge`.
template <bool LEFT, typename WORD, typename V>
__device__ __forceinline__ V neighbour(V own, const Edge& edge)
{
    const uint32_t bits = edge.word >> edge.shift;
    typename WORD::memory element;
    __builtin_memcpy(&element, &bits, sizeof(element));
    const V from_edge = WORD::of(element), shifted = static_cast<V>(from_lane(own, LEFT));
    return (threadIdx.x & (kWave - 1)) == (LEFT ? 0 : kWave - 1) ? from_edge : shifted;
}

// The same with the element asked for here, behind a branch: a trip to memory of its own, but the forms that ask in front of their loads or without a
// branch are up to 5 % slower at stride 2 (binary16 [16384, 112, 112] forward 93 -> 98 us, binary32 3x3 / 2 / 0 backward 163 -> 170).
template <bool LEFT, typename WORD, typename V, typename M, typename I>
__device__ __forceinline__ V neighbour(V own, bool inside, const M* p, I at)
{
    constexpr int kEdge = LEFT ? 0 : kWave - 1;
    V from_edge = 0;
    if constexpr (sizeof(I) == 8) {
        const int64_t edge_at = read_lane_i64(at, kEdge);
        if (__builtin_amdgcn_readlane(static_cast<int>(inside), kEdge) != 0) from_edge = WORD::of(load_uniform_element(p + edge_at));
        const V shifted = static_cast<V>(from_lane(own, LEFT));
        return (threadIdx.x & (kWave - 1)) == kEdge ? from_edge : shifted;
    } else {
        Edge edge = {0, 0};
        if (__builtin_amdgcn_readlane(static_cast<int>(inside), kEdge) != 0) edge = edge_element<LEFT>(p, at, true);
        return neighbour<LEFT, WORD>(own, edge);
    }
}

// The first `count` (1 .. N - 1) of N values or positions, as pieces of 4, 2 and 1: at most three stores.
template <int N, typename T, typename V>
__device__ __forceinline__ void store_first(T* dst, V v, int count)
{
    typedef T pair __attribute__((ext_vector_type(2), aligned(sizeof(T))));
    typedef T quad __attribute__((ext_vector_type(4), aligned(sizeof(T))));
    T t0 = v[0], t1 = v[1];
    if constexpr (N == 8) {
        if (count & 4) {
            quad w;
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = v[k];
            *reinterpret_cast<quad*>(dst) = w;
            dst += 4;
        }
        t0 = count & 4 ? v[4] : t0;
        t1 = count & 4 ? v[5] : t1;
    }
    T last = t0;
    if constexpr (N >= 4) {
        if (count & 2) {
            pair w;
            w[0] = t0;
            w[1] = t1;
            *reinterpret_cast<pair*>(dst) = w;
            dst += 2;
        }
        const T second = N == 8 && (count & 4) ? v[N == 8 ? 6 : 2] : v[2];
        last = count & 2 ? second : t0;
    }
    if (count & 1) *dst = last;
}

__device__ __forceinline__ void store_first_codes(uint8_t* dst, uint64_t codes, int count)
{
    typedef uint32_t word __attribute__((aligned(1)));
    typedef uint16_t half __attribute__((aligned(1)));
    if (count & 4) {
        *reinterpret_cast<word*>(dst) = static_cast<uint32_t>(codes);
        dst += 4;
        codes >>= 32;
    }
    if (count & 2) {
        *reinterpret_cast<half*>(dst) = static_cast<uint16_t>(codes);
        dst += 2;
        codes >>= 16;
    }
    if (count & 1) *dst = static_cast<uint8_t>(codes);
}

// How the forward kernel carries a value: as its bit pattern (a selection of floating-point values by their
// comparison becomes a maximum instruction, which returns +0 where the first of two zeros is -0).
// Binary16 at stride 2 is widened to binary32 first: every value is compared twice or more, and a
// comparison of halves has to extract them (32 -> 29 us at 3x3 / 2 / 1 on [4096, 113, 113]); at stride 1 the
// registers of three widened rows cost more (70 -> 85 us).
template <typename T, int S>
struct Carrier;
template <int S>
struct Carrier<float, S> {
    typedef uint32_t raw;
    typedef raw memory;
    typedef uint32_t type;
    static __device__ __forceinline__ type of(raw u) { return u; }
    static __device__ __forceinline__ float value(type u) { return __uint_as_float(u); }
    static __device__ __forceinline__ raw back(type u) { return u; }
};
template <>
struct Carrier<_Float16, 1> {
    typedef uint16_t raw;
    typedef raw memory;
    typedef uint16_t type;
    static __device__ __forceinline__ type of(raw u) { return u; }
    static __device__ __forceinline__ _Float16 value(type u)
    {
        _Float16 h;
        __builtin_memcpy(&h, &u, 2);
        return h;
    }
    static __device__ __forceinline__ raw back(type u) { return u; }
};
template <>
struct Carrier<_Float16, 2> {
    typedef uint16_t raw;
    typedef raw memory;
    typedef uint32_t type;
    static __device__ __forceinline__ type of(raw u)
    {
        uint32_t w = __float_as_uint(static_cast<float>(Carrier<_Float16, 1>::value(u)));   // exact
        asm("" : "+v"(w));   // a pattern, not a value, to the compiler
        return w;
    }
    static __device__ __forceinline__ float value(type u) { return __uint_as_float(u); }
    static __device__ __forceinline__ raw back(type u)
    {
        asm("" : "+v"(u));
        const _Float16 h = static_cast<_Float16>(__uint_as_float(u));
        raw r;
        __builtin_memcpy(&r, &h, 2);
        return r;
    }
};

// Forward.  Rows and columns outside the image read as the nearest ones inside (their addresses are
// clamped).  A copy to the right of or below its original never wins, because only a larger value
// replaces the running maximum; one to the left or above wins in its original's place, and the
// position moves to the original (which is the first of the equal values inside the image).
// PH, PW: padding of the rows and of the columns.  NT: non-temporal stores.
// BRIEF: fewer instructions around the window and all loads in flight before the first comparison (see forward_brief).
template <typename T, int K, int PH, int PW, int S, bool NT, bool BRIEF>
__global__ __launch_bounds__(kBlock) void maxpool2d_forward_rows_kernel(const T* __restrict__ x, Pool g, RowPool q,
                                                                        T* __restrict__ y, uint8_t* __restrict__ argmax)
{
    static_assert(K == 3 || PW == 0, "a padded column is the first or the last of three");
    typedef Carrier<T, S> C;
    typedef typename C::raw raw;
    typedef raw vec_in __attribute__((ext_vector_type(16 / sizeof(T)), aligned(sizeof(T))));
    typedef raw vec_out __attribute__((ext_vector_type(16 / sizeof(T) / S), aligned(sizeof(T))));
    typedef typename RowVec<T, S>::codes vec_codes;
    constexpr int E = 16 / sizeof(T), NO = E / S;
    constexpr bool kLeft = PW == 1, kRight = K == 3 && (PW == 0 || S == 1);   // columns needed from the neighbours
    typedef typename std::conditional<BRIEF, uint32_t, int64_t>::type Index;
    uint32_t c;
    int32_t i;
    bool live;
    Index at[K], o;   // the lane's first element of every window row, and its first output
    const raw* xr = reinterpret_cast<const raw*>(x);
    raw* yr = reinterpret_cast<raw*>(y);
    int64_t elems = q.elems;   // from xr on
    if constexpr (BRIEF) {
        const RowLane l = row_lane(q.total, q.chunks, q.by_chunks, q.rows, q.by_rows);
        c = l.c;
        i = l.row;
        live = l.live;
        const uint32_t W = static_cast<uint32_t>(g.W);
        at[0] = (row_from_plane0(l, S, g.H, q.rows) - PH) * W + E * c;
#pragma unroll
        for (int a = 1; a < K; ++a) at[a] = at[a - 1] + W;
        if (PH == 1) {   // only the row above the first and the one below the last are outside
            at[0] += i == 0 ? W : 0u;
            at[K - 1] -= S * i - PH + K - 1 >= g.H ? W : 0u;
        }
        o = NO * l.at - __umul24(l.down, NO * q.chunks - static_cast<uint32_t>(g.OW));   // columns that the lanes of a row cover beyond its own: few
        const int64_t base = static_cast<int64_t>(l.plane0) * (static_cast<int64_t>(g.H) * g.W), out_base = static_cast<int64_t>(l.strip0) * g.OW;
        xr += base;
        elems -= base;
        yr += out_base;
        argmax += out_base;
    } else {
        const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
        live = idx < q.total;
        const uint32_t id = live ? idx : q.total - 1;   // every lane takes part in the shift
        const uint32_t strip = fastdiv(id, q.by_chunks);           // output row over all planes
        c = id - strip * q.chunks;
        const uint32_t plane = fastdiv(strip, q.by_rows);
        i = static_cast<int32_t>(strip - plane * q.rows);
#pragma unroll
        for (int a = 0; a < K; ++a) {
            const int32_t r = min(max(S * i - PH + a, 0), g.H - 1);
            at[a] = (static_cast<int64_t>(plane) * g.H + r) * g.W + static_cast<int64_t>(E) * c;
        }
        o = static_cast<int64_t>(strip) * g.OW + NO * static_cast<int32_t>(c);
    }
    typename C::type v[K][E + 2];   // slot 1 + t: column E c + t; slots 0 and E + 1: the neighbours' columns
    if (BRIEF ? __any(at[K - 1] + E > elements_up_to_32_bits(elems)) : __any(at[K - 1] + E > elems)) {
#pragma unroll
        for (int a = 0; a < K; ++a)
#pragma unroll
            for (int t = 0; t < E; ++t) v[a][1 + t] = C::of(xr[min(static_cast<int64_t>(at[a]) + t, elems - 1)]);
    } else {
        vec_in w[K];
#pragma unroll
        for (int a = 0; a < K; ++a) w[a] = *reinterpret_cast<const vec_in*>(xr + at[a]);
        // left alone, the compiler puts the comparisons of a row in front of the next row's load
        if constexpr (BRIEF && (sizeof(T) == 4 || S == 1)) asm volatile("" : "+v"(w[0]), "+v"(w[1]), "+v"(w[K - 1]));
#pragma unroll
        for (int a = 0; a < K; ++a)
#pragma unroll
            for (int t = 0; t < E; ++t) v[a][1 + t] = C::of(w[a][t]);
    }
    if (kLeft) {
#pragma unroll
        for (int a = 0; a < K; ++a) {
            if constexpr (BRIEF && S == 1) v[a][0] = neighbour<true, C>(v[a][E], edge_element<true>(xr, at[a] - 1, c > 0));
            else v[a][0] = neighbour<true, C>(v[a][E], c > 0, xr, at[a] - 1);
            v[a][0] = c > 0 ? v[a][0] : v[a][1];   // the padded column
        }
    }
    if (kRight) {
#pragma unroll
        for (int a = 0; a < K; ++a) {
            if constexpr (BRIEF && S == 1) v[a][E + 1] = neighbour<false, C>(v[a][1], edge_element<false>(xr, at[a] + E, c + 1 < q.chunks));
            else v[a][E + 1] = neighbour<false, C>(v[a][1], c + 1 < q.chunks, xr, at[a] + E);
        }
    }
    const int32_t j0 = NO * static_cast<int32_t>(c);
    vec_out out;
    uint64_t codes = 0;
#pragma unroll
    for (int e = 0; e < NO; ++e) {
        // column S (j0 + e) - PW + b = E c - 1 + slot
        constexpr int kFirst = 1 - PW;
        const bool past = PW == 1 && S * (j0 + e) + 1 >= g.W;   // the window's last column is padding
        typename C::type best = v[0][S * e + kFirst];
        uint32_t best_k = 0;
#pragma unroll
        for (int a = 0; a < K; ++a)
#pragma unroll
            for (int b = 0; b < K; ++b) {
                if (a == 0 && b == 0) continue;
                typename C::type val = v[a][S * e + b + kFirst];
                if (PW == 1 && b == K - 1) val = past ? v[a][S * e + b - 1 + kFirst] : val;
                const bool take = C::value(val) > C::value(best);
                best = take ? val : best;
                best_k = take ? static_cast<uint32_t>(a * K + b) : best_k;
            }
        if (PW == 1 && e == 0) best_k += c == 0 && (best_k == 0 || best_k == 3 || best_k == 6) ? 1u : 0u;
        if (PH == 1) best_k += i == 0 && best_k < K ? K : 0u;
        out[e] = C::back(best);
        codes |= static_cast<uint64_t>(best_k) << (8 * e);
    }
    const int left = g.OW - j0;   // output columns from j0 on
    if (!live || left <= 0) return;
    if (left >= NO) {
        if (NT) {
            __builtin_nontemporal_store(out, reinterpret_cast<vec_out*>(yr + o));
            __builtin_nontemporal_store(static_cast<vec_codes>(codes), reinterpret_cast<vec_codes*>(argmax + o));
        } else {
            *reinterpret_cast<vec_out*>(yr + o) = out;
            *reinterpret_cast<vec_codes*>(argmax + o) = static_cast<vec_codes>(codes);
        }
    } else {
        store_first<NO>(yr + o, out, left);
        store_first_codes(argmax + o, codes, left);
    }
}

// Backward.  A lane produces E columns of S input rows, S q + rr.  The output rows whose windows reach
// them are q (K = 2), q and q + 1 (stride 2, padding 1), q - 1 and q (stride 2, K = 3, padding 0), and
// q - 1 .. q + 1 (stride 1).  The additions run over ascending output row, then column.
// NT: non-temporal stores.  BRIEF: fewer instructions around the windows, what the edge lanes need of their neighbours asked for in front of the loads
// (stride 1) and all loads in flight before the first use (binary16); see backward_brief.
template <typename T, int K, int P, int S, bool NT, bool BRIEF>
__global__ __launch_bounds__(kBlock) void maxpool2d_backward_rows_kernel(const uint8_t* __restrict__ argmax,
                                                                         const T* __restrict__ grad_y, Pool g, RowPool q,
                                                                         T* __restrict__ grad_x)
{
    typedef typename RowVec<T, S>::in vec_in;
    typedef typename RowVec<T, S>::out vec_out;
    typedef typename RowVec<T, S>::codes vec_codes;
    constexpr int E = 16 / sizeof(T), NO = E / S;
    constexpr int MR = S == 1 ? 3 : (K == 3 ? 2 : 1);                  // output rows
    constexpr int kFirstRow = K == 3 && (P == 0 || S == 1) ? -1 : 0;   // the first of them, relative to q
    constexpr bool kLeft = K == 3 && (P == 0 || S == 1), kRight = P == 1;
    constexpr uint32_t kNone = 0x100;                                  // no window position
    typedef typename std::conditional<BRIEF, uint32_t, int64_t>::type Index;
    uint32_t gy[MR][NO + 2];     // slot 1 + t: output column j0 + t
    uint32_t code[MR][NO + 2];
    uint32_t c, plane = 0;       // plane: the ordinary form's
    int32_t j0, stretch;         // the lane's first output column; its stretch of S input rows
    bool live;
    Index at[MR], to = 0;        // the lane's first element of every output row; of its first input row, BRIEF
    bool row_ok[MR];
    int64_t elems = q.elems;     // from grad_y and argmax on
    if constexpr (BRIEF) {
        const RowLane l = row_lane(q.total, q.chunks, q.by_chunks, q.rows, q.by_rows);
        c = l.c;
        j0 = NO * static_cast<int32_t>(c);
        stretch = l.row;
        live = l.live;
        const uint32_t OW = static_cast<uint32_t>(g.OW);
        at[0] = (row_from_plane0(l, 1, g.OH, q.rows) + static_cast<uint32_t>(kFirstRow)) * OW + NO * c;
#pragma unroll
        for (int u = 1; u < MR; ++u) at[u] = at[0] + static_cast<uint32_t>(u) * OW;
#pragma unroll
        for (int u = 0; u < MR; ++u) {
            const int32_t i = stretch + kFirstRow + u;
            row_ok[u] = i >= 0 && i < g.OH;
            // a row that does not exist is the one above the first or the one below the last
            at[u] = row_ok[u] ? at[u] : (kFirstRow + u < 0 ? at[u] + OW : at[u] - OW);
        }
        to = row_from_plane0(l, S, g.H, q.rows) * static_cast<uint32_t>(g.W) + E * c;
        const int64_t base = static_cast<int64_t>(l.plane0) * (static_cast<int64_t>(g.OH) * g.OW);
        grad_y += base;
        argmax += base;
        elems -= base;
        grad_x += static_cast<int64_t>(l.plane0) * (static_cast<int64_t>(g.H) * g.W);
    } else {
        const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
        live = idx < q.total;
        const uint32_t id = live ? idx : q.total - 1;
        const uint32_t strip = fastdiv(id, q.by_chunks);           // stretch of S input rows over all planes
        c = id - strip * q.chunks;
        plane = fastdiv(strip, q.by_rows);
        stretch = static_cast<int32_t>(strip - plane * q.rows);
        j0 = NO * static_cast<int32_t>(c);
#pragma unroll
        for (int u = 0; u < MR; ++u) {
            const int32_t i = stretch + kFirstRow + u;
            row_ok[u] = i >= 0 && i < g.OH;
            at[u] = (static_cast<int64_t>(plane) * g.OH + min(max(i, 0), g.OH - 1)) * g.OW + j0;
        }
    }
    Edge edge_gy[MR][2] = {}, edge_code[MR][2] = {};   // to the left, to the right
    if constexpr (BRIEF && S == 1) {
        const bool left_there = c > 0 && j0 - 1 < g.OW, right_there = c + 1 < q.chunks && j0 + NO < g.OW;
#pragma unroll
        for (int u = 0; u < MR; ++u) {
            edge_gy[u][0] = edge_element<true>(grad_y, at[u] - 1, left_there);
            edge_code[u][0] = edge_element<true>(argmax, at[u] - 1, left_there);
            edge_gy[u][1] = edge_element<false>(grad_y, at[u] + NO, right_there);
            edge_code[u][1] = edge_element<false>(argmax, at[u] + NO, right_there);
        }
    }
    if (BRIEF ? __any(at[MR - 1] + NO > elements_up_to_32_bits(elems)) : __any(at[MR - 1] + NO > elems)) {
#pragma unroll
        for (int u = 0; u < MR; ++u)
#pragma unroll
            for (int t = 0; t < NO; ++t) {
                const int64_t o = min(static_cast<int64_t>(at[u]) + t, elems - 1);
                gy[u][1 + t] = GradientWord<T>::of(grad_y[o]);
                code[u][1 + t] = argmax[o];
            }
    } else {
        vec_out w[MR];
        uint64_t cw[MR];
#pragma unroll
        for (int u = 0; u < MR; ++u) {
            w[u] = *reinterpret_cast<const vec_out*>(grad_y + at[u]);
            cw[u] = *reinterpret_cast<const vec_codes*>(argmax + at[u]);
        }
        if constexpr (BRIEF && sizeof(T) == 2 && MR == 3) asm volatile("" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(cw[0]), "+v"(cw[1]), "+v"(cw[2]));
        else if constexpr (BRIEF && sizeof(T) == 2 && MR == 2) asm volatile("" : "+v"(w[0]), "+v"(w[1]), "+v"(cw[0]), "+v"(cw[1]));
#pragma unroll
        for (int u = 0; u < MR; ++u)
#pragma unroll
            for (int t = 0; t < NO; ++t) {
                gy[u][1 + t] = GradientWord<T>::of(w[u][t]);
                code[u][1 + t] = static_cast<uint32_t>(cw[u] >> (8 * t)) & 0xffu;
            }
    }
#pragma unroll
    for (int u = 0; u < MR; ++u) {
        // the neighbours' columns first, as stored; then what does not exist is no position
        const bool left_there = c > 0 && j0 - 1 < g.OW, right_there = c + 1 < q.chunks && j0 + NO < g.OW;
        if (kLeft) {
            if constexpr (BRIEF && S == 1) gy[u][0] = neighbour<true, GradientWord<T>>(gy[u][NO], edge_gy[u][0]);
            else gy[u][0] = neighbour<true, GradientWord<T>>(gy[u][NO], left_there, grad_y, at[u] - 1);
            if constexpr (BRIEF && S == 1) code[u][0] = neighbour<true, PositionWord>(code[u][NO], edge_code[u][0]);
            else code[u][0] = neighbour<true, PositionWord>(code[u][NO], left_there, argmax, at[u] - 1);
            code[u][0] = row_ok[u] && left_there ? code[u][0] : kNone;
        }
        if (kRight) {
            if constexpr (BRIEF && S == 1) gy[u][NO + 1] = neighbour<false, GradientWord<T>>(gy[u][1], edge_gy[u][1]);
            else gy[u][NO + 1] = neighbour<false, GradientWord<T>>(gy[u][1], right_there, grad_y, at[u] + NO);
            if constexpr (BRIEF && S == 1) code[u][NO + 1] = neighbour<false, PositionWord>(code[u][1], edge_code[u][1]);
            else code[u][NO + 1] = neighbour<false, PositionWord>(code[u][1], right_there, argmax, at[u] + NO);
            code[u][NO + 1] = row_ok[u] && right_there ? code[u][NO + 1] : kNone;
        }
#pragma unroll
        for (int t = 0; t < NO; ++t) code[u][1 + t] = row_ok[u] && j0 + t < g.OW ? code[u][1 + t] : kNone;
    }
    const int left = g.W - E * static_cast<int32_t>(c);   // input columns from the lane's first on, > 0
    vec_in rows[S];   // all of them before the first store: two rows share lines, which meet if their stores are close
#pragma unroll
    for (int rr = 0; rr < S; ++rr) {
        vec_in out;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            float acc = 0.0f;
#pragma unroll
            for (int u = 0; u < MR; ++u) {                          // ascending output row
                const int a = rr + P - S * (kFirstRow + u);         // row of input row S q + rr in its window
                if (a < 0 || a >= K) continue;
#pragma unroll
                for (int t = kLeft ? -1 : 0; t < NO + (kRight ? 1 : 0); ++t) {   // ascending output column
                    const int b = e + P - S * t;
                    if (b < 0 || b >= K) continue;
                    acc += code[u][1 + t] == static_cast<uint32_t>(a * K + b) ? __uint_as_float(gy[u][1 + t]) : 0.0f;  // + 0 changes nothing
                }
            }
            out[e] = static_cast<T>(acc);
        }
        if (S > 1) asm volatile("" : "+v"(out));
        rows[rr] = out;
    }
#pragma unroll
    for (int rr = 0; rr < S; ++rr) {
        const vec_in out = rows[rr];
        const int32_t r = S * stretch + rr;
        if (!live || r >= g.H) continue;
        T* dst = grad_x;
        if constexpr (BRIEF) dst += to + static_cast<uint32_t>(rr) * static_cast<uint32_t>(g.W);
        else dst += (static_cast<int64_t>(plane) * g.H + r) * g.W + static_cast<int64_t>(E) * c;   // at the start it costs 1 to 2 % (binary32 3x3/2/0)
        if (left >= E) {
            if (NT) __builtin_nontemporal_store(out, reinterpret_cast<vec_in*>(dst));
            else *reinterpret_cast<vec_in*>(dst) = out;
        } else {
            store_first<E>(dst, out, left);
        }
    }
}

// Backward of 2x2 windows without overlap for small results: an input lies in one window, so a lane produces 16 bytes
// of ONE input row.  Twice the wavefronts of the kernel above with half the chain each, which is what counts as long as the
// result takes no longer than they do (10 MiB: 9.0 against 10.5 us binary32, 9.9 against 11.4 binary16); beyond it, reading
// every gradient twice does (20 MiB alike, 60 MiB up to 50 % behind).
template <typename T>
__global__ __launch_bounds__(kBlock) void maxpool2d_backward_2x2_kernel(const uint8_t* __restrict__ argmax,
                                                                        const T* __restrict__ grad_y, Pool g, RowPool q,
                                                                        T* __restrict__ grad_x)
{
    typedef typename RowVec<T, 2>::in vec_in;
    typedef typename RowVec<T, 2>::out vec_out;
    typedef typename RowVec<T, 2>::codes vec_codes;
    constexpr int E = 16 / sizeof(T), NO = E / 2;
    constexpr uint32_t kNone = 0x100;                          // no window position
    const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
    if (idx >= q.total) return;
    const uint32_t strip = fastdiv(idx, q.by_chunks);          // input row over all planes
    const uint32_t c = idx - strip * q.chunks;
    const uint32_t plane = fastdiv(strip, q.by_rows);
    const int32_t r = static_cast<int32_t>(strip - plane * q.rows), i = r >> 1;
    const int32_t j0 = NO * static_cast<int32_t>(c);
    const int64_t at = (static_cast<int64_t>(plane) * g.OH + min(i, g.OH - 1)) * g.OW + j0;
    float gy[NO];
    uint32_t code[NO];
    if (at + NO > q.elems) {
#pragma unroll
        for (int t = 0; t < NO; ++t) {
            const int64_t o = min(at + t, q.elems - 1);
            gy[t] = static_cast<float>(grad_y[o]);
            code[t] = argmax[o];
        }
    } else {
        const vec_out w = *reinterpret_cast<const vec_out*>(grad_y + at);
        const uint64_t cw = *reinterpret_cast<const vec_codes*>(argmax + at);
#pragma unroll
        for (int t = 0; t < NO; ++t) {
            gy[t] = static_cast<float>(w[t]);
            code[t] = static_cast<uint32_t>(cw >> (8 * t)) & 0xffu;
        }
    }
    const uint32_t first = 2 * (static_cast<uint32_t>(r) & 1u);   // position of the row's even columns
    vec_in out;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const uint32_t k = i < g.OH && j0 + e / 2 < g.OW ? code[e / 2] : kNone;
        float acc = 0.0f;
        acc += k == first + e % 2 ? gy[e / 2] : 0.0f;
        out[e] = static_cast<T>(acc);
    }
    T* dst = grad_x + static_cast<int64_t>(strip) * g.W + static_cast<int64_t>(E) * c;
    const int left = g.W - E * static_cast<int32_t>(c);
    if (left >= E) __builtin_nontemporal_store(out, reinterpret_cast<vec_in*>(dst));
    else store_first<E>(dst, out, left);
}

}  // namespace

// Blocks of kWavesPerBlock wavefronts that each take 64 lanes of 16 bytes, along x and then y (a grid has
// fewer than 2^32 lanes along x).
static dim3 relu_blocks(int64_t n, int64_t element_bytes)
{
    const int64_t per_block = int64_t(kBlock) * 16 / element_bytes, blocks = (n + per_block - 1) / per_block;
    const int64_t along_x = blocks < (int64_t(1) << 22) ? blocks : int64_t(1) << 22;
    return dim3(static_cast<unsigned>(along_x), static_cast<unsigned>((blocks + along_x - 1) / along_x));
}

// Whether y is stored through the caches: the next layer reads it, and a result that fits the 256 MiB Infinity Cache beside what
// that layer reads and writes is found there.  Non-temporal stores -> these, medians:
//   ReLU, pooling of its result and a pass over that, in a step with 768 MiB of other traffic between its two directions (us)
//                               24 MiB        48 MiB        64 MiB        80 MiB        96 MiB        112 MiB       128 MiB
//     binary32 112 x 112 3/2/1  27.1 -> 27.1  41.2 -> 40.6  50.7 -> 49.9  62.2 -> 59.8  70.5 -> 67.8  80.0 -> 78.2  90.4 -> 86.6
//     binary32  51 x  14 3/1/1  39.0 -> 39.0  63.6 -> 63.3  81.0 -> 80.0  97.5 -> 96.8 114.9 ->113.9 131.7 ->132.1 148.5 ->152.8
//     binary16 113 x 113 3/2/1  29.7 -> 29.4  44.5 -> 43.9  54.4 -> 53.3  64.9 -> 64.0  74.2 -> 72.8  83.3 -> 82.2  93.4 -> 91.3
//     binary16  57 x  57 3/1/1  46.7 -> 46.3  75.0 -> 75.2  95.6 -> 95.2 115.8 ->115.5 136.4 ->136.7 158.7 ->159.2 177.9 ->182.2
//   (binary32 57 x 57 3/1/1 and 144 MiB 173.3 -> 170.2, 51 x 14 169.1 -> 175.9)
//   six layers of a pass, ReLU and a pass over its result, per layer, both types: from 24 to 112 MiB -1.5 to -4.6 %, at 128 MiB -1 %; with a residual read as
//   well -0.4 to -5 %, at 128 MiB binary32 +1 %; where the pass in front updates its tensor in place +0.4 to +3.3 %
// A call whose result nothing reads, over one to four tensors in turn: 24 MiB 6 to 15 % behind, 32 MiB 4 to 19 %, 40 MiB 1 to 11 %, 48 MiB -1 to +6 %, 64 to 112 MiB
// -2 to +4 %.  Hence from the size at which the reader gains about what such a call loses, to the largest at which no image loses more than its runs differ.
// Pooling stores past the caches in both directions: forward, its reader gains 0 to 2 us and a call by itself loses 0 to 3 (64 to 144 MiB); backward, binary16
// gains nothing, and binary32 2 to 5 % in a step at the cost of up to 44 % alone (80 MiB, four tensors in turn 18.3 -> 25.9 us).
static bool relu_through_caches(int64_t bytes) { return bytes >= int64_t(48) << 20 && bytes <= int64_t(112) << 20; }

int launch_relu_forward(const void* x, int dtype, int64_t n, void* y, uint8_t* mask, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t mask_words = (n + 255) / 256 * 8;
    uint32_t* words = reinterpret_cast<uint32_t*>(mask);
    const auto typed = [&](const auto* from, auto* to) {
        typedef std::remove_pointer_t<decltype(to)> T;
        const dim3 blocks = relu_blocks(n, sizeof(T));
        if (relu_through_caches(n * static_cast<int64_t>(sizeof(T)))) launch(relu_forward_kernel<T, false>, blocks, kBlock, s, from, n, mask_words, to, words);
        else launch(relu_forward_kernel<T, true>, blocks, kBlock, s, from, n, mask_words, to, words);
    };
    if (dtype == ACTQ_F32) typed(static_cast<const float*>(x), static_cast<float*>(y));
    else typed(static_cast<const _Float16*>(x), static_cast<_Float16*>(y));
    return launched("actq_relu_forward");
}

int launch_relu_backward(const uint8_t* mask, const void* grad_y, int dtype, int64_t n, void* grad_x, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t mask_words = (n + 255) / 256 * 8;
    if (dtype == ACTQ_F32) {
        launch(relu_backward_kernel<float>, relu_blocks(n, 4), kBlock, s,
            reinterpret_cast<const uint32_t*>(mask), mask_words, static_cast<const float*>(grad_y), n, static_cast<float*>(grad_x));
    } else {
        launch(relu_backward_kernel<_Float16>, relu_blocks(n, 2), kBlock, s,
            reinterpret_cast<const uint32_t*>(mask), mask_words, static_cast<const _Float16*>(grad_y), n, static_cast<_Float16*>(grad_x));
    }
    return launched("actq_relu_backward");
}

static Pool make_pool(const PoolShape& p, int64_t planes, int64_t per_plane, dim3* grid)
{
    Pool g;
    g.H = p.H; g.W = p.W; g.OH = p.OH; g.OW = p.OW;
    g.kh = p.kh; g.kw = p.kw; g.sh = p.sh; g.sw = p.sw;
    g.ph = p.ph; g.pw = p.pw; g.dh = p.dh; g.dw = p.dw;
    g.by_OW = make_fastdiv(static_cast<uint32_t>(p.OW));
    g.by_W = make_fastdiv(static_cast<uint32_t>(p.W));
    g.by_sh = make_fastdiv(static_cast<uint32_t>(p.sh));
    g.by_sw = make_fastdiv(static_cast<uint32_t>(p.sw));
    g.by_dh = make_fastdiv(static_cast<uint32_t>(p.dh));
    g.by_dw = make_fastdiv(static_cast<uint32_t>(p.dw));
    const int64_t gy = planes < 65535 ? planes : 65535;
    g.grid_y = static_cast<uint32_t>(gy);
    *grid = dim3(static_cast<unsigned>((per_plane + kBlock - 1) / kBlock), static_cast<unsigned>(gy),
                 static_cast<unsigned>((planes + gy - 1) / gy));
    return g;
}

constexpr int kPoolBwdBlock = 256;   // threads per block of the streaming backward kernel [128 .. 1024 alike]

// Backward path of its own for even extents (3x3 / stride 2 / padding 1 and 2x2 / stride 2 / padding 0, H = 2 OH
// and W = 2 OW, rows a multiple of 32 bytes long): planes and rows flatten into one index without any row or
// column being special but at the ends of a plane, and every load and store is aligned.
struct StreamPool {
    uint32_t chunks_per_row;   // W / E
    FastDiv by_chunks, by_rows;  // by_rows: division by OH
    uint32_t rows_per_plane;   // OH
    uint32_t total;            // planes * OH * chunks_per_row
};

// A lane owns the NO = E / 2 output columns of one output row q (counted over all planes) that lie over its
// 16 bytes of input columns, and produces the two input rows 2q and 2q + 1 there: every gradient and
// position is loaded once per output row that needs it, in whole cache lines, and the results
// leave as two 128-bit stores.  With a 3x3 window input row 2q + 1 also lies in the window of
// output row q + 1, and the lane's last column in that of the first output column of the lane to
// its right, which arrives by a wavefront shift (lane 63 takes it through the scalar data path).
// The additions run over ascending output row, then column, as in the kernels above.
__device__ __forceinline__ uint32_t from_right_lane(uint32_t v)
{
    constexpr int kWaveShiftLeft1 = 0x130;
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), kWaveShiftLeft1, 0xf, 0xf, false));
}

// JOIN: both rows before either store.
template <typename T, int K, int P, bool JOIN>
__global__ __launch_bounds__(kPoolBwdBlock) void maxpool2d_backward_stream_kernel(const uint8_t* __restrict__ argmax,
                                                                           const T* __restrict__ grad_y, Pool g,
                                                                           StreamPool q, T* __restrict__ grad_x)
{
    constexpr int E = 16 / sizeof(T);    // input columns per lane
    constexpr int NO = E / 2;            // output columns per lane
    constexpr int MR = K == 3 ? 2 : 1;   // output rows whose windows reach the lane's two input rows
    typedef T vec_in __attribute__((ext_vector_type(E)));
    typedef T vec_out __attribute__((ext_vector_type(NO)));
    typedef typename std::conditional<NO == 2, uint16_t, uint32_t>::type code_word;
    const uint32_t idx = blockIdx.x * kPoolBwdBlock + threadIdx.x;
    const bool live = idx < q.total;
    const uint32_t id = live ? idx : q.total - 1;   // every lane takes part in the shift
    const uint32_t strip = fastdiv(id, q.by_chunks);             // output row over all planes
    const uint32_t ch = id - strip * q.chunks_per_row;
    const uint32_t plane = fastdiv(strip, q.by_rows);
    const bool bottom = strip - plane * q.rows_per_plane == q.rows_per_plane - 1;
    const bool right_ok = ch + 1 < q.chunks_per_row;
    const int lane = threadIdx.x & (kWave - 1);
    float gy[MR][NO + 1];
    uint32_t code[MR][NO + 1];
    bool valid[MR];
#pragma unroll
    for (int u = 0; u < MR; ++u) {
        valid[u] = !(u == 1 && bottom);   // below the plane's last output row there is nothing
        const int64_t at = (static_cast<int64_t>(strip) + (valid[u] ? u : 0)) * g.OW + static_cast<int64_t>(NO) * ch;
        const vec_out w = *reinterpret_cast<const vec_out*>(grad_y + at);
        const uint32_t cw = *reinterpret_cast<const code_word*>(argmax + at);
#pragma unroll
        for (int t = 0; t < NO; ++t) {
            gy[u][t] = static_cast<float>(w[t]);
            code[u][t] = (cw >> (8 * t)) & 0xffu;
        }
        gy[u][NO] = 0.0f;
        code[u][NO] = 0;
        if (K == 3) {
            gy[u][NO] = __uint_as_float(from_right_lane(__float_as_uint(gy[u][0])));
            code[u][NO] = from_right_lane(code[u][0]);
            // lane 63: the element after its own, as aligned 32-bit words through the scalar data path
            const uint32_t at_lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(at), kWave - 1);
            const uint32_t at_hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(static_cast<uint64_t>(at) >> 32), kWave - 1);
            const bool last_right_ok = __builtin_amdgcn_readlane(static_cast<uint32_t>(right_ok), kWave - 1) != 0;
            const int64_t next = static_cast<int64_t>((static_cast<uint64_t>(at_hi) << 32) | at_lo) + NO;
            float edge_g = 0.0f;
            uint32_t edge_c = 0;
            if (last_right_ok) {
                if (sizeof(T) == 4) {
                    edge_g = __uint_as_float(load_uniform(reinterpret_cast<const uint32_t*>(grad_y) + next));
                } else {
                    // NO = 4: the element is 8-byte aligned, so it is the low half of its word
                    const uint32_t word = load_uniform(reinterpret_cast<const uint32_t*>(grad_y) + (next >> 1));
                    const uint16_t lo = static_cast<uint16_t>(word);
                    _Float16 h;
                    __builtin_memcpy(&h, &lo, 2);
                    edge_g = static_cast<float>(h);
                }
                const uint32_t word = load_uniform(reinterpret_cast<const uint32_t*>(argmax) + (next >> 2));
                edge_c = (word >> (8 * (static_cast<uint32_t>(next) & 3u))) & 0xffu;
            }
            gy[u][NO] = lane == kWave - 1 ? edge_g : gy[u][NO];
            code[u][NO] = lane == kWave - 1 ? edge_c : code[u][NO];
        }
    }
    vec_in rows[2];
    T* dst = grad_x + 2 * static_cast<int64_t>(strip) * g.W + static_cast<int64_t>(E) * ch;
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
        vec_in out;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            float acc = 0.0f;
#pragma unroll
            for (int u = 0; u < MR; ++u) {            // ascending output row
                const int a = rr + P - 2 * u;         // row of input row 2q + rr in the window of output row q + u
                if (a < 0 || a >= K) continue;
#pragma unroll
                for (int t = 0; t <= NO; ++t) {       // ascending output column
                    const int b = e + P - 2 * t;      // column E ch + e in the window of output column NO ch + t
                    if (b < 0 || b >= K) continue;
                    const bool ok = valid[u] && (t < NO || right_ok);
                    acc += ok && code[u][t] == static_cast<uint32_t>(a * K + b) ? gy[u][t] : 0.0f;  // + 0 changes nothing
                }
            }
            out[e] = static_cast<T>(acc);
        }
        if (JOIN) asm volatile("" : "+v"(out));
        rows[rr] = out;
        if (!JOIN && live) __builtin_nontemporal_store(out, reinterpret_cast<vec_in*>(dst + rr * g.W));
    }
    if (JOIN && live) {
        __builtin_nontemporal_store(rows[0], reinterpret_cast<vec_in*>(dst));
        __builtin_nontemporal_store(rows[1], reinterpret_cast<vec_in*>(dst + g.W));
    }
}

static bool aligned_to(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

static bool quad_geometry(const PoolShape& p) {
    return p.kh == p.kw && (p.kh == 2 || p.kh == 3) && p.sh == p.sw && (p.sh == 1 || p.sh == 2) && p.dh == 1 && p.dw == 1;
}

// The lanes of the row kernels: `rows` rows per plane of `columns` columns that lanes of E columns must cover;
// false if a launch cannot hold them.
static bool row_pool(int64_t planes, int64_t rows, int64_t columns, int E, int64_t elems, RowPool* q)
{
    const int64_t chunks = (columns + E - 1) / E, total = planes * rows * chunks;
    if (total >= (int64_t(1) << 31)) return false;
    q->chunks = static_cast<uint32_t>(chunks);
    q->by_chunks = make_fastdiv(q->chunks);
    q->by_rows = make_fastdiv(static_cast<uint32_t>(rows));
    q->rows = static_cast<uint32_t>(rows);
    q->total = static_cast<uint32_t>(total);
    q->elems = elems;
    return true;
}

static bool row_geometry(const PoolShape& p)
{
    if (p.kh != p.kw || p.sh != p.sw || p.ph != p.pw || p.dh != 1 || p.dw != 1) return false;
    return p.sh == 2 ? (p.kh == 3 && p.ph <= 1) || (p.kh == 2 && p.ph == 0) : p.sh == 1 && p.kh == 3 && p.ph == 1;
}

// Which backward kernel a row geometry takes.  The times are those of a call as a training step makes it: the gradient has
// just been written, the positions and the result's old lines are not in the caches (1 GiB has gone through them).  (Over a few tensors in
// turn part of the result stays in the 256 MiB Infinity Cache and other kernels win.)  What decides is how the stores meet the
// 128-byte lines of the result: a line whose pieces leave in two instructions far apart, or in two XCDs, is written twice.
struct BackwardRule {
    bool single;   // 2x2: a lane owns one input row
    bool stream;   // otherwise: the kernel for even extents and aligned rows, or the row kernel
    bool join;     // the stream kernel computes both rows of a lane before it stores either
    bool nt;       // the row kernel's stores are non-temporal
};

static BackwardRule backward_rule(int64_t planes, const PoolShape& p, int64_t element_bytes)
{
    BackwardRule r = {false, false, false, false};
    if (!row_geometry(p)) return r;
    const int64_t row = p.W * element_bytes, mib = planes * p.H * row >> 20;   // of the result
    const bool even = p.sh == 2 && 2 * p.OH == p.H && 2 * p.OW == p.W && p.W % 8 == 0;
    if (p.kh == 3) {
        // 3x3 / 2 / 1: the stream kernel but for the shortest rows, which lie many to a line (binary16, 100 to 300 MiB: rows of 32 bytes are 7 to 20 %
        // faster with the row kernel, of 48 bytes 5 to 9 % slower, of 112 bytes 13 % at 100 MiB, of 256 bytes 15 % at 60).
        r.stream = even && p.ph == 1 && row >= (element_bytes == 2 ? 48 : 32);
        // Rows that end inside a line share it with the next row, and the two pieces meet (binary16, 100 MiB: rows of 80 bytes 47 %, of
        // 112 bytes 40 %, of 224 bytes 5 %; binary32 rows of 64 and 96 bytes 15 and 35 %; whole lines lose up to 6 %).
        r.join = row % 128 != 0;
    } else if (p.W % 4 == 0 && mib < 20) {
        r.single = true;
    } else {
        // 2x2: always on whole 64 bytes (against the row kernel with the better stores, binary16 at 100 MiB: rows of 64 bytes 14 %, of 128 11 %, of
        // 192 21 %, binary32 14 to 21 %).  Rows with other ends lose more the larger the result, the short ones first (binary16, rows of 112 bytes:
        // 40 MiB 7 % ahead, 60 alike, 100 11 % behind, 300 40 %; of 224 bytes: 60 MiB 3 % ahead, 150 2 % behind, 200 9 %).
        r.stream = even && (row % 64 == 0 || mib < (row < 128 ? 48 : 160));
    }
    // Long rows and rows of whole sectors (2x2 from 192 bytes on, where rows of 96 bytes lose 15 to 50 %): binary16, 100 MiB, 2x2 rows of 450 bytes
    // 12 %, of 600 12 %, 3x3 / 2 / 1 of 600 18 %, 3x3 / 2 / 0 of 2000 21 %; binary32 2x2 rows of 900 bytes 12 %.  Shorter rows lose: binary32 2x2 rows of
    // 112 bytes 46 %, of 240 bytes 10 %.
    r.nt = row >= 256 || row % 128 == 0 || (row % 32 == 0 && row >= (p.kh == 3 ? 96 : 192));
    return r;
}

// Windows that are padded along one axis only, stride 2: 3x3 beside the rows' ends, 2x2 above and below.
// Forward, the rows are only clamped, so these take the same kernel (against one output per lane, [4096, 112, 112]:
// binary32 85 -> 50 and 55 -> 48 us, binary16 77 -> 27 and 49 -> 25 us).
static bool one_sided_row_geometry(const PoolShape& p)
{
    if (p.kh != p.kw || p.sh != 2 || p.sw != 2 || p.dh != 1 || p.dw != 1) return false;
    return (p.kh == 3 && p.ph == 0 && p.pw == 1) || (p.kh == 2 && p.ph == 1 && p.pw == 0);
}

// Whether a row kernel takes its BRIEF form.  Where no lane has a neighbour in another wavefront (the lanes of a row divide 64), the ordinary form asks for no
// words at the edges, and there is no trip to memory behind the loads that the loads together could make up for.
static bool wavefronts_hold_rows(const RowPool& q) { return q.chunks <= kWave && kWave % q.chunks == 0; }

// Forward, the loads together pay from the size on at which HBM sets the pace (a few tensors in turn, us, ordinary -> BRIEF):
//   binary32  3x3/1/1 [16384, 112, 112] 407 -> 348, [8192, 56, 56] 53.3 -> 46.4, [522, 55, 394] 27.4 -> 23.7; 6 MB -2 to +2 %, lanes that divide 64 (rows of
//             15, 31, 63, 125) 0 to +9 %
//             3x3/2/1 [16384, 112, 112] 180 -> 168, [8192, 56, 56] 26.3 -> 24.3, [2048, 57, 57] alike; below, up to +7 % ([3, 23, 23] 2.12 -> 2.27)
//             3x3/2/0 [4096, 113, 113] 50.5 -> 47.7; 30 MB -2 to +5 %
//   binary16  3x3/1/1 [16384, 112, 112] 250 -> 230, [65536, 28, 28] 72 -> 68, [4096, 112, 112] 62 -> 58; odd rows -3 to +5 % (100 MB: 27 columns +5, 113 -3)
//             3x3/2/1 [16384, 112, 112] 94.5 -> 91.6, [4096, 112, 112] 26.8 -> 26.0; 30 MB -2 to +1 %, 6 MB up to +3 %; 3x3/2/0 alike or +1 to +5 %
static bool forward_brief(int64_t planes, const PoolShape& p, const RowPool& q, int64_t element_bytes)
{
    if (p.kh != 3 || p.W >= (1 << 22)) return false;   // 2x2 windows gain nothing; a lane's stretch is found with 24-bit products
    const int64_t mib = planes * p.H * p.W * element_bytes >> 20;
    if (element_bytes == 2) return p.ph == 1 && (p.sh == 1 ? mib >= 24 && p.W % 2 == 0 : mib >= 64);
    return !wavefronts_hold_rows(q) && mib >= (p.ph == 1 ? 24 : 64);
}

// Backward, the words at the edges in front of the loads spare a trip to memory that small gradients wait for:
//   3x3/1/1   binary32 [64, 31, 47] 3.51 -> 2.97, [28, 258, 258] 7.51 -> 6.37, [8192, 56, 56] 50.1 -> 46.8, [16384, 112, 112] 397 -> 357; lanes that divide 64
//             -1 to -3 % up to 14 MB, +3 to +4 % from 25 MB on
//             binary16 [2, 27, 264] 3.94 -> 3.06, [2197, 50, 50] 13.2 -> 11.2, [4096, 113, 113] 91 -> 85, [16384, 112, 112] 302 -> 272; odd rows of 7 to 27
//             columns -1 to -10 % up to 14 MB, 0 to +4 % from 25 MB on
//   stride 2  binary16, 8 to 25 MB -3 to -9 % (8 MB of [225, 225] planes -4, 25 MB -6 to -9), below +-1.5; 30 MB -5 to +6, 100 MB -3 to +5 %
//             (3x3/2/1: [79, 79] planes +4, [56351, 37, 37] 81.5 -> 84.4).  Binary32 gains nothing at best (3x3/2/1 of 30 MB up to +7 %).
static bool backward_brief(int64_t planes, const PoolShape& p, const RowPool& q, int64_t element_bytes)
{
    if (p.kh != 3 || p.W >= (1 << 22)) return false;
    const int64_t mib = planes * p.H * p.W * element_bytes >> 20;
    if (p.sh == 2) return element_bytes == 2 && mib < 24;
    return mib < 16 || (element_bytes == 2 ? p.W % 2 == 0 || p.W >= 32 : !wavefronts_hold_rows(q));
}

template <typename T>
static void maxpool_forward_typed(const T* x, int64_t planes, const PoolShape& p, T* y, uint8_t* argmax, hipStream_t s)
{
    dim3 grid;
    constexpr int kE = 16 / static_cast<int>(sizeof(T));
    RowPool rows;
    // the columns that lanes must hold: those over the outputs, and with K = 3 and no padding one more
    const int64_t columns = static_cast<int64_t>(p.sw) * p.OW + (p.kh == 3 && p.pw == 0 ? 1 : 0);
    if ((row_geometry(p) || one_sided_row_geometry(p)) && row_pool(planes, p.OH, columns, kE, planes * p.H * p.W, &rows)) {
        dim3 unused;
        const Pool g = make_pool(p, planes, 1, &unused);
        const unsigned blocks = (rows.total + kBlock - 1) / kBlock;
        // Non-temporal stores of y and the positions but on rows of other lengths than whole 16 bytes (binary16 3x3/1 on [65536, 28, 28] 74 -> 78 us
        // with them; binary32 2x2 as in a step, where x has just been written and the layer behind reads y: [6158, 113, 113] alone 88 -> 96 us,
        // [2052, 113, 113] with a pass over y 33 -> 39).  binary32 3x3 keeps them there too: over a few tensors in turn [4096, 111, 120]
        // 50 -> 46 us and 3x3/1 on [1026, 113, 113] 35 -> 29, in a step alike alone and 5 to 10 % behind with the pass over y.  On whole 16 bytes,
        // over a few tensors in turn: binary16 2x2/2 27.9 -> 25.8 us on [4096, 112, 112], 3x3/2 54.9 -> 52.8 us on [4096, 160, 160]; with the pass
        // over y, results that would have stayed in the Infinity Cache cost 10 to 20 % more.
        const bool nt = sizeof(T) == 4 ? p.kh == 3 || p.W % 4 == 0 : p.W % 8 == 0;
        const bool brief = forward_brief(planes, p, rows, sizeof(T));
        // What the rules ask for and a geometry does not have takes the form that it has: every choice launches.
#define ACTQ_POOL_ROWS(K, PH, PW, S)                                                                                                                   \
    do {                                                                                                                                               \
        constexpr bool kBrief = K == 3 && (sizeof(T) == 4 || PH == 1), kOrdinaryStores = sizeof(T) == 2 || K == 2;                                     \
        const auto with = [&](auto store, auto form) {                                                                                                 \
            launch(maxpool2d_forward_rows_kernel<T, K, PH, PW, S, decltype(store)::value, decltype(form)::value>, blocks, kBlock, s, x, g, rows, y, argmax);\
        };                                                                                                                                             \
        const auto form = [&](auto store) {                                                                                                            \
            if (kBrief && brief) with(store, std::bool_constant<kBrief>());                                                                            \
            else with(store, std::false_type());                                                                                                       \
        };                                                                                                                                             \
        if (nt || !kOrdinaryStores) form(std::true_type());                                                                                            \
        else form(std::bool_constant<!kOrdinaryStores>());                                                                                             \
    } while (0)
        if (p.sh == 1) ACTQ_POOL_ROWS(3, 1, 1, 1);
        else if (p.kh == 2 && p.ph == 0) ACTQ_POOL_ROWS(2, 0, 0, 2);
        else if (p.kh == 2) ACTQ_POOL_ROWS(2, 1, 0, 2);
        else if (p.pw == 0) ACTQ_POOL_ROWS(3, 0, 0, 2);
        else if (p.ph == 0) ACTQ_POOL_ROWS(3, 0, 1, 2);
        else ACTQ_POOL_ROWS(3, 1, 1, 2);
#undef ACTQ_POOL_ROWS
        return;
    }
    const Pool g = make_pool(p, planes, static_cast<int64_t>(p.OH) * p.OW, &grid);
    if (p.kh == 3 && p.kw == 3) launch(maxpool2d_forward_kernel<T, 3, 3>, grid, kBlock, s, x, planes, g, y, argmax);
    else if (p.kh == 2 && p.kw == 2) launch(maxpool2d_forward_kernel<T, 2, 2>, grid, kBlock, s, x, planes, g, y, argmax);
    else launch(maxpool2d_forward_kernel<T, 0, 0>, grid, kBlock, s, x, planes, g, y, argmax);
}

template <typename T>
static void maxpool_backward_typed(const uint8_t* argmax, const T* grad_y, int64_t planes, const PoolShape& p,
                                   T* grad_x, hipStream_t s)
{
    dim3 grid;
    constexpr int kE = 16 / static_cast<int>(sizeof(T));
    const BackwardRule rule = backward_rule(planes, p, sizeof(T));
    const bool stream_geometry = rule.stream && aligned_to(grad_x, 16) && aligned_to(grad_y, 16) && aligned_to(argmax, 4) &&
                                 planes * p.OH * (p.W / kE) < (int64_t(1) << 31);
    if (stream_geometry) {
        StreamPool q;
        q.chunks_per_row = static_cast<uint32_t>(p.W / kE);
        q.by_chunks = make_fastdiv(q.chunks_per_row);
        q.rows_per_plane = static_cast<uint32_t>(p.OH);
        q.by_rows = make_fastdiv(q.rows_per_plane);
        q.total = static_cast<uint32_t>(planes * q.rows_per_plane * q.chunks_per_row);
        dim3 unused;
        const Pool g = make_pool(p, planes, 1, &unused);
        const unsigned blocks = (q.total + kPoolBwdBlock - 1) / kPoolBwdBlock;
        if (p.kh == 2) launch(maxpool2d_backward_stream_kernel<T, 2, 0, false>, blocks, kPoolBwdBlock, s, argmax, grad_y, g, q, grad_x);
        else if (rule.join) launch(maxpool2d_backward_stream_kernel<T, 3, 1, true>, blocks, kPoolBwdBlock, s, argmax, grad_y, g, q, grad_x);
        else launch(maxpool2d_backward_stream_kernel<T, 3, 1, false>, blocks, kPoolBwdBlock, s, argmax, grad_y, g, q, grad_x);
        return;
    }
    RowPool rows;
    const int64_t rows_per_lane = rule.single ? 1 : p.sh;
    if (row_geometry(p) && row_pool(planes, (static_cast<int64_t>(p.H) + rows_per_lane - 1) / rows_per_lane, p.W, kE, planes * p.OH * p.OW, &rows)) {
        dim3 unused;
        const Pool g = make_pool(p, planes, 1, &unused);
        const unsigned blocks = (rows.total + kBlock - 1) / kBlock;
        if (rule.single) {
            launch(maxpool2d_backward_2x2_kernel<T>, blocks, kBlock, s, argmax, grad_y, g, rows, grad_x);
            return;
        }
        const bool brief = backward_brief(planes, p, rows, sizeof(T));
#define ACTQ_POOL_ROWS(K, P, S)                                                                                                                        \
    do {                                                                                                                                               \
        constexpr bool kBrief = K == 3 && (S == 1 || sizeof(T) == 2);                                                                                  \
        const auto with = [&](auto store, auto form) {                                                                                                 \
            launch(maxpool2d_backward_rows_kernel<T, K, P, S, decltype(store)::value, decltype(form)::value>, blocks, kBlock, s, argmax, grad_y, g, rows, grad_x);\
        };                                                                                                                                             \
        const auto form = [&](auto store) {                                                                                                            \
            if (kBrief && brief) with(store, std::bool_constant<kBrief>());                                                                            \
            else with(store, std::false_type());                                                                                                       \
        };                                                                                                                                             \
        if (rule.nt) form(std::true_type());                                                                                                           \
        else form(std::false_type());                                                                                                                  \
    } while (0)
        if (p.sh == 1) ACTQ_POOL_ROWS(3, 1, 1);
        else if (p.kh == 2) ACTQ_POOL_ROWS(2, 0, 2);
        else if (p.ph == 1) ACTQ_POOL_ROWS(3, 1, 2);
        else ACTQ_POOL_ROWS(3, 0, 2);
#undef ACTQ_POOL_ROWS
        return;
    }
    if (quad_geometry(p)) {
        QuadGeometry q;
        q.quads_per_row = (p.W + 3) / 4;
        q.by_quads = make_fastdiv(static_cast<uint32_t>(q.quads_per_row));
        q.vector_ok = p.W % 4 == 0 && aligned_to(grad_x, 4 * sizeof(T));
        const Pool g = make_pool(p, planes, static_cast<int64_t>(p.H) * q.quads_per_row, &grid);
#define ACTQ_POOL_BWD(K, S) launch(maxpool2d_backward_quad_kernel<T, K, S>, grid, kBlock, s, argmax, grad_y, planes, g, q, grad_x)
        if (p.kh == 3 && p.sh == 2) ACTQ_POOL_BWD(3, 2);
        else if (p.kh == 3) ACTQ_POOL_BWD(3, 1);
        else if (p.sh == 2) ACTQ_POOL_BWD(2, 2);
        else ACTQ_POOL_BWD(2, 1);
#undef ACTQ_POOL_BWD
        return;
    }
    const Pool g = make_pool(p, planes, static_cast<int64_t>(p.H) * p.W, &grid);
    // how many output rows / columns can contain one input location
    const int64_t reach_h = (static_cast<int64_t>(p.dh) * (p.kh - 1) + p.sh) / p.sh;
    const int64_t reach_w = (static_cast<int64_t>(p.dw) * (p.kw - 1) + p.sw) / p.sw;
    const int64_t reach = reach_h > reach_w ? reach_h : reach_w;
    if (reach <= 1) launch(maxpool2d_backward_kernel<T, 1>, grid, kBlock, s, argmax, grad_y, planes, g, grad_x);
    else if (reach == 2) launch(maxpool2d_backward_kernel<T, 2>, grid, kBlock, s, argmax, grad_y, planes, g, grad_x);
    else if (reach == 3) launch(maxpool2d_backward_kernel<T, 3>, grid, kBlock, s, argmax, grad_y, planes, g, grad_x);
    else launch(maxpool2d_backward_kernel<T, 0>, grid, kBlock, s, argmax, grad_y, planes, g, grad_x);
}

// The row kernels number their lanes in 31 bits; larger tensors (34 GB and more) take several launches over ranges of planes
// (3x3 / 1 / 1 on binary16 [1369572, 112, 112] with a lane per element: forward 64 ms, backward 78; in two launches 19.7 and 25.0).
// `each` gets the first plane and the number of planes.
template <typename T, typename Each>
static void over_planes(int64_t planes, const PoolShape& p, const Each& each)
{
    constexpr int64_t kE = 16 / static_cast<int64_t>(sizeof(T));
    const int64_t height = p.H > p.OH ? p.H : p.OH, width = p.W > p.sw * static_cast<int64_t>(p.OW) ? p.W : p.sw * static_cast<int64_t>(p.OW);
    const int64_t most = ((int64_t(1) << 31) - 1) / (height * ((width + 1 + kE - 1) / kE));   // a bound on the lanes of either direction
    int64_t step = planes;
    if (most >= 1 && (row_geometry(p) || one_sided_row_geometry(p))) {
        const int64_t launches = (planes + most - 1) / most;
        step = (planes + launches - 1) / launches;
    }
    for (int64_t at = 0; at < planes; at += step) each(at, planes - at < step ? planes - at : step);
}

int launch_maxpool2d_forward(const void* x, int dtype, int64_t planes, const PoolShape& p, void* y,
                             uint8_t* argmax, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t in = static_cast<int64_t>(p.H) * p.W, out = static_cast<int64_t>(p.OH) * p.OW;
    const auto typed = [&](const auto* from, auto* to) {
        over_planes<std::remove_pointer_t<decltype(to)>>(planes, p, [&](int64_t at, int64_t count) {
            maxpool_forward_typed(from + at * in, count, p, to + at * out, argmax + at * out, s);
        });
    };
    if (dtype == ACTQ_F32) typed(static_cast<const float*>(x), static_cast<float*>(y));
    else typed(static_cast<const _Float16*>(x), static_cast<_Float16*>(y));
    return launched("actq_maxpool2d_forward");
}

int launch_maxpool2d_backward(const uint8_t* argmax, const void* grad_y, int dtype, int64_t planes,
                              const PoolShape& p, void* grad_x, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t in = static_cast<int64_t>(p.H) * p.W, out = static_cast<int64_t>(p.OH) * p.OW;
    const auto typed = [&](const auto* from, auto* to) {
        over_planes<std::remove_pointer_t<decltype(to)>>(planes, p, [&](int64_t at, int64_t count) {
            maxpool_backward_typed(argmax + at * out, from + at * out, count, p, to + at * in, s);
        });
    };
    if (dtype == ACTQ_F32) typed(static_cast<const float*>(grad_y), static_cast<float*>(grad_x));
    else typed(static_cast<const _Float16*>(grad_y), static_cast<_Float16*>(grad_x));
    return launched("actq_maxpool2d_backward");
}

}  // namespace actq
