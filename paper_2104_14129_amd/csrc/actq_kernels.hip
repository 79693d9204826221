// HIP kernels of libactq for gfx950 (MI355X): per-group min/range, stochastic rounding
// with Philox4x32-10 noise, bit-stream packing, and unpack + dequantize (ActNN,
// Sec. 4.1 and Sec. 5.1).
//
// Work decomposition.  The group size is 256 = one 64-lane wavefront x 4 consecutive
// elements per lane, so one 128-bit load per lane brings in a whole group.  A *tile* is
// four consecutive groups of one sample (4 KiB of binary32 input, four loads in flight per
// lane); tiles never cross a sample, so the width b_n is uniform over a tile and every
// branch on it is divergence-free.  One wavefront handles one tile and exits: on this part
// many short-lived wavefronts stream HBM faster than a few long-lived ones.
//
// The path is bound by HBM only if the integer work of the noise generator stays hidden, so
// the rest is kept off the vector ALU as far as possible:
//   * the statistics reduce the minimum and maximum of the four groups *together*: eight
//     partial values per lane are folded by a transposing butterfly (v_permlane32_swap,
//     v_permlane16_swap, DPP row_ror:8) that halves the number of live values at every step,
//     so the whole tile costs 18 cross-lane operations instead of 48;
//   * the quantizer loads its tile in address order and deals it through the LDS so that a lane
//     holds a contiguous piece of one group (quantize_run_f16, quantize_tile), and the lane keeps
//     its noise, its share of the reduction and its bytes of the bit stream to itself.
// Every kernel exists for samples of whole groups and for samples that end inside a group
// (RAGGED): those are read and written with the same 128-bit accesses at the alignment of an
// element, and only the tile in which a sample ends is fetched element by element.  (A path of
// guarded elements for all tiles took 2 to 3.5 times as long, the write side of binary16 most.)
//
// Beyond the arithmetic, four things about the memory system decide the speed (all measured
// on tensors that do not fit the caches):
//   * small writes that reach HBM in the middle of a read stream are expensive out of all
//     proportion (the statistics, 0.8 % of the bytes, cost 10 % of the time): they are issued
//     as ordinary cached stores and the tiles are dealt to the eight XCDs in long runs, so that
//     whole lines of them collect in one L2 (wave_unit);
//   * a write stream is fastest when every XCD writes every eighth 4 KiB page of it (the
//     dequantizer's order), and a branch between the loads and the stores of a wavefront makes
//     the compiler serialise the stores (dequantize_groups);
//   * the scalar loads at the start of a wavefront are issued in batches (ACTQ_SCALAR_BATCH*);
//   * loads must cover whole cache lines per instruction: four 128-bit loads whose lanes are 64
//     bytes apart cost the binary16 quantizer a third of its time (quantize_run_f16).
//
// This file must be compiled with -ffp-contract=off: the scaling step is a subtraction
// and a multiplication that are rounded separately.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "actq_internal.h"

namespace actq {
namespace {

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;
constexpr int kBlock = kWave * kWavesPerBlock;
constexpr int kTileGroups = 4;
constexpr int kMaxMulti = ACTQ_MAX_TENSORS_PER_CALL;  // tensors of one multi-tensor launch

// Launch shapes of the statistics, quantizer and dequantizer kernels, for one tensor as for several.
// Each value was chosen by A/B runs on the 53-tensor ResNet-50 sweep at batch 256,
// alternatives in brackets.
constexpr int kDqGroupsF32 = 4;         // dequantizer: groups per wavefront, binary32 output [2, 1: slower]
constexpr int kDqGroupsF16 = 8;         //              binary16 output: the same 4 KiB per wavefront
constexpr int kDqBlock = 256;           //              threads per block [512 alike; 1024, 128, 64 slower]
constexpr int kDqXcdMap = 1;            //              tiles dealt to the XCDs modulo 8 [plain order: 13 % slower]
constexpr int kDqRaggedRun = 16;        //              ragged samples: consecutive workgroups' tiles per XCD
constexpr int kGsBlock = 256;           // statistics: threads per block [64 .. 1024: alike or slower]
constexpr int kGsXcdMap = 0;
constexpr int kGsRun = 16;              //             consecutive workgroups' tiles per XCD [1: 5 % slower; 8, 32 near; not powers of two: slower]
constexpr int kGsRunHalf = 2;           //             binary16 tensors of whole tiles (group_stats_launch)
constexpr int kQpXcdMap = 0;            // quantizer [tiles modulo 8: slower]
constexpr int kQpRun = 16;              //           [1: 3 % slower; 32 alike]

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------
// Cross-lane helpers (DPP within a row of 16 lanes, v_readlane across rows).

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v)
{
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xf, 0xf, true));
}

constexpr int kDppXor1 = 0xB1;         // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;         // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // lane i <-> 7-i inside each 8 lanes
constexpr int kDppXor8 = 0x128;        // row_ror:8, lane i <-> i^8 inside each 16 lanes

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// min over lanes {l, l^32} of a (kept in lanes 0..31) and of b (kept in lanes 32..63)
__device__ __forceinline__ float fold32(float a, float b)
{
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return fminf(__uint_as_float(r.x), __uint_as_float(r.y));
}

// min over lanes {l, l^16} of a (kept in rows 0 and 2) and of b (kept in rows 1 and 3)
__device__ __forceinline__ float fold16(float a, float b)
{
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return fminf(__uint_as_float(r.x), __uint_as_float(r.y));
}

// Joint reduction of the four groups of a tile.  lo[u] / hi[u] are the lane-local minimum
// and maximum of group u.  On return every lane of row u (lanes 16u..16u+15) holds the
// wavefront-wide minimum and maximum of group u.  Inputs are finite.
__device__ __forceinline__ void tile_min_max(const float (&lo)[4], const float (&hi)[4], int lane,
                                             float& row_min, float& row_max)
{
    // max(x) = -min(-x): all eight values are folded with min; value 2u is lo[u], 2u+1 is -hi[u]
    float c[4];
    c[0] = fold32(lo[0], lo[2]);    // values 0 | 4
    c[1] = fold32(-hi[0], -hi[2]);  // values 1 | 5
    c[2] = fold32(lo[1], lo[3]);    // values 2 | 6
    c[3] = fold32(-hi[1], -hi[3]);  // values 3 | 7
    float d[2];
    d[0] = fold16(c[0], c[2]);      // value (lane>>4)*2
    d[1] = fold16(c[1], c[3]);      // value (lane>>4)*2 + 1
    const bool upper = (lane & 8) != 0;
    const float keep = upper ? d[1] : d[0];
    const float give = upper ? d[0] : d[1];
    float e = fminf(keep, dpp_f32<kDppXor8>(give));  // value lane>>3, still to fold over lane bits 0..2
    e = fminf(e, dpp_f32<kDppXor1>(e));
    e = fminf(e, dpp_f32<kDppXor2>(e));
    e = fminf(e, dpp_f32<kDppHalfMirror>(e));
    const float other = dpp_f32<kDppXor8>(e);
    row_min = upper ? other : e;
    row_max = -(upper ? e : other);
}

// ------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11), state in registers.  The two three-way exclusive-ors
// of a round are one gfx950 three-input bit operation each (truth table 0x96 = a ^ b ^ c).

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&out)[4])
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t prod_a = static_cast<uint64_t>(c0) * 0xD2511F53u;
        const uint64_t prod_b = static_cast<uint64_t>(c2) * 0xCD9E8D57u;
        const uint32_t y0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(prod_b >> 32), c1, k0, 0x96);
        const uint32_t y2 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(prod_a >> 32), c3, k1, 0x96);
        c1 = static_cast<uint32_t>(prod_b);
        c3 = static_cast<uint32_t>(prod_a);
        c0 = y0;
        c2 = y2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}

// ------------------------------------------------------------------------------------
// Four consecutive elements of one lane, widened to binary32.  ALIGNED: the tensor's samples are whole
// groups, so every quadruple has the alignment of its own size.  Otherwise (a sample ends in a part of
// a group) it has that of an element only; the memory instructions are the same ones, global accesses
// of any width may start at any byte on this target.

// LAYOUT of the samples: whole groups, or a part of a group at the end (RAGGED), in which case they are a
// whole number of 128-byte lines long or not.
enum Layout { kWholeGroups, kRaggedLines, kRagged };

template <typename T>
struct Io;

template <>
struct Io<float> {
    typedef f32x4 quad;
    typedef f32x4 __attribute__((aligned(4))) quad_unaligned;
    static __device__ __forceinline__ float narrow(float v) { return v; }
};

template <>
struct Io<_Float16> {
    typedef f16x4 quad;
    typedef f16x4 __attribute__((aligned(2))) quad_unaligned;
    // binary32 -> binary16, round to nearest even, of a value that has already been rounded
    // to binary32.  The empty asm keeps the compiler from merging the conversion into the
    // producing multiply-add (a mixed-precision fma rounds once, straight to binary16, and
    // differs from the two-step result in rare half-way cases).
    static __device__ __forceinline__ _Float16 narrow(float v)
    {
        asm("" : "+v"(v));
        return static_cast<_Float16>(v);
    }
};

template <typename T, bool ALIGNED, bool NT>
__device__ __forceinline__ void load4(const T* p, float (&v)[4])
{
    typedef typename std::conditional<ALIGNED, typename Io<T>::quad, typename Io<T>::quad_unaligned>::type source;
    typename Io<T>::quad t;
    if constexpr (NT) t = __builtin_nontemporal_load(reinterpret_cast<const source*>(p));
    else t = *reinterpret_cast<const source*>(p);
    v[0] = static_cast<float>(t.x); v[1] = static_cast<float>(t.y);
    v[2] = static_cast<float>(t.z); v[3] = static_cast<float>(t.w);
}

template <typename T, int LAYOUT>
__device__ __forceinline__ void store4(T* p, const float (&v)[4])
{
    typename Io<T>::quad t;
    t.x = Io<T>::narrow(v[0]); t.y = Io<T>::narrow(v[1]); t.z = Io<T>::narrow(v[2]); t.w = Io<T>::narrow(v[3]);
    if constexpr (LAYOUT == kWholeGroups) __builtin_nontemporal_store(t, reinterpret_cast<typename Io<T>::quad*>(p));
    else if constexpr (LAYOUT == kRaggedLines) __builtin_nontemporal_store(t, reinterpret_cast<typename Io<T>::quad_unaligned*>(p));
    else *reinterpret_cast<typename Io<T>::quad_unaligned*>(p) = t;
}

// Lane-local minimum and maximum of each group.
__device__ __forceinline__ void lane_min_max(const float (&v)[kTileGroups][4], float (&lo)[kTileGroups], float (&hi)[kTileGroups])
{
#pragma unroll
    for (int u = 0; u < kTileGroups; ++u) {
        lo[u] = fminf(fminf(v[u][0], v[u][1]), fminf(v[u][2], v[u][3]));
        hi[u] = fmaxf(fmaxf(v[u][0], v[u][1]), fmaxf(v[u][2], v[u][3]));
    }
}

// Loads through the constant address space: for memory that no kernel of this library writes
// while it reads it (widths, offsets, and the headers in the dequantizer).  A wavefront-uniform
// load of this kind goes through the scalar data path whatever the compiler can prove about
// aliasing, which keeps four loads per tile off the vector memory pipeline.
template <typename V>
__device__ __forceinline__ V load_readonly(const V* p)
{
    typedef const V __attribute__((address_space(4))) * constant_ptr;
    return *(constant_ptr)(reinterpret_cast<uintptr_t>(p));
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t __attribute__((aligned(1))) word_a1;   // words that start at any byte
typedef u32x2 __attribute__((aligned(1))) words_a1;

// True if the sample's byte range [off, off + bytes) is 32-byte aligned and inside the stream.
__device__ __forceinline__ bool range_ok(uint64_t off, uint64_t bytes, uint64_t capacity)
{
    return (off & 31u) == 0 && off <= capacity && bytes <= capacity - off;
}

// bfloat16 header (Sec. 4.1, last paragraph): the zero point is rounded down and the range,
// taken from the rounded zero point, is rounded up, so every element still scales into [0, B].
// Both return the 16 bits of the bfloat16 value.
__device__ __forceinline__ uint32_t bf16_floor_bits(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u >> 16) + (((u & 0xffffu) != 0 && (u >> 31) != 0) ? 1u : 0u);
}

__device__ __forceinline__ uint32_t bf16_ceil_bits(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u >> 16) + (((u & 0xffffu) != 0 && (u >> 31) == 0) ? 1u : 0u);
}

// A zero the compiler cannot see through, in a vector register: added to a wavefront-uniform
// index it keeps the load on the vector memory path.
__device__ __forceinline__ uint32_t vector_zero()
{
    uint32_t z;
    asm volatile("v_mov_b32 %0, 0" : "=v"(z));
    return z;
}

// Header of group `index` as (Z, step R / B).  HDR: 0 = stored as such in binary32; 1 = (Z, R) in
// bfloat16; 2 = one (Z, R) pair in binary32 for the whole tensor, the step being 0 when R is 0
// or B / R overflows (the degenerate rule of the quantizer).
// This one through the vector memory path: every lane loads the same address (binary32 output;
// scalar loads are 10 % slower there on cold data).
template <int HDR>
__device__ __forceinline__ f32x2 load_header_vector(const void* __restrict__ header, int64_t index, float kB, uint32_t vzero)
{
    if (HDR == 2) {
        const f32x2 zr = static_cast<const f32x2*>(header)[vzero];
        f32x2 h;
        h.x = zr.x;
        h.y = (zr.y != 0.0f && __builtin_isfinite(kB / zr.y)) ? zr.y / kB : 0.0f;
        return h;
    }
    if (HDR == 1) {
        const uint32_t w = static_cast<const uint32_t*>(header)[index + vzero];
        f32x2 h;
        h.x = __uint_as_float(w << 16);
        h.y = __uint_as_float(w & 0xffff0000u) / kB;
        return h;
    }
    return static_cast<const f32x2*>(header)[index + vzero];
}

// The same header through the scalar data path, `index` being uniform (binary16 output).
template <int HDR>
__device__ __forceinline__ f32x2 load_header(const void* __restrict__ header, int64_t index, float kB)
{
    if (HDR == 2) {
        const f32x2 zr = load_readonly(static_cast<const f32x2*>(header));
        f32x2 h;
        h.x = zr.x;
        h.y = (zr.y != 0.0f && __builtin_isfinite(kB / zr.y)) ? zr.y / kB : 0.0f;
        return h;
    }
    if (HDR == 1) {
        const uint32_t w = load_readonly(static_cast<const uint32_t*>(header) + index);
        f32x2 h;
        h.x = __uint_as_float(w << 16);
        h.y = __uint_as_float(w & 0xffff0000u) / kB;  // IEEE division, as the step R / B is defined
        return h;
    }
    return load_readonly(static_cast<const f32x2*>(header) + index);
}

// ------------------------------------------------------------------------------------
// Sec. 4.1 + Sec. 5.1: scale, round stochastically, pack.

// Orders the compiler's view of a wavefront-private LDS hand-over (write by one lane, read
// by another lane of the same wavefront).  The hardware executes one wavefront's LDS
// instructions in order, so no instruction is emitted.
__device__ __forceinline__ void wave_lds_handover()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------------------------------
// The zero point, factor and header of a group from its minimum and maximum.  HDR: 0 = (Z, R / B) in
// binary32; 1 = (Z, R) in bfloat16, Z rounded down and R, taken from the rounded Z, rounded up; 2 = one
// (Z, R) for the whole tensor, given by the caller: the group's own extremes are not used.
struct GroupScale {
    float zero, inv;
    f32x2 header;      // HDR 0
    uint32_t header16; // HDR 1
};

// LANES lanes share a group; with HDR 0 one IEEE division gives both quotients, B / R in the lower half
// of them and R / B in the upper half, and a lane permutation (TRADE) exchanges the results.
template <int HDR, int LANES, int TRADE>
__device__ __forceinline__ GroupScale group_scale(float mn, float mx, float kB, int lane, const void* header)
{
    GroupScale s;
    if (HDR == 0) {
        const float range = mx - mn;
        const bool inv_side = (lane & (LANES / 2)) == 0;
        const float quotient = (inv_side ? kB : range) / (inv_side ? range : kB);
        const float traded = dpp_f32<TRADE>(quotient);
        s.zero = mn;
        s.inv = inv_side ? quotient : traded;
        float scale = inv_side ? traded : quotient;
        if (!(range != 0.0f) || !__builtin_isfinite(s.inv)) {   // constant group, or B / R overflows
            s.inv = 0.0f;
            scale = 0.0f;
        }
        s.header.x = mn;
        s.header.y = scale;
        s.header16 = 0;
    } else {
        uint32_t zb = 0, rb = 0;
        float range;
        if (HDR == 1) {
            zb = bf16_floor_bits(mn);
            s.zero = __uint_as_float(zb << 16);
            rb = bf16_ceil_bits(mx - s.zero);
            range = __uint_as_float(rb << 16);
            if (!__builtin_isfinite(range)) range = 0.0f;  // rounding up overflowed: degenerate
        } else {
            const f32x2 zr = load_readonly(static_cast<const f32x2*>(header));
            s.zero = zr.x;
            range = zr.y;
        }
        s.inv = kB / range;
        if (!(range != 0.0f) || !__builtin_isfinite(s.inv)) {
            s.inv = 0.0f;
            rb = 0;
        }
        s.header16 = zb | (rb << 16);
        s.header.x = s.header.y = 0.0f;
    }
    return s;
}

// An ordinary (cached) store: the headers of neighbouring tiles meet in the L2 and leave as whole lines
// (non-temporal ones reached HBM piecemeal, +2 % on the ResNet-50 sweep).
template <int HDR>
__device__ __forceinline__ void store_header(void* header, int64_t group, const GroupScale& s)
{
    if (HDR == 0) static_cast<f32x2*>(header)[group] = s.header;
    if (HDR == 1) static_cast<uint32_t*>(header)[group] = s.header16;
}

// Clears the codes past the end of a sample: word k of a lane that holds `count` valid codes of B bits.
template <int B>
__device__ __forceinline__ uint32_t valid_bits(int count, int k)
{
    const int n = count * B - 32 * k;
    return n >= 32 ? ~0u : (n <= 0 ? 0u : (1u << n) - 1u);
}

// ------------------------------------------------------------------------------------
// binary16 input with 16-bit noise and a header per group: a lane-to-element map of its own.
//
// With two bytes per element the quantizer is bound by the vector ALU (every SIMD issues all
// the time), so this path exists to issue fewer instructions for the same arithmetic:
//   * a lane works on 32 consecutive elements, so a group is eight lanes and a wavefront
//     takes a run of EIGHT groups: what is paid once per group and lane (the reduction across
//     lanes, the two IEEE divisions, addresses, the header) is spread over twice the elements
//     of a tile of four groups (quantize_tile).  32 elements are exactly what four Philox calls serve with
//     16-bit noise: a lane uses all words of its own calls and nothing is traded between
//     lanes.  The run's four kilobytes are loaded in address order and dealt to the lanes
//     through the LDS (LDS instructions do not take vector-ALU issue slots);
//   * a lane's 32 codes are 4 B consecutive bytes of the bit stream for every width B, stored
//     by the lane itself: the codes do not pass through the LDS;
//   * minimum and maximum are taken on the packed binary16 pairs as they arrive (min and max
//     of binary16 values are exact in binary16) with the three-operand packed instructions,
//     folded into one packed pair (min, -max) per lane, so the reduction over the eight
//     lanes works on one register with three lane permutations;
//   * the subtraction x - Z reads the binary16 half of the loaded word directly (a
//     mixed-precision fma with the factor 1: fl32(x * 1 - Z) is the separately rounded
//     subtraction), which removes the conversions to binary32 and the half extractions;
//   * the clamp of the scaled value to B = 2^b - 1 is skipped for b <= 7, where it cannot
//     change a code: with r the range and q = fl(B / r) (normal for any binary16 range),
//     fl((x - Z) q) <= fl(r q) <= fl(B (1 + 2^-24)) <= B + ulp(B), and with ulp(B) <= 2^-17
//     the sum B + ulp(B) + (1 - 2^-16) is a binary32 number below B + 1, so the floor is B
//     with or without the clamp.  (For b = 8 one ulp is 2^-16 and the sum reaches 256: the
//     clamp is kept.)  The bfloat16 header changes none of this: x - Z <= R there, too, because R
//     is rounded up from max - Z, and a range that is not 0 is at least 2^-24.
// The last run of a sample may hold fewer than eight groups: its spare lanes re-read the sample's
// last group and store nothing.  RAGGED: the sample may end inside a group, so no run but a sample's
// last one is short, the samples are aligned to an element only, and the last run is fetched element
// by element, each one past the end as a copy of the sample's last (which leaves the group's minimum
// and maximum alone); its codes are cleared.

constexpr int kQpGroupsF16 = 8;   // groups per wavefront
constexpr int kQpStageSlots = 272;   // 16-byte LDS slots per wavefront: the run's 256 pieces and one spare per sixteen

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f16x2 as_f16x2(uint32_t u)
{
    f16x2 v;
    __builtin_memcpy(&v, &u, 4);
    return v;
}

__device__ __forceinline__ uint32_t as_u32(f16x2 v)
{
    uint32_t u;
    __builtin_memcpy(&u, &v, 4);
    return u;
}

template <int CTRL>
__device__ __forceinline__ f16x2 dpp_f16x2(f16x2 v)
{
    return as_f16x2(dpp_u32<CTRL>(as_u32(v)));
}

// Minimum over each eight consecutive lanes, per packed half, in every one of the eight.
__device__ __forceinline__ f16x2 eight_lane_min(f16x2 p)
{
    p = __builtin_elementwise_minimum(p, dpp_f16x2<kDppXor1>(p));
    p = __builtin_elementwise_minimum(p, dpp_f16x2<kDppXor2>(p));
    p = __builtin_elementwise_minimum(p, dpp_f16x2<kDppHalfMirror>(p));
    return p;
}

// fl32(half - z) for the low (HIGH = false) or high half of `word`: one instruction, the half is
// widened by the operand selector.  `one` is 1.0f in a register.
template <bool HIGH>
__device__ __forceinline__ float half_minus(uint32_t word, float one, float neg_z)
{
    float r;
    if (HIGH) asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(word), "v"(one), "v"(neg_z));
    else asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(word), "v"(one), "v"(neg_z));
    return r;
}

// Code of the lane's element j (half j & 1 of loaded word j >> 1, the noise in the same half of
// noise word j >> 1).
template <int B>
__device__ __forceinline__ uint32_t code_f16(const uint32_t (&xw)[16], const uint32_t (&rnd)[16], int j, float one,
                                             float neg_mn, float inv)
{
    constexpr float kB = static_cast<float>((1 << B) - 1);
    const float centred = (j & 1) ? half_minus<true>(xw[j >> 1], one, neg_mn) : half_minus<false>(xw[j >> 1], one, neg_mn);
    float scaled = centred * inv;
    if (B == 8) scaled = fminf(scaled, kB);
    const uint32_t noise = (j & 1) ? rnd[j >> 1] >> 16 : rnd[j >> 1] & 0xffffu;
    return static_cast<uint32_t>(__builtin_fmaf(static_cast<float>(noise), 1.52587890625e-05f, scaled));
}

// The lane's 32 codes, packed LSB first into the B words of `out`.
template <int B>
__device__ __forceinline__ void encode_lane_f16(const uint32_t (&xw)[16], const uint32_t (&rnd)[16], float neg_mn, float inv,
                                                uint32_t (&out)[8])
{
    const float one = 1.0f;
    if constexpr ((B & (B - 1)) == 0) {
        // whole codes per word: word by word, last code first
        constexpr int kPerWord = 32 / B;
#pragma unroll
        for (int w = 0; w < B; ++w) {
            uint32_t acc = 0;
#pragma unroll
            for (int k = kPerWord - 1; k >= 0; --k) {
                const uint32_t q = code_f16<B>(xw, rnd, w * kPerWord + k, one, neg_mn, inv);
                if (k == kPerWord - 1) acc = q;
                else asm("v_lshl_or_b32 %0, %1, %2, %3" : "=v"(acc) : "v"(acc), "n"(B), "v"(q));   // (acc << B) | q, kept one instruction per code
            }
            out[w] = acc;
        }
    } else {
        // codes straddle words
#pragma unroll
        for (int w = 0; w < 8; ++w) out[w] = 0;
#pragma unroll
        for (int j = 0; j < 32; ++j) {
            const uint32_t q = code_f16<B>(xw, rnd, j, one, neg_mn, inv);
            const int w = (j * B) >> 5, sh = (j * B) & 31;
            out[w] |= q << sh;
            if (sh + B > 32) out[w + 1] |= q >> (32 - sh);
            if ((j & 7) == 7) __builtin_amdgcn_sched_barrier(0);   // eight codes at a time keep the temporaries in registers
        }
    }
}

// 4 B bytes of a lane (words w[0 .. B-1]) to a 4-byte aligned address.
template <int B>
__device__ __forceinline__ void store_lane_words(uint8_t* dst, const uint32_t (&w)[8])
{
    typedef u32x4 __attribute__((aligned(4))) u32x4_a4;
    typedef u32x2 __attribute__((aligned(4))) u32x2_a4;
    constexpr int kQuads = B / 4, kRest = B % 4;
#pragma unroll
    for (int h = 0; h < kQuads; ++h) {
        u32x4 v;
        v.x = w[4 * h + 0];
        v.y = w[4 * h + 1];
        v.z = w[4 * h + 2];
        v.w = w[4 * h + 3];
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4_a4*>(dst + 16 * h));
    }
    uint8_t* rest = dst + 16 * kQuads;
    if constexpr (kRest == 1) __builtin_nontemporal_store(w[4 * kQuads], reinterpret_cast<uint32_t*>(rest));
    if constexpr (kRest == 2) {
        u32x2 v;
        v.x = w[4 * kQuads];
        v.y = w[4 * kQuads + 1];
        __builtin_nontemporal_store(v, reinterpret_cast<u32x2_a4*>(rest));
    }
    if constexpr (kRest == 3) {
        u32x2 v;
        v.x = w[4 * kQuads];
        v.y = w[4 * kQuads + 1];
        __builtin_nontemporal_store(v, reinterpret_cast<u32x2_a4*>(rest));
        __builtin_nontemporal_store(w[4 * kQuads + 2], reinterpret_cast<uint32_t*>(rest + 8));
    }
}

template <int B>
__device__ __forceinline__ void encode_store_f16(const uint32_t (&xw)[16], const uint32_t (&rnd)[16], float neg_mn, float inv,
                                                 bool valid, uint8_t* dst, bool clear, int count)
{
    uint32_t w[8];
    encode_lane_f16<B>(xw, rnd, neg_mn, inv, w);
    if (clear) {
#pragma unroll
        for (int k = 0; k < B; ++k) w[k] &= valid_bits<B>(count, k);
    }
    // the words are final here, for every lane: left alone, the compiler moves the encoding under the
    // store's condition but keeps the 32 subtractions in front of it, and their results do not fit the registers
#pragma unroll
    for (int k = 0; k < B; ++k) asm volatile("" : "+v"(w[k]));
    if (valid) store_lane_words<B>(dst, w);
}

// Sixteen bytes at the alignment of an element.
template <typename T> struct Piece;
template <> struct Piece<float> { typedef u32x4 __attribute__((aligned(4))) type; };
template <> struct Piece<_Float16> { typedef u32x4 __attribute__((aligned(2))) type; };

// The 16-byte piece of a short tile that starts at element `first`: elements past the last valid one
// (index `last`) are copies of it.
__device__ __forceinline__ u32x4 guarded_piece(const float* tile, uint32_t first, uint32_t last)
{
    u32x4 v;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = __float_as_uint(tile[min(first + k, last)]);
    return v;
}

__device__ __forceinline__ u32x4 guarded_piece(const _Float16* tile, uint32_t first, uint32_t last)
{
    u32x4 v;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f16x2 h;
        h[0] = tile[min(first + 2 * k, last)];
        h[1] = tile[min(first + 2 * k + 1, last)];
        v[k] = as_u32(h);
    }
    return v;
}

// What a wavefront of the quantizer needs beside its tile.
struct QuantizeArgs {
    uint32_t k0, k1, tag0, tag1;   // Philox key and the tensor's tag
    uint32_t noise_sample;         // index of the sample in the noise counter
    const uint8_t* bits;
    const uint64_t* offsets;
    uint8_t* packed;
    uint64_t capacity;
    void* header;
};

// A run of up to eight groups starting at g0 of sample n.  A sample whose width or byte range is
// invalid is skipped, nothing is written.
template <int HDR, bool RAGGED>
__device__ __forceinline__ void quantize_run_f16(const _Float16* __restrict__ xs, uint32_t n, uint32_t g0, uint64_t D, uint32_t ng,
                                                 int lane, const QuantizeArgs& a, u32x4* stage)
{
    // lane l works on elements 32 (l & 7) .. + 31 of group g0 + (l >> 3): bytes 64 l .. 64 l + 63 of the run
    uint32_t g = g0 + (static_cast<uint32_t>(lane) >> 3);
    const bool valid = g < ng;
    g = valid ? g : ng - 1;
    const uint32_t chunk = (g << 3) + (static_cast<uint32_t>(lane) & 7u);   // 64-byte piece of the sample, four noise counters
    // A run arrives in the order of the addresses (load p takes kilobyte p, lane l its bytes
    // 16 l .. 16 l + 15) and is dealt to the lanes through the LDS further down; loading a lane's own
    // 64 bytes directly costs a third of the kernel's time (121 against 78 us on the ResNet-50 stem
    // tensor: four loads whose lanes are 64 bytes apart touch 32 cache lines each).  Past the end of a
    // sample of whole groups its last piece is repeated, for lanes that store nothing (until then the
    // shorter run was loaded lane by lane: [26212, 1280] 26.8 -> 20.6 us, and in tiles of four groups,
    // binary32 [43688, 768] 45.1 -> 26.7 us).
    const bool full = !RAGGED || (static_cast<uint64_t>(g0 + kQpGroupsF16) << 8) <= D;   // the same for the whole wavefront
    u32x4 x[4];
    if (RAGGED) {
        const _Float16* run = xs + (static_cast<int64_t>(g0) << 8);
        if (full) {
#pragma unroll
            for (int p = 0; p < 4; ++p) x[p] = __builtin_nontemporal_load(reinterpret_cast<const Piece<_Float16>::type*>(run) + (64 * p + lane));
        } else {
            const uint32_t last = static_cast<uint32_t>(D - (static_cast<uint64_t>(g0) << 8)) - 1u;
#pragma unroll
            for (int p = 0; p < 4; ++p) x[p] = guarded_piece(run, static_cast<uint32_t>(8 * (64 * p + lane)), last);
        }
    } else {
        const u32x4* src = reinterpret_cast<const u32x4*>(xs) + (static_cast<int64_t>(g0) << 5);
        const uint32_t last = ((ng - g0) << 5) - 1u;   // the sample's last 16-byte piece
#pragma unroll
        for (int p = 0; p < 4; ++p) x[p] = __builtin_nontemporal_load(src + min(static_cast<uint32_t>(64 * p + lane), last));
    }
    uint32_t width_word = load_readonly(reinterpret_cast<const uint32_t*>(a.bits) + (n >> 2));
    uint64_t off = load_readonly(a.offsets + n);
    // noise: counter = feature index / 8 = 4 chunk and the three after it
    uint32_t rnd[16];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        uint32_t r[4];
        philox4x32_10(4 * chunk + p, a.noise_sample, a.tag0, a.tag1, a.k0, a.k1, r);
#pragma unroll
        for (int k = 0; k < 4; ++k) rnd[4 * p + k] = r[k];
        // one call after the other (interleaved, the four calls' temporaries cost the eighth wavefront per
        // SIMD), and here, in the shadow of the loads, not behind the look at the sample's width
        asm volatile("" : "+v"(rnd[4 * p]), "+v"(rnd[4 * p + 1]), "+v"(rnd[4 * p + 2]), "+v"(rnd[4 * p + 3]));
        __builtin_amdgcn_sched_barrier(0);
    }
    // 16-byte piece i of the run sits at slot i + i / 16: one spare slot per 256 bytes, so that the
    // sixteen lanes the LDS serves at a time hit every bank once on the way in and on the way out
#pragma unroll
    for (int p = 0; p < 4; ++p) stage[68 * p + lane + (lane >> 4)] = x[p];
    wave_lds_handover();
#pragma unroll
    for (int p = 0; p < 4; ++p) x[p] = stage[4 * lane + p + (lane >> 2)];
    uint32_t xw[16];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        xw[4 * p + 0] = x[p].x;
        xw[4 * p + 1] = x[p].y;
        xw[4 * p + 2] = x[p].z;
        xw[4 * p + 3] = x[p].w;
    }
    // lane-local minimum and maximum per packed half, then (min, -max) as one pair over the eight lanes
    f16x2 lo2 = as_f16x2(xw[0]), hi2 = as_f16x2(xw[0]);
#pragma unroll
    for (int k = 1; k < 16; ++k) {
        lo2 = __builtin_elementwise_minimum(lo2, as_f16x2(xw[k]));
        hi2 = __builtin_elementwise_maximum(hi2, as_f16x2(xw[k]));
    }
    f16x2 low, high;
    low[0] = lo2[0]; low[1] = -hi2[0];
    high[0] = lo2[1]; high[1] = -hi2[1];
    const f16x2 fold = eight_lane_min(__builtin_elementwise_minimum(low, high));
    const float mn = static_cast<float>(fold[0]) + 0.0f;   // -0.0 -> +0.0
    const float mx = -static_cast<float>(fold[1]);
    asm volatile("" : "+s"(width_word), "+s"(off));   // the scalar loads are waited for here, behind the noise
    const uint32_t b = (width_word >> ((n & 3u) * 8u)) & 0xffu;
    if (b < 1 || b > 8 || !range_ok(off, static_cast<uint64_t>(ng) * 32u * b, a.capacity)) return;
    const GroupScale s = group_scale<HDR, 8, kDppHalfMirror>(mn, mx, static_cast<float>((1u << b) - 1u), lane, nullptr);
    uint8_t* dst = a.packed + off + static_cast<uint64_t>(chunk) * (4u * b);
    const bool clear = RAGGED && !full;
    const int64_t behind = static_cast<int64_t>(D) - 32 * static_cast<int64_t>(chunk);
    const int count = clear ? static_cast<int>(max(int64_t(0), min(int64_t(32), behind))) : 32;
    switch (b) {
        case 1: encode_store_f16<1>(xw, rnd, -s.zero, s.inv, valid, dst, clear, count); break;
        case 2: encode_store_f16<2>(xw, rnd, -s.zero, s.inv, valid, dst, clear, count); break;
        case 3: encode_store_f16<3>(xw, rnd, -s.zero, s.inv, valid, dst, clear, count); break;
        case 4: encode_store_f16<4>(xw, rnd, -s.zero, s.inv, valid, dst, clear, count); break;
        case 5: encode_store_f16<5>(xw, rnd, -s.zero, s.inv, valid, dst, clear, count); break;
        case 6: encode_store_f16<6>(xw, rnd, -s.zero, s.inv, valid, dst, clear, count); break;
        case 7: encode_store_f16<7>(xw, rnd, -s.zero, s.inv, valid, dst, clear, count); break;
        default: encode_store_f16<8>(xw, rnd, -s.zero, s.inv, valid, dst, clear, count); break;
    }
    if (valid && (lane & 7) == 0) store_header<HDR>(a.header, static_cast<int64_t>(n) * ng + g, s);
}

// ------------------------------------------------------------------------------------
// Everything else -- binary32 input, 24-bit noise, the per-tensor header -- with the same idea for
// tiles of four groups.
//
// A lane works on SIXTEEN consecutive elements, a group is one row of sixteen lanes and a
// wavefront takes the tile's four groups: the tile is loaded in address order and dealt to the
// lanes through the LDS exactly as above.  Sixteen elements are what two Philox calls serve with
// 16-bit noise and four with 24-bit noise, so again nothing is traded between lanes; the
// reduction is four row-local lane permutations on the lane's own minimum and maximum; the
// division pair is per row.  A lane's sixteen codes are 2 B consecutive bytes of the bit stream:
// two neighbouring lanes join theirs (for odd B the odd lane's bits are moved up by sixteen) and
// the even lane stores the 4 B bytes.
// The clamp stays for every width: B / R can be subnormal for a binary32 range, and then the
// bound used above for binary16 input does not hold, nor does it for a range the caller gives.
// Minimum over the sixteen lanes of each row, in every lane of the row.
__device__ __forceinline__ float row_min_f32(float v)
{
    v = fminf(v, dpp_f32<kDppXor1>(v));
    v = fminf(v, dpp_f32<kDppXor2>(v));
    v = fminf(v, dpp_f32<kDppHalfMirror>(v));
    v = fminf(v, dpp_f32<kDppXor8>(v));
    return v;
}

// Code of element j of the lane.  16-bit noise: half j & 1 of noise word j >> 1; 24-bit noise: the
// upper 24 bits of noise word j.
template <int NOISE_BITS, int B>
__device__ __forceinline__ uint32_t tile_code(float x, const uint32_t* rnd, int j, float mn, float inv)
{
    constexpr float kB = static_cast<float>((1 << B) - 1);
    const float centred = x - mn;
    float scaled = centred * inv;
    scaled = fminf(scaled, kB);  // the two roundings can overshoot B by an ulp
    if (NOISE_BITS == 16) {
        const uint32_t noise = (j & 1) ? rnd[j >> 1] >> 16 : rnd[j >> 1] & 0xffffu;
        return static_cast<uint32_t>(__builtin_fmaf(static_cast<float>(noise), 1.52587890625e-05f, scaled));
    }
    const float frac = __builtin_amdgcn_fractf(scaled);  // exact for scaled >= 0
    const uint32_t q = static_cast<uint32_t>(scaled);    // truncation = floor
    return q + ((static_cast<float>(rnd[j] >> 8) < frac * 16777216.0f) ? 1u : 0u);
}

// The lane's sixteen codes, packed LSB first: 16 B bits in out[0 .. (B + 1) / 2 - 1], upper bits zero.
template <int NOISE_BITS, int B>
__device__ __forceinline__ void encode_lane_tile(const float (&v)[16], const uint32_t* rnd, float mn, float inv, uint32_t (&out)[4])
{
#pragma unroll
    for (int w = 0; w < 4; ++w) out[w] = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const uint32_t q = tile_code<NOISE_BITS, B>(v[j], rnd, j, mn, inv);
        const int w = (j * B) >> 5, sh = (j * B) & 31;
        out[w] |= q << sh;
        if (sh + B > 32) out[w + 1] |= q >> (32 - sh);
    }
}

template <int NOISE_BITS, int B>
__device__ __forceinline__ void encode_store_tile(const float (&v)[16], const uint32_t* rnd, float mn, float inv,
                                                  bool valid, int lane, uint8_t* dst_pair, bool clear, int count)
{
    uint32_t own[4];
    encode_lane_tile<NOISE_BITS, B>(v, rnd, mn, inv, own);
    constexpr int kOwn = (B + 1) / 2;   // words that hold the lane's 16 B bits
    if (clear) {
#pragma unroll
        for (int k = 0; k < kOwn; ++k) own[k] &= valid_bits<B>(count, k);
    }
    uint32_t nb[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < kOwn; ++k) nb[k] = dpp_u32<kDppXor1>(own[k]);   // the neighbour's words (used by the even lane)
    uint32_t w[8];
    if (B % 2 == 0) {
#pragma unroll
        for (int k = 0; k < kOwn; ++k) {
            w[k] = own[k];
            w[kOwn + k] = nb[k];
        }
    } else {
        // own bits end in the middle of word kOwn - 1: the neighbour's follow from bit 16 of it
#pragma unroll
        for (int k = 0; k < kOwn - 1; ++k) w[k] = own[k];
        w[kOwn - 1] = own[kOwn - 1] | (nb[0] << 16);
#pragma unroll
        for (int k = 0; k + 1 < kOwn; ++k) w[kOwn + k] = __builtin_amdgcn_alignbit(nb[k + 1], nb[k], 16);
    }
    // the words are final here, for every lane (see encode_store_f16)
#pragma unroll
    for (int k = 0; k < B; ++k) asm volatile("" : "+v"(w[k]));
    if (valid && (lane & 1) == 0) store_lane_words<B>(dst_pair, w);
}

// The tile of up to four groups starting at g0 of sample n.  A sample whose width or byte
// range is invalid is skipped, nothing is written.
template <typename T, int NOISE_BITS, int HDR, bool RAGGED>
__device__ __forceinline__ void quantize_tile(const T* __restrict__ xs, uint32_t n, uint32_t g0, uint64_t D, uint32_t ng,
                                              int lane, const QuantizeArgs& a, u32x4* stage)
{
    constexpr int kE = 16 / static_cast<int>(sizeof(T));   // elements per 16-byte piece
    constexpr int kP = 16 / kE;                            // pieces per lane
    // lane l works on elements 16 (l & 15) .. + 15 of group g0 + (l >> 4)
    uint32_t g = g0 + (static_cast<uint32_t>(lane) >> 4);
    const bool valid = g < ng;
    g = valid ? g : ng - 1;
    const uint32_t chunk = (g << 4) + (static_cast<uint32_t>(lane) & 15u);   // sixteen elements of the sample
    const bool full = !RAGGED || (static_cast<uint64_t>(g0 + kTileGroups) << 8) <= D;   // the same for the whole wavefront
    u32x4 x[kP];
    if (RAGGED) {
        const T* tile = xs + (static_cast<int64_t>(g0) << 8);
        if (full) {
#pragma unroll
            for (int p = 0; p < kP; ++p) x[p] = __builtin_nontemporal_load(reinterpret_cast<const typename Piece<T>::type*>(tile) + (64 * p + lane));
        } else {
            const uint32_t last = static_cast<uint32_t>(D - (static_cast<uint64_t>(g0) << 8)) - 1u;
#pragma unroll
            for (int p = 0; p < kP; ++p) x[p] = guarded_piece(tile, static_cast<uint32_t>(kE * (64 * p + lane)), last);
        }
    } else {
        const u32x4* src = reinterpret_cast<const u32x4*>(xs) + static_cast<int64_t>(g0) * (16 * kP);
        const uint32_t last = (ng - g0) * (16 * kP) - 1u;   // the sample's last 16-byte piece
#pragma unroll
        for (int p = 0; p < kP; ++p) x[p] = __builtin_nontemporal_load(src + min(static_cast<uint32_t>(64 * p + lane), last));
    }
    uint32_t width_word = load_readonly(reinterpret_cast<const uint32_t*>(a.bits) + (n >> 2));
    uint64_t off = load_readonly(a.offsets + n);
    // noise: counter = feature index / 8 (16-bit noise: two calls) or / 4 (24-bit noise: four calls)
    constexpr int kCalls = NOISE_BITS == 16 ? 2 : 4;
    uint32_t rnd[4 * kCalls];
#pragma unroll
    for (int p = 0; p < kCalls; ++p) {
        uint32_t r[4];
        philox4x32_10(kCalls * chunk + p, a.noise_sample, a.tag0, a.tag1, a.k0, a.k1, r);
#pragma unroll
        for (int k = 0; k < 4; ++k) rnd[4 * p + k] = r[k];
        // one call after the other, in the shadow of the loads (see quantize_run_f16)
        asm volatile("" : "+v"(rnd[4 * p]), "+v"(rnd[4 * p + 1]), "+v"(rnd[4 * p + 2]), "+v"(rnd[4 * p + 3]));
        __builtin_amdgcn_sched_barrier(0);
    }
    // piece i of the tile at slot i + i / 16 (see quantize_run_f16)
#pragma unroll
    for (int p = 0; p < kP; ++p) stage[68 * p + lane + (lane >> 4)] = x[p];
    wave_lds_handover();
#pragma unroll
    for (int p = 0; p < kP; ++p) x[p] = stage[kP * lane + p + lane * kP / 16];
    float v[16];
#pragma unroll
    for (int p = 0; p < kP; ++p)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (sizeof(T) == 4) {
                v[4 * p + k] = __uint_as_float(x[p][k]);
            } else {
                const f16x2 h = as_f16x2(x[p][k]);
                v[(8 * p + 2 * k) & 15] = static_cast<float>(h[0]);
                v[(8 * p + 2 * k + 1) & 15] = static_cast<float>(h[1]);
            }
        }
    float mn = 0.0f, mx = 0.0f;
    if (HDR != 2) {
        float lo = v[0], hi = v[0];
#pragma unroll
        for (int k = 1; k < 16; ++k) {
            lo = fminf(lo, v[k]);
            hi = fmaxf(hi, v[k]);
        }
        mn = row_min_f32(lo) + 0.0f;   // -0.0 -> +0.0
        mx = -row_min_f32(-hi);
    }
    asm volatile("" : "+s"(width_word), "+s"(off));   // the scalar loads are waited for here, behind the noise
    const uint32_t b = (width_word >> ((n & 3u) * 8u)) & 0xffu;
    if (b < 1 || b > 8 || !range_ok(off, static_cast<uint64_t>(ng) * 32u * b, a.capacity)) return;
    const GroupScale s = group_scale<HDR, 16, kDppXor8>(mn, mx, static_cast<float>((1u << b) - 1u), lane, a.header);
    // the even lane of a pair stores both lanes' bytes: 4 b bytes from byte 2 b chunk of the sample's stream
    uint8_t* dst = a.packed + off + static_cast<uint64_t>(chunk) * (2u * b);
    const bool clear = RAGGED && !full;
    const int64_t behind = static_cast<int64_t>(D) - 16 * static_cast<int64_t>(chunk);
    const int count = clear ? static_cast<int>(max(int64_t(0), min(int64_t(16), behind))) : 16;
    switch (b) {
        case 1: encode_store_tile<NOISE_BITS, 1>(v, rnd, s.zero, s.inv, valid, lane, dst, clear, count); break;
        case 2: encode_store_tile<NOISE_BITS, 2>(v, rnd, s.zero, s.inv, valid, lane, dst, clear, count); break;
        case 3: encode_store_tile<NOISE_BITS, 3>(v, rnd, s.zero, s.inv, valid, lane, dst, clear, count); break;
        case 4: encode_store_tile<NOISE_BITS, 4>(v, rnd, s.zero, s.inv, valid, lane, dst, clear, count); break;
        case 5: encode_store_tile<NOISE_BITS, 5>(v, rnd, s.zero, s.inv, valid, lane, dst, clear, count); break;
        case 6: encode_store_tile<NOISE_BITS, 6>(v, rnd, s.zero, s.inv, valid, lane, dst, clear, count); break;
        case 7: encode_store_tile<NOISE_BITS, 7>(v, rnd, s.zero, s.inv, valid, lane, dst, clear, count); break;
        default: encode_store_tile<NOISE_BITS, 8>(v, rnd, s.zero, s.inv, valid, lane, dst, clear, count); break;
    }
    if (HDR != 2 && valid && (lane & 15) == 0) store_header<HDR>(a.header, static_cast<int64_t>(n) * ng + g, s);
}

// ------------------------------------------------------------------------------------
// Sec. 4.1: h^ = code * scale + Z.

// binary32 at eight bits, where a fifth of the traffic are codes that come in: the last store of a wavefront
// goes out when the others have been acknowledged ([128, 802816] 85 -> 82 us).  At two bits the same wait
// costs 9 %; binary16 is paced by its loads instead (dequantize_pairs_f16).
__device__ __forceinline__ void wait_for_stores()
{
    constexpr int kVmcnt0 = 0x0F70;   // vmcnt(0), the other counters as they are
    __builtin_amdgcn_s_waitcnt(kVmcnt0);
}

// Ends the code of one width with something no other width's code ends with.  Left alone, the compiler
// shares the last store of all widths behind a jump, and there it waits for every load and store that
// any of them may have in flight (139 -> 152 us at B = 2 with the bfloat16 header on binary32 [256, 802816]).
template <int B>
__device__ __forceinline__ void end_of_width()
{
    asm volatile("; end of width %0" ::"n"(B));
}

// NG consecutive groups of one sample.  FULL: all of them are present and whole, and the code is
// straight-line: every load is issued before the first store and nothing branches in between.  (A
// branch around a load or a store makes the compiler wait for *all* outstanding vector memory
// operations where the paths join -- and on this target a store counts until it is acknowledged, so
// the stores of a wavefront would go out one at a time.)  Otherwise (the last run of a sample)
// groups past the end repeat the loads of the sample's last group, all values are computed, and
// then what exists is stored.
template <typename T, int LAYOUT, bool FULL, int B, int HDR, int NG>
__device__ __forceinline__ void dequantize_groups(const uint8_t* __restrict__ src_sample,
                                                  const void* __restrict__ header, T* __restrict__ os,
                                                  int64_t D, uint32_t n, uint32_t g0, uint32_t ng, int lane, uint32_t* stage)
{
    // A lane's four codes are the 4 * B bits that start at bit 4 * B * lane of the group.  If B divides 8
    // they lie inside one aligned 32-bit word.  Otherwise they lie inside the word that starts at the byte
    // of their first bit (at most 28 bits, 4 of them skipped), kept inside the group at its end; a full run
    // then brings its bit stream (NG * 32 * B contiguous bytes) in with coalesced word loads and picks
    // those words from the wavefront's LDS slice (direct loads at any byte: 287 -> 354 us at B = 3 on
    // binary32 [256, 1605632]).
    constexpr uint32_t code_mask = (1u << B) - 1u;
    constexpr bool kAligned = (8 % B) == 0;
    constexpr bool kStaged = FULL && !kAligned;
    const uint32_t first_bit = static_cast<uint32_t>(lane) * (4u * B);
    const uint32_t byte = kAligned ? first_bit >> 5 << 2 : min(first_bit >> 3, 32u * B - 4u);
    const uint32_t shift = first_bit - 8u * byte;
    uint32_t word[NG];
    f32x2 hd[NG];
    const uint32_t vzero = vector_zero();
    // bases of the run: the groups are constant offsets from them (address arithmetic per group cost 2 %)
    const uint8_t* run_src = src_sample + static_cast<uint64_t>(g0) * (32 * B);
    const int64_t hdr0 = static_cast<int64_t>(n) * ng + g0;
    const int64_t d_run = (static_cast<int64_t>(g0) << 8) + lane * 4;
    T* run_out = os + d_run;
    const uint32_t last = ng - 1u - g0;
#pragma unroll
    for (int u = 0; u < NG; ++u) {
        const uint32_t at = FULL ? static_cast<uint32_t>(u) : min(static_cast<uint32_t>(u), last);
        const uint8_t* src = run_src + at * (32u * B) + byte;
        if constexpr (kStaged) word[u] = 0;
        else if constexpr (kAligned) word[u] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(src));
        else word[u] = __builtin_nontemporal_load(reinterpret_cast<const word_a1*>(src));
        const int64_t index = hdr0 + at;
        hd[u] = load_header_vector<HDR>(header, index, static_cast<float>(code_mask), vzero);
    }
    if constexpr (kStaged) {
        constexpr int kWords = NG * 8 * B;
        constexpr int kLoads = (kWords + 63) / 64;
        static_assert(kLoads * 64 <= 256, "the slice holds 256 words");
        uint32_t in[kLoads];
#pragma unroll
        for (int j = 0; j < kLoads; ++j)   // lanes past the end re-read the last word
            in[j] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(run_src) + min(j * 64 + lane, kWords - 1));
#pragma unroll
        for (int j = 0; j < kLoads; ++j) stage[j * 64 + lane] = in[j];
        wave_lds_handover();
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            const uint32_t at = u * (8 * B) + (first_bit >> 5);
            // past the last word of the run the neighbour is not used: those lanes' bits end with the word
            word[u] = __builtin_amdgcn_alignbit(stage[at + 1 < 256u ? at + 1 : 255u], stage[at], first_bit & 31u);
        }
        wave_lds_handover();
    }
    // The divisions of the bfloat16 header come before the first store: with two of them behind it the stores leave
    // less evenly (b = 2 on [128, 802816]: 78 against 73.7 us).  Samples that end inside a group, stored in another
    // order, are 6 % slower with it ([256, 501861] 100 -> 107 us).
    if constexpr (FULL && HDR == 1 && LAYOUT == kWholeGroups) {
#pragma unroll
        for (int u = 0; u < NG; ++u) asm volatile("" : "+v"(hd[u].y));
    }
    float o[NG][4];
#pragma unroll
    for (int u = 0; u < NG; ++u) {
        const uint32_t piece = kStaged ? word[u] : word[u] >> shift;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t q = (piece >> (k * B)) & code_mask;
            o[u][k] = __builtin_fmaf(static_cast<float>(q), hd[u].y, hd[u].x);
        }
        if (FULL && B == 8 && u == NG - 1) wait_for_stores();
        if (FULL) store4<T, LAYOUT>(run_out + u * 256, o[u]);
    }
    if (FULL) {
        end_of_width<B>();
        return;
    }
#pragma unroll
    for (int u = 0; u < NG; ++u) asm volatile("" : "+v"(o[u][0]), "+v"(o[u][1]), "+v"(o[u][2]), "+v"(o[u][3]));
#pragma unroll
    for (int u = 0; u < NG; ++u) {
        const int64_t d0 = d_run + u * 256;
        if (d0 + 4 <= D) {
            store4<T, LAYOUT>(run_out + u * 256, o[u]);
        } else if (LAYOUT != kWholeGroups) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (d0 + k < D) run_out[u * 256 + k] = Io<T>::narrow(o[u][k]);
        }
    }
}

// binary16 output: a lane that owned four elements would store only 8 bytes, so here a lane
// takes eight consecutive elements (16 bytes) and the wavefront covers two groups per step
// (lanes 0..31 the even group, lanes 32..63 the odd one).  Unpacking is free to choose its
// lane-to-element map: nothing is reduced across lanes.
template <int LAYOUT, bool FULL, int B, int HDR, int NP>
__device__ __forceinline__ void dequantize_pairs_f16(const uint8_t* __restrict__ src_sample,
                                                     const void* __restrict__ header,
                                                     _Float16* __restrict__ os, int64_t D, uint32_t n, uint32_t g0,
                                                     uint32_t ng, int lane)
{
    typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
    typedef f16x8 __attribute__((aligned(2))) f16x8_unaligned;
    const auto store = [](_Float16* at, f16x8 v) {
        if constexpr (LAYOUT == kWholeGroups) __builtin_nontemporal_store(v, reinterpret_cast<f16x8*>(at));
        else if constexpr (LAYOUT == kRaggedLines) __builtin_nontemporal_store(v, reinterpret_cast<f16x8_unaligned*>(at));
        else *reinterpret_cast<f16x8_unaligned*>(at) = v;
    };
    constexpr uint32_t code_mask = (1u << B) - 1u;
    const uint32_t half = static_cast<uint32_t>(lane) >> 5;   // which group of the pair
    const uint32_t li = static_cast<uint32_t>(lane) & 31u;    // position inside the group: elements 8*li .. 8*li+7
    // The lane's 8 * B bits are bytes li * B .. + B - 1 of the group: one 32-bit word (B <= 4) or 64-bit
    // word (B > 4) holds them.  The word is the aligned one around them where there is one, otherwise it
    // starts with them, kept inside the group at its end.
    constexpr bool kWide = B > 4;
    const uint32_t byte = B == 8 ? li * 8u : (kWide ? min(li * B, 32u * B - 8u) : (B == 3 ? min(li * B, 32u * B - 4u) : li * B & ~3u));
    const uint32_t shift = 8u * (li * B - byte);
    uint32_t code[NP], code_hi[NP];   // the high word for B > 4 only
    f32x2 hd[NP];
    // bases of the run, as above
    const uint8_t* run_src = src_sample + static_cast<uint64_t>(g0) * (32 * B);
    const int64_t hdr0 = static_cast<int64_t>(n) * ng + g0;
    const int64_t d_run = (static_cast<int64_t>(g0 + half) << 8) + li * 8;
    _Float16* run_out = os + d_run;
    const uint32_t last = ng - 1u - g0;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint32_t at = FULL ? 2 * p + half : min(2 * p + half, last);
        const uint8_t* src = run_src + (FULL ? static_cast<uint32_t>(2 * p) * (32u * B) + (half * (32u * B) + byte) : at * (32u * B) + byte);
        if constexpr (kWide) {
            u32x2 w;
            if constexpr (B == 8) w = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(src));
            else w = __builtin_nontemporal_load(reinterpret_cast<const words_a1*>(src));
            code[p] = w.x;
            code_hi[p] = w.y;
        } else if constexpr (B == 3) {
            code[p] = __builtin_nontemporal_load(reinterpret_cast<const word_a1*>(src));
            code_hi[p] = 0;
        } else {
            code[p] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(src));
            code_hi[p] = 0;
        }
        // both groups' headers through the scalar data path (their indices are uniform), then the
        // lane's half picks one: a per-lane load would be a second vector load in front of each store
        const uint32_t even = 2 * p, odd = 2 * p + 1;
        const f32x2 hd_even = load_header<HDR>(header, hdr0 + (FULL ? even : min(even, last)), static_cast<float>(code_mask));
        const f32x2 hd_odd = load_header<HDR>(header, hdr0 + (FULL ? odd : min(odd, last)), static_cast<float>(code_mask));
        hd[p].x = half ? hd_odd.x : hd_even.x;
        hd[p].y = half ? hd_odd.y : hd_even.y;
        // At eight bits, where a third of the traffic are codes, a pair's loads stay one behind the other and its
        // store leaves when they are there (all loads first, all waited for: [256, 802816] 98.5 against 96.3 us with
        // the binary32 header, 98.0 against 95.9 with the bfloat16 header; [128, 802816] 51.7 against 50.5).
        if (FULL && B == 8) __builtin_amdgcn_sched_barrier(0);
    }
    // Otherwise all loads are waited for before the first store: the four stores of a wavefront then leave together.
    // (As each load arrives: 76.9 against 73.6 us at B = 1, 78.3 against 76.9 us with mixed widths on [256, 802816].)
    if constexpr (NP == 4 && B != 8) asm volatile("" : "+v"(code[0]), "+v"(code[1]), "+v"(code[2]), "+v"(code[3]));
    f16x8 o[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint64_t mine = kWide ? ((static_cast<uint64_t>(code_hi[p]) << 32) | code[p]) >> shift : static_cast<uint64_t>(code[p] >> shift);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t q = static_cast<uint32_t>(mine >> (k * B)) & code_mask;
            o[p][k] = Io<_Float16>::narrow(__builtin_fmaf(static_cast<float>(q), hd[p].y, hd[p].x));
        }
        if (FULL) store(run_out + p * 512, o[p]);
    }
    if (FULL) {
        end_of_width<B>();
        return;
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        u32x4 w;
        __builtin_memcpy(&w, &o[p], 16);
        asm volatile("" : "+v"(w));
        __builtin_memcpy(&o[p], &w, 16);
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int64_t d0 = d_run + p * 512;
        if (d0 + 8 <= D) {
            store(run_out + p * 512, o[p]);
        } else if (LAYOUT != kWholeGroups) {
#pragma unroll
            for (int k = 0; k < 7; ++k)
                if (d0 + k < D) run_out[p * 512 + k] = o[p][k];
        }
    }
}

// The run of up to NG groups that starts at g0.  One or two groups that are left of a sample of whole groups are a run
// of their own length: with NG loads and headers of which most repeat the last group's, and a branch before each store,
// samples of one group took longer than those of four by more than the accesses explain (mixed widths, 134 MB of
// binary32: [131072, 256] 61.6 -> 48.0 us, [65536, 512] 41.7 -> 34.1, [26212, 1280] 39.5 -> 36.5; binary16 with the
// bfloat16 header 57.1 -> 37.0 and 33.0 -> 23.4 us).
template <typename T, int LAYOUT, int B, int HDR, int NG>
__device__ __forceinline__ void dequantize_run(const uint8_t* __restrict__ src_sample,
                                               const void* __restrict__ header, T* __restrict__ os,
                                               int64_t D, uint32_t n, uint32_t g0, uint32_t ng, int lane, uint32_t* stage)
{
    const bool full = (static_cast<int64_t>(g0 + NG) << 8) <= D;
    if constexpr (sizeof(T) == 2) {
        static_assert(NG % 2 == 0, "pairs of groups");
        if (full) dequantize_pairs_f16<LAYOUT, true, B, HDR, NG / 2>(src_sample, header, os, D, n, g0, ng, lane);
        else if (LAYOUT == kWholeGroups && ng - g0 <= 2)
            dequantize_pairs_f16<LAYOUT, false, B, HDR, 1>(src_sample, header, os, D, n, g0, ng, lane);
        else dequantize_pairs_f16<LAYOUT, false, B, HDR, NG / 2>(src_sample, header, os, D, n, g0, ng, lane);
    } else {
        if (full) dequantize_groups<T, LAYOUT, true, B, HDR, NG>(src_sample, header, os, D, n, g0, ng, lane, stage);
        else if (LAYOUT == kWholeGroups && ng - g0 == 1)
            dequantize_groups<T, LAYOUT, true, B, HDR, 1>(src_sample, header, os, D, n, g0, ng, lane, stage);
        else if (LAYOUT == kWholeGroups && ng - g0 == 2)
            dequantize_groups<T, LAYOUT, true, B, HDR, 2>(src_sample, header, os, D, n, g0, ng, lane, stage);
        else dequantize_groups<T, LAYOUT, false, B, HDR, NG>(src_sample, header, os, D, n, g0, ng, lane, stage);
    }
}

// ------------------------------------------------------------------------------------
// Several tensors in one launch.  A network saves dozens of activations of very different
// sizes (a ResNet-50 step: 53, from 26 MB to 822 MB at batch 256); one launch per tensor leaves
// the chip draining and refilling 53 times per pass, and the small tensors cannot fill it at
// all.  Here blockIdx.y is the tensor and blockIdx.x runs over its tiles, sample after sample
// (in an order that depends on the kernel, see wave_unit), so the launch walks HBM like
// back-to-back single-tensor launches, without the gaps.  grid.x is sized for the largest
// tensor of the call and the surplus blocks of smaller ones exit at once, so a call should
// group tensors of similar size.  The start of a wavefront is short: one batch of scalar loads
// for the tensor's item from the kernel arguments, one for the sample's width and offset, then
// the data; a multiply-high division splits the linear tile index into sample and tile.
// (Measured alternatives on the 53-tensor sweep: samples in grid.y with all tensors' tiles side
// by side in grid.x -- 53 concurrent streams -- made every kernel 5-20 % slower than single
// launches; one linear grid over all tensors with a ballot over prefix sums to find the tensor
// costs a vector load at the start of every wavefront, which the write-bound dequantizer does
// not hide: 83 against 73 us on the stage-1 tensor.)
// A single tensor is a launch with a table of one (against samples in grid.y: group_stats 65 -> 63 us,
// unpack_dequantize 79.3 -> 72.9 us on the stage-1 tensor).  All tensors have the same N, dtype and header
// format.  RAGGED kernels take a tensor whose samples end in a part of a group (single tensors only).

struct MultiItem {
    const void* x;            // input of group_stats / quantize_pack
    void* out;                // output of unpack_dequantize
    float* gmin;              // outputs of group_stats
    float* grange;
    void* header;
    const uint8_t* bits;
    const uint64_t* offsets;
    int64_t D;
    FastDiv by_tiles;         // division by the tiles of one sample
    uint32_t tiles;           // tiles of one sample
    uint32_t total_tiles;     // N * tiles
};

// The table travels by value in the kernel arguments; a table of one (most calls) is a launch of its own
// kind, because 40 items are 3.2 kB of arguments, 0.5 us of the 4 us that a launch costs the host.
template <int CAPACITY>
struct MultiTable {
    uint32_t first_sample;    // index of the table's first sample in the noise counter
    uint32_t first_tile;      // of every tensor, where a launch starts
    MultiItem item[CAPACITY];
};

// Linear work index of wavefront `wave` of block `bx`.  Blocks are handed to the eight XCDs in
// turn, so block bx runs on XCD bx % 8 (grid.x is a multiple of 8 * RUN).
// XCD_MAP 0: RUN consecutive blocks' worth of units (RUN * WAVES units) stay on one XCD -- RUN = 1
//   is the plain order, block bx takes units bx * WAVES ...  A longer run keeps whole cache lines
//   of the small per-group outputs inside one XCD's L2, so that they reach HBM as fewer, fuller writes.
// XCD_MAP 1: every run of 8 blocks shares 8 * WAVES consecutive units and block bx takes the
//   units congruent to bx modulo 8: each XCD then writes every eighth unit of the stream.
template <int WAVES, int XCD_MAP, int RUN = 1>
__device__ __forceinline__ uint32_t wave_unit(uint32_t bx, uint32_t wave)
{
    if (XCD_MAP == 1) return (bx >> 3) * (8 * WAVES) + (bx & 7u) + 8 * wave;
    if (RUN > 1) {
        const uint32_t k = bx >> 3;   // position among the blocks of this XCD
        return (((k / RUN) * 8 + (bx & 7u)) * RUN + (k % RUN)) * WAVES + wave;
    }
    return bx * WAVES + wave;
}

// Makes the listed scalar values live at this point of the program: every scalar load that
// produces them has been issued, and is waited for, here -- as one batch.  Left to itself the
// compiler fetches each field of a table item, and each of widths and offsets, right where it
// is first used, which strings four to six dependent scalar memory round trips in front of the
// first vector load of a wavefront.
#define ACTQ_SCALAR_BATCH2(a, b) asm volatile("" : "+s"(a), "+s"(b))
#define ACTQ_SCALAR_BATCH10(a, b, c, d, e, f, g, h, i, j) \
    asm volatile("" : "+s"(a), "+s"(b), "+s"(c), "+s"(d), "+s"(e), "+s"(f), "+s"(g), "+s"(h), "+s"(i), "+s"(j))

// What a wavefront of a multi-tensor launch knows after one batch of scalar loads from the
// table: its sample and its run of groups inside the sample, and the tensor's pointers.
struct MultiCursor {
    uint32_t n, tile;        // sample, run of groups inside the sample
    uint64_t D;
    uintptr_t x, out, header, gmin, grange, bits, offsets;
};

// A pointer that went through an integer register has lost its address space, and the compiler
// would emit flat memory instructions for it (which also tick the LDS counter).  Everything the
// table points to is device memory: the pointer is rebuilt as a global one, and the conversion
// to a generic pointer lets the compiler carry that knowledge to every use.
template <typename P>
__device__ __forceinline__ P* device_pointer(uintptr_t a)
{
    typedef P __attribute__((address_space(1))) * global_pointer;
    return (P*)((global_pointer)a);
}

// False: the wavefront has no work.  XCD_MAP: the order of wave_unit.
template <int WAVES_PER_BLOCK, int XCD_MAP, int RUN, int CAPACITY>
__device__ __forceinline__ bool multi_cursor(const MultiTable<CAPACITY>& t, uint32_t wave, MultiCursor& c)
{
    const MultiItem& it = t.item[CAPACITY == 1 ? 0 : blockIdx.y];
    const uint32_t lin = t.first_tile + wave_unit<WAVES_PER_BLOCK, XCD_MAP, RUN>(blockIdx.x, wave);
    // tiles: low word the runs per sample, high word all runs of the tensor
    uint64_t tiles = (static_cast<uint64_t>(it.total_tiles) << 32) | it.tiles;
    uint64_t div = (static_cast<uint64_t>(it.by_tiles.s) << 32) | it.by_tiles.m;
    c.D = static_cast<uint64_t>(it.D);
    c.x = reinterpret_cast<uintptr_t>(it.x);
    c.out = reinterpret_cast<uintptr_t>(it.out);
    c.header = reinterpret_cast<uintptr_t>(it.header);
    c.gmin = reinterpret_cast<uintptr_t>(it.gmin);
    c.grange = reinterpret_cast<uintptr_t>(it.grange);
    c.bits = reinterpret_cast<uintptr_t>(it.bits);
    c.offsets = reinterpret_cast<uintptr_t>(it.offsets);
    ACTQ_SCALAR_BATCH10(tiles, div, c.D, c.x, c.out, c.header, c.gmin, c.grange, c.bits, c.offsets);
    if (lin >= static_cast<uint32_t>(tiles >> 32)) return false;
    c.n = (__umulhi(lin, static_cast<uint32_t>(div)) + lin) >> static_cast<uint32_t>(div >> 32);
    c.tile = lin - c.n * static_cast<uint32_t>(tiles);
    return true;
}

// Width and byte offset of the cursor's sample, as one batch of scalar loads.
__device__ __forceinline__ void sample_width_offset(const MultiCursor& c, uint32_t& b, uint64_t& off)
{
    uint32_t width_word = load_readonly(reinterpret_cast<const uint32_t*>(c.bits) + (c.n >> 2));
    off = load_readonly(reinterpret_cast<const uint64_t*>(c.offsets) + c.n);
    ACTQ_SCALAR_BATCH2(width_word, off);
    b = (width_word >> ((c.n & 3u) * 8u)) & 0xffu;
}


// Sec. 4.1: Z = min, R = max - min per group; one tile of four groups per wavefront.  NT: non-temporal loads.  RUN: consecutive workgroups' tiles per XCD.
template <typename T, bool RAGGED, bool NT, int CAPACITY, int RUN = kGsRun>
__global__ __launch_bounds__(kGsBlock) void group_stats_multi_kernel(MultiTable<CAPACITY> t)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));
    MultiCursor c;
    if (!multi_cursor<kGsBlock / kWave, kGsXcdMap, RUN, CAPACITY>(t, wave, c)) return;
    const uint32_t ng = static_cast<uint32_t>((c.D + (kGroup - 1)) >> 8);
    const uint32_t g0 = c.tile * kTileGroups;
    const T* tile = device_pointer<const T>(c.x) + (static_cast<int64_t>(c.n) * static_cast<int64_t>(c.D) + (static_cast<int64_t>(g0) << 8));
    float v[kTileGroups][4];
    if (!RAGGED || (static_cast<uint64_t>(g0 + kTileGroups) << 8) <= c.D) {
#pragma unroll
        for (int u = 0; u < kTileGroups; ++u)   // a group past the end of the sample re-reads the tile's first (its results are not stored)
            load4<T, !RAGGED, NT>(tile + ((RAGGED || g0 + u < ng ? u << 8 : 0) + lane * 4), v[u]);
    } else {
        // the tile in which the sample ends: elements past the end are copies of its last one
        const uint32_t last = static_cast<uint32_t>(c.D - (static_cast<uint64_t>(g0) << 8)) - 1u;
#pragma unroll
        for (int u = 0; u < kTileGroups; ++u)
#pragma unroll
            for (int k = 0; k < 4; ++k) v[u][k] = static_cast<float>(tile[min(static_cast<uint32_t>((u << 8) + lane * 4 + k), last)]);
    }
    float lo[kTileGroups], hi[kTileGroups];
    lane_min_max(v, lo, hi);
    float mn, mx;
    tile_min_max(lo, hi, lane, mn, mx);
    mn += 0.0f;  // -0.0 -> +0.0
    const uint32_t g = g0 + (static_cast<uint32_t>(lane) >> 4);
    if ((lane & 15) == 0 && g < ng) {
        const int64_t gi = static_cast<int64_t>(c.n) * ng + g;
        device_pointer<float>(c.gmin)[gi] = mn;
        device_pointer<float>(c.grange)[gi] = (mx - mn) + 0.0f;  // a zero range is +0.0 whichever zeros the extremes were
    }
}

template <int CAPACITY>
__device__ __forceinline__ QuantizeArgs quantize_args(const MultiTable<CAPACITY>& t, const MultiCursor& c, uint32_t k0, uint32_t k1, uint64_t tag,
                                                      uint8_t* packed, uint64_t capacity)
{
    const uint64_t tensor_tag = tag + blockIdx.y;  // every tensor of the launch draws its own noise
    QuantizeArgs a;
    a.k0 = k0;
    a.k1 = k1;
    a.tag0 = static_cast<uint32_t>(tensor_tag);
    a.tag1 = static_cast<uint32_t>(tensor_tag >> 32);
    a.noise_sample = t.first_sample + c.n;
    a.bits = device_pointer<const uint8_t>(c.bits);
    a.offsets = device_pointer<const uint64_t>(c.offsets);
    a.packed = packed;
    a.capacity = capacity;
    a.header = device_pointer<void>(c.header);
    return a;
}

// Runs of kQpGroupsF16 groups (the table is built for runs of that length).  Eight wavefronts per SIMD
// are asked for: the kernel lives on other wavefronts' issue slots while one waits for its loads.
template <int HDR, bool RAGGED, int CAPACITY>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void quantize_pack_run_kernel(
    MultiTable<CAPACITY> t, uint32_t k0, uint32_t k1, uint64_t tag, uint8_t* __restrict__ packed, uint64_t capacity)
{
    __shared__ u32x4 stage_all[kWavesPerBlock][kQpStageSlots];
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));
    MultiCursor c;
    if (!multi_cursor<kWavesPerBlock, kQpXcdMap, kQpRun, CAPACITY>(t, wave, c)) return;
    quantize_run_f16<HDR, RAGGED>(device_pointer<const _Float16>(c.x) + static_cast<int64_t>(c.n) * static_cast<int64_t>(c.D), c.n,
                                  c.tile * kQpGroupsF16, c.D, static_cast<uint32_t>((c.D + (kGroup - 1)) >> 8), lane,
                                  quantize_args(t, c, k0, k1, tag, packed, capacity), stage_all[wave]);
}

// One tile of four groups per wavefront.
template <typename T, int NOISE_BITS, int HDR, bool RAGGED, int CAPACITY>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void quantize_pack_tile_kernel(
    MultiTable<CAPACITY> t, uint32_t k0, uint32_t k1, uint64_t tag, uint8_t* __restrict__ packed, uint64_t capacity)
{
    __shared__ u32x4 stage_all[kWavesPerBlock][kQpStageSlots];
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));
    MultiCursor c;
    if (!multi_cursor<kWavesPerBlock, kQpXcdMap, kQpRun, CAPACITY>(t, wave, c)) return;
    quantize_tile<T, NOISE_BITS, HDR, RAGGED>(device_pointer<const T>(c.x) + static_cast<int64_t>(c.n) * static_cast<int64_t>(c.D), c.n,
                                              c.tile * kTileGroups, c.D, static_cast<uint32_t>((c.D + (kGroup - 1)) >> 8), lane,
                                              quantize_args(t, c, k0, k1, tag, packed, capacity), stage_all[wave]);
}

// Ragged samples shift the pages that tiles and XCDs share, so the tiles are dealt in runs (like the
// quantizer's), and where tiles share lines, too, the stores are ordinary cached ones: the two halves of
// a line meet in an L2.  Binary32, [256, 501860] at B = 2: 120 us with the order and the non-temporal stores of
// whole groups, 118 with the runs, 110 with cached stores, 100 with both; whole lines ([256, 51744]): 13.0 us,
// 12.3 with the runs, 13.1 with both.
template <typename T, int HDR, int NG, int LAYOUT, int CAPACITY>
__global__ __launch_bounds__(kDqBlock) void unpack_dequantize_multi_kernel(MultiTable<CAPACITY> t, const uint8_t* __restrict__ packed,
                                                                           uint64_t capacity)
{
    constexpr bool kRun = LAYOUT != kWholeGroups;
    __shared__ uint32_t stage_all[sizeof(T) == 4 ? kDqBlock / kWave : 1][256];   // a slice per wavefront (odd widths, binary32)
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));
    uint32_t* stage = stage_all[sizeof(T) == 4 ? wave : 0];
    MultiCursor c;
    if (!multi_cursor<kDqBlock / kWave, kRun ? 0 : kDqXcdMap, kRun ? kDqRaggedRun : 1, CAPACITY>(t, wave, c)) return;
    uint32_t b;
    uint64_t off;
    sample_width_offset(c, b, off);
    const uint32_t ng = static_cast<uint32_t>((c.D + (kGroup - 1)) >> 8);
    const uint32_t n = c.n;
    const int64_t D = static_cast<int64_t>(c.D);
    T* os = device_pointer<T>(c.out) + static_cast<int64_t>(n) * D;
    const void* header = device_pointer<const void>(c.header);
    if (!range_ok(off, static_cast<uint64_t>(ng) * 32u * b, capacity)) return;
    const uint8_t* src = packed + off;
    const uint32_t g0 = c.tile * NG;
    switch (b) {
        case 1: dequantize_run<T, LAYOUT, 1, HDR, NG>(src, header, os, D, n, g0, ng, lane, stage); break;
        case 2: dequantize_run<T, LAYOUT, 2, HDR, NG>(src, header, os, D, n, g0, ng, lane, stage); break;
        case 3: dequantize_run<T, LAYOUT, 3, HDR, NG>(src, header, os, D, n, g0, ng, lane, stage); break;
        case 4: dequantize_run<T, LAYOUT, 4, HDR, NG>(src, header, os, D, n, g0, ng, lane, stage); break;
        case 5: dequantize_run<T, LAYOUT, 5, HDR, NG>(src, header, os, D, n, g0, ng, lane, stage); break;
        case 6: dequantize_run<T, LAYOUT, 6, HDR, NG>(src, header, os, D, n, g0, ng, lane, stage); break;
        case 7: dequantize_run<T, LAYOUT, 7, HDR, NG>(src, header, os, D, n, g0, ng, lane, stage); break;
        case 8: dequantize_run<T, LAYOUT, 8, HDR, NG>(src, header, os, D, n, g0, ng, lane, stage); break;
        default: return;
    }
}

// ------------------------------------------------------------------------------------
// One range and zero point for the whole tensor (the per-tensor baseline of Sec. 4.1 and
// Sec. 6.1): Z = min, R = max - min over all elements.  Three tiny launches on the caller's
// stream: set the two result words to the identity, reduce (a fixed number of wavefronts
// stride over the tensor; each block folds its minimum and maximum and issues two atomics),
// and convert.  Minimum and maximum do not depend on the order of the operations, so the
// atomics do not make the result vary.  While the reduction runs the two words hold order-
// preserving integer images of the floats (sign bit flipped for non-negative values, all
// bits flipped for negative ones), on which unsigned min / max order like the floats.

__device__ __forceinline__ uint32_t float_to_ordered(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float ordered_to_float(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__global__ void tensor_stats_init_kernel(uint32_t* zr)
{
    if (threadIdx.x == 0) {
        zr[0] = 0xffffffffu;  // above every value's image
        zr[1] = 0u;           // below every value's image
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void tensor_stats_reduce_kernel(const T* __restrict__ x, int64_t n, uint32_t* zr)
{
    __shared__ float part_lo[kWavesPerBlock], part_hi[kWavesPerBlock];
    constexpr int kE = 16 / sizeof(T);  // elements per 128-bit load
    const int64_t chunks = n / kE;      // whole 128-bit chunks; x is 16-byte aligned
    float lo = __builtin_inff(), hi = -__builtin_inff();
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t c = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; c < chunks; c += stride) {
        if constexpr (sizeof(T) == 4) {
            const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(x) + c);
            lo = fminf(fminf(lo, v.x), fminf(fminf(v.y, v.z), v.w));
            hi = fmaxf(fmaxf(hi, v.x), fmaxf(fmaxf(v.y, v.z), v.w));
        } else {
            typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
            const f16x8 v = __builtin_nontemporal_load(reinterpret_cast<const f16x8*>(x) + c);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                lo = fminf(lo, static_cast<float>(v[k]));
                hi = fmaxf(hi, static_cast<float>(v[k]));
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < n - chunks * kE) {  // the last, partial chunk
        const float v = static_cast<float>(x[chunks * kE + threadIdx.x]);
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, d));
        hi = fmaxf(hi, __shfl_xor(hi, d));
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        part_lo[threadIdx.x >> 6] = lo;
        part_hi[threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kWavesPerBlock; ++w) {
            lo = fminf(lo, part_lo[w]);
            hi = fmaxf(hi, part_hi[w]);
        }
        atomicMin(zr, float_to_ordered(lo));
        atomicMax(zr + 1, float_to_ordered(hi));
    }
}

__global__ void tensor_stats_finish_kernel(uint32_t* zr)
{
    if (threadIdx.x == 0) {
        const float mn = ordered_to_float(zr[0]) + 0.0f;  // -0.0 -> +0.0
        const float mx = ordered_to_float(zr[1]);
        zr[0] = __float_as_uint(mn);
        zr[1] = __float_as_uint((mx - mn) + 0.0f);  // a zero range is +0.0
    }
}

// ------------------------------------------------------------------------------------
// Sec. 4.2, Eq. (8): w_n = (G / 6) * ||grad_n||^2 * sum_g R_ng^2.  One block per sample over the
// group ranges (1/256 of the tensor's size).  The block is as wide as the sample needs (up to
// 1024 lanes) and every lane keeps four independent partial sums, so that a sample with many
// groups has enough loads in flight; the partial sums are combined in a fixed order, so the
// result is reproducible.
constexpr int kSensMaxBlock = 1024;

__global__ __launch_bounds__(kSensMaxBlock) void sample_sensitivity_kernel(const float* __restrict__ grange,
                                                                           uint32_t N, uint32_t ng, uint32_t grid_x,
                                                                           float coeff, const float* __restrict__ grad2,
                                                                           float* __restrict__ w)
{
    __shared__ float partial[kSensMaxBlock / kWave];
    const uint32_t n = blockIdx.y * grid_x + blockIdx.x;
    if (n >= N) return;
    const float* r = grange + static_cast<int64_t>(n) * ng;
    const uint32_t threads = blockDim.x;
    // asked for now, needed at the end
    float norm2 = 1.0f;
    if (grad2) norm2 = grad2[n];
    float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
    uint32_t g = threadIdx.x;
    for (; g + 3 * threads < ng; g += 4 * threads) {
        const float r0 = r[g], r1 = r[g + threads], r2 = r[g + 2 * threads], r3 = r[g + 3 * threads];
        a0 = __builtin_fmaf(r0, r0, a0);
        a1 = __builtin_fmaf(r1, r1, a1);
        a2 = __builtin_fmaf(r2, r2, a2);
        a3 = __builtin_fmaf(r3, r3, a3);
    }
    for (; g < ng; g += threads) a0 = __builtin_fmaf(r[g], r[g], a0);
    float acc = (a0 + a1) + (a2 + a3);
    // lanes, then wavefronts, in a fixed order
    acc += dpp_f32<kDppXor1>(acc);
    acc += dpp_f32<kDppXor2>(acc);
    acc += dpp_f32<kDppHalfMirror>(acc);
    acc += dpp_f32<kDppXor8>(acc);
    acc += __shfl_xor(acc, 16);
    acc += __shfl_xor(acc, 32);
    float total = 0.0f;
    if (threads == kWave) {
        total += acc;
    } else {
        if ((threadIdx.x & (kWave - 1)) == 0) partial[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x == 0)
            for (uint32_t k = 0; k < threads / kWave; ++k) total += partial[k];
    }
    if (threadIdx.x == 0) w[n] = coeff * total * norm2;
}

// ------------------------------------------------------------------------------------
// Sec. 4.3 on the device: the greedy allocation without the host in the loop.
//
// The greedy applies moves (item i, step r of the width ladder) in ascending order of
// (price, i, r) until enough bits are freed, and an item's prices never decrease along the
// ladder.  Its result is therefore fixed by the price of the last applied move, the threshold:
// every move strictly cheaper is applied, and the moves of exactly that price are applied in
// (i, r) order until the budget holds.  One workgroup finds the threshold and works out of LDS;
// a prefix sum then turns the widths into byte offsets.
//
// What bounds it: one workgroup has one compute unit, and most phases are chains of dependent instructions, LDS round trips
// and barriers.  A radix selection over the 64-bit patterns of all prices (eight passes of eight bits) took 154 us for 13,568
// items with all eight widths, 101 us with {1, 2, 4, 8}, and 10 us for 128 items.  Hence:
//   * a small problem (allocate_bits_small_kernel: up to 1024 items, 2048 of one size or of few moves) has every price in registers and takes one
//     histogram over the range of the prices: the bin that holds the threshold has a handful of moves, which are ranked;
//   * a large one (allocate_bits_kernel) does not price its moves at all at first.  A price is
//     (w / D) * c_r to within a few units in the last place, so a histogram of the ITEMS over
//     w / D gives bounds of the bits freed below any price t: sum_r dw_r * (elements of the items
//     with w / D < t / c_r).  A search over t on that table leaves a bracket that holds the
//     threshold and, typically, one or two hundred of the 95,000 moves; only the items of those are priced
//     exactly, and the widths of all other items follow from comparing w / D with t / c_r;
//   * many (nearly) equal prices are left to select_price, which narrows a bracket [lo, hi] of price patterns until at most
//     64 candidates are left.
// The order of w / D is taken from the upper 32 bits of its binary64 pattern (20 bits of mantissa),
// computed to within one unit.  Every comparison on it leaves a margin of two units: what passes is
// cheaper (dearer) by one unit at least, 2^-21, and the rounding errors of t / c_r and of the price
// are below 2^-50.  What lies inside the margin is decided by exact prices.  Both the bits freed
// below the bracket and the widths of the items are taken per bin of the table, not per item.

constexpr int kAllocBlock = 1024;
constexpr int kAllocWavesMax = kAllocBlock / kWave;
constexpr int kMaxSteps = 7;
// Items per thread of the small kernel from 1025 items on.  Of one size: 2048 with all widths 12.5 against 14.4 us with the large kernel, with
// {1, 2, 4, 8} 9.7 against 13.2.
constexpr int kSmallItems = 2;
// With sizes of their own only up to this many moves.  Large kernel -> small one (us), log-normal sensitivities / all equal / all zero / half of them zero:
//   {1, 8}         1025 items 13.3 -> 8.5 / 19.0 -> 10.6 / 18.5 -> 8.4 / 13.2 -> 11.9    2048 items 13.4 -> 9.6 / 20.6 -> 12.2 / 20.6 -> 8.5 / 13.8 -> 13.8
//   {1, 2, 4}      1025 items 13.6 -> 9.1 / 19.0 -> 11.4 / 20.1 -> 8.7 / 13.2 -> 12.5    2048 items 13.4 -> 10.3 / 20.6 -> 13.8 / 22.5 -> 8.8 / 13.8 -> 14.5
//   {1, 2, 4, 8}   1025 items 13.3 -> 10.3 / 19.3 -> 12.1 / 21.9 -> 8.7 / 13.3 -> 13.5   1300 items 13.6 -> 10.1 / 20.0 -> 13.0 / 23.9 -> 9.0 / 13.6 -> 14.3
// Beyond, the bin of the threshold may hold more moves than are ranked: 2048 items, {1, 2, 4, 8}, log-normal 13.5 -> 13.7 or 17.8 by the draw, 1500 with all
// widths 14.2 -> 18.5.
constexpr int64_t kSmallMoves = 4 * kAllocBlock;
constexpr int kAllocBins = 4096;      // bins of the large kernel's table over w / D
constexpr int kAllocList = 1024;      // items with undecided steps the large kernel lists: one per thread
// Beyond this many items a bin holds so many that the list of all items in undecided bins overflows, and their moves are priced in every
// turn: each item is tested by itself then.  Log-normal sensitivities, all listed -> tested (us): 150,000 with all widths 400 -> 248 where the
// list overflows and 214 -> 230 where it does not, 200,000 490 -> 302, 400,000 with {1, 2, 4, 8} 965 -> 594.
constexpr int64_t kAllocFilter = 131072;
constexpr int kSearchRounds = 5;      // of the large kernel's search over its table, at most
constexpr int kSearchWaves = 8;       // wavefronts that search, eight prices each [16: slower, they share the SIMDs]
constexpr int kAllocQuads = 4;        // quadruples of consecutive items per thread kept in registers: 16,384 items in all

// What the budget is compared with.
struct AllocBudget {
    uint64_t bits;
    uint32_t widest, narrowest;   // allowed widths
};

struct AllocArgs {
    int64_t M;
    int64_t D;               // element count of every item when D_items is null
    const int64_t* D_items;  // per-item element counts, or null
    AllocBudget total;
    Ladder lad;
    double inverse[kMaxSteps];   // 1 / lad.price[r]
    uint32_t width_nibbles;      // lad.width[k] in bits 4 k .. 4 k + 3
};

// DPP row_shr:K with zero fill: lane i of a row of 16 receives lane i - K, or 0 when there is none.
template <int K>
__device__ __forceinline__ uint64_t row_shift_right(uint64_t v)
{
    const uint32_t lo = dpp_u32<0x110 + K>(static_cast<uint32_t>(v));
    const uint32_t hi = dpp_u32<0x110 + K>(static_cast<uint32_t>(v >> 32));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

template <int CTRL>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v)
{
    const uint32_t lo = dpp_u32<CTRL>(static_cast<uint32_t>(v));
    const uint32_t hi = dpp_u32<CTRL>(static_cast<uint32_t>(v >> 32));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ uint64_t read_lane(uint64_t v, int src)
{
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(v)), src));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(v >> 32)), src));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ uint32_t read_lane(uint32_t v, int src)
{
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), src));
}

// Inclusive prefix sum inside each row of sixteen lanes.
__device__ __forceinline__ uint32_t row_inclusive_scan(uint32_t v)
{
    v += dpp_u32<0x111>(v);   // row_shr:1, 2, 4, 8 with zero fill
    v += dpp_u32<0x112>(v);
    v += dpp_u32<0x114>(v);
    v += dpp_u32<0x118>(v);
    return v;
}

__device__ __forceinline__ uint64_t row_inclusive_scan(uint64_t v)
{
    v += row_shift_right<1>(v);
    v += row_shift_right<2>(v);
    v += row_shift_right<4>(v);
    v += row_shift_right<8>(v);
    return v;
}

// Inclusive prefix sum over the 64 lanes: the rows' own, then the totals of the preceding rows,
// read from the rows' last lanes.
__device__ __forceinline__ uint64_t wave_inclusive_scan(uint64_t v, int lane)
{
    v = row_inclusive_scan(v);
    const uint64_t t0 = read_lane(v, 15), t1 = read_lane(v, 31), t2 = read_lane(v, 47);
    const int row = lane >> 4;
    uint64_t before = 0;
    before += row > 0 ? t0 : 0;
    before += row > 1 ? t1 : 0;
    before += row > 2 ? t2 : 0;
    return v + before;
}

__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v, int)
{
    v = row_inclusive_scan(v);
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x142, 0xa, 0xf, false));   // row_bcast:15 to rows 1 and 3
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x143, 0xc, 0xf, false));   // row_bcast:31 to rows 2 and 3
    return v;
}

struct Add { template <typename V> __device__ V operator()(V a, V b) const { return a + b; } };
struct Min { template <typename V> __device__ V operator()(V a, V b) const { return a < b ? a : b; } };
struct Max { template <typename V> __device__ V operator()(V a, V b) const { return a > b ? a : b; } };
struct Or { template <typename V> __device__ V operator()(V a, V b) const { return a | b; } };

// Reduction over each row of sixteen lanes, in every lane of it.
template <typename Op>
__device__ __forceinline__ uint64_t row_reduce(uint64_t v, Op op)
{
    v = op(v, dpp_u64<kDppXor1>(v));
    v = op(v, dpp_u64<kDppXor2>(v));
    v = op(v, dpp_u64<kDppHalfMirror>(v));
    v = op(v, dpp_u64<kDppXor8>(v));
    return v;
}

template <typename Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v, Op op)
{
    v = op(v, dpp_u32<kDppXor1>(v));
    v = op(v, dpp_u32<kDppXor2>(v));
    v = op(v, dpp_u32<kDppHalfMirror>(v));
    v = op(v, dpp_u32<kDppXor8>(v));
    const auto lane = [&](int src) { return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), src)); };
    return op(op(lane(0), lane(16)), op(lane(32), lane(48)));
}

template <typename Op>
__device__ __forceinline__ uint64_t wave_reduce(uint64_t v, Op op)
{
    v = row_reduce(v, op);
    return op(op(read_lane(v, 0), read_lane(v, 16)), op(read_lane(v, 32), read_lane(v, 48)));
}

// Reduction over each row of sixteen lanes of 32-bit values, read from its first lane.
template <typename Op>
__device__ __forceinline__ uint32_t row_result(uint32_t v, Op op)
{
    v = op(v, dpp_u32<kDppXor1>(v));
    v = op(v, dpp_u32<kDppXor2>(v));
    v = op(v, dpp_u32<kDppHalfMirror>(v));
    v = op(v, dpp_u32<kDppXor8>(v));
    return read_lane(v, 0);
}

// Second half of a reduction over the workgroup, behind a barrier: the wavefronts' results.
template <typename Op>
__device__ __forceinline__ uint64_t combine_waves(const uint64_t* of_wave, int waves, uint64_t identity, Op op)
{
    const int k = threadIdx.x & 15;
    return read_lane(row_reduce(k < waves ? of_wave[k] : identity, op), 0);
}

// Exclusive prefix sum over the workgroup in thread order; `total` receives the sum.  One barrier;
// `of_wave` (one entry per wavefront) must not be in use by anything else until the next barrier.
template <typename V>
__device__ __forceinline__ V block_exclusive_scan(V v, V* of_wave, V& total)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int waves = blockDim.x >> 6;
    const V incl = wave_inclusive_scan(v, lane);
    if (lane == kWave - 1) of_wave[wave] = incl;
    __syncthreads();
    const int k = lane & 15;
    const V own = k < waves ? of_wave[k] : V(0);
    const V upto = row_inclusive_scan(own);
    total = read_lane(upto, 15);
    return read_lane(upto, wave) - read_lane(own, wave) + incl - v;
}

// price of one step of item (w, D): two separately rounded double operations; -0.0 becomes +0.0
__device__ __forceinline__ uint64_t price_bits(float w, int64_t D, double step_price)
{
    const double key = (static_cast<double>(w) * step_price) / static_cast<double>(D) + 0.0;
    return static_cast<uint64_t>(__double_as_longlong(key));
}

// The threshold among candidate moves: its price pattern, the bits freed by all cheaper moves of
// the problem, and how many moves have exactly this price.
struct Threshold {
    uint64_t price, below, ties;
};

constexpr int kSelectBins = 256;

struct SelectLds {
    uint64_t hist[2][kSelectBins];   // both cleared by the caller, as is `count`
    uint64_t key[kWave], amount[kWave];
    uint64_t least[kAllocWavesMax], most[kAllocWavesMax];   // per wavefront
    uint64_t count[2];               // moves: up to 7 * 2^31
};

// `each(f)` calls f(price, bits freed) for the thread's candidates.  All candidates of the workgroup:
// n of them (n >= 1) with prices in [lo, hi]; the moves that are not candidates are either cheaper
// than the threshold (they free `below` bits) or dearer.  Uniform over the workgroup, and so is
// every branch around the barriers.
template <typename Each>
__device__ Threshold select_price(const Each& each, uint64_t n, uint64_t lo, uint64_t hi, uint64_t need, uint64_t below,
                                  SelectLds& s)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    for (int turn = 0;; turn ^= 1) {
        if (lo == hi) return Threshold{lo, below, n};
        if (n > kWave) {
            const uint64_t span = hi - lo;
            const int bits = 64 - __builtin_clzll(span);
            const int shift = bits > 8 ? bits - 8 : 0;   // (span >> shift) < 256
            uint64_t* h = s.hist[turn];
            each([&](uint64_t key, uint64_t freed) {
                if (key >= lo && key <= hi)
                    __hip_atomic_fetch_add(&h[(key - lo) >> shift], freed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            });
            __syncthreads();
            // Every wavefront finds, for itself, the bin in which the running sum of freed bits
            // first reaches `need`.  Exactly one lane holds it.
            uint64_t hb[4], mine = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) { hb[k] = h[4 * lane + k]; mine += hb[k]; }
            const uint64_t incl = wave_inclusive_scan(mine, lane);
            uint64_t run = below + incl - mine;
            const bool winner = run < need && run + mine >= need;
            int digit = 4 * lane;
            bool found = false;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                found = found || run + hb[k] >= need;
                if (!found) { run += hb[k]; ++digit; }
            }
            const uint64_t vote = __ballot(winner);
            const int src = vote ? __builtin_ctzll(vote) : 0;
            digit = __builtin_amdgcn_readlane(digit, src);
            below = read_lane(run, src);
            const uint64_t top = lo + ((static_cast<uint64_t>(digit) + 1) << shift) - 1;
            lo += static_cast<uint64_t>(digit) << shift;
            hi = top < hi && top >= lo ? top : hi;
        }
        // what is left, counted, and listed if it is little
        each([&](uint64_t key, uint64_t freed) {
            if (key >= lo && key <= hi) {
                const uint64_t at = __hip_atomic_fetch_add(&s.count[turn], uint64_t(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (at < kWave) {
                    s.key[at] = key;
                    s.amount[at] = freed;
                }
            }
        });
        // the other turn's words: all threads are past the barrier behind their last use
        for (int k = tid; k < kSelectBins; k += blockDim.x) s.hist[turn ^ 1][k] = 0;
        if (tid == 0) s.count[turn ^ 1] = 0;
        __syncthreads();
        n = s.count[turn];
        if (n <= kWave) break;
        // Many moves in one bin: the bracket shrinks to their prices.  Equal ones (items of the same size and sensitivity)
        // are told apart from nearly equal ones here and not bit by bit (256 items of sensitivity 1, all widths: 20.2 -> 12.1 us).
        uint64_t least = ~uint64_t(0), most = 0;
        each([&](uint64_t key, uint64_t) {
            if (key >= lo && key <= hi) {
                least = key < least ? key : least;
                most = key > most ? key : most;
            }
        });
        least = wave_reduce(least, Min());
        most = wave_reduce(most, Max());
        if (lane == 0) {
            s.least[tid >> 6] = least;
            s.most[tid >> 6] = most;
        }
        __syncthreads();
        lo = combine_waves(s.least, blockDim.x >> 6, ~uint64_t(0), Min());
        hi = combine_waves(s.most, blockDim.x >> 6, 0, Max());
    }
    // at most one move per lane: sums over the cheaper and over the not dearer ones of the list
    const bool live = lane < static_cast<int>(n);
    const uint64_t key = live ? s.key[lane] : ~uint64_t(0);
    uint64_t cheaper = 0, upto = 0, ties = 0;
    for (int k = 0; k < static_cast<int>(n); ++k) {
        const uint64_t other = s.key[k], freed = s.amount[k];
        cheaper += other < key ? freed : 0;
        upto += other <= key ? freed : 0;
        ties += other == key ? 1 : 0;
    }
    const uint64_t vote = __ballot(live && below + cheaper < need && below + upto >= need);
    const int src = vote ? __builtin_ctzll(vote) : 0;
    return Threshold{read_lane(key, src), below + read_lane(cheaper, src), read_lane(ties, src)};
}

// The sensitivity finite and not negative (see valid_sensitivity_bits), 0 < D < 2^34.
__device__ __forceinline__ bool valid_weight(float w)
{
    constexpr int kZeroOrPositive = 0x1E0;   // either zero, positive subnormal, positive normal
    return __builtin_amdgcn_classf(w, kZeroOrPositive);
}

__device__ __forceinline__ bool valid_item(float w, int64_t D)
{
    const uint32_t low = static_cast<uint32_t>(D), high = static_cast<uint32_t>(static_cast<uint64_t>(D) >> 32);
    return valid_weight(w) & (high < 4u) & ((low | high) != 0u);
}

__device__ __forceinline__ uint64_t stream_bytes(int64_t D, int width)
{
    return (static_cast<uint64_t>(D) + kGroup - 1) / kGroup * 32u * static_cast<uint64_t>(width);
}

// What the totals decide before any search.
struct AllocVerdict {
    bool search, loose;
    uint64_t need;    // bits that must be freed, > 0 if there is a search
    int64_t status;
};

__host__ __device__ inline AllocVerdict alloc_verdict(uint64_t elems, bool invalid, const AllocBudget& b)
{
    AllocVerdict v;
    v.loose = !invalid && elems * b.widest <= b.bits;
    const bool infeasible = !invalid && elems * b.narrowest > b.bits;
    v.search = !invalid && !v.loose && !infeasible;
    v.need = elems * b.widest - b.bits;
    v.status = invalid ? ACTQ_EINVAL : (infeasible ? ACTQ_EINFEASIBLE : ACTQ_OK);
    return v;
}

// Width and price of rung k for an index that differs between lanes: the widths are nibbles of one
// word, the prices are picked from scalar registers.
__device__ __forceinline__ int ladder_width(const AllocArgs& a, int k) { return static_cast<int>((a.width_nibbles >> (4 * k)) & 15u); }

__device__ __forceinline__ double ladder_price(const Ladder& lad, int k)
{
    double v = lad.price[0];
#pragma unroll
    for (int j = 1; j < kMaxSteps; ++j) v = k == j ? lad.price[j] : v;
    return v;
}

constexpr int kSmallBins = 512;

// The bin of `hist` in which the running sum of freed bits, from `start` on, reaches `need`; `below`: the sum before it.  Every
// wavefront for itself; exactly one lane holds the bin.
template <typename Amount>
__device__ __forceinline__ uint32_t winning_bin(const Amount* hist, Amount need, Amount start, int lane, Amount& below)
{
    constexpr int kPer = kSmallBins / kWave;
    Amount hb[kPer], mine = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) { hb[k] = hist[kPer * lane + k]; mine += hb[k]; }
    Amount run = start + wave_inclusive_scan(mine, lane) - mine;
    const uint64_t vote = __ballot(run < need && run + mine >= need);
    uint32_t digit = static_cast<uint32_t>(kPer * lane);
    bool found = false;
#pragma unroll
    for (int k = 0; k + 1 < kPer; ++k) {
        found = found || run + hb[k] >= need;
        run += found ? Amount(0) : hb[k];
        digit += found ? 0u : 1u;
    }
    const int src = vote ? __builtin_ctzll(vote) : 0;
    below = read_lane(run, src);
    return read_lane(digit, src);
}

// The threshold among n <= 64 moves, one per lane, ranked from registers: its price, the bits freed by the cheaper moves and
// the number of moves of this price.  Every wavefront for itself.
template <typename Amount>
__device__ __forceinline__ void rank_moves(const uint64_t* keys, const Amount* amounts, int n, Amount need, Amount start, int lane,
                                           uint64_t& price, Amount& below, uint64_t& count)
{
    const bool listed = lane < n;
    const uint64_t own = listed ? keys[lane] : ~uint64_t(0);
    const Amount frees = listed ? amounts[lane] : Amount(0);
    // moves of one price (items of one size and sensitivity) need no ranking: 64 items of sensitivity one with {1, 2, 4, 8} 9.6 -> 6.3 us, with all
    // widths 10.1 -> 6.6 (call to call)
    const uint64_t one = read_lane(own, 0);
    if (__ballot(listed && own != one) == 0) {
        price = one;
        below = start;
        count = static_cast<uint64_t>(n);
        return;
    }
    Amount cheaper = 0, upto = 0;
    uint32_t ties = 0;
#pragma unroll 4
    for (int k = 0; k < ((n + 3) & ~3); ++k) {   // lanes past the list free nothing and have no price
        const uint64_t other = read_lane(own, k);
        const Amount freed = read_lane(frees, k);
        cheaper += other < own ? freed : Amount(0);
        upto += other <= own ? freed : Amount(0);
        ties += other == own ? 1u : 0u;
    }
    const uint64_t vote = __ballot(listed && start + cheaper < need && start + upto >= need);
    const int src = vote ? __builtin_ctzll(vote) : 0;
    price = read_lane(own, src);
    below = start + read_lane(cheaper, src);
    count = read_lane(ties, src);
}

// The threshold among n moves, which `each(f)` enumerates, with many (nearly) equal prices: the bracket starts at the smallest and the
// largest of them, and equal ones need no more than that.  Called by the whole workgroup.
template <typename Each>
__device__ __forceinline__ Threshold select_among(const Each& each, uint64_t n, uint64_t need, uint64_t below, SelectLds& s)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), waves = blockDim.x >> 6;
    uint64_t least = ~uint64_t(0), most = 0;
    each([&](uint64_t key, uint64_t) {
        least = key < least ? key : least;
        most = key > most ? key : most;
    });
    least = wave_reduce(least, Min());
    most = wave_reduce(most, Max());
    for (int k = tid; k < 2 * kSelectBins; k += blockDim.x) (&s.hist[0][0])[k] = 0;
    if (tid < 2) s.count[tid] = 0;
    if (lane == 0) {
        s.least[tid >> 6] = least;
        s.most[tid >> 6] = most;
    }
    __syncthreads();
    return select_price(each, n, combine_waves(s.least, waves, ~uint64_t(0), Min()), combine_waves(s.most, waves, 0, Max()), need, below, s);
}

// What the small kernel is told.  Items of one size: the totals are known on the host, and with them what they decide and how
// much is to be freed, in units of D bits.
struct SmallAllocArgs {
    int32_t M, steps;
    uint32_t width_nibbles;      // lad.width[k] in bits 4 k .. 4 k + 3
    uint32_t need;               // items of one size: units to free
    int32_t status;              // items of one size: ACTQ_OK or ACTQ_EINFEASIBLE
    uint32_t search, loose;
    uint64_t unit_bytes;         // items of one size: stream bytes per bit of width
    int64_t D;                   // element count of every item when D_items is null
    double reciprocal;           // 1 / D
    const int64_t* D_items;      // per-item element counts, or null
    AllocBudget total;           // per-item sizes
    double price[kMaxSteps];     // of step r, for a unit of w / D; ascending
};

// (w c) / d as one IEEE division gives it, from y = 1 / d rounded to nearest (d an integer below 2^34, w c between 2^-165 and
// 2^128 or zero: nothing over- or underflows).  The first correction makes the quotient one of the two binary64 numbers around
// the true one, the second picks the nearer (Markstein's theorem on quotients by a correctly rounded reciprocal).
__device__ __forceinline__ uint64_t quotient_bits(double a, double d, double y)
{
    double q = a * y;
    q = __builtin_fma(__builtin_fma(-q, d, a), y, q);
    q = __builtin_fma(__builtin_fma(-q, d, a), y, q);
    return static_cast<uint64_t>(__double_as_longlong(q + 0.0));   // -0.0 becomes +0.0
}

// ITEMS consecutive items per thread, all their prices in registers.  UNIFORM: items of one size.
// A problem of this size is one chain of dependent instructions in a few wavefronts, so what counts is their number: prices by a
// reciprocal instead of a division each, minimum and maximum of the prices from the upper halves of their patterns, freed bits as
// 32-bit multiples of the common size, one histogram that leaves a handful of moves, and those ranked from registers.  Many (nearly)
// equal prices go on to select_among.  Kernel durations with a thread per move and the prices in LDS, and so, items of one size:
// 4 with {1, 2, 4, 8} 4.8 -> 3.6 us, 128 5.3 -> 3.7, 256 with all widths 7.7 -> 4.4, 1024 16.1 -> 7.6, 2048 23.0 -> 12.5;
// per-item sizes: 300 with all widths 8.8 -> 5.6, 1024 17.2 -> 12.0.  (Call to call, with the arguments as one batch: 4 items 3.1, 128 3.6, 256 with
// all widths 4.0, 1024 6.9.)
template <bool UNIFORM, int ITEMS>
__global__ __launch_bounds__(kAllocBlock) void allocate_bits_small_kernel(const float* __restrict__ w, SmallAllocArgs a,
                                                                          uint8_t* __restrict__ bits,
                                                                          uint64_t* __restrict__ offsets,
                                                                          int64_t* __restrict__ result)
{
    typedef typename std::conditional<UNIFORM, uint32_t, uint64_t>::type Amount;   // freed bits: units of D, or bits
    __shared__ Amount hist[kSmallBins];
    __shared__ uint64_t list_key[kWave];
    __shared__ Amount list_amount[kWave];
    __shared__ uint32_t list_count;
    __shared__ uint32_t wave_lo[kAllocWavesMax], wave_hi[kAllocWavesMax];
    __shared__ uint64_t wave_elems[kAllocWavesMax], wave_ties[kAllocWavesMax];
    __shared__ Amount wave_sum[kAllocWavesMax];
    __shared__ SelectLds sel;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), threads = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = threads >> 6;
    const int M = a.M, steps = a.steps;
    // 180 bytes of arguments, as one batch: left alone they are eleven loads, each waited for where it is first used (128 items 4.07 -> 3.66 us)
    asm volatile("" : : "s"(w), "s"(a.M), "s"(a.steps), "s"(a.width_nibbles), "s"(a.need), "s"(a.status), "s"(a.search), "s"(a.loose), "s"(a.unit_bytes), "s"(a.D),
                 "s"(a.reciprocal), "s"(a.D_items), "s"(a.price[0]), "s"(a.price[1]), "s"(a.price[2]), "s"(a.price[3]), "s"(a.price[4]), "s"(a.price[5]),
                 "s"(a.price[6]), "s"(bits), "s"(offsets), "s"(result));
    const int first = tid * ITEMS;   // the thread's items, consecutive ones
    const auto width_of = [&](int k) { return static_cast<int>((a.width_nibbles >> (4 * k)) & 15u); };
    float wi[ITEMS];
    int64_t Di[ITEMS];
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const int i = first + q < M ? first + q : M - 1;
        wi[q] = w[i];
        Di[q] = UNIFORM ? a.D : a.D_items[i];
    }
    for (int k = tid; k < kSmallBins; k += threads) hist[k] = 0;
    if (tid == 0) list_count = 0;
    uint64_t key[ITEMS][kMaxSteps];   // steps that do not exist: no price
    uint32_t lo = ~0u, hi = 0;        // upper halves of the prices; invalid items: bit 31 of hi
    uint64_t elems = 0;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const bool live = first + q < M;
        const bool ok = UNIFORM ? valid_sensitivity_bits(__float_as_uint(wi[q])) : valid_item(wi[q], Di[q]);
        if (!UNIFORM) {
            elems += live && ok ? static_cast<uint64_t>(Di[q]) : uint64_t(0);
            if (Di[q] <= 0 || Di[q] >= (int64_t(1) << 34)) Di[q] = 1;   // invalid input: stay memory-safe
        }
        const double d = static_cast<double>(Di[q]), y = UNIFORM ? a.reciprocal : 1.0 / d, weight = static_cast<double>(wi[q]);
        uint32_t top = 0;
#pragma unroll
        for (int r = 0; r < kMaxSteps; ++r) {
            key[q][r] = ~uint64_t(0);
            if (r < steps) {
                const uint64_t k = quotient_bits(weight * a.price[r], d, y);
                key[q][r] = live ? k : ~uint64_t(0);
                top = static_cast<uint32_t>(k >> 32);   // the last step is the dearest
            }
        }
        const uint32_t least = static_cast<uint32_t>(key[q][0] >> 32);
        lo = least < lo ? least : lo;
        top = ok ? top : 0x80000000u;
        hi = live && top > hi ? top : hi;
    }
    lo = wave_reduce(lo, Min());
    hi = wave_reduce(hi, Max());
    if (!UNIFORM) elems = wave_reduce(elems, Add());
    if (waves > 1) {
        if (lane == 0) {
            wave_lo[wave] = lo;
            wave_hi[wave] = hi;
            if (!UNIFORM) wave_elems[wave] = elems;
        }
        __syncthreads();
        const int k = lane & 15, at = k < waves ? k : 0;
        lo = row_result(wave_lo[at], Min());
        hi = row_result(wave_hi[at], Max());
        if (!UNIFORM) elems = combine_waves(wave_elems, waves, 0, Add());
    } else {
        __syncthreads();   // the histogram is cleared
    }
    const bool invalid = (hi >> 31) != 0;
    bool search = a.search != 0, loose = a.loose != 0;
    int64_t status = a.status;
    Amount need = static_cast<Amount>(a.need);
    if (!UNIFORM) {
        const AllocVerdict v = alloc_verdict(elems, false, a.total);
        search = v.search;
        loose = v.loose;
        status = v.status;
        need = static_cast<Amount>(v.need);
    }
    if (invalid) {
        search = loose = false;
        status = ACTQ_EINVAL;
    }
    const auto freed_by = [&](int q, int from, int to) {   // by going from rung `from` to rung `to`
        return static_cast<Amount>(UNIFORM ? 1 : Di[q]) * static_cast<Amount>(width_of(from) - width_of(to));
    };

    uint64_t threshold = 0;    // the price of the last move,
    Amount below = 0;          // the bits freed by all cheaper ones,
    uint64_t at_threshold = 0; // and how many moves have exactly this price
    if (search) {
        // the bin in which the running sum of freed bits reaches `need`
        const uint32_t span = hi - lo;
        int shift = 23 - __builtin_clz(span | 1u);   // (span >> shift) < 512
        shift = shift > 0 ? shift : 0;
        const auto bin_of = [&](uint64_t k) { return (static_cast<uint32_t>(k >> 32) - lo) >> shift; };
        uint32_t digit = 0, here = 0;
        int n = M * steps;
        if (span != 0) {
#pragma unroll
            for (int q = 0; q < ITEMS; ++q)
#pragma unroll
                for (int r = 0; r < kMaxSteps; ++r)
                    if (r < steps && first + q < M)
                        __hip_atomic_fetch_add(&hist[bin_of(key[q][r])], freed_by(q, r, r + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __syncthreads();
            digit = winning_bin(hist, need, Amount(0), lane, below);
        }
        // its moves
#pragma unroll
        for (int q = 0; q < ITEMS; ++q)
#pragma unroll
            for (int r = 0; r < kMaxSteps; ++r)
                if (r < steps) here |= first + q < M && bin_of(key[q][r]) == digit ? 1u << (q * kMaxSteps + r) : 0u;
        if (span != 0) {
            if (here != 0) {
                uint32_t at = __hip_atomic_fetch_add(&list_count, static_cast<uint32_t>(__builtin_popcount(here)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
                for (int q = 0; q < ITEMS; ++q)
#pragma unroll
                    for (int r = 0; r < kMaxSteps; ++r)
                        if (here >> (q * kMaxSteps + r) & 1u) {
                            if (at < kWave) {
                                list_key[at] = key[q][r];
                                list_amount[at] = freed_by(q, r, r + 1);
                            }
                            ++at;
                        }
            }
            __syncthreads();
            n = __builtin_amdgcn_readfirstlane(static_cast<int>(list_count));
        }
        if (span != 0 && n <= kWave) {
            rank_moves(list_key, list_amount, n, need, below, lane, threshold, below, at_threshold);
        } else {
            const auto each = [&](auto f) {
#pragma unroll
                for (int q = 0; q < ITEMS; ++q)
#pragma unroll
                    for (int r = 0; r < kMaxSteps; ++r)
                        if (here >> (q * kMaxSteps + r) & 1u) f(key[q][r], static_cast<uint64_t>(freed_by(q, r, r + 1)));
            };
            const Threshold t = select_among(each, static_cast<uint64_t>(n), static_cast<uint64_t>(need), static_cast<uint64_t>(below), sel);
            threshold = t.price;
            below = static_cast<Amount>(t.below);
            at_threshold = t.ties;
        }
    }
    int rung[ITEMS], ties[ITEMS];
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        rung[q] = loose ? 0 : steps;
        ties[q] = 0;
        if (search) {
            rung[q] = 0;
#pragma unroll
            for (int r = 0; r < kMaxSteps; ++r) {
                rung[q] += key[q][r] < threshold ? 1 : 0;
                ties[q] += key[q][r] == threshold ? 1 : 0;
            }
        }
    }
    if (at_threshold > 1) {
        // the moves at the threshold in (item, step) order, until the budget holds
        const uint64_t rest = static_cast<uint64_t>(need - below);
        uint64_t sum = 0, unused;
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) sum += static_cast<uint64_t>(freed_by(q, rung[q], rung[q] + ties[q]));
        uint64_t before = block_exclusive_scan(sum, wave_ties, unused);
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            uint64_t freed = before;
            before += static_cast<uint64_t>(freed_by(q, rung[q], rung[q] + ties[q]));
            for (; ties[q] > 0 && freed < rest; --ties[q], ++rung[q]) freed += static_cast<uint64_t>(freed_by(q, rung[q], rung[q] + 1));
        }
    } else {
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) rung[q] += ties[q];   // the one move at the threshold is applied
    }
    // offsets: widths (items of one size) or bytes, summed in item order
    Amount size[ITEMS], sum = 0, total;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const int width = width_of(rung[q]);
        size[q] = first + q < M ? static_cast<Amount>(UNIFORM ? static_cast<uint64_t>(width) : stream_bytes(Di[q], width)) : Amount(0);
        sum += size[q];
    }
    Amount before = block_exclusive_scan(sum, wave_sum, total);
    const uint64_t unit = UNIFORM ? a.unit_bytes : 1;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        if (first + q < M) {
            bits[first + q] = static_cast<uint8_t>(width_of(rung[q]));
            offsets[first + q] = static_cast<uint64_t>(before) * unit;
        }
        before += size[q];
    }
    if (tid == 0) {
        result[0] = static_cast<int64_t>(static_cast<uint64_t>(total) * unit);
        result[1] = status;
    }
}

// Upper 32 bits of the binary64 pattern of w / D, one unit off at most: the reciprocal of D in binary32
// (relative error below 2^-22 with the rounding of D) is four times finer than a unit, and costs a
// tenth of a binary64 division.  A valid sensitivity is not negative; -0.0 counts as 0.
__device__ __forceinline__ double reciprocal_of(int64_t D)
{
    uint32_t low = static_cast<uint32_t>(D), high = static_cast<uint32_t>(static_cast<uint64_t>(D) >> 32);
    asm("" : "+v"(low), "+v"(high));   // two words to the compiler, which makes one long conversion of the 64 bits
    const float d = __builtin_fmaf(static_cast<float>(high), 4294967296.0f, static_cast<float>(low));
    return static_cast<double>(__builtin_amdgcn_rcpf(d));
}

__device__ __forceinline__ uint32_t ratio_by(float w, double reciprocal)
{
    const double q = static_cast<double>(w) * reciprocal;
    return static_cast<uint32_t>(static_cast<uint64_t>(__double_as_longlong(q)) >> 32) & 0x7fffffffu;
}

__device__ __forceinline__ uint32_t ratio_of(float w, int64_t D) { return ratio_by(w, reciprocal_of(D)); }

// Upper 32 bits of (price with the upper 32 bits `t` and zeros below) / c_r.
__device__ __forceinline__ uint32_t ratio_at(uint64_t price, double inverse)
{
    return static_cast<uint32_t>(static_cast<uint64_t>(__double_as_longlong(__longlong_as_double(static_cast<long long>(price)) * inverse)) >> 32);
}

// For a bracket [lo, hi) of prices: how item ratios compare with lo / c_r and hi / c_r, every r.
// A step r of an item is certainly cheaper than lo if ratio + 2 < below[r], and certainly not
// cheaper than hi if ratio > above[r].
struct RatioBracket {
    uint32_t below[kMaxSteps], above[kMaxSteps];
};

// The bins [0, below[r]) hold only items whose step r is certainly cheaper than the bracket, the bins from above[r] on
// only items whose step is certainly not; both fall with r.
struct BinBracket {
    uint32_t below[kMaxSteps], above[kMaxSteps];
};

// For items with ratio u: the steps before `first` are cheaper than the bracket, steps [first, last) are undecided.
__device__ __forceinline__ void bracket_steps(const RatioBracket& b, int steps, uint32_t u, int& first, int& last)
{
    first = 0;
    last = 0;
#pragma unroll
    for (int r = 0; r < kMaxSteps; ++r) {
        first += u + 2u < b.below[r] ? 1 : 0;
        last += r < steps && u <= b.above[r] ? 1 : 0;
    }
}

// The rung of an item near the threshold, and its moves of exactly that price.
__device__ __forceinline__ void settle_item(float wi, int64_t Di, const AllocArgs& a, const RatioBracket& br, int steps, uint64_t price, int& rung, int& ties)
{
    int first, last;
    bracket_steps(br, steps, ratio_of(wi, Di), first, last);
    rung = first;
    ties = 0;
    for (int r = first; r < last; ++r) {
        const uint64_t key = price_bits(wi, Di, ladder_price(a.lad, r));
        rung += key < price ? 1 : 0;
        ties += key == price ? 1 : 0;
    }
}

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int64_t i64x2_a8 __attribute__((ext_vector_type(2), aligned(8)));
typedef int64_t i64x4 __attribute__((ext_vector_type(4)));
typedef int64_t i64x4_a8 __attribute__((ext_vector_type(4), aligned(8)));

// Any M.  A thread's items come in quadruples of consecutive ones, 4096 items per round; the bins (ratios, before there are
// bins) and group counts of the first kAllocQuads rounds stay in registers.  M >= 4: the small kernel takes fewer.
// The items in a bin with undecided steps are listed, one per thread, and from there on they are the small kernel's problem:
// exact prices in registers, a histogram over the bracket, the bin that holds the threshold, its few moves ranked.  More of
// them than the list holds are priced again in every turn of select_price, which the ties end.
// What bounds it is instructions: sixteen wavefronts share four SIMDs, so a phase costs four times the instructions of one wavefront,
// whether they do different work or the same.  Hence items of one size in a row are looked at together, sums are in 32 bits where
// they fit, the search gives a lane a price and a step (one wavefront with the steps one behind the other: 4.8 -> 3.2 thousand
// cycles), bins are classified by scalar comparisons (3.9 -> 1.9), a list takes one LDS operation per wavefront, and the bin and the rank of the
// threshold are found by one wavefront for all (6.8 -> 4.4).  Thousands of cycles of 34 for 13,568 items with all widths: loads 2.4, ratios and totals 6.6,
// table 3.2, prefix sums 1.1, search 3.2, bins 1.9, list 3.4, exact prices 2.4, threshold 4.4, units and scan 3.4, stores 2.
// 2049 items of the ResNet-50's sizes with all widths 14.1 -> 12.5 us, 13,568 19.5 -> 16.1 ({1, 2, 4, 8}: 18.7 -> 15.7; sizes drawn at random 21.0 -> 18.3),
// 40,960 59.1 -> 53.4, 150,000 240 -> 228; 13,568 of sensitivity one 42.4 -> 34.2, of zero 118 -> 112; none of 828 problems slower.
__global__ __launch_bounds__(kAllocBlock) void allocate_bits_kernel(const float* __restrict__ w, AllocArgs a,
                                                                    uint8_t* __restrict__ bits,
                                                                    uint64_t* __restrict__ offsets,
                                                                    int64_t* __restrict__ result)
{
    constexpr int kQ = 4, kCached = kAllocQuads * kQ;
    constexpr int64_t kRound = int64_t(kAllocBlock) * kQ;
    // elements of the items per bin of w / D, then their prefix sums: 32-bit multiples of 2^scale if they are that small
    __shared__ uint64_t table[kAllocBins + 2];
    __shared__ uint32_t step_class[kAllocBins / 4];   // per bin, a byte: steps certainly cheaper than the bracket, and 8 if any step is undecided
    __shared__ uint32_t list_item[kAllocList];        // items with undecided steps
    __shared__ uint8_t list_rung[kAllocList];         // their rungs, and their moves at the threshold in the upper half
    __shared__ uint64_t hist[kSmallBins];             // bits freed by the undecided moves per bin of the bracket
    __shared__ uint64_t rank_key[kWave], rank_amount[kWave];
    __shared__ SelectLds sel;
    __shared__ uint64_t wave_a[kAllocWavesMax], wave_b[kAllocWavesMax], wave_c[kAllocWavesMax];
    __shared__ uint32_t wave_scan[kAllocWavesMax];
    __shared__ uint64_t wave_round[2][kAllocWavesMax], wave_bytes[kAllocQuads * kAllocWavesMax];
    __shared__ uint32_t list_count, rank_count;       // items: fewer than 2^31
    __shared__ uint64_t move_count;                   // moves: up to 7 * 2^31
    __shared__ uint32_t wave_lo[kAllocWavesMax], wave_hi[kAllocWavesMax], wave_or[kAllocWavesMax];
    __shared__ uint64_t all_cheaper;
    __shared__ uint32_t last_short[kSearchRounds], first_enough[kSearchRounds];
    __shared__ Threshold found;                       // by one wavefront for all: sixteen that do the same take turns on four SIMDs
    __shared__ uint32_t found_digit;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int waves = kAllocWavesMax;
    const int steps = a.lad.count - 1;
    const int64_t M = a.M;
    // the lines of the arguments that the search needs are on their way before it
    asm volatile("" : : "s"(a.lad.price[0]), "s"(a.inverse[0]));
    const auto item = [&](int j) { return (j / kQ) * kRound + tid * kQ + j % kQ; };
    const auto elements = [&](int64_t i) { return a.D_items ? a.D_items[i] : a.D; };

    // Ratios, totals and validation.  An empty slot has D = 0 and the largest ratio.
    constexpr uint32_t kNone = 0x7fffffffu;
    uint32_t ratio[kCached];
    int64_t size[kCached];
    uint64_t my_elems = 0;
    uint32_t lo_less1 = kNone - 1u, hi_ratio = 0;   // over the positive ratios, the smallest less 1; bit 31 of hi_ratio: an invalid item
    uint32_t all_sizes = 0;                    // lower words, or-ed
    float weight[kCached];
    // Whole quadruples per load (a load instruction costs its 64 addresses, not its bytes); one that
    // reaches past the end is taken from the last four items and shifted into place below.
    f32x4 weight4[kAllocQuads];
    i64x4 size4[kAllocQuads];
#pragma unroll
    for (int k = 0; k < kAllocQuads; ++k) {
        const int64_t i0 = item(k * kQ), at = i0 < M - kQ ? i0 : M - kQ;
        weight4[k] = *reinterpret_cast<const f32x4_a4*>(w + at);
        if (a.D_items) size4[k] = *reinterpret_cast<const i64x4_a8*>(a.D_items + at);
        else size4[k] = i64x4{a.D, a.D, a.D, a.D};
    }
    for (int k = tid; k < kAllocBins + 2; k += kAllocBlock) table[k] = 0;
    if (tid < kSmallBins) hist[tid] = 0;
    if (tid == 0) {
        list_count = 0;
        rank_count = 0;
        move_count = 0;
        all_cheaper = 0;
    }
    if (tid < kSearchRounds) {
        last_short[tid] = 0;
        first_enough[tid] = ~0u;
    }
#pragma unroll
    for (int k = 0; k < kAllocQuads; ++k) {
        // all loads before the first use of one: left alone, the compiler moves each under the branch of its round, one latency behind the other
        asm volatile("" : "+v"(weight4[k]), "+v"(size4[k][0]), "+v"(size4[k][1]), "+v"(size4[k][2]), "+v"(size4[k][3]));
        if ((k + 1) * kRound > M) {
            const int64_t past = item(k * kQ) - (M - kQ);   // 1, 2, 3: the quadruple is shifted by that much; from 4 on it is empty
            const bool one = past > 0 && (past & 1) != 0, two = past > 0 && (past & 2) != 0;
            weight4[k] = one ? __builtin_shufflevector(weight4[k], weight4[k], 1, 2, 3, 3) : weight4[k];
            weight4[k] = two ? __builtin_shufflevector(weight4[k], weight4[k], 2, 3, 3, 3) : weight4[k];
            size4[k] = one ? __builtin_shufflevector(size4[k], size4[k], 1, 2, 3, 3) : size4[k];
            size4[k] = two ? __builtin_shufflevector(size4[k], size4[k], 2, 3, 3, 3) : size4[k];
        }
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            weight[k * kQ + q] = weight4[k][q];
            size[k * kQ + q] = size4[k][q];
        }
    }
    // The ratio of an item; straight-line code, every item of a wavefront takes it.
    const auto count_item = [&](bool live, float wi, int64_t& Di) {
        const bool ok = live & valid_item(wi, Di);
        const uint32_t u = ratio_of(wi, Di), counted = ok ? u : kNone, less1 = counted - 1u;   // 0 becomes the largest
        lo_less1 = less1 < lo_less1 ? less1 : lo_less1;
        const uint32_t top = ok ? u : (live ? 0x80000000u : 0u);
        hi_ratio = top > hi_ratio ? top : hi_ratio;
        Di = ok ? Di : 0;
        my_elems += static_cast<uint64_t>(Di);
        all_sizes |= static_cast<uint32_t>(Di);
        return counted;
    };
    uint32_t alike_rounds = 0;   // quadruples of one size in the whole wavefront
    // rounds in which this wavefront has items: the others cost it nothing
    const auto in_round = [&](int k) { return k * kRound + wave * (kWave * kQ) < M; };
#pragma unroll
    for (int k = 0; k < kAllocQuads; ++k) {
        if (!in_round(k)) {
#pragma unroll
            for (int j = k * kQ; j < (k + 1) * kQ; ++j) {
                ratio[j] = kNone;
                size[j] = 0;
            }
            continue;
        }
        // Quadruples of one size in the whole wavefront (a layer's samples are neighbours): the size is looked at once
        // (four items 108 -> 52 instructions, the bound of this phase: one compute unit issues for all of them).  An invalid item
        // keeps its size here: it leaves the kernel no search that could use it.
        const int64_t D = size[k * kQ];
        const bool alike = size[k * kQ + 1] == D && size[k * kQ + 2] == D && size[k * kQ + 3] == D && item(k * kQ) + kQ <= M;
        if (__all(alike)) {
            const bool size_ok = valid_item(1.0f, D);
            const double reciprocal = reciprocal_of(D);
#pragma unroll
            for (int j = k * kQ; j < (k + 1) * kQ; ++j) {
                const uint32_t u = ratio_by(weight[j], reciprocal), less1 = u - 1u;
                const uint32_t top = (valid_weight(weight[j]) & size_ok) ? u : 0x80000000u;
                lo_less1 = less1 < lo_less1 ? less1 : lo_less1;
                hi_ratio = top > hi_ratio ? top : hi_ratio;
                ratio[j] = u;
            }
            my_elems += static_cast<uint64_t>(D) * kQ;
            all_sizes |= static_cast<uint32_t>(D);
            alike_rounds |= 1u << k;
            continue;
        }
#pragma unroll
        for (int j = k * kQ; j < (k + 1) * kQ; ++j) {
            const int32_t left = static_cast<int32_t>(M < (int64_t(1) << 30) ? M : int64_t(1) << 30) - (j / kQ) * static_cast<int32_t>(kRound);
            ratio[j] = count_item(tid * kQ + j % kQ < left, weight[j], size[j]);
        }
        __builtin_amdgcn_sched_barrier(0);   // a quadruple at a time: the temporaries stay in registers
    }
    // items beyond the registers: recomputed in every pass
    const auto further_quads = [&](auto f) {   // f(first item, first of them that counts, sensitivities, sizes)
        for (int64_t i0 = kAllocQuads * kRound + tid * kQ; i0 < M; i0 += kRound) {
            const int64_t at = i0 < M - kQ ? i0 : M - kQ;
            const f32x4 x = *reinterpret_cast<const f32x4_a4*>(w + at);
            i64x4 y = {a.D, a.D, a.D, a.D};
            if (a.D_items) y = *reinterpret_cast<const i64x4_a8*>(a.D_items + at);
            f(at, static_cast<int>(i0 - at), x, y);
        }
    };
    const auto further = [&](auto f) {
        further_quads([&](int64_t at, int from, f32x4 x, i64x4 y) {
#pragma unroll
            for (int q = 0; q < kQ; ++q)
                if (q >= from) f(at + q, x[q], y[q]);
        });
    };
    further_quads([&](int64_t, int from, f32x4 x, i64x4 y) {
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            int64_t Di = y[q];
            (void)count_item(q >= from, x[q], Di);
        }
    });
    {
        const uint64_t e = wave_reduce(my_elems, Add());
        const uint32_t l = wave_reduce(lo_less1, Min()), h = wave_reduce(hi_ratio, Max()), o = wave_reduce(all_sizes, Or());
        if (lane == 0) {
            wave_a[wave] = e;
            wave_lo[wave] = l;
            wave_hi[wave] = h;
            wave_or[wave] = o;
        }
    }
    __syncthreads();
    const uint64_t elems = combine_waves(wave_a, waves, 0, Add());
    const uint32_t first_ratio = row_result(wave_lo[lane & 15], Min()) + 1u;
    const uint32_t last_ratio = row_result(wave_hi[lane & 15], Max());   // 0: every price is 0
    const uint32_t sizes = row_result(wave_or[lane & 15], Or());
    const bool invalid = (last_ratio >> 31) != 0;
    const AllocVerdict v = alloc_verdict(elems, invalid, a.total);
    // 2^scale divides every size
    const int scale = sizes ? __builtin_ctz(sizes) : 31;
    const bool narrow = (elems >> scale) >> 32 == 0;
    // and sums of freed bits are below 2^32 in these units: fewer than eight bits per element
    const bool short_sums = (elems >> scale) >> 29 == 0;
    uint32_t* const table32 = reinterpret_cast<uint32_t*>(table);

    Threshold t = {0, 0, 0};
    RatioBracket br;
    // the bins of the table: bin 0 the ratio 0, then equal steps from the smallest positive ratio
    const uint32_t span = last_ratio > first_ratio ? last_ratio - first_ratio : 0u;
    int shift = span ? 32 - __builtin_clz(span) - 12 : 0;
    shift = shift > 0 ? shift : 0;
    if ((span >> shift) > static_cast<uint32_t>(kAllocBins - 2)) ++shift;
    // a positive ratio is 2^-183 at least, its pattern far above the 2^20 that a bin holds at most
    const uint32_t origin = first_ratio - (1u << shift);
    const auto bin_of = [&](uint32_t u) {   // an empty slot's ratio gives some bin, too
        const uint32_t bin = __builtin_elementwise_sub_sat(u, origin) >> shift;
        return bin < static_cast<uint32_t>(kAllocBins) ? bin : static_cast<uint32_t>(kAllocBins - 1);
    };
    const auto class_of = [&](uint32_t bin) { return static_cast<uint32_t>(reinterpret_cast<const uint8_t*>(step_class)[bin]); };
    uint32_t price_lo = 0, price_hi = 0;    // the bracket: upper halves of price patterns
    // rungs and tied moves of the items in registers, four bits each
    uint64_t rungs = 0, tied = 0;
    if (v.search) {
        const auto add_item = [&](uint32_t bin, int64_t D) {
            if (narrow) __hip_atomic_fetch_add(&table32[bin], __builtin_amdgcn_alignbit(static_cast<uint32_t>(static_cast<uint64_t>(D) >> 32), static_cast<uint32_t>(D), scale), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            else __hip_atomic_fetch_add(&table[bin], static_cast<uint64_t>(D), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
#pragma unroll
        for (int k = 0; k < kAllocQuads; ++k) {
            if (!in_round(k)) continue;
#pragma unroll
            for (int j = k * kQ; j < (k + 1) * kQ; ++j) {
                ratio[j] = bin_of(ratio[j]);   // bins from here on
                add_item(ratio[j], size[j]);         // an empty slot adds nothing
            }
        }
        further([&](int64_t, float wi, int64_t Di) { add_item(bin_of(ratio_of(wi, Di)), Di); });
        __syncthreads();
        // elements of the items in the bins before a bin
        const auto to_prefix = [&](auto* entry, auto* of_wave) {
            typedef typename std::remove_reference<decltype(*entry)>::type V;
            V own[4], mine = 0, total;
#pragma unroll
            for (int k = 0; k < 4; ++k) { own[k] = entry[4 * tid + k]; mine += own[k]; }
            V run = block_exclusive_scan(mine, of_wave, total);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                entry[4 * tid + k] = run;
                run += own[k];
            }
            if (tid == kAllocBlock - 1) entry[kAllocBins] = run;
        };
        if (narrow) to_prefix(table32, wave_scan);
        else to_prefix(table, wave_round[0]);
        __syncthreads();

        // ---- the bracket: both bounds of the bits freed below 64 prices at a time, eight per wavefront, a lane per price and step
        // lane r of eight: step r
        double inverse = 0.0;
        uint32_t dw = 0;
#pragma unroll
        for (int r = 0; r < kMaxSteps; ++r) {
            inverse = (lane & 7) == r ? a.inverse[r] : inverse;
            dw = (lane & 7) == r && r < steps ? static_cast<uint32_t>(a.lad.width[r] - a.lad.width[r + 1]) : dw;
        }
        {
            // price patterns' upper halves; nothing positive is cheaper than `start`, nothing is dearer than `end`
            const uint64_t lowest = static_cast<uint64_t>(first_ratio) << 32, highest = static_cast<uint64_t>(last_ratio + 1) << 32;
            const uint32_t p_lo = static_cast<uint32_t>(static_cast<uint64_t>(__double_as_longlong(__longlong_as_double(static_cast<long long>(lowest)) * a.lad.price[0])) >> 32);
            const uint32_t p_hi = static_cast<uint32_t>(static_cast<uint64_t>(__double_as_longlong(__longlong_as_double(static_cast<long long>(highest)) * ladder_price(a.lad, steps - 1))) >> 32);
            const uint32_t start = last_ratio ? (p_lo > 4u ? p_lo - 4u : 0u) : 0u, end = last_ratio ? p_hi + 4u : 4u;
            const uint32_t candidate = static_cast<uint32_t>(8 * wave + (lane >> 3));
            const auto price_at = [](uint32_t from, uint32_t width, uint32_t k) {
                return from + static_cast<uint32_t>(static_cast<uint64_t>(width) * k >> 6);
            };
            uint32_t lo = 0, hi = end, left = start, right = end;
            for (int round = 0; round < kSearchRounds; ++round) {
                const uint32_t width = right - left;
                if (wave < kSearchWaves) {
                    const uint32_t u = ratio_at(static_cast<uint64_t>(price_at(left, width, candidate)) << 32, inverse);   // 0 for a step that does not exist
                    // items of ratio < u - 2 only: whole bins before the one that holds it
                    const uint32_t x = u > 2u ? u - 2u : 0u;
                    const uint32_t bl = x <= first_ratio ? 1u : 1u + ((x - first_ratio) >> shift);
                    const uint32_t b_least = x == 0 ? 0u : (bl < static_cast<uint32_t>(kAllocBins) ? bl : static_cast<uint32_t>(kAllocBins));
                    // every item of ratio <= u + 2: whole bins up to the one that holds it
                    const uint32_t y = u + 2u;
                    const uint32_t bm = y < first_ratio ? 1u : 2u + ((y - first_ratio) >> shift);
                    const uint32_t b_most = bm < static_cast<uint32_t>(kAllocBins) ? bm : static_cast<uint32_t>(kAllocBins);
                    // bits freed by the moves cheaper than the price: lower and upper bound, over the steps; lanes whose price is too low and high enough
                    uint64_t not_yet, enough;
                    if (short_sums) {
                        uint32_t least = dw * table32[b_least], most = dw * table32[b_most];
                        least += dpp_u32<kDppXor1>(least);
                        most += dpp_u32<kDppXor1>(most);
                        least += dpp_u32<kDppXor2>(least);
                        most += dpp_u32<kDppXor2>(most);
                        least += dpp_u32<kDppHalfMirror>(least);
                        most += dpp_u32<kDppHalfMirror>(most);
                        const uint32_t need = static_cast<uint32_t>((v.need + ((uint64_t(1) << scale) - 1)) >> scale);
                        not_yet = __ballot(most < need);
                        enough = __ballot(least >= need);
                    } else {
                        uint64_t least = static_cast<uint64_t>(dw) * (narrow ? static_cast<uint64_t>(table32[b_least]) << scale : table[b_least]);
                        uint64_t most = static_cast<uint64_t>(dw) * (narrow ? static_cast<uint64_t>(table32[b_most]) << scale : table[b_most]);
                        least += dpp_u64<kDppXor1>(least);
                        most += dpp_u64<kDppXor1>(most);
                        least += dpp_u64<kDppXor2>(least);
                        most += dpp_u64<kDppXor2>(most);
                        least += dpp_u64<kDppHalfMirror>(least);
                        most += dpp_u64<kDppHalfMirror>(most);
                        not_yet = __ballot(most < v.need);
                        enough = __ballot(least >= v.need);
                    }
                    if (lane == 0) {
                        if (not_yet) __hip_atomic_fetch_max(&last_short[round], 1u + 8u * wave + static_cast<uint32_t>(63 - __builtin_clzll(not_yet)) / 8u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        if (enough) __hip_atomic_fetch_min(&first_enough[round], 8u * wave + static_cast<uint32_t>(__builtin_ctzll(enough)) / 8u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
                __syncthreads();
                const uint32_t before = read_lane(last_short[round], 0), from = read_lane(first_enough[round], 0);
                if (before != 0) lo = price_at(left, width, before - 1u);
                if (from != ~0u) hi = price_at(left, width, from);
                left = lo > start ? lo : start;
                right = hi;
                // Finer than a bin the table cannot tell.  With few items per bin the turn that would leave one bin instead of four costs more
                // than their items; with many the list would not hold them (150,000 items 240 -> 455 us).
                if (((right - left) >> shift) < (M <= kAllocQuads * kRound ? 4u : 1u) || right - left > width / 2u) break;
            }
            price_lo = lo;
            price_hi = hi;
        }

        // ---- what the bracket decides, per bin
        BinBracket bins;
        uint64_t my_below = 0;   // bits freed by moves that are cheaper than the bracket
        {
            const bool step = lane < steps;   // lane r: step r
            // a ladder with fewer steps: the unused ones are never cheaper (`above` is not looked at)
            const uint32_t below = step ? ratio_at(static_cast<uint64_t>(price_lo) << 32, inverse) : 0u;
            const uint32_t above = step ? ratio_at(static_cast<uint64_t>(price_hi) << 32, inverse) + 2u : 0u;
            // bin b > 0 holds the ratios first_ratio + ((b - 1) << shift) .. first_ratio + (b << shift) - 1
            uint32_t bin_below = below > first_ratio + 2u ? 1u + ((below - first_ratio - 2u) >> shift) : 1u;
            bin_below = below > 2u ? bin_below : 0u;
            uint32_t bin_above = above >= first_ratio ? 2u + ((above - first_ratio) >> shift) : 1u;
            bin_below = bin_below < static_cast<uint32_t>(kAllocBins) ? bin_below : static_cast<uint32_t>(kAllocBins);
            bin_above = step ? bin_above : 0u;
#pragma unroll
            for (int r = 0; r < kMaxSteps; ++r) {
                br.below[r] = read_lane(below, r);
                br.above[r] = read_lane(above, r);
                bins.below[r] = read_lane(bin_below, r);
                bins.above[r] = read_lane(bin_above, r);
            }
            if (wave == 0 && step)
                my_below = static_cast<uint64_t>(dw) * (narrow ? static_cast<uint64_t>(table32[bin_below]) << scale : table[bin_below]);
        }
        {
            // a wavefront has 256 neighbouring bins, and most boundaries lie outside of them: scalar comparisons
            const uint32_t base = static_cast<uint32_t>(wave) * (4 * kWave), own = 4u * static_cast<uint32_t>(lane);
            uint32_t first = 0, last = 0;   // four bins, a byte each
            const auto count_bins = [&](uint32_t& counts, uint32_t boundary) {   // the bins before it
                if (boundary <= base) return;
                if (boundary >= base + 4 * kWave) {
                    counts += 0x01010101u;
                    return;
                }
                const uint32_t before = __builtin_elementwise_sub_sat(boundary - base, own);
                counts += before >= 4u ? 0x01010101u : 0x01010101u & ((1u << (8u * before)) - 1u);
            };
#pragma unroll
            for (int r = 0; r < kMaxSteps; ++r) {
                count_bins(first, bins.below[r]);
                count_bins(last, bins.above[r]);
            }
            const uint32_t classes = first | ((last - first + 0x07070707u) & 0x08080808u);   // first <= last < 8
            step_class[tid] = classes;
        }
        __syncthreads();

        // ---- the items in a bin with undecided steps, listed; beyond kAllocFilter, those with undecided steps of their own
        uint32_t undecided = 0, listed_at = 0;
        const bool filter = M > kAllocFilter;
#pragma unroll
        for (int k = 0; k < kAllocQuads; ++k) {
            if (!in_round(k)) continue;
#pragma unroll
            for (int j = k * kQ; j < (k + 1) * kQ; ++j) {
                const uint32_t cls = class_of(ratio[j]);
                undecided |= (cls >> 3) << j;
                rungs |= static_cast<uint64_t>(cls & 7u) << (4 * j);
            }
            const int64_t live = M - item(k * kQ);   // an invalid size has left no search: the slots with items are those of the first M
            if (live < kQ) undecided &= live > 0 ? (1u << (k * kQ + static_cast<int>(live))) - 1u : (1u << (k * kQ)) - 1u;
        }
        const auto steps_freed = [&](int64_t Di, int from, int to) {   // bits freed by going from rung `from` to rung `to`
            return static_cast<uint64_t>(Di) * static_cast<uint64_t>(ladder_width(a, from) - ladder_width(a, to));
        };
        if (filter) {
            for (uint32_t m = undecided; m != 0; m &= m - 1) {
                const int j = __builtin_ctz(m);
                const int64_t i = item(j), Di = elements(i);
                int first, last;
                bracket_steps(br, steps, ratio_of(w[i], Di), first, last);
                if (first != last) continue;
                undecided &= ~(1u << j);
                my_below += steps_freed(Di, static_cast<int>(rungs >> (4 * j)) & 15, first);   // those before are counted with its bin
                rungs = (rungs & ~(uint64_t(15) << (4 * j))) | (static_cast<uint64_t>(first) << (4 * j));
            }
        }
        // places in the list: one LDS operation per wavefront
        const auto places = [&](uint32_t mask, uint32_t* total) {
            const uint32_t own = static_cast<uint32_t>(__builtin_popcount(mask)), upto = wave_inclusive_scan(own, lane);
            const uint32_t of_wave = read_lane(upto, kWave - 1);
            uint32_t from = 0;
            if (of_wave != 0) {
                if (lane == 0) from = __hip_atomic_fetch_add(total, of_wave, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                from = read_lane(from, 0);
            }
            return from + upto - own;
        };
        listed_at = places(undecided, &list_count);
        if (undecided != 0) {
            uint32_t at = listed_at;
            for (uint32_t m = undecided; m != 0; m &= m - 1, ++at)
                if (at < static_cast<uint32_t>(kAllocList)) list_item[at] = static_cast<uint32_t>(item(__builtin_ctz(m)));
        }
        uint64_t decided = 0;   // the same of the items beyond the registers: only the list leaves them out
        const auto list_further = [&](auto tested) {
            bool full = false;   // this thread has seen the list past its end: it is not used
            further([&](int64_t i, float wi, int64_t Di) {
                if (tested && full) return;
                const uint32_t u = ratio_of(wi, Di), cls = class_of(bin_of(u));
                if (!(cls & 8u)) return;
                if (tested) {
                    int first, last;
                    bracket_steps(br, steps, u, first, last);
                    if (first == last) {
                        decided += steps_freed(Di, static_cast<int>(cls & 7u), first);
                        return;
                    }
                }
                const uint32_t at = __hip_atomic_fetch_add(&list_count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                full = at >= static_cast<uint32_t>(kAllocList);
                if (!full) list_item[at] = static_cast<uint32_t>(i);
            });
        };
        if (filter) list_further(std::true_type());
        else list_further(std::false_type());
        __syncthreads();
        const uint32_t listed = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(list_count)));
        if (listed <= static_cast<uint32_t>(kAllocList)) {
            // a thread per item: its undecided moves, priced exactly, into the bins of the bracket
            uint64_t key[kMaxSteps];   // upper half below price_lo: cheaper, from price_hi on: dearer than the threshold
            uint32_t here = 0;
            const bool mine = static_cast<uint32_t>(tid) < listed;
            const uint32_t spread = price_hi - price_lo - 1u;   // price_lo < price_hi
            int fine = 23 - __builtin_clz(spread | 1u);         // (spread >> fine) < 512
            fine = fine > 0 ? fine : 0;
            int64_t Di = 0;
            my_below += decided;
            if (mine) {
                const int64_t i = list_item[tid];
                const float wi = w[i];
                Di = elements(i);
                const uint32_t cls = class_of(bin_of(ratio_of(wi, Di)));
                const double d = static_cast<double>(Di), y = 1.0 / d, of_item = static_cast<double>(wi);
#pragma unroll
                for (int r = 0; r < kMaxSteps; ++r) {
                    key[r] = r < steps ? quotient_bits(of_item * a.lad.price[r], d, y) : ~uint64_t(0);
                    const uint32_t top = static_cast<uint32_t>(key[r] >> 32);
                    const uint64_t freed = static_cast<uint64_t>(Di) * static_cast<uint64_t>(a.lad.width[r] - a.lad.width[r + 1]);
                    // cheaper steps of the item beyond those counted with its bin
                    if (top < price_lo && static_cast<uint32_t>(r) >= (cls & 7u)) my_below += freed;
                    if (top >= price_lo && top < price_hi) {
                        here |= 1u << r;
                        __hip_atomic_fetch_add(&hist[(top - price_lo) >> fine], freed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
            }
            if (__ballot(my_below != 0) != 0) {
                const uint64_t b = wave_reduce(my_below, Add());
                if (lane == 0) __hip_atomic_fetch_add(&all_cheaper, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __syncthreads();
            if (wave == 0) {
                uint64_t below_bin;
                const uint32_t of_need = winning_bin(hist, v.need, all_cheaper, lane, below_bin);
                if (lane == 0) {
                    found_digit = of_need;
                    found.below = below_bin;
                }
            }
            __syncthreads();
            const uint32_t digit = read_lane(found_digit, 0);
            const uint64_t below = read_lane(found.below, 0);
            // the moves in the bin that holds the threshold
            uint32_t chosen = 0;
#pragma unroll
            for (int r = 0; r < kMaxSteps; ++r)
                chosen |= (here >> r & 1u) && ((static_cast<uint32_t>(key[r] >> 32) - price_lo) >> fine) == digit ? 1u << r : 0u;
            uint32_t at = places(chosen, &rank_count);
            if (chosen != 0) {
#pragma unroll
                for (int r = 0; r < kMaxSteps; ++r)
                    if (chosen >> r & 1u) {
                        if (at < static_cast<uint32_t>(kWave)) {
                            rank_key[at] = key[r];
                            rank_amount[at] = static_cast<uint64_t>(Di) * static_cast<uint64_t>(a.lad.width[r] - a.lad.width[r + 1]);
                        }
                        ++at;
                    }
            }
            __syncthreads();
            const int n = __builtin_amdgcn_readfirstlane(static_cast<int>(rank_count));
            if (n <= kWave) {
                if (wave == 0) {
                    Threshold own;
                    rank_moves(rank_key, rank_amount, n, v.need, below, lane, own.price, own.below, own.ties);
                    if (lane == 0) found = own;
                }
                __syncthreads();
                t.price = read_lane(found.price, 0);
                t.below = read_lane(found.below, 0);
                t.ties = read_lane(found.ties, 0);
            } else {
                const auto each = [&](auto f) {
#pragma unroll
                    for (int r = 0; r < kMaxSteps; ++r)
                        if (chosen >> r & 1u) f(key[r], static_cast<uint64_t>(Di) * static_cast<uint64_t>(a.lad.width[r] - a.lad.width[r + 1]));
                };
                t = select_among(each, static_cast<uint64_t>(n), v.need, below, sel);
            }
            if (mine) {
                uint32_t rung = 0, ties = 0;
#pragma unroll
                for (int r = 0; r < kMaxSteps; ++r) {
                    rung += key[r] < t.price ? 1u : 0u;
                    ties += key[r] == t.price ? 1u : 0u;
                }
                if (t.ties == 1) { rung += ties; ties = 0; }   // the one move at the threshold is applied
                list_rung[tid] = static_cast<uint8_t>(rung | ties << 4);
            }
            __syncthreads();
            for (uint32_t m = undecided; m != 0; m &= m - 1, ++listed_at) {
                const int j = __builtin_ctz(m);
                const uint32_t state = list_rung[listed_at];
                rungs = (rungs & ~(uint64_t(15) << (4 * j))) | (static_cast<uint64_t>(state & 15u) << (4 * j));
                tied |= static_cast<uint64_t>(state >> 4) << (4 * j);
            }
        } else {
            // many (nearly) equal prices: the undecided moves, priced again in every turn; before(D, class) once per item that is looked at
            const auto walk_items = [&](auto f, auto before) {
                const auto moves_of = [&](float wi, int64_t Di, uint32_t cls, uint32_t u) {
                    int first, last;
                    bracket_steps(br, steps, u, first, last);
                    before(Di, static_cast<int>(cls & 7u), first);
                    for (int r = first; r < last; ++r)
                        f(price_bits(wi, Di, ladder_price(a.lad, r)),
                          static_cast<uint64_t>(Di) * static_cast<uint64_t>(ladder_width(a, r) - ladder_width(a, r + 1)));
                };
                for (uint32_t m = undecided; m != 0; m &= m - 1) {
                    const int64_t i = item(__builtin_ctz(m));
                    const float wi = w[i];
                    const int64_t Di = elements(i);
                    const uint32_t u = ratio_of(wi, Di);
                    moves_of(wi, Di, class_of(bin_of(u)), u);
                }
                further_quads([&](int64_t, int from, f32x4 x, i64x4 y) {
#pragma unroll 1
                    for (int q = 0; q < kQ; ++q) {   // rolled: this is inlined five times
                        const float wi = x[0];
                        const int64_t Di = y[0];
                        x = __builtin_shufflevector(x, x, 1, 2, 3, 3);
                        y = __builtin_shufflevector(y, y, 1, 2, 3, 3);
                        if (q < from) continue;
                        const uint32_t u = ratio_of(wi, Di), cls = class_of(bin_of(u));
                        if (cls & 8u) moves_of(wi, Di, cls, u);
                    }
                });
            };
            const auto walk = [&](auto f) { walk_items(f, [](int64_t, int, int) {}); };
            for (int k = tid; k < 2 * kSelectBins; k += kAllocBlock) (&sel.hist[0][0])[k] = 0;
            if (tid < 2) sel.count[tid] = 0;
            uint64_t lo = ~uint64_t(0), hi = 0, moves = 0;
            walk_items([&](uint64_t key, uint64_t) {
                ++moves;
                lo = key < lo ? key : lo;
                hi = key > hi ? key : hi;
            }, [&](int64_t Di, int of_bin, int of_item) {   // cheaper steps of the item beyond those counted with its bin
                my_below += static_cast<uint64_t>(Di) * static_cast<uint64_t>(ladder_width(a, of_bin) - ladder_width(a, of_item));
            });
            const uint64_t b = wave_reduce(my_below, Add());
            lo = wave_reduce(lo, Min());
            hi = wave_reduce(hi, Max());
            moves = wave_reduce(moves, Add());
            if (lane == 0) {
                wave_a[wave] = b;
                wave_b[wave] = lo;
                wave_c[wave] = hi;
                if (moves != 0) __hip_atomic_fetch_add(&move_count, moves, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __syncthreads();
            t = select_price(walk, move_count, combine_waves(wave_b, waves, ~uint64_t(0), Min()), combine_waves(wave_c, waves, 0, Max()),
                             v.need, combine_waves(wave_a, waves, 0, Add()), sel);
            for (uint32_t m = undecided; m != 0; m &= m - 1) {
                const int j = __builtin_ctz(m);
                const int64_t i = item(j);
                int rung, ties;
                settle_item(w[i], elements(i), a, br, steps, t.price, rung, ties);
                if (t.ties == 1) { rung += ties; ties = 0; }
                rungs = (rungs & ~(uint64_t(15) << (4 * j))) | (static_cast<uint64_t>(rung) << (4 * j));
                tied |= static_cast<uint64_t>(ties) << (4 * j);
            }
        }
    } else if (!v.loose) {
        rungs = 0x1111111111111111ull * static_cast<uint64_t>(steps);
    }

    // ---- offsets, in item order
    const uint64_t rest = v.need - t.below;   // bits still to free among the moves priced exactly at the threshold
    uint64_t tie_carry = 0, byte_carry = 0;
    const auto apply_ties = [&](int64_t Di, int& rung, int ties, uint64_t freed) {
        for (; ties > 0 && freed < rest; --ties, ++rung)
            freed += static_cast<uint64_t>(Di) * static_cast<uint64_t>(ladder_width(a, rung) - ladder_width(a, rung + 1));
    };
    const auto tie_bits = [&](int64_t Di, int rung, int ties) {
        return static_cast<uint64_t>(Di) * static_cast<uint64_t>(ladder_width(a, rung) - ladder_width(a, rung + ties));
    };
    if (t.ties > 1) {
#pragma unroll
        for (int k = 0; k < kAllocQuads; ++k) {
            if (k * kRound >= M) break;
            uint64_t of_item[kQ], sum = 0, total;
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
                const int j = k * kQ + q;
                of_item[q] = tie_bits(size[j], static_cast<int>(rungs >> (4 * j)) & 15, static_cast<int>(tied >> (4 * j)) & 15);
                sum += of_item[q];
            }
            uint64_t before = tie_carry + block_exclusive_scan(sum, wave_round[k & 1], total);
            tie_carry += total;
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
                const int j = k * kQ + q;
                int rung = static_cast<int>(rungs >> (4 * j)) & 15;
                apply_ties(size[j], rung, static_cast<int>(tied >> (4 * j)) & 15, before);
                before += of_item[q];
                rungs = (rungs & ~(uint64_t(15) << (4 * j))) | (static_cast<uint64_t>(rung) << (4 * j));
            }
        }
    }
    const bool word_stores = (reinterpret_cast<uintptr_t>(bits) & 3u) == 0;
    // widths and offsets of the quadruple from i0 on; units: 32 bytes of the stream per item
    const auto store_quad = [&](int64_t i0, uint32_t widths, const uint32_t (&units)[kQ], uint64_t off) {
        uint64_t at[kQ];
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            at[q] = off;
            off += static_cast<uint64_t>(units[q]) * 32u;
        }
        if (i0 + kQ <= M && word_stores) {
            *reinterpret_cast<uint32_t*>(bits + i0) = widths;
            i64x2_a8 x, y;
            x[0] = static_cast<int64_t>(at[0]);
            x[1] = static_cast<int64_t>(at[1]);
            y[0] = static_cast<int64_t>(at[2]);
            y[1] = static_cast<int64_t>(at[3]);
            *reinterpret_cast<i64x2_a8*>(offsets + i0) = x;
            *reinterpret_cast<i64x2_a8*>(offsets + i0 + 2) = y;
            return;
        }
#pragma unroll
        for (int q = 0; q < kQ; ++q)
            if (i0 + q < M) {
                bits[i0 + q] = static_cast<uint8_t>(widths >> (8 * q));
                offsets[i0 + q] = at[q];
            }
    };
    // groups of an item: below 2^26, so that a quadruple's units stay below 2^31
    const auto groups_of = [](int64_t D) {
        const uint64_t up = static_cast<uint64_t>(D) + (kGroup - 1);
        return __builtin_amdgcn_alignbit(static_cast<uint32_t>(up >> 32), static_cast<uint32_t>(up), 8);
    };
    // The sums of all rounds in registers go through one barrier.  In 32 bits where all groups together allow it (a scan of a wavefront in
    // 64 bits takes eight times as many instructions).
    if (invalid) {   // invalid input: stay memory-safe, with the sizes as they are where they can be
        alike_rounds = 0;
#pragma unroll
        for (int j = 0; j < kCached; ++j) {
            const int64_t i = item(j);
            int64_t Di = i < M ? elements(i) : 0;
            if (Di <= 0 || Di >= (int64_t(1) << 34)) Di = i < M ? 1 : 0;
            size[j] = Di;
        }
    }
    const auto store_rounds = [&](auto zero) {
        typedef decltype(zero) V;   // units: 32 bytes of the stream
        V upto[kAllocQuads];
        uint32_t units[kCached], own[kAllocQuads], widths[kAllocQuads];
        V* const of_waves = reinterpret_cast<V*>(wave_bytes);
#pragma unroll
        for (int k = 0; k < kAllocQuads; ++k) {
            own[k] = 0;
            widths[k] = 0;
            upto[k] = 0;
            if (in_round(k)) {
                uint32_t groups[kQ];
                groups[0] = groups_of(size[k * kQ]);
                if (alike_rounds >> k & 1u) {
                    groups[1] = groups[2] = groups[3] = groups[0];
                } else {
#pragma unroll
                    for (int q = 1; q < kQ; ++q) groups[q] = groups_of(size[k * kQ + q]);
                }
#pragma unroll
                for (int q = 0; q < kQ; ++q) {
                    const int j = k * kQ + q;
                    const uint32_t b = static_cast<uint32_t>(ladder_width(a, static_cast<int>(rungs >> (4 * j)) & 15));
                    units[j] = groups[q] * b;
                    own[k] += units[j];
                    widths[k] |= b << (8 * q);
                }
                upto[k] = wave_inclusive_scan(static_cast<V>(own[k]), lane);
            }
            if (lane == kWave - 1) of_waves[k * kAllocWavesMax + wave] = upto[k];
        }
        __syncthreads();
        const V of_wave = of_waves[lane];   // row k of the lanes: round k
        const V scan = row_inclusive_scan(of_wave);
#pragma unroll
        for (int k = 0; k < kAllocQuads; ++k) {
            const uint64_t off = byte_carry + 32u * static_cast<uint64_t>(read_lane(scan, 16 * k + wave) - read_lane(of_wave, 16 * k + wave) + upto[k] - own[k]);
            byte_carry += 32u * static_cast<uint64_t>(read_lane(scan, 16 * k + 15));
            if (!in_round(k)) continue;
            const uint32_t quad[kQ] = {units[k * kQ], units[k * kQ + 1], units[k * kQ + 2], units[k * kQ + 3]};
            store_quad(item(k * kQ), widths[k], quad, off);
        }
    };
    if (!invalid && (elems >> 8) + static_cast<uint64_t>(M) < (uint64_t(1) << 29)) store_rounds(uint32_t(0));
    else store_rounds(uint64_t(0));
    // items beyond the registers, round by round
    for (int64_t base = kAllocQuads * kRound; base < M; base += kRound) {
        int64_t D4[kQ];
        int rung[kQ], ties[kQ];
        uint64_t tie4[kQ], sum = 0, total;
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int64_t i = base + tid * kQ + q;
            D4[q] = i < M ? elements(i) : 0;
            if (D4[q] <= 0 || D4[q] >= (int64_t(1) << 34)) D4[q] = i < M ? 1 : 0;
            rung[q] = v.loose ? 0 : steps;
            ties[q] = 0;
            if (v.search && i < M) {
                const float wi = w[i];
                const uint32_t cls = class_of(bin_of(ratio_of(wi, D4[q])));
                rung[q] = static_cast<int>(cls & 7u);
                if (cls & 8u) settle_item(wi, D4[q], a, br, steps, t.price, rung[q], ties[q]);
            }
            tie4[q] = tie_bits(D4[q], rung[q], ties[q]);
            sum += tie4[q];
        }
        if (t.ties > 1) {
            uint64_t before = tie_carry + block_exclusive_scan(sum, wave_round[0], total);
            tie_carry += total;
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
                apply_ties(D4[q], rung[q], ties[q], before);
                before += tie4[q];
            }
        } else {
#pragma unroll
            for (int q = 0; q < kQ; ++q) rung[q] += ties[q];   // the one move at the threshold is applied
        }
        uint32_t units[kQ], widths = 0;
        uint64_t all = 0;
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const uint32_t b = static_cast<uint32_t>(ladder_width(a, rung[q]));
            units[q] = groups_of(D4[q]) * b;
            all += units[q];
            widths |= b << (8 * q);
        }
        const uint64_t off = byte_carry + 32u * block_exclusive_scan(all, wave_round[1], total);
        byte_carry += 32u * total;
        store_quad(base + tid * kQ, widths, units, off);
        if (t.ties <= 1) __syncthreads();   // wave_round[1] has been read by everyone
    }
    if (tid == 0) {
        result[0] = static_cast<int64_t>(byte_carry);
        result[1] = v.status;
    }
}

// ------------------------------------------------------------------------------------
// Host-side launch geometry.

int check_launch(const char* who)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(ACTQ_EHIP, "%s: launch failed: %s", who, hipGetErrorString(e));
    return ACTQ_OK;
}

}  // namespace

// Groups a wavefront of the quantizer takes: binary16 input with 16-bit noise and a header per group
// has a kernel of its own that works on runs of eight.
static bool quantize_by_runs(int dtype, int noise_bits, int hdr) { return dtype == ACTQ_F16 && noise_bits == 16 && hdr != ACTQ_HDR_TENSOR; }

static int quantize_groups_per_wave(int dtype, int noise_bits, int hdr)
{
    return quantize_by_runs(dtype, noise_bits, hdr) ? kQpGroupsF16 : kTileGroups;
}

// Fills the table but for its first tile; `most` receives the tiles of the largest tensor.
template <int CAPACITY>
static int make_multi_table(const char* who, const actq_tensor* tensors, int32_t count, int64_t N, int64_t first_sample,
                            MultiTable<CAPACITY>* t, int groups_per_wave, uint64_t* most)
{
    t->first_sample = static_cast<uint32_t>(first_sample);
    *most = 0;
    for (int32_t i = 0; i < count; ++i) {
        const int64_t ng = (tensors[i].D + kGroup - 1) / kGroup;
        const uint64_t per_sample = static_cast<uint64_t>((ng + groups_per_wave - 1) / groups_per_wave);
        const uint64_t tiles = per_sample * static_cast<uint64_t>(N);
        if (tiles >= (uint64_t(1) << 31)) return fail(ACTQ_EINVAL, "%s: tensor %d has too many tiles for one launch", who, i);
        if (tiles > *most) *most = tiles;
        MultiItem& it = t->item[i];
        it.x = tensors[i].x;
        it.out = tensors[i].out;
        it.gmin = tensors[i].gmin;
        it.grange = tensors[i].grange;
        it.header = tensors[i].header;
        it.bits = tensors[i].bits;
        it.offsets = tensors[i].offsets;
        it.D = tensors[i].D;
        it.by_tiles = make_fastdiv(static_cast<uint32_t>(per_sample));
        it.tiles = static_cast<uint32_t>(per_sample);
        it.total_tiles = static_cast<uint32_t>(tiles);
    }
    return ACTQ_OK;
}

// A launch has fewer than 2^32 lanes along x, that is 2^26 tiles; kLaunchTiles are whole runs in every order.
constexpr uint64_t kLaunchTiles = uint64_t(1) << 25;

// launch(grid, first tile) for as many launches as `most` tiles need.
template <typename F>
static int each_launch(const char* who, uint64_t most, int32_t count, int waves_per_block, int run, F launch)
{
    // whole runs of 8 * run blocks (`run` blocks per XCD): every order of wave_unit covers a run exactly
    const uint64_t blocks_per_run = 8u * static_cast<uint64_t>(run);
    const uint64_t per_run = blocks_per_run * static_cast<uint64_t>(waves_per_block);
    for (uint64_t first = 0; first < most; first += kLaunchTiles) {
        const uint64_t tiles = most - first < kLaunchTiles ? most - first : kLaunchTiles;
        launch(dim3(static_cast<unsigned>((tiles + per_run - 1) / per_run * blocks_per_run), static_cast<unsigned>(count)),
               static_cast<uint32_t>(first));
        if (int rc = check_launch(who)) return rc;
    }
    return ACTQ_OK;
}

// Whether the statistics leave a tensor of this many bytes in the 256 MiB Infinity Cache, where the quantizer finds (part of) it:
// ordinary loads instead of non-temporal ones.  Compression of one tensor of 64 samples with non-temporal loads (us) and how it changes with
// ordinary ones; "made": a pass writes the tensor in front, behind 768 MiB of other traffic; "in turn": four tensors.
//               24 MiB       48 MiB       80 MiB       144 MiB      176 MiB      208 MiB
// f32, made     23.3 -0.4%   28.4 +0.1%   42.2 -1.2%   61.5 -1.2%   73.1 +4.2%   83.0 +9.6%
// f32, in turn  23.5 +2.5%   28.9 +1.0%   42.7 -1.5%   63.0 -0.5%   73.1 +0.2%   83.1 -0.6%
// f16, made     23.4 +1.5%   34.9 -1.0%   44.7 -2.7%   65.1 -4.0%   75.8 +2.8%   87.6 +6.6%
// f16, in turn  23.3 +0.3%   34.2 +0.3%   44.4 -1.3%   65.1 -2.8%   76.0 -3.5%   87.0 -4.4%
// Samples that end inside a group, made: f32 -4.1, -3.9, -4.7, -4.4, +3.0, +7.4 %; f16 -3.6, -5.6, -7.0, -10.1, -6.6, -4.2 %.  With a pass over the tensor
// behind its compression f32 -4.6, -3.8, -3.4, -1.4, +2.1, +5.6 %.  The statistics by themselves, in turn, are behind: f32 from 64 MiB on 7 to 28 %, f16 6 to 19 %.
// The limit is the largest size at which the compression of a tensor that was just made does not lose; below 80 MiB f32 in turn loses up to 3 %.
// Tensor sets keep non-temporal loads: the statistics of all their tensors run in front of the first codes, and sets that fit the cache as a whole are not measured.
static bool stays_cached(int64_t bytes) { return bytes <= int64_t(144) << 20; }

// Launches with a table of CAPACITY items; ragged samples come as single tensors only.
template <int CAPACITY>
static int group_stats_launch(const char* who, const actq_tensor* tensors, int32_t count, int dtype, int64_t N, bool ragged, hipStream_t s)
{
    MultiTable<CAPACITY> t;
    uint64_t most;
    if (int rc = make_multi_table(who, tensors, count, N, 0, &t, kTileGroups, &most)) return rc;
    return each_launch(who, most, count, kGsBlock / kWave, kGsRun, [&](dim3 grid, uint32_t first) {
        t.first_tile = first;
        const auto typed = [&](auto element, auto nt) {
            typedef decltype(element) T;
            constexpr bool kNt = decltype(nt)::value;
            if constexpr (CAPACITY == 1) {
                if (ragged) {
                    launch(group_stats_multi_kernel<T, true, kNt, 1>, grid, kGsBlock, s, t);
                    return;
                }
                // Binary16, samples of whole tiles, non-temporal loads: every second workgroup fills a line of 128 bytes of either result, and runs of no more
                // workgroups read 16 KiB per XCD in turn: [256, 802816] 59.4 -> 57.1 us, [13032, 15360] 58.0 -> 55.6, all 1.5 to 5 % less.  Elsewhere lines are
                // shared by XCDs, [7551, 23808] 52.8 -> 56.7, and binary32 loses ([128, 802816] 57.8 -> 60.2); sets of tensors -4 to +1 %.  With ordinary loads
                // runs of two are up to 3 % behind from 100 MB on ([14352, 5120] 23.8 -> 24.5) and 0.05 to 0.1 of 2 us on the smallest tensors.
                if constexpr (std::is_same<T, _Float16>::value && kNt) {
                    if (tensors[0].D % (kTileGroups * kGroup) == 0) {
                        launch(group_stats_multi_kernel<T, false, kNt, 1, kGsRunHalf>, grid, kGsBlock, s, t);
                        return;
                    }
                }
            }
            launch(group_stats_multi_kernel<T, false, kNt, CAPACITY>, grid, kGsBlock, s, t);
        };
        if constexpr (CAPACITY == 1) {
            if (stays_cached(N * tensors[0].D * (dtype == ACTQ_F32 ? 4 : 2))) {
                if (dtype == ACTQ_F32) typed(float(), std::false_type());
                else typed(_Float16(), std::false_type());
                return;
            }
        }
        if (dtype == ACTQ_F32) typed(float(), std::true_type());
        else typed(_Float16(), std::true_type());
    });
}

struct QuantizeCall {
    uint64_t seed, tag;
    int noise_bits, hdr;
    uint8_t* packed;
    uint64_t capacity;
};

template <typename T, int NOISE_BITS, int HDR, int CAPACITY>
static void quantize_tile_launch(bool ragged, const MultiTable<CAPACITY>& t, dim3 grid, const QuantizeCall& c, hipStream_t s)
{
    const uint32_t k0 = static_cast<uint32_t>(c.seed), k1 = static_cast<uint32_t>(c.seed >> 32);
    if constexpr (CAPACITY == 1) {
        if (ragged) {
            launch(quantize_pack_tile_kernel<T, NOISE_BITS, HDR, true, 1>, grid, kBlock, s, t, k0, k1, c.tag, c.packed, c.capacity);
            return;
        }
    }
    launch(quantize_pack_tile_kernel<T, NOISE_BITS, HDR, false, CAPACITY>, grid, kBlock, s, t, k0, k1, c.tag, c.packed, c.capacity);
}

template <int HDR, int CAPACITY>
static void quantize_run_launch(bool ragged, const MultiTable<CAPACITY>& t, dim3 grid, const QuantizeCall& c, hipStream_t s)
{
    const uint32_t k0 = static_cast<uint32_t>(c.seed), k1 = static_cast<uint32_t>(c.seed >> 32);
    if constexpr (CAPACITY == 1) {
        if (ragged) {
            launch(quantize_pack_run_kernel<HDR, true, 1>, grid, kBlock, s, t, k0, k1, c.tag, c.packed, c.capacity);
            return;
        }
    }
    launch(quantize_pack_run_kernel<HDR, false, CAPACITY>, grid, kBlock, s, t, k0, k1, c.tag, c.packed, c.capacity);
}

template <int CAPACITY>
static int quantize_launch(const char* who, const actq_tensor* tensors, int32_t count, int dtype, int64_t N, int64_t first_sample,
                           bool ragged, const QuantizeCall& c, hipStream_t s)
{
    MultiTable<CAPACITY> t;
    uint64_t most;
    if (int rc = make_multi_table(who, tensors, count, N, first_sample, &t, quantize_groups_per_wave(dtype, c.noise_bits, c.hdr), &most)) return rc;
    return each_launch(who, most, count, kWavesPerBlock, kQpRun, [&](dim3 grid, uint32_t first) {
        t.first_tile = first;
        if (dtype == ACTQ_F32) {
            if (c.noise_bits == 16) {
                if (c.hdr == ACTQ_HDR_F32) quantize_tile_launch<float, 16, 0>(ragged, t, grid, c, s);
                else if (c.hdr == ACTQ_HDR_BF16) quantize_tile_launch<float, 16, 1>(ragged, t, grid, c, s);
                else quantize_tile_launch<float, 16, 2>(ragged, t, grid, c, s);
            } else {
                if (c.hdr == ACTQ_HDR_F32) quantize_tile_launch<float, 24, 0>(ragged, t, grid, c, s);
                else if (c.hdr == ACTQ_HDR_BF16) quantize_tile_launch<float, 24, 1>(ragged, t, grid, c, s);
                else quantize_tile_launch<float, 24, 2>(ragged, t, grid, c, s);
            }
        } else if (c.noise_bits == 16) {
            if (c.hdr == ACTQ_HDR_F32) quantize_run_launch<0>(ragged, t, grid, c, s);
            else if (c.hdr == ACTQ_HDR_BF16) quantize_run_launch<1>(ragged, t, grid, c, s);
            else quantize_tile_launch<_Float16, 16, 2>(ragged, t, grid, c, s);
        } else {
            if (c.hdr == ACTQ_HDR_F32) quantize_tile_launch<_Float16, 24, 0>(ragged, t, grid, c, s);
            else if (c.hdr == ACTQ_HDR_BF16) quantize_tile_launch<_Float16, 24, 1>(ragged, t, grid, c, s);
            else quantize_tile_launch<_Float16, 24, 2>(ragged, t, grid, c, s);
        }
    });
}

template <typename T, int NG, int HDR, int CAPACITY>
static void dequantize_typed_launch(int layout, const MultiTable<CAPACITY>& t, dim3 grid, const uint8_t* pk, uint64_t capacity, hipStream_t s)
{
    if constexpr (CAPACITY == 1) {
        if (layout == kRaggedLines) {
            launch(unpack_dequantize_multi_kernel<T, HDR, NG, kRaggedLines, 1>, grid, kDqBlock, s, t, pk, capacity);
            return;
        }
        if (layout == kRagged) {
            launch(unpack_dequantize_multi_kernel<T, HDR, NG, kRagged, 1>, grid, kDqBlock, s, t, pk, capacity);
            return;
        }
    }
    launch(unpack_dequantize_multi_kernel<T, HDR, NG, kWholeGroups, CAPACITY>, grid, kDqBlock, s, t, pk, capacity);
}

template <typename T, int NG, int CAPACITY>
static int dequantize_launch(const char* who, const actq_tensor* tensors, int32_t count, const void* packed, uint64_t capacity, int hdr,
                             int64_t N, int layout, hipStream_t s)
{
    MultiTable<CAPACITY> t;
    uint64_t most;
    if (int rc = make_multi_table(who, tensors, count, N, 0, &t, NG, &most)) return rc;
    const uint8_t* pk = static_cast<const uint8_t*>(packed);
    return each_launch(who, most, count, kDqBlock / kWave, layout == kWholeGroups ? 1 : kDqRaggedRun, [&](dim3 grid, uint32_t first) {
        t.first_tile = first;
        if (hdr == ACTQ_HDR_F32) dequantize_typed_launch<T, NG, 0>(layout, t, grid, pk, capacity, s);
        else if (hdr == ACTQ_HDR_BF16) dequantize_typed_launch<T, NG, 1>(layout, t, grid, pk, capacity, s);
        else dequantize_typed_launch<T, NG, 2>(layout, t, grid, pk, capacity, s);
    });
}

// A single tensor is a table of one.  A table counts fewer than 2^31 tiles per tensor: a tensor with more
// (2^31 samples of a group each, say) goes sample range by sample range.  f(first sample, samples) is one.
template <typename F>
static int by_sample_ranges(int64_t N, int64_t D, int groups_per_wave, F f)
{
    const int64_t ng = (D + kGroup - 1) / kGroup;
    const int64_t per_sample = (ng + groups_per_wave - 1) / groups_per_wave;
    const int64_t most = ((int64_t(1) << 31) - 1) / per_sample / 4 * 4;   // multiples of four keep the widths 4-byte aligned
    for (int64_t n0 = 0; n0 < N; n0 += most)
        if (int rc = f(n0, N - n0 < most ? N - n0 : most)) return rc;
    return ACTQ_OK;
}

template <typename P>
static P* advance(P* p, int64_t bytes)
{
    return p ? reinterpret_cast<P*>(reinterpret_cast<uintptr_t>(p) + static_cast<uintptr_t>(bytes)) : p;
}

static int64_t element_bytes(int dtype) { return dtype == ACTQ_F32 ? 4 : 2; }

static int64_t header_bytes_of(int hdr, int64_t groups) { return hdr == ACTQ_HDR_TENSOR ? 0 : groups * (hdr == ACTQ_HDR_BF16 ? 4 : 8); }

int launch_group_stats(const void* x, int dtype, int64_t N, int64_t D, float* gmin, float* grange,
                       void* stream)
{
    const int64_t ng = (D + kGroup - 1) / kGroup;
    return by_sample_ranges(N, D, kTileGroups, [&](int64_t n0, int64_t count) {
        actq_tensor one = {};
        one.x = advance(x, n0 * D * element_bytes(dtype));
        one.gmin = gmin + n0 * ng;
        one.grange = grange + n0 * ng;
        one.D = D;
        return group_stats_launch<1>("actq_group_stats", &one, 1, dtype, count, D % kGroup != 0, static_cast<hipStream_t>(stream));
    });
}

int launch_quantize_pack(const void* x, int dtype, int64_t N, int64_t D, const uint8_t* bits,
                         const uint64_t* offsets, uint64_t seed, uint64_t tag, int noise_bits,
                         void* packed, uint64_t capacity, void* header, int hdr, void* stream)
{
    const int64_t ng = (D + kGroup - 1) / kGroup;
    const QuantizeCall call = {seed, tag, noise_bits, hdr, static_cast<uint8_t*>(packed), capacity};
    return by_sample_ranges(N, D, quantize_groups_per_wave(dtype, noise_bits, hdr), [&](int64_t n0, int64_t count) {
        actq_tensor one = {};
        one.x = advance(x, n0 * D * element_bytes(dtype));
        one.header = advance(header, header_bytes_of(hdr, n0 * ng));
        one.bits = bits + n0;
        one.offsets = offsets + n0;
        one.D = D;
        return quantize_launch<1>("actq_quantize_pack", &one, 1, dtype, count, n0, D % kGroup != 0, call, static_cast<hipStream_t>(stream));
    });
}

int launch_unpack_dequantize(const void* packed, uint64_t capacity, const void* header, int hdr,
                             const uint8_t* bits, const uint64_t* offsets, int64_t N, int64_t D,
                             void* out, int out_dtype, void* stream)
{
    const int64_t ng = (D + kGroup - 1) / kGroup;
    const bool lines = D * element_bytes(out_dtype) % 128 == 0 && reinterpret_cast<uintptr_t>(out) % 128 == 0;
    // Samples of whole groups whose last tile is short.  Where they are an even number of tiles, XCDs that take every eighth tile do not get alike: of two
    // tiles per sample, a long and a short one, every second XCD gets the short ones and is nearly idle.  Where they are an odd number of groups, hardly a
    // tile begins where 4 KiB of the output do.  From 48 MiB on such tensors take the order of the samples that end inside a group, runs of sixteen workgroups
    // per XCD, where that was faster at every width (us; widths the same everywhere or mixed with that mean, either header):
    //   an even number of tiles up to six, of whose room an eighth (binary32: a quarter) is empty, at any width: binary16 [20507, 2560] 31.3 -> 24.4, at eight
    //     bits 33.8 -> 27.5, [3627, 7168] 13.1 -> 12.6, at four 13.3 -> 13.4; binary32 [29296, 1280] 40.2 -> 32.9, at eight 38.4 -> 33.9, but at six with the
    //     binary32 header [78125, 1280] 92 -> 97.  Less empty room, or more tiles: [3385, 7680] 12.2 -> 12.7, binary32 [30048, 3328] at a mean of four 82.1 -> 86.3;
    //   odd numbers of groups, and binary32 with an eighth empty, at up to 3.25 bits per element: binary16 [32552, 4352] 0.85 to 0.99 of the time, [64, 817408]
    //     23.7 -> 22.7, at three bits everywhere [5974, 4352] 14.6 -> 15.0; binary32 [11268, 3328] 36.7 -> 31.1, [16276, 2304] 35.8 -> 31.4, at worst
    //     [18601, 5376] 79.5 -> 81.3.  At four bits and more [43402, 2304] 74 -> 84, binary16 at five [5974, 4352] 15.0 -> 16.3, though mixed widths gain
    //     up to there.  The widths are on the device; what the stream may take is known;
    //   long binary32 samples up to 160 MiB: [45, 817408] 0.91 to 0.99 of the time, [122, 817408] with mixed widths 71.8 -> 78.3.
    // Up to 16 MB the runs keep too few XCDs busy (+25 % at worst), at 26 MB -16 to +14 %; samples of at most half a tile 0 to +84 %.
    const bool half = out_dtype == ACTQ_F16;
    const int64_t per_tile = half ? kDqGroupsF16 : kDqGroupsF32, tiles = (ng + per_tile - 1) / per_tile, room = tiles * per_tile, output = N * D * element_bytes(out_dtype);
    const bool idle = tiles % 2 == 0 && tiles <= 6 && 8 * (room - ng) >= room;
    const bool at_any_width = idle && (half || 4 * (room - ng) >= room);
    const bool narrow = capacity <= static_cast<uint64_t>(N) * static_cast<uint64_t>(ng) * 104;   // bytes of a group at 3.25 bits
    const bool at_narrow_widths = (idle || ng % 2 == 1) && (half || ng <= 128 || output <= int64_t(160) << 20);
    const bool runs = lines && ng > per_tile / 2 && output >= int64_t(48) << 20 && (at_any_width || (narrow && at_narrow_widths));
    const int layout = D % kGroup == 0 && !runs ? kWholeGroups : (lines ? kRaggedLines : kRagged);
    hipStream_t s = static_cast<hipStream_t>(stream);
    return by_sample_ranges(N, D, out_dtype == ACTQ_F16 ? kDqGroupsF16 : kDqGroupsF32, [&](int64_t n0, int64_t count) {
        actq_tensor one = {};
        one.out = advance(out, n0 * D * element_bytes(out_dtype));
        one.header = const_cast<void*>(advance(header, header_bytes_of(hdr, n0 * ng)));
        one.bits = bits + n0;
        one.offsets = offsets + n0;
        one.D = D;
        if (out_dtype == ACTQ_F32) return dequantize_launch<float, kDqGroupsF32, 1>("actq_unpack_dequantize", &one, 1, packed, capacity, hdr, count, layout, s);
        return dequantize_launch<_Float16, kDqGroupsF16, 1>("actq_unpack_dequantize", &one, 1, packed, capacity, hdr, count, layout, s);
    });
}

int launch_group_stats_multi(const actq_tensor* tensors, int32_t count, int dtype, int64_t N, void* stream)
{
    const char* who = "actq_group_stats_multi";
    hipStream_t s = static_cast<hipStream_t>(stream);
    return count == 1 ? group_stats_launch<1>(who, tensors, count, dtype, N, false, s)
                      : group_stats_launch<kMaxMulti>(who, tensors, count, dtype, N, false, s);
}

int launch_quantize_pack_multi(const actq_tensor* tensors, int32_t count, int dtype, int64_t N, uint64_t seed,
                               uint64_t tag, int noise_bits, void* packed, uint64_t capacity, int hdr, void* stream)
{
    const char* who = "actq_quantize_pack_multi";
    hipStream_t s = static_cast<hipStream_t>(stream);
    const QuantizeCall call = {seed, tag, noise_bits, hdr, static_cast<uint8_t*>(packed), capacity};
    return count == 1 ? quantize_launch<1>(who, tensors, count, dtype, N, 0, false, call, s)
                      : quantize_launch<kMaxMulti>(who, tensors, count, dtype, N, 0, false, call, s);
}

template <int CAPACITY>
static int dequantize_multi(const actq_tensor* tensors, int32_t count, const void* packed, uint64_t capacity, int hdr, int64_t N,
                            int out_dtype, hipStream_t s)
{
    const char* who = "actq_unpack_dequantize_multi";
    if (out_dtype == ACTQ_F32) return dequantize_launch<float, kDqGroupsF32, CAPACITY>(who, tensors, count, packed, capacity, hdr, N, kWholeGroups, s);
    return dequantize_launch<_Float16, kDqGroupsF16, CAPACITY>(who, tensors, count, packed, capacity, hdr, N, kWholeGroups, s);
}

int launch_unpack_dequantize_multi(const actq_tensor* tensors, int32_t count, const void* packed, uint64_t capacity,
                                   int hdr, int64_t N, int out_dtype, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    return count == 1 ? dequantize_multi<1>(tensors, count, packed, capacity, hdr, N, out_dtype, s)
                      : dequantize_multi<kMaxMulti>(tensors, count, packed, capacity, hdr, N, out_dtype, s);
}

int launch_allocate_bits(const float* w, const int64_t* D_items, int64_t D, int64_t M, int64_t budget_bits,
                         const Ladder& lad, uint8_t* bits, uint64_t* offsets, int64_t* result, void* stream)
{
    uint32_t width_nibbles = 0;
    for (int k = 0; k < lad.count; ++k) width_nibbles |= static_cast<uint32_t>(lad.width[k]) << (4 * k);
    const AllocBudget total = {static_cast<uint64_t>(budget_bits), static_cast<uint32_t>(lad.width[0]), static_cast<uint32_t>(lad.width[lad.count - 1])};
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool two = M > kAllocBlock;   // items per thread
    if (!two || (M <= kSmallItems * kAllocBlock && (!D_items || M * (lad.count - 1) <= kSmallMoves))) {
        SmallAllocArgs a = {};
        a.M = static_cast<int32_t>(M);
        a.steps = lad.count - 1;
        a.width_nibbles = width_nibbles;
        a.D = D;
        a.D_items = D_items;
        a.total = total;
        for (int r = 0; r < kMaxSteps; ++r) a.price[r] = lad.price[r];
        if (!D_items) {
            const AllocVerdict v = alloc_verdict(static_cast<uint64_t>(M) * static_cast<uint64_t>(D), false, total);
            a.search = v.search;
            a.loose = v.loose;
            a.status = static_cast<int32_t>(v.status);
            a.need = v.search ? static_cast<uint32_t>((v.need + static_cast<uint64_t>(D) - 1) / static_cast<uint64_t>(D)) : 0u;
            a.unit_bytes = static_cast<uint64_t>((D + kGroup - 1) / kGroup) * (kGroup / 8);
            a.reciprocal = 1.0 / static_cast<double>(D);
        }
        const int64_t lanes = (M + kWave - 1) / kWave * kWave;
        const unsigned block = static_cast<unsigned>(lanes < kAllocBlock ? lanes : kAllocBlock);
        if (D_items && two) launch(allocate_bits_small_kernel<false, kSmallItems>, 1, block, s, w, a, bits, offsets, result);
        else if (D_items) launch(allocate_bits_small_kernel<false, 1>, 1, block, s, w, a, bits, offsets, result);
        else if (two) launch(allocate_bits_small_kernel<true, kSmallItems>, 1, block, s, w, a, bits, offsets, result);
        else launch(allocate_bits_small_kernel<true, 1>, 1, block, s, w, a, bits, offsets, result);
    } else {
        AllocArgs a;
        a.M = M;
        a.D = D;
        a.D_items = D_items;
        a.total = total;
        a.lad = lad;
        for (int r = 0; r < kMaxSteps; ++r) a.inverse[r] = r + 1 < lad.count ? 1.0 / lad.price[r] : 0.0;
        a.width_nibbles = width_nibbles;
        launch(allocate_bits_kernel, 1, kAllocBlock, s, w, a, bits, offsets, result);
    }
    return check_launch("actq_allocate_bits_device");
}

int launch_tensor_stats(const void* x, int dtype, int64_t n, float* zr, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint32_t* words = reinterpret_cast<uint32_t*>(zr);
    const int64_t chunks = n / (dtype == ACTQ_F32 ? 4 : 8);
    int64_t blocks = (chunks + kBlock - 1) / kBlock;
    if (blocks < 1) blocks = 1;
    if (blocks > 2048) blocks = 2048;  // eight resident blocks per compute unit: 4096 atomics in all
    launch(tensor_stats_init_kernel, 1, kWave, s, words);
    if (dtype == ACTQ_F32)
        launch(tensor_stats_reduce_kernel<float>, static_cast<unsigned>(blocks), kBlock, s, static_cast<const float*>(x), n, words);
    else
        launch(tensor_stats_reduce_kernel<_Float16>, static_cast<unsigned>(blocks), kBlock, s, static_cast<const _Float16*>(x), n, words);
    launch(tensor_stats_finish_kernel, 1, kWave, s, words);
    return check_launch("actq_tensor_stats");
}

int launch_sample_sensitivity(const float* grange, int64_t N, int64_t ng, int32_t G, const float* grad2,
                              float* w, void* stream)
{
    const uint32_t gx = N < 65535 ? static_cast<uint32_t>(N) : 65535u;
    const uint32_t gy = static_cast<uint32_t>((N + gx - 1) / gx);
    if (gy > 65535u) return fail(ACTQ_EINVAL, "actq_sample_sensitivity: too many samples for one launch");
    // one lane per group up to 1024 lanes, whole wavefronts
    const int64_t lanes = (ng + kWave - 1) / kWave * kWave;
    const unsigned block = static_cast<unsigned>(lanes < kSensMaxBlock ? lanes : kSensMaxBlock);
    launch(sample_sensitivity_kernel, dim3(gx, gy), block, static_cast<hipStream_t>(stream),
        grange, static_cast<uint32_t>(N), static_cast<uint32_t>(ng), gx, static_cast<float>(G) / 6.0f, grad2, w);
    return check_launch("actq_sample_sensitivity");
}

}  // namespace actq
