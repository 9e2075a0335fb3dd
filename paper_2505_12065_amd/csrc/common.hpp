// Device-side building blocks shared by the flat-scan and graph-search kernels
// (gfx950 / CDNA4 only: 64-wide wavefronts, MFMA, LDS).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <limits.h>
#include <math.h>
#include <utility>

#include "plan.hpp"

namespace ann {

typedef uint32_t u4 __attribute__((ext_vector_type(4)));       // one raw 16-byte chunk
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));

// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>): a loop the compiler
// cannot decline to unroll, so register arrays indexed by it stay in registers
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_impl(static_cast<F &&>(f), std::make_integer_sequence<int, N>{});
}

// Blocks are dealt to the 8 XCDs (each with its own L2) round-robin.  The number of this block in an order in which every
// XCD has a run of neighbours: work that shares data is numbered side by side and is then fetched into one L2.
__device__ __forceinline__ int xcd_block() {
    const int per = gridDim.x >> 3, more = gridDim.x & 7, xcd = blockIdx.x & 7;
    return xcd * per + min(xcd, more) + (int)(blockIdx.x >> 3);
}

struct F16 { static constexpr int bytes = 2; };
struct BF16 { static constexpr int bytes = 2; };
struct F32 { static constexpr int bytes = 4; };

// ---- order -------------------------------------------------------------------------------
// (s, id) precedes (s2, id2): larger score first, equal scores by lower id.
__device__ __forceinline__ bool precedes(float s, int id, float s2, int id2) {
    return s > s2 || (s == s2 && id < id2);
}

constexpr int EMPTY_ID = INT_MAX;   // id of an unused list slot (its score is -inf)

// Sorted list of the KP best (score, id) pairs, held in registers (every index
// is a compile-time constant after unrolling).
template <int KP>
struct TopList {
    float s[KP];
    int id[KP];

    __device__ __forceinline__ void init() {
#pragma unroll
        for (int i = 0; i < KP; ++i) { s[i] = -INFINITY; id[i] = EMPTY_ID; }
    }
    // true when (v, vid) would enter the list
    __device__ __forceinline__ bool admits(float v, int vid) const {
        return precedes(v, vid, s[KP - 1], id[KP - 1]);
    }
    // insert (v, vid); a pair that does not precede the last entry is dropped
    __device__ __forceinline__ void insert(float v, int vid) {
        bool before[KP];
#pragma unroll
        for (int i = 0; i < KP; ++i) before[i] = precedes(v, vid, s[i], id[i]);
#pragma unroll
        for (int i = KP - 1; i > 0; --i) {
            s[i] = before[i - 1] ? s[i - 1] : (before[i] ? v : s[i]);
            id[i] = before[i - 1] ? id[i - 1] : (before[i] ? vid : id[i]);
        }
        s[0] = before[0] ? v : s[0];
        id[0] = before[0] ? vid : id[0];
    }
};

// ---- selection across lanes ------------------------------------------------------------------
// (score, id) -> 64-bit key whose unsigned order is the list order: larger score first, equal
// scores by lower id.  -0 is folded into +0 so that equal scores compare equal; an empty slot
// (-inf, EMPTY_ID) maps to the smallest key any list entry can have.
__device__ __forceinline__ uint64_t order_key(float s, int id) {
    uint32_t b = __float_as_uint(s + 0.0f);
    b = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    return ((uint64_t)b << 32) | (uint32_t)~id;
}
__device__ __forceinline__ void order_key_decode(uint64_t key, float &s, int &id) {
    uint32_t b = (uint32_t)(key >> 32);
    b = (b & 0x80000000u) ? (b ^ 0x80000000u) : ~b;
    s = __uint_as_float(b);
    id = (int)~(uint32_t)key;
}

// Lane exchanges inside a wave without a trip through the LDS crossbar: data-parallel-primitive moves inside
// rows of 16 lanes, row swaps (gfx950) between them.
template <int CTRL>
__device__ __forceinline__ int dpp_move(int x) {
    return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xf, 0xf, false);
}
constexpr int DPP_SWAP1 = 0xB1;                           // quad_perm [1,0,3,2]
constexpr int DPP_SWAP2 = 0x4E;                           // quad_perm [2,3,0,1]
constexpr int DPP_SWAP3 = 0x1B;                           // quad_perm [3,2,1,0]
constexpr int DPP_HALF_MIRROR = 0x141;                    // lane i of each 8 <- lane 7 - i
constexpr int DPP_MIRROR = 0x140;                         // lane i of each 16 <- lane 15 - i
constexpr int DPP_ROR8 = 0x128;                           // lane i of each 16 <- lane i ^ 8

// the values of lane and lane ^ MASK (MASK 16 or 32), in either order: enough for a maximum or a minimum
template <int MASK>
__device__ __forceinline__ void row_pair(uint32_t x, uint32_t &a, uint32_t &b) {
    static_assert(MASK == 16 || MASK == 32, "rows of 16 lanes");
    if constexpr (MASK == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        a = r[0]; b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        a = r[0]; b = r[1];
    }
}
// lane <- lane ^ MASK, MASK a power of two below 16
template <int MASK>
__device__ __forceinline__ uint32_t lane_swap(uint32_t x) {
    static_assert(MASK == 1 || MASK == 2 || MASK == 4 || MASK == 8, "inside a row of 16 lanes");
    if constexpr (MASK == 1) return (uint32_t)dpp_move<DPP_SWAP1>((int)x);
    else if constexpr (MASK == 2) return (uint32_t)dpp_move<DPP_SWAP2>((int)x);
    else if constexpr (MASK == 4) return (uint32_t)dpp_move<DPP_SWAP3>(dpp_move<DPP_HALF_MIRROR>((int)x));
    else return (uint32_t)dpp_move<DPP_ROR8>((int)x);
}

// maximum of x over the lanes whose numbers differ only in the bits LO <= bit < HI, in every one of them
template <int LO, int HI>
__device__ __forceinline__ uint64_t group_max(uint64_t x) {
    auto step = [&](uint32_t lo, uint32_t hi) {
        const uint64_t o = ((uint64_t)hi << 32) | lo;
        x = o > x ? o : x;
    };
    if constexpr (LO <= 1 && HI > 1) step(lane_swap<1>((uint32_t)x), lane_swap<1>((uint32_t)(x >> 32)));
    if constexpr (LO <= 2 && HI > 2) step(lane_swap<2>((uint32_t)x), lane_swap<2>((uint32_t)(x >> 32)));
    if constexpr (LO <= 4 && HI > 4) step(lane_swap<4>((uint32_t)x), lane_swap<4>((uint32_t)(x >> 32)));
    if constexpr (LO <= 8 && HI > 8) step(lane_swap<8>((uint32_t)x), lane_swap<8>((uint32_t)(x >> 32)));
    auto rows = [&](auto mc) {
        uint32_t l0, l1, h0, h1;
        row_pair<decltype(mc)::value>((uint32_t)x, l0, l1);
        row_pair<decltype(mc)::value>((uint32_t)(x >> 32), h0, h1);
        const uint64_t a = ((uint64_t)h0 << 32) | l0, b = ((uint64_t)h1 << 32) | l1;
        x = a > b ? a : b;
    };
    if constexpr (LO <= 16 && HI > 16) rows(std::integral_constant<int, 16>{});
    if constexpr (LO <= 32 && HI > 32) rows(std::integral_constant<int, 32>{});
    return x;
}

// x sorted over the lanes of each aligned group of G lanes (32 or 64), largest first: a bitonic network of 15 or
// 21 compare-and-exchange steps, four vector instructions each.
template <int G>
__device__ __forceinline__ uint32_t group_sort_desc(uint32_t x) {
    const int lane = threadIdx.x & (WAVE - 1);
    auto step = [&](auto kc, auto jc) {
        constexpr int K = decltype(kc)::value, J = decltype(jc)::value;
        // inside a block of K lanes whose bit K is clear the larger value goes to the lower lane
        const bool larger = ((lane & J) == 0) == ((lane & K) == 0 || K == G);
        uint32_t a = x, b;
        if constexpr (J >= 16) row_pair<J>(x, a, b);
        else b = lane_swap<J>(x);
        x = larger ? (a > b ? a : b) : (a > b ? b : a);
    };
    auto merge = [&](auto kc) {
        constexpr int K = decltype(kc)::value;
        if constexpr (K >= 64) step(kc, std::integral_constant<int, 32>{});
        if constexpr (K >= 32) step(kc, std::integral_constant<int, 16>{});
        if constexpr (K >= 16) step(kc, std::integral_constant<int, 8>{});
        if constexpr (K >= 8) step(kc, std::integral_constant<int, 4>{});
        if constexpr (K >= 4) step(kc, std::integral_constant<int, 2>{});
        step(kc, std::integral_constant<int, 1>{});
    };
    merge(std::integral_constant<int, 2>{});
    merge(std::integral_constant<int, 4>{});
    merge(std::integral_constant<int, 8>{});
    merge(std::integral_constant<int, 16>{});
    merge(std::integral_constant<int, 32>{});
    if constexpr (G == 64) merge(std::integral_constant<int, 64>{});
    return x;
}

// out <- the KP best entries of the sorted lists `in` held by the lanes whose numbers differ
// only in the bits LO <= bit < HI (LO, HI powers of two; HI = 64: up to the whole wave);
// every lane of such a group receives the same result.  KP rounds of "largest list head wins and
// is popped": a round costs one max-reduction instead of a full list merge.  An entry held
// by several lanes is taken once.
template <int KP, int LP, int LO, int HI>
__device__ __forceinline__ void group_top(const TopList<LP> &in, TopList<KP> &out) {
    uint64_t key[LP];
#pragma unroll
    for (int i = 0; i < LP; ++i) key[i] = order_key(in.s[i], in.id[i]);
    const uint64_t empty = order_key(-INFINITY, EMPTY_ID);
#pragma unroll
    for (int r = 0; r < KP; ++r) {
        const uint64_t m = group_max<LO, HI>(key[0]);
        if (key[0] == m) {
#pragma unroll
            for (int i = 0; i + 1 < LP; ++i) key[i] = key[i + 1];
            key[LP - 1] = empty;
        }
        order_key_decode(m, out.s[r], out.id[r]);
    }
}

// ---- 16-byte chunks -----------------------------------------------------------------------
__device__ __forceinline__ u4 load_chunk(const void *p) { return *reinterpret_cast<const u4 *>(p); }

__device__ __forceinline__ u4 zero_chunk() { u4 z = {0u, 0u, 0u, 0u}; return z; }

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

// acc + <x, q> over one 16-byte chunk of each operand, fp32 accumulation: 16-bit inputs by v_dot2c_f32_{f16,bf16}, two exact
// products added to the fp32 accumulator per instruction, fp32 by FMA.  Four accumulators, one per 4 bytes of the chunk:
// four independent chains (a dependent chain of dot instructions issues several times slower than independent ones), for
// lanes that add up many chunks one after the other.  The caller adds the four.
template <class T>
__device__ __forceinline__ void dot_chunk4(u4 x, u4 q, f4 &acc);

template <>
__device__ __forceinline__ void dot_chunk4<F16>(u4 x, u4 q, f4 &acc) {
    const h8 a = __builtin_bit_cast(h8, x), b = __builtin_bit_cast(h8, q);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        acc[i] = __builtin_amdgcn_fdot2(h2{a[2 * i], a[2 * i + 1]}, h2{b[2 * i], b[2 * i + 1]}, acc[i], false);
}

template <>
__device__ __forceinline__ void dot_chunk4<BF16>(u4 x, u4 q, f4 &acc) {
    const b8 a = __builtin_bit_cast(b8, x), b = __builtin_bit_cast(b8, q);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        acc[i] = __builtin_amdgcn_fdot2_f32_bf16(bf2{a[2 * i], a[2 * i + 1]}, bf2{b[2 * i], b[2 * i + 1]}, acc[i], false);
}

template <>
__device__ __forceinline__ void dot_chunk4<F32>(u4 x, u4 q, f4 &acc) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = fmaf(__uint_as_float(x[i]), __uint_as_float(q[i]), acc[i]);
}

// ---- MFMA ---------------------------------------------------------------------------------
// D[16x16] += A[16x32] * B[32x16].  Lane l supplies A[l % 16][8*(l/16) .. +8) and
// B[8*(l/16) .. +8)[l % 16]; it receives D[4*(l/16) + i][l % 16], i = 0..3.
template <class T>
__device__ __forceinline__ f4 mfma16(u4 a, u4 b, f4 c);

template <>
__device__ __forceinline__ f4 mfma16<F16>(u4 a, u4 b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}
template <>
__device__ __forceinline__ f4 mfma16<BF16>(u4 a, u4 b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0);
}

// Sums of products of 16 rows with 16 columns over 64-byte steps, on the 16x16 matrix instructions.  Step s of an
// operand is one 16-byte chunk per lane: chunk 4 s + l/16 of row (column) l % 16, made ready by `operand`.
template <class T>
struct TileSum {                                          // 16 bits: one instruction of 32 columns per step
    f4 a;
    static __device__ __forceinline__ u4 operand(u4 x) { return x; }
    __device__ __forceinline__ void clear() { a = f4{0.f, 0.f, 0.f, 0.f}; }
    __device__ __forceinline__ void step(int, u4 x, u4 y) { a = mfma16<T>(x, y, a); }
    __device__ __forceinline__ f4 sum() const { return a; }
};
// fp32: the 16x16x4 instruction is a chain of four fused multiply-adds in column order (checked bit for bit), so it
// takes one chunk of 4 columns; `operand` turns the lane's chunk round (a 4 x 4 transpose between the four registers
// and the four rows of 16 lanes: register j of lane l then holds column l/16 of chunk 4 s + j).  Eight partial
// sums, of chunks c = 0 .. 7 modulo 8, added pairwise at the end: chains an eighth as long as a single sum's.
template <>
struct TileSum<F32> {
    f4 a[8];
    static __device__ __forceinline__ u4 operand(u4 x) {
        auto r = __builtin_amdgcn_permlane32_swap(x[0], x[2], false, false);
        x[0] = r[0]; x[2] = r[1];
        r = __builtin_amdgcn_permlane32_swap(x[1], x[3], false, false);
        x[1] = r[0]; x[3] = r[1];
        r = __builtin_amdgcn_permlane16_swap(x[0], x[1], false, false);
        x[0] = r[0]; x[1] = r[1];
        r = __builtin_amdgcn_permlane16_swap(x[2], x[3], false, false);
        x[2] = r[0]; x[3] = r[1];
        return x;
    }
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int c = 0; c < 8; ++c) a[c] = f4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void step(int s, u4 x, u4 y) {            // (s & 1 a constant after unrolling)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f4 &c = a[(s & 1) * 4 + j];
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x[j]), __uint_as_float(y[j]), c, 0, 0, 0);
        }
    }
    __device__ __forceinline__ f4 sum() const { return ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])); }
};

// D[32x32] += A[32x16] * B[16x32].  Lane l supplies A[l % 32][8*(l/32) .. +8) and
// B[8*(l/32) .. +8)[l % 32]; it receives D[8*(i/4) + 4*(l/32) + i%4][l % 32], i = 0..15.
template <class T>
__device__ __forceinline__ f16v mfma32(u4 a, u4 b, f16v c);

template <>
__device__ __forceinline__ f16v mfma32<F16>(u4 a, u4 b, f16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}
template <>
__device__ __forceinline__ f16v mfma32<BF16>(u4 a, u4 b, f16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0);
}

// Continuation of an exact search: with a boundary pair per query, only rows that come strictly
// after (s[q], id[q]) in the order are candidates of query q.  Null pointers: no boundary.
// A search that takes the corpus in parts counts rows from the start of the part, which is row `base`.
struct After {
    const float *s = nullptr;
    const int *id = nullptr;
    int base = 0;
};
// The score of a row for the selection: unchanged when the row comes after the boundary (or the
// boundary score is NaN: nothing excluded), NaN otherwise, and a NaN score is never listed.
__device__ __forceinline__ float after_boundary(float s, int id, float bs, int bid) {
    const bool keep = bs > s || (bs == s && bid < id) || bs != bs;
    return keep ? s : __builtin_nanf("");
}

// One (score, id) pair as stored in the partial-result workspace.
struct Cand {
    float s;
    int id;
};

}  // namespace ann
