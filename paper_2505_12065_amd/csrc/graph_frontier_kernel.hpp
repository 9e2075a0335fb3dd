// Approximate retrieval on graphs of at most 32 slots per node: best-first search whose candidate list is never written down
// (Sections 2.1 and 3.3, Appendix B.3 of the paper; semantics in ann.h and graph_kernel.hpp).
//
// The method's list is at any time the ef best of the nodes scored so far, and the search expands its best unexpanded entry
// until there is none.  Let u be the best unexpanded of ALL scored nodes.  Everything that precedes u has been expanded, so
// u is in the list exactly if fewer than ef expanded nodes precede it.  The search is therefore
//
//      expand the best unexpanded node, until ef expanded nodes precede it or there is none,
//
// and what it needs is not an ordered list of ef entries but a priority queue of unexpanded nodes, of which only the head
// has to be in order.  The queue:
//   * the 64 best unexpanded nodes, in order, one 64-bit key per lane (in the registers of every wave: each wave does the same
//     work on its own copy, nothing is exchanged);
//   * the others in a pool in LDS, in no order; when the lanes run low the 64 best of it are fetched;
//   * the expanded nodes, in LDS, in the order in which they were expanded.
// Pool and expanded nodes share one array of ef + some entries, one from each end.  When they meet, a bound is searched for
// that at least ef scored nodes reach (by halving) and what lies below it leaves; new nodes below it are not taken in.
//
// One workgroup serves one query, in steps of several expansions:
//   select   the first lanes: u_0, u_1, ..., the next nodes to expand unless a neighbour scored on the way beats one of them
//   gather   their adjacency rows; neighbours scored before are left out, the rest is numbered in order (every wave does
//            this for itself); as many u's as fit 63 neighbours take part, the first always does
//   score    one row group of 8 lanes per neighbour, all rows in flight at once; a neighbour that the step before scored without
//            committing it brings its key along, the others fill the row groups without a gap; the keys go round through LDS: the one barrier of a step (a second after the
//            marks where the visited set is in memory)
//   commit   u_0 is expanded; u_j as well if no neighbour of u_0 .. u_{j-1} precedes it.  Those are the expansions that the
//            search one by one makes, in its order, with its visited set.  What was scored for the others is dropped.
//   insert   the neighbours of the committed nodes: into the lanes one by one if they are few, in the order of their ranks, a share of
//            which every wave finds, if not (one more barrier).
//
// Bound by the chain inside a step: 6.3 k clocks at 200 k x 768 fp16, ef = 2048, B = 256 (wait for the adjacency rows 0.6, visited bits
// and numbering 0.5, lookup of kept keys 0.3, rows 2.2, barrier 0.3, commit 0.5, insert 0.8, queue and pool 0.6, marks 0.4) at 2.2
// expansions a step for the slowest query; 8.4 k at ef = 64, where 40 rows take 3.1 and the insertion of as many keys 1.6.  A load
// instruction of 16 bytes a lane takes the memory path 16 clocks, for one row of eight or for all: 24 rows spread over eight waves
// keep it as busy as 64 (0.80 us a step from the L2, 0.41 without gaps; 8 rows 0.80 / 0.23).  Without gaps, us: B = 256, ef = 2048 2457 / 2266;
// B = 1, ef = 64 with its coarse search 108 / 99.5; maturity exit, rows of 768 bytes, B = 256, ef = 64 and 256 0.97 to 1.00 times as long.
// The ordered list in LDS that this replaces cost 12 to 15 k clocks a step: 64 list positions looked up, one list in two parts merged, cut
// and rebuilt (200 k x 768, B = 256, ef = 2048 5190 us; more, and the maturity exit, at frontier_pays).
// Off the chain of a step (together 200 k x 768, R = 32: B = 256, ef = 2048 2164 / 2120 us, B = 512, ef = 256 712 / 672; 200 k x 256, B = 32, ef = 512 628 / 569; B = 1,
// ef = 64 with its coarse search 134 / 130, eight queries): the ranks of many new keys come from compares with a lane's key (eight
// reads of 16 bytes a lane, by eight waves, kept the LDS busy for as long as the compares took); loads that only warm the caches are waited for with the next
// adjacency rows instead of before the barrier; the marks, LDS atomics by every wave, some 500 clocks of that queue, go ahead of the insertion,
// which hardly reads the LDS, by eight waves (by four, two workgroups a compute unit, that is 1 % longer).  One of them alone undone, ranks / waits /
// marks, % longer: B = 1, ef = 64 3.9 / 0.8 / 1.3, B = 256, ef = 2048 1.5 / 1.5 / 0.2, B = 512, ef = 256 4.2 / 0.5 / -0.1; 200 k x 256, B = 32, ef = 512 3.0 / 2.0 / 1.1; with the
// maturity exit, 200 k x 384, B = 256, ef = 256 -0.5 / -1.1 / -0.9, and 0.5 with the average by all waves (200 k x 768, R = 24, B = 10, ef = 400 1.9).
// Keeping the keys of uncommitted neighbours takes the rows a step loads from 54 to 26 at ef = 2048; 64-bit compares instead
// of maxima of doubles in the networks and insertions cost 4 % of a short list.  Not faster: 8 waves and two workgroups per compute
// unit (413 us against 309 at B = 512, ef = 64: 128 registers a lane), the smallest place a neighbour stops found by LDS atomics before the
// barrier (0.95 k clocks more there, 0.5 fewer after it); the place where the commits stop found by ballots (1.5 % longer: a compare, a ballot
// and scalar work in a row are 28 clocks, a lane move 14); visited bits set by one wave and kept keys looked up with them, which take one more
// barrier a step (8 % longer by eight waves: the two of a SIMD come to it 250 clocks apart).
#pragma once

#include "graph_kernel.hpp"

namespace ann {

// order-preserving image of a score (larger is better), 0 for a NaN, which is never listed; -0 counts as +0
__device__ __forceinline__ uint32_t score_key(float s) {
    const uint32_t b = __float_as_uint(s + 0.0f);
    const uint32_t k = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    return s == s ? k : 0u;
}
__device__ __forceinline__ float key_score(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k);
}
// A node's key, 63 bits: the score's image, the node's number turned round.  Larger precedes.  0: none; image 0: a NaN score.
// Read as a double a key is 0 or positive and finite (the largest exponent belongs to NaN scores), and doubles of one sign are
// ordered like their bits: the networks below take maxima and minima of doubles, one instruction each.
constexpr int KEY_SHIFT = 31;
constexpr uint64_t KEY_MOST = 0x7fefffffffffffffull;      // larger than any key
constexpr uint64_t KEY_LISTED = 1ull << KEY_SHIFT;        // no score that is a number has a smaller key
__device__ __forceinline__ uint64_t node_key(float s, int v) { return ((uint64_t)score_key(s) << KEY_SHIFT) | ((uint32_t)~v & 0x7fffffffu); }
__device__ __forceinline__ int key_node(uint64_t k) { return (int)(~(uint32_t)k & 0x7fffffffu); }
__device__ __forceinline__ uint32_t key_image(uint64_t k) { return (uint32_t)(k >> KEY_SHIFT); }
// (through asm: the compiler's own form first sees to signalling NaNs, of which there are none)
__device__ __forceinline__ uint64_t key_max(uint64_t a, uint64_t b) {
    uint64_t r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ uint64_t key_min(uint64_t a, uint64_t b) {
    uint64_t r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ __forceinline__ uint64_t make64(uint32_t lo, uint32_t hi) { return ((uint64_t)hi << 32) | lo; }
__device__ __forceinline__ uint64_t read_lane(uint64_t x, int l) {
    return make64((uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l), (uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), l));
}
constexpr uint64_t UNKNOWN = ~0ull;                       // of a neighbour that a step has not scored
// lanes of m below this one
__device__ __forceinline__ int rank_in(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// x with lane l (a constant after unrolling) replaced
__device__ __forceinline__ int write_lane(int x, int value, int l) {
    asm("v_writelane_b32 %0, %1, %2" : "+v"(x) : "s"(value), "n"(l));
    return x;
}
// lane i <- lane i - 1, lane 0 <- first; lane i <- lane i + 1, lane 63 <- 0
__device__ __forceinline__ uint64_t lanes_up(uint64_t x, uint64_t first) {
    return make64((uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)first, (int)(uint32_t)x, 0x138, 0xf, 0xf, false),
                  (uint32_t)__builtin_amdgcn_update_dpp((int)(first >> 32), (int)(x >> 32), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ uint64_t lanes_down(uint64_t x) {
    return make64((uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, 0x130, 0xf, 0xf, false),
                  (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(x >> 32), 0x130, 0xf, 0xf, false));
}
// lane i <- lane i + n, 0 past the end
__device__ __forceinline__ uint64_t lanes_down_by(uint64_t x, int n, int lane) {
    const int from = (lane + n) * 4;
    const uint64_t o = make64((uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)x),
                              (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(x >> 32)));
    return lane + n < 64 ? o : 0ull;
}
// lane l <- the smallest of lanes 0 .. l
__device__ __forceinline__ uint32_t lanes_min(uint32_t x) {
    auto with = [&](auto ctrl, auto rows) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        x = min(x, o);
    };
    with(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});      // lane - 1 of the row of 16, - 2, - 4, - 8
    with(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
    with(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
    with(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
    with(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});      // the last lane of row 0 (2) to row 1 (3)
    with(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});      // lane 31 to rows 2 and 3
    return x;
}
// maximum over the wave, in every lane (no NaN among them)
__device__ __forceinline__ float wave_max(float x) {
    auto with = [&](int o) { x = fmaxf(x, __int_as_float(o)); };
    with(dpp_move<DPP_SWAP1>(__float_as_int(x)));
    with(dpp_move<DPP_SWAP2>(__float_as_int(x)));
    with(dpp_move<DPP_HALF_MIRROR>(__float_as_int(x)));
    with(dpp_move<DPP_MIRROR>(__float_as_int(x)));
    uint32_t a, b;
    row_pair<16>(__float_as_uint(x), a, b);
    x = fmaxf(__uint_as_float(a), __uint_as_float(b));
    row_pair<32>(__float_as_uint(x), a, b);
    return fmaxf(__uint_as_float(a), __uint_as_float(b));
}
// minimum over the wave, in every lane
__device__ __forceinline__ int wave_min(int x) {
    x = min(x, dpp_move<DPP_SWAP1>(x));
    x = min(x, dpp_move<DPP_SWAP2>(x));
    x = min(x, dpp_move<DPP_HALF_MIRROR>(x));
    x = min(x, dpp_move<DPP_MIRROR>(x));
    return min(min(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
               min(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

// One stage of a sorting network: lanes l and l ^ J compare, and the larger key goes to the lanes of LARGER.
template <int J, uint64_t LARGER>
__device__ __forceinline__ uint64_t compare_lanes(uint64_t x) {
    uint64_t a, b;
    if constexpr (J >= 16) {
        uint32_t l0, l1, h0, h1;
        row_pair<J>((uint32_t)x, l0, l1);
        row_pair<J>((uint32_t)(x >> 32), h0, h1);
        a = make64(l0, h0);
        b = make64(l1, h1);
    } else {
        a = x;
        b = make64(lane_swap<J>((uint32_t)x), lane_swap<J>((uint32_t)(x >> 32)));
    }
    const uint64_t most = key_max(a, b), least = key_min(a, b);
    return __builtin_amdgcn_inverse_ballot_w64(LARGER) ? most : least;
}
constexpr uint64_t lanes_without(int bit) {               // lanes whose number has `bit` clear
    uint64_t m = 0;
    for (int l = 0; l < 64; ++l) m |= (l & bit) ? 0ull : 1ull << l;
    return m;
}
// a bitonic sequence over the lanes -> descending
__device__ __forceinline__ uint64_t clean_desc(uint64_t x) {
    x = compare_lanes<32, lanes_without(32)>(x);
    x = compare_lanes<16, lanes_without(16)>(x);
    x = compare_lanes<8, lanes_without(8)>(x);
    x = compare_lanes<4, lanes_without(4)>(x);
    x = compare_lanes<2, lanes_without(2)>(x);
    return compare_lanes<1, lanes_without(1)>(x);
}
// any keys -> ascending over the lanes (inside a block of K lanes the larger goes up where bit K is clear)
__device__ __forceinline__ uint64_t sort_asc(uint64_t x) {
    auto stage = [&](auto kc, auto jc) {
        constexpr int K = decltype(kc)::value, J = decltype(jc)::value;
        constexpr uint64_t up = K == 64 ? ~0ull : lanes_without(K);
        x = compare_lanes<J, (lanes_without(J) & ~up) | (~lanes_without(J) & up)>(x);
    };
    auto merge = [&](auto kc) {
        constexpr int K = decltype(kc)::value;
        if constexpr (K >= 64) stage(kc, std::integral_constant<int, 32>{});
        if constexpr (K >= 32) stage(kc, std::integral_constant<int, 16>{});
        if constexpr (K >= 16) stage(kc, std::integral_constant<int, 8>{});
        if constexpr (K >= 8) stage(kc, std::integral_constant<int, 4>{});
        if constexpr (K >= 4) stage(kc, std::integral_constant<int, 2>{});
        stage(kc, std::integral_constant<int, 1>{});
    };
    merge(std::integral_constant<int, 2>{});
    merge(std::integral_constant<int, 4>{});
    merge(std::integral_constant<int, 8>{});
    merge(std::integral_constant<int, 16>{});
    merge(std::integral_constant<int, 32>{});
    merge(std::integral_constant<int, 64>{});
    return x;
}
// descending over the lanes <- key put into its place; the last lane's key falls out
__device__ __forceinline__ uint64_t insert_desc(uint64_t x, uint64_t key) { return key_max(x, key_min(lanes_up(x, KEY_MOST), key)); }
// the same, ascending
__device__ __forceinline__ uint64_t insert_asc(uint64_t x, uint64_t key) { return key_min(x, key_max(lanes_up(x, 0ull), key)); }
// Descending over the lanes <- the 64 best of itself and the keys of the lanes in `from`.  Returns what does not stay, one
// key per lane, in no order, 0: none.
__device__ __forceinline__ uint64_t insert_many(uint64_t &x, uint64_t key, bool from) {
    const uint64_t b = sort_asc(from ? key : 0ull);
    const uint64_t low = key_min(x, b);
    x = clean_desc(key_max(x, b));
    return low;
}

// <q, x_v> by the 8 lanes of a row group; every lane of the group gets the sum.  Lane `sub` takes chunks sub, sub + 8, ...;
// all of a lane's loads of a row are issued before the first is used.  Rows are cut into runs of 32 chunks, four loads a lane:
// up to three whole ones at constant offsets, and a last one that may end inside (its lanes past the end load the row's
// last chunk and leave the product out).  QREG: the lane's share of the first 128 chunks of the query stays in registers.
template <class T, bool QREG>
struct FrontierScorer {
    static constexpr int RUN = 4 * LANES_PER_ROW;
    u4 x[16];
    u4 qr[QREG ? 16 : 1];
    const char *base;                                     // of the corpus, the lane's first chunk
    const u4 *qs;                                         // the query in LDS
    int sub, nch, row_bytes, whole, left;                 // whole runs (at most three); chunks of the last run, 0 .. 32

    __device__ __forceinline__ FrontierScorer(const void *X, const u4 *qs_, int nch_, int sub_) : qs(qs_), sub(sub_), nch(nch_) {
        base = static_cast<const char *>(X) + sub * 16;
        row_bytes = nch * 16;
        whole = min(nch / RUN, 3);
        left = min(nch - whole * RUN, RUN);
        if constexpr (QREG) {
#pragma unroll
            for (int u = 0; u < 16; ++u) qr[u] = qs[min(sub + (u < 12 ? u : 4 * whole + u - 12) * LANES_PER_ROW, nch - 1)];
        }
    }
    __device__ __forceinline__ u4 q_chunk(int u) const {
        if constexpr (QREG) return qr[u];
        else return qs[min(sub + (u < 12 ? u : 4 * whole + u - 12) * LANES_PER_ROW, nch - 1)];
    }
    // (scalars through an empty asm: their comparisons are made where they are needed, not kept in registers)
    static __device__ __forceinline__ int fresh(int a) { asm volatile("" : "+s"(a)); return a; }
    static __device__ __forceinline__ int fresh_lane(int a) { asm volatile("" : "+v"(a)); return a; }
    __device__ __forceinline__ const char *row(int v) const { return base + (uint64_t)(uint32_t)v * (uint32_t)row_bytes; }
    __device__ __forceinline__ void issue(int v) {
        const char *p = row(v);
        const int w = fresh(whole), l = fresh(left);
#pragma unroll
        for (int g = 0; g < 3; ++g)
            if (w > g) {
#pragma unroll
                for (int u = 4 * g; u < 4 * g + 4; ++u) x[u] = load_chunk(p + u * LANES_PER_ROW * 16);
            }
        if (l > 0) {
            const int own = fresh_lane(sub), most = l - 1 - own;          // (a lane past the end goes back to the last chunk)
            const char *e = p + w * (RUN * 16);
#pragma unroll
            for (int u = 0; u < 2; ++u) x[12 + u] = load_chunk(e + min(u * LANES_PER_ROW, most) * 16);
            if (l > 2 * LANES_PER_ROW) {
#pragma unroll
                for (int u = 2; u < 4; ++u) x[12 + u] = load_chunk(e + min(u * LANES_PER_ROW, most) * 16);
            }
        }
    }
    __device__ __forceinline__ float dots(int v) {
        f4 acc = {0.f, 0.f, 0.f, 0.f};                    // four independent chains, added at the end
        const int w = fresh(whole), l = fresh(left);
#pragma unroll
        for (int g = 0; g < 3; ++g)
            if (w > g) {
#pragma unroll
                for (int u = 4 * g; u < 4 * g + 4; ++u) dot_chunk4<T>(x[u], q_chunk(u), acc);
            }
        if (l > 0) {
            const int lim = l - fresh_lane(sub);
            auto part = [&](int u) {
                f4 t = acc;
                dot_chunk4<T>(x[12 + u], q_chunk(12 + u), t);
                acc = u * LANES_PER_ROW < lim ? t : acc;
            };
            part(0);
            part(1);
            if (l > 2 * LANES_PER_ROW) {
                part(2);
                part(3);
            }
        }
        if (fresh(nch) > 4 * RUN) {                       // longer rows: another 128 chunks at a time, the query from LDS
            const char *p = row(v);
            for (int c = 4 * RUN; c < nch; c += 4 * RUN) {
                const int lim = nch - c - fresh_lane(sub);
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    if (c + g * RUN < nch) {
#pragma unroll
                        for (int u = 4 * g; u < 4 * g + 4; ++u) x[u] = load_chunk(p + (c + min(u * LANES_PER_ROW, lim - 1)) * 16);
                    }
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    if (c + g * RUN < nch) {
#pragma unroll
                        for (int u = 4 * g; u < 4 * g + 4; ++u) {
                            f4 t = acc;
                            dot_chunk4<T>(x[u], qs[c + sub + min(u * LANES_PER_ROW, lim - 1)], t);
                            acc = u * LANES_PER_ROW < lim ? t : acc;
                        }
                    }
            }
        }
        return group_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
    }
};

// TIGHT: see settle, and the end
template <class T, int NW, int W, int VIS, bool NS, bool QREG, int OCC, bool TIGHT = false>
__global__ __launch_bounds__(NW * WAVE, OCC) void graph_frontier_kernel(
    FrontierArgs args) {
    const int64_t N = args.N;
    const int d = args.d, R = args.R, ef = args.ef;
    const int32_t *__restrict__ graph = args.graph;
    const FrontierLds &L = args.L;
    const NonStall &ns = args.ns;
    // (what is needed at the end only is read again there: scalar registers are short)
    auto late = [] {
        typedef __attribute__((address_space(4))) const FrontierArgs Late;
        Late *p = (Late *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(p));
        return p;
    };
    constexpr int NT = NW * WAVE, GROUPS = NT / LANES_PER_ROW, MOST = FRONTIER_MOST, FEW = 6, LOW = 4, HASHES = FrontierLds::HASHES;
    constexpr int AHEAD = 16;                             // nodes of the queue whose adjacency rows are kept at hand
    constexpr int ENTS = FRONTIER_MOST + 1, SETS = ENTS / GROUPS;        // neighbours of a step; of a row group, which scores one of them
    static_assert(ENTS == 64 && (SETS == 1 || SETS == 2), "a lane per neighbour");
    extern __shared__ __align__(16) unsigned char smem[];
    uint64_t *ck = reinterpret_cast<uint64_t *>(smem + FrontierLds::CK);               // [2][64] keys of a step's neighbours
    uint64_t *sorted = reinterpret_cast<uint64_t *>(smem + FrontierLds::SORTED);       // [64]
    int *at_hash = reinterpret_cast<int *>(smem + FrontierLds::HASH);                  // [2][HASHES] where a neighbour is among them
    int *ctl = reinterpret_cast<int *>(smem + FrontierLds::CTL);                       // [2][8] a count of every wave; the ready word; [2] the moving average
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int *ent = reinterpret_cast<int *>(smem + FrontierLds::WAVES + wave * FrontierLds::WAVE_BYTES);   // [64] this wave's list of the neighbours, and [64]
    int *ent_u = ent + FrontierLds::WAVE_BYTES / 8;                                                   // whose they are (and a place for the rest)
    auto again_of = [&](int w) {                          // [2] which neighbours of wave w's share an earlier one names, behind its list
        return reinterpret_cast<uint32_t *>(smem + FrontierLds::WAVES + w * FrontierLds::WAVE_BYTES + FrontierLds::WAVE_BYTES - 12);
    };
    uint64_t *tops = reinterpret_cast<uint64_t *>(smem + FrontierLds::WAVES);           // [NW][64], in the place of the waves' lists
    uint64_t *A = reinterpret_cast<uint64_t *>(smem + L.keys);                         // [cap] expanded from the left, pool from the right
    uint32_t *bits = reinterpret_cast<uint32_t *>(smem + L.vis);
    u4 *qs = reinterpret_cast<u4 *>(smem + L.q);
    const int b = blockIdx.x, cap = L.cap;
    const int32_t *my_entries = ns.entries ? ns.entries + (size_t)b * ns.n_entries : nullptr;
    const int E = ns.entries ? ns.n_entries : 1;
    const int nch = d * T::bytes / 16;                    // 16-byte chunks per row
    uint32_t *gbits = VIS == FRONTIER_VIS_GLOBAL ? ns.visited + (size_t)b * ns.words : nullptr;   // zero on entry
    const int sub = lane & (LANES_PER_ROW - 1);           // lane's position inside its row group
    const int grp = tid / LANES_PER_ROW;                  // takes the grp-th neighbour that is not known

    for (int c = tid; c < nch; c += NT) qs[c] = load_chunk(static_cast<const char *>(args.Q) + ((size_t)b * nch + c) * 16);
    if constexpr (VIS == FRONTIER_VIS_LDS)
        for (int i = tid; i < L.vis_words / 4; i += NT) reinterpret_cast<u4 *>(bits)[i] = zero_chunk();
    for (int i = tid; i < 128; i += NT) ck[i] = 0;
    for (int i = tid; i < 2 * HASHES; i += NT) at_hash[i] = 0;
    __syncthreads();

    FrontierScorer<T, QREG> rows(args.X, qs, nch, sub);
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    auto hash_of = [](int v) { return (int)(((uint32_t)v * 2654435761u) >> (32 - FrontierLds::HASH_BITS)); };
    auto lanes_below = [](int n) { return n >= 64 ? ~0ull : (1ull << n) - 1ull; };

    uint64_t t = 0;                                       // the best unexpanded nodes, descending over the lanes
    uint64_t floor_key = 0;                               // t takes what exceeds it (0: the pool is empty, t takes all)
    uint64_t bound = KEY_LISTED;                          // no node below it can be among the ef best any more (NaN: never is)
    int n_t = 0, n_pool = 0, live = 0, n_exp = 0;         // nodes in t; places of the pool, and those not empty; expanded nodes kept
    int n_expand = 0, n_dist = 0, early = 0;
    int buf = 0;

    // Every wave writes A itself, the same keys to the same places: what a wave reads there needs no barrier unless
    // the waves have shared the work of writing.
    auto to_pool = [&](uint64_t key, bool from) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(from);
        if (from) A[cap - 1 - (n_pool + rank_in(m))] = key;
        const int n = __builtin_popcountll(m);
        n_pool += n;
        live += n;
    };
    // t <- the 64 best of t and `asc`, ascending over the lanes, n of them; the others go to the pool
    auto merge = [&](uint64_t asc, int n) {
        const uint64_t low = key_min(t, asc);
        t = clean_desc(key_max(t, asc));
        n_t += n;
        if (n_t > 64) {
            floor_key = read_lane(t, 63);
            n_t = 64;
            if (ef <= 64) bound = floor_key;              // (what lies below is not among the ef best: no pool)
            else to_pool(low, low != 0);
        }
    };
    // The 64 best of what `at(i)`, i < n, gives (0: nothing) and, in wave 0, `own`, descending over the lanes: a share per wave, then
    // the shares are merged.  Takes the place of the waves' lists: nothing in them is of use here, and the caller has a barrier
    // follow before they are written again.
    auto best_of = [&](int n, uint64_t own, auto &&at) {
        uint64_t best = wave == 0 ? own : 0;
        for (int c = wave * WAVE; c < n; c += NT) {
            const uint64_t key = c + lane < n ? at(c + lane) : 0ull;
            const uint64_t least = read_lane(best, 63);
            uint64_t m = __builtin_amdgcn_ballot_w64(key > least);
            if (__builtin_popcountll(m) > FEW) insert_many(best, key, key > least);
            else
                for (; m != 0; m &= m - 1) best = insert_desc(best, read_lane(key, __builtin_ctzll(m)));
        }
        barrier();
        tops[wave * WAVE + lane] = best;
        barrier();
        // pairs of waves, pairs of pairs, ...: both sides of a pair end with the same
#pragma unroll
        for (int w = 1; w < NW; w *= 2) {
            const uint64_t o = tops[(wave ^ w) * WAVE + 63 - lane];       // ascending
            best = clean_desc(key_max(best, o));
            if (2 * w < NW) {
                barrier();                                // (all have read)
                tops[wave * WAVE + lane] = best;
                barrier();
            }
        }
        return best;
    };
    // t <- the 64 best unexpanded nodes
    auto refill = [&] {
        barrier();
        t = best_of(n_pool, t, [&](int i) { return A[cap - 1 - i]; });
        const uint64_t last = read_lane(t, 63);
        const int had = n_t;
        n_t = __builtin_popcountll(__builtin_amdgcn_ballot_w64(t != 0));
        live -= n_t - had;
        floor_key = last;
        if (live == 0) {
            floor_key = 0;
            n_pool = 0;
        }
        for (int i = tid; i < n_pool; i += NT)
            if (A[cap - 1 - i] >= floor_key) A[cap - 1 - i] = 0;
        barrier();
    };
    // sum over the workgroup of a number that is the same in all lanes of a wave
    int parity = 0;
    auto add_waves = [&](int x, int *before) {
        if (lane == 0) ctl[parity * 8 + wave] = x;
        barrier();
        int sum = 0, b4 = 0;
        for (int w = 0; w < NW; ++w) {
            const int c = __builtin_amdgcn_readfirstlane(ctl[parity * 8 + w]);
            b4 += w < wave ? c : 0;
            sum += c;
        }
        parity ^= 1;
        *before = b4;
        return sum;
    };
    // keys below `bound` and empty places leave one side of A; returns how many stay
    auto compact = [&](int n, auto &&ref) {
        int kept = 0;
        for (int c = 0; c < n; c += NT) {
            const uint64_t key = c + tid < n ? ref(c + tid) : 0ull;
            const uint64_t m = __builtin_amdgcn_ballot_w64(key >= bound);
            int before;
            const int all = add_waves(__builtin_popcountll(m), &before);
            if (key >= bound) ref(kept + before + rank_in(m)) = key;
            kept += all;
        }
        return kept;
    };
    auto prune = [&] {
        barrier();
        int unused;
        // The first HELD keys of a thread stay in registers while the bound is searched for, some 15 times through them all (from
        // LDS each time a bound took 45 k clocks at ef = 2048, now 23 k).
        constexpr int HELD = NS || !QREG ? 2 : 8;
        const int n = n_exp + n_pool;
        auto at = [&](int i) { return i < n ? A[i < n_exp ? i : cap - 1 - (i - n_exp)] : 0ull; };
        uint64_t held[HELD];
#pragma unroll
        for (int u = 0; u < HELD; ++u) held[u] = at(u * NT + tid);
        auto count = [&](uint64_t from) {                 // scored nodes that reach `from`, which is not 0
            int c = wave == 0 ? __builtin_popcountll(__builtin_amdgcn_ballot_w64(t >= from)) : 0;
#pragma unroll
            for (int u = 0; u < HELD; ++u) c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(held[u] >= from));
            for (int i = HELD * NT + wave * WAVE; i < n; i += NT) c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(at(i + lane) >= from));
            return add_waves(c, &unused);
        };
        uint64_t lo = bound, hi = KEY_MOST;                // at least ef reach lo (or all that there are), fewer reach hi
        for (uint64_t mid = lo;; mid = lo + ((hi - lo) >> 1)) {
            const int c = count(mid);
            if (c >= ef) lo = mid;
            else hi = mid;
            if ((c >= ef && c <= ef + L.spare) || hi <= lo + 1) break;
        }
        bound = lo;
        n_exp = compact(n_exp, [&](int i) -> uint64_t & { return A[i]; });
        n_pool = live = compact(n_pool, [&](int i) -> uint64_t & { return A[cap - 1 - i]; });
        if (live == 0) floor_key = 0;
        barrier();
    };
    // expanded nodes that precede `key`
    auto expanded_before = [&](uint64_t key) {
        int c = 0;
        for (int i = 0; i < n_exp; i += WAVE)
            c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(i + lane < n_exp && A[min(i + lane, n_exp - 1)] > key));
        return c;
    };
    auto mark = [&](uint64_t key, bool from) {
        const int v = key_node(key);
        from = from && (unsigned)v < (unsigned)N;
        if constexpr (VIS == FRONTIER_VIS_LDS) {
            if (from) atomicOr(&bits[v >> 5], 1u << (v & 31));            // (every wave, for itself)
        } else {
            if (from && wave == 0) atomicOr(&gbits[v >> 5], 1u << (v & 31));
        }
    };

    // ---- maturity exit: best and worst entries of the list -------------------------------------------------
    const bool track = NS && (ns.tau < INFINITY || ns.stats != nullptr || ns.ema != nullptr);
    float ema = 0.f, due = 0.f;                           // samples that have not entered the average yet, one per lane
    int n_due = 0;
    auto average = [&](float r, int from, int to) {       // samples from .. to - 1 enter
        auto take = [&](int q) {
            const float one = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r), q));
            ema = fmaf(ns.alpha, one - ema, ema);
        };
        int p = from;
        for (; p + 4 <= to; p += 4) {
            take(p);
            take(p + 1);
            take(p + 2);
            take(p + 3);
        }
        for (; p < to; ++p) take(p);
    };
    uint64_t best_key = 0;                                // of all scored nodes
    uint32_t low_key = ~0u;                               // the worst score of the list while it is not full
    int listed = 0;                                       // entries of the list
    // a full list: its n_s lowest keys, ascending over the lanes, KEY_MOST behind them
    uint64_t S = KEY_MOST;
    int n_s = 0;
    bool s_all = false;                                   // S is the whole list
    uint64_t worst = 0;                                   // a full list's worst entry: keys below it are not in the list
    auto lowest = [&] {
        barrier();
        auto turned = [&](uint64_t key) { return key != 0 && key >= worst ? ~key & 0x7fffffffffffffffull : 0ull; };
        const uint64_t own = clean_desc(sort_asc(turned(t)));             // (an ascending run is a bitonic sequence)
        const uint64_t best = best_of(n_exp + n_pool, own, [&](int i) { return turned(i < n_exp ? A[i] : A[cap - 1 - (i - n_exp)]); });
        S = best != 0 ? ~best & 0x7fffffffffffffffull : KEY_MOST;
        n_s = __builtin_popcountll(__builtin_amdgcn_ballot_w64(best != 0));
        s_all = n_s == listed;
        barrier();                                        // (the waves' lists are written again)
    };

    // the entry nodes (at most 32, one row group each); ids that are no nodes and ids named by an earlier slot are left out
    {
        int v0 = -1;
        if (grp < E) {
            v0 = my_entries ? my_entries[grp] : args.entry;
            if ((unsigned)v0 >= (unsigned)N) v0 = -1;
            for (int j = 0; j < grp && v0 >= 0; ++j)
                if (my_entries[j] == v0) v0 = -1;
        }
        float s0 = 0.f;
        if (v0 >= 0) {
            rows.issue(v0);
            s0 = rows.dots(v0);
        }
        if (sub == 0 && grp < 32) ck[grp] = v0 >= 0 ? node_key(s0, v0) : 0ull;
        barrier();
        const uint64_t key = lane < 32 ? ck[lane] : 0ull;
        buf = 1;
        mark(key, key != 0);
        n_dist = __builtin_popcountll(__builtin_amdgcn_ballot_w64(key != 0));
        const uint64_t in = __builtin_amdgcn_ballot_w64(key >= bound);
        merge(sort_asc(key >= bound ? key : 0ull), __builtin_popcountll(in));
        if (NS && n_t > 0) {
            best_key = read_lane(t, 0);
            listed = min(ef, __builtin_popcountll(in));
            const uint64_t last = read_lane(t, listed - 1);
            low_key = key_image(last);
            worst = listed == ef ? last : 0;              // (there may be more entries than the list holds)
        }
        if constexpr (VIS == FRONTIER_VIS_GLOBAL) __syncthreads();
    }

    // gather: lane l asks for slot l % 32 of the adjacency rows of u_(2r + l / 32)
    int n_sel, nb[W / 2], none[W / 2];
    const char *my_slot = reinterpret_cast<const char *>(graph + min(lane & 31, R - 1));
    const int no_slot = (lane & 31) < R ? 0 : -1;
    auto request = [&] {
        n_sel = min(n_t, W);
        const int node_of = t != 0 ? key_node(t) : -1;
#pragma unroll
        for (int r = 0; r < W / 2; ++r) {
            const int ua = __builtin_amdgcn_readlane(node_of, 2 * r), ub = __builtin_amdgcn_readlane(node_of, 2 * r + 1);
            const int u = lane < 32 ? ua : ub;            // (-1: there is none; node 0's row is read instead)
            nb[r] = *reinterpret_cast<const int *>(my_slot + (uint64_t)(uint32_t)max(u, 0) * (uint32_t)(R * 4));
            none[r] = u | no_slot;
        }
    };
    auto settle = [&] {
        // (a step leaves up to 64 + W nodes there, the end another 64: TIGHT sees to those there)
        if (n_exp + n_pool + (TIGHT ? 64 : 128) + W > cap) prune();
        if (n_t < LOW && live > 0) refill();
    };
    settle();
    request();
    int touched = 0, ahead = 0;                           // (loads for the caches' sake: waited for with the next adjacency rows, which come after them)
    for (;;) {
        if (n_t == 0) break;                              // nothing left to expand
        if (n_exp >= ef && expanded_before(read_lane(t, 0)) >= ef) break;

        const int nodes = (int)N;
        uint32_t word[W / 2];
#pragma unroll
        for (int r = 0; r < W / 2; ++r) {
            nb[r] = none[r] < 0 ? -1 : nb[r];
            const uint32_t at = min((uint32_t)nb[r], (uint32_t)(nodes - 1)) >> 5;
            if constexpr (VIS == FRONTIER_VIS_LDS) word[r] = bits[at];
            else word[r] = __hip_atomic_load(&gbits[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("" ::"v"(touched), "v"(ahead));
        // lane j of upto: neighbours of u_0 .. u_j.  (No branches: what does not take part goes to a place nobody reads.)
        int upto = 0, sum = 0;
#pragma unroll
        for (int r = 0; r < W / 2; ++r) {
            const bool fresh = (uint32_t)nb[r] < (uint32_t)nodes && ((word[r] >> (nb[r] & 31)) & 1u) == 0;
            const uint64_t m = __builtin_amdgcn_ballot_w64(fresh);
            const int at = sum + rank_in(m);
            const int to = fresh ? min(at, 64) : 64;
            ent[to] = nb[r];
            ent_u[to] = 2 * r + (lane >> 5);
            sum += __builtin_popcount((uint32_t)m);
            upto = write_lane(upto, sum, 2 * r);
            sum += __builtin_popcount((uint32_t)(m >> 32));
            upto = write_lane(upto, sum, 2 * r + 1);
        }
        int n_part = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < n_sel && upto <= MOST));   // u's that take part
        const int n_ent = __builtin_amdgcn_readlane(upto, n_part - 1);                                   // neighbours of the step

        // ---- score ---------------------------------------------------------------------------------------------
        // Lane i of every wave looks after neighbour i.  One that the step before has scored but not committed brings its key
        // along; the rest goes to the row groups without a gap, since a load instruction takes the memory path as long for one row as for
        // eight.  More than there are groups are left unknown.  (The rank takes a trip through the LDS before the first row is asked for.  Against a row
        // group for every place of the list, eight waves, times as long: rows of 1.5 KB 0.91 to 0.97 at any R; of 768 bytes 0.93 to 0.98 for 256 queries, 0.94 to
        // 1.01 for 16, 1.01 to 1.03 for one; of up to 512 bytes 0.94 to 1.02, 0.96 to 1.04, 0.96 to 1.04, the upper ends at R <= 8 and rows of up to 256 bytes.
        // By ds_permute and two lane moves instead of the LDS 1.3 % longer on average; chosen by a flag at run time 2 to 3 %.  A name given twice takes a
        // row group as often as it is named: on graphs of overlapping rows 0.99 to 1.01 by eight waves, 0.85 to 0.97 by four.)
        const int mine = ent[lane], from_u = ent_u[lane];                 // whose the neighbour of this lane is
        const uint64_t kept = ck[(buf ^ 1) * 64 + at_hash[(buf ^ 1) * HASHES + hash_of(mine)]];
        const bool known = lane < n_ent && key_node(kept) == mine, need = lane < n_ent && !known;
        const uint64_t need_m = __builtin_amdgcn_ballot_w64(need);
        const int n_need = __builtin_popcountll(need_m), rank = rank_in(need_m);
        if (need) ent_u[rank] = mine;
        const int todo = grp < n_need ? ent_u[grp] : -1;
        if (todo >= 0) {
            rows.issue(todo);
            // (its adjacency row into the near caches: it is likely a node of the next steps)
            touched = graph[(size_t)todo * R + min(sub * 4, R - 1)];
        }
        // A neighbour named twice in the step belongs to the first that names it: eight lanes, eight apart, look at those before one of
        // this wave's share.
        {
            const int part = lane >> 3;
            const int4 oa = *reinterpret_cast<const int4 *>(ent + part * 8), ob = *reinterpret_cast<const int4 *>(ent + part * 8 + 4);
            uint32_t word = 0;
#pragma unroll
            for (int h = 0; h < SETS; ++h) {
                const int i = (wave * SETS + h) * 8 + sub, i0 = part * 8, e = ent[i];
                const int dup = ((int)(i0 + 0 < i) & (int)(oa.x == e)) | ((int)(i0 + 1 < i) & (int)(oa.y == e)) |
                                ((int)(i0 + 2 < i) & (int)(oa.z == e)) | ((int)(i0 + 3 < i) & (int)(oa.w == e)) |
                                ((int)(i0 + 4 < i) & (int)(ob.x == e)) | ((int)(i0 + 5 < i) & (int)(ob.y == e)) |
                                ((int)(i0 + 6 < i) & (int)(ob.z == e)) | ((int)(i0 + 7 < i) & (int)(ob.w == e));
                uint64_t m = __builtin_amdgcn_ballot_w64(dup != 0);
                m |= m >> 32;
                m |= m >> 16;
                m |= m >> 8;
                word |= ((uint32_t)m & 0xffu) << (8 * h);
            }
            if (lane == 0) again_of(wave)[buf] = word;
        }
        // The samples of the step before enter the average, some 40 clocks each and one after the other: by the last of eight waves alone, which has
        // the fewest rows, while these come in (50 k x 768, R = 24, B = 10, ef = 400 846 us by all waves after the request of the
        // next adjacency rows, 810).  Of four waves each has rows in most steps (B = 500 by the last 1140, by all 1122).
        if (NS && track && NW == 8 && wave == NW - 1) {
            average(due, 0, n_due);
            if (lane == 0) ctl[17 + buf] = __float_as_int(ema);
        }
        if (todo >= 0) {
            const uint64_t own = node_key(rows.dots(todo), todo);
            if (sub == 0) {
                ck[buf * 64 + grp] = own;
                at_hash[buf * HASHES + hash_of(todo)] = grp;
            }
        }
        if (wave == NW - 1) {                             // (the last wave has the fewest rows)
            // The adjacency rows of the queue's next nodes into the L2, out of which the rows drive what is not asked for again
            // (frontier_ahead says where that pays).  Not before there is a pool (what is scored lately is there), nor with the maturity
            // exit, where it changes nothing (200 k x 384, B = 256, ef = 64, 256, 1024 116.7 / 115.9, 246.8 / 246.2, 763.6 / 763.2 us with).
            if (!NS && frontier_ahead(NW) && live > 0 && lane >= W && lane < AHEAD && t != 0) ahead = graph[(size_t)key_node(t) * R];
            if (known) {
                const int slot = n_need + rank_in(__builtin_amdgcn_ballot_w64(known));
                ck[buf * 64 + slot] = kept;
                at_hash[buf * HASHES + hash_of(mine)] = slot;
            }
        }
        barrier();

        // ---- commit ------------------------------------------------------------------------------------------
        uint64_t key = need ? ck[buf * 64 + rank] : known ? kept : 0ull;
        if constexpr (SETS == 2) key = need && rank >= GROUPS ? UNKNOWN : key;
        key = again_of(lane / (8 * SETS))[buf] >> (lane & (8 * SETS - 1)) & 1u ? 0ull : key;
        if (NS && track && NW == 8) ema = __int_as_float(__builtin_amdgcn_readfirstlane(ctl[17 + buf]));
        buf ^= 1;
        // A neighbour stops the expansions from the first whose node it precedes, but none up to its own; one that is unknown stops
        // its own.
        int C;
        {
            int c = 1;                                    // (u_0 is expanded anyway; keys descend: a count is a place)
#pragma unroll
            for (int j = 1; j < W; ++j) c += (int)(read_lane(t, j) > key);
            c = max(c, from_u + 1);
            if constexpr (SETS == 2) c = key == UNKNOWN ? from_u : c;
            C = min(n_part, wave_min(key != 0 ? c : W));
        }
        if constexpr (SETS == 2) key = key == UNKNOWN ? 0ull : key;
        if (n_exp + C > ef)                               // a u that ef expanded nodes precede is not expanded
            for (int j = 1; j < C; ++j)
                if (n_exp + j >= ef && expanded_before(read_lane(t, j)) + j >= ef) C = j;
        bool leave = false;
        if (NS && track) {
            // The relative quality of every newly scored node against the best and worst entries of the list as its
            // expansion starts, into the moving average in slot order, expansion by expansion.  The best entry is the same
            // for all of them (a new best one would have ended the step).
            const uint32_t c_k = key_image(key);
            // (what does not precede the worst entry does not get into a full list)
            const uint64_t all = __builtin_amdgcn_ballot_w64(c_k != 0 && (listed < ef || key > worst));
            const int most_in = listed + __builtin_popcountll(all & lanes_below(__builtin_amdgcn_readlane(upto, C - 1)));
            const bool filling = listed < ef && most_in <= ef;            // even with all of them: the worst entry is a running minimum
            if (!filling && !s_all && most_in - ef >= n_s) lowest();
            const float s_best = key_score(key_image(best_key)), c_s = key_score(c_k);
            uint32_t low = c_k != 0 ? c_k : ~0u;          // lane l: smallest of lanes 0 .. l
            if (filling) low = lanes_min(low);
            int n_in = 0, from = 0, out = 0;
            uint32_t worst_k = 0;                         // the list's worst entry as the expansion of this lane's node starts
            if (filling) {
                for (int j = 0; j < C; ++j) {
                    const int to = __builtin_amdgcn_readlane(upto, j);
                    const uint32_t w = min(low_key, from > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)low, from - 1) : ~0u);
                    worst_k = lane >= from && lane < to ? w : worst_k;
                    from = to;
                }
            } else {
                // The list and the new keys of the earlier expansions together: the worst entry is the one with as many
                // below it as there are too many.  (Keys that would not have got in are below it as well.)  S takes the new
                // keys that lie in its range; what lies above its highest need not be known.
                const uint64_t top = s_all ? KEY_MOST : read_lane(S, n_s - 1);
                const uint64_t ranged = all & __builtin_amdgcn_ballot_w64(key < top);
                for (int j = 0; j < C; ++j) {
                    const int to = __builtin_amdgcn_readlane(upto, j);
                    const uint64_t of_j = lanes_below(to) & ~lanes_below(from);
                    const uint32_t w = key_image(read_lane(S, out));
                    worst_k = (of_j >> lane) & 1 ? w : worst_k;
                    n_in += __builtin_popcountll(all & of_j);
                    for (uint64_t i = ranged & of_j; i != 0; i &= i - 1) {
                        S = insert_asc(S, read_lane(key, __builtin_ctzll(i)));
                        ++n_s;
                    }
                    out = max(0, listed + n_in - ef);     // entries of S that have left
                    from = to;
                }
                s_all = s_all && n_s <= 64;
                n_s = min(n_s, 64);
            }
            float r = NAN;                                // NaN: no sample; -inf: one, but best == worst
            const float s_worst = key_score(worst_k);
            if (lane < from && c_k != 0) r = s_best != s_worst ? (s_best - c_s) / (s_best - s_worst) : -INFINITY;
            const uint32_t mag = __float_as_uint(r) & 0x7fffffffu;
            const bool sample = mag < 0x7f800000u;
            const uint64_t samples = __builtin_amdgcn_ballot_w64(sample);
            // the samples side by side: lane p gets the p-th
            ent[sample ? rank_in(samples) : 64] = __float_as_int(r);      // (the neighbours are not read any more)
            const float in_order = __int_as_float(ent[lane]);
            // Most steps cannot take the average past tau whatever the order of their samples: then it is brought up to date
            // while the next adjacency rows are on their way.
            n_due = __builtin_popcountll(samples);
            due = in_order;
            const float most = wave_max(sample ? r : -INFINITY);
            // (the last term: more than 63 roundings can add)
            if (!(ema + (float)n_due * ns.alpha * fmaxf(most - ema, 0.f) * 1.001f + 1e-5f * (fabsf(ema) + fabsf(ns.tau)) <= ns.tau)) {
                n_due = 0;
                int p = 0;
                for (int j = 0; j < C; ++j) {
                    const int end = __builtin_popcountll(samples & lanes_below(__builtin_amdgcn_readlane(upto, j)));
                    average(in_order, p, end);
                    p = end;
                    if (ema > ns.tau) {                       // mature: leave as soon as the engine is ready
                        int ready = 1;
                        const int32_t *at = late()->ns.ready;
                        if (at) {
                            barrier();
                            if (tid == 0) ctl[16] = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                            __syncthreads();
                            ready = __builtin_amdgcn_readfirstlane(ctl[16]);
                        }
                        if (ready) {
                            early = 1;
                            leave = true;
                            C = j + 1;
                        }
                    }
                }
            }
            from = __builtin_amdgcn_readlane(upto, C - 1);
            n_dist += __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < from && key != 0));
            if (filling) n_in = __builtin_popcountll(all & lanes_below(from));
            if (filling) {
                low_key = min(low_key, from > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)low, from - 1) : ~0u);
            } else {
                const uint64_t moved = lanes_down_by(S, out, lane);       // (all lanes take part)
                S = lane + out < 64 ? moved : KEY_MOST;   // what has left the list leaves S
                n_s -= out;
                worst = read_lane(S, 0);
            }
            listed = min(ef, listed + n_in);
        }
        // ---- insert; the next rows are asked for as soon as their nodes are known ------------------------------
        const int n_com = __builtin_amdgcn_readlane(upto, C - 1);         // neighbours of committed nodes
        const bool in = lane < n_com;
        if constexpr (NW == 8) mark(key, in && key != 0);
        n_expand += C;
        if (lane < C) A[n_exp + lane] = t;
        n_exp += C;
        n_t -= C;
        if (C > 2) t = lanes_down_by(t, C, lane);
        else for (int i = 0; i < C; ++i) t = lanes_down(t);
        const bool taken = in && key >= bound, high = taken && key > floor_key;
        const uint64_t high_m = __builtin_amdgcn_ballot_w64(high);
        if (__builtin_amdgcn_ballot_w64(taken && !high) != 0) to_pool(key, taken && !high);
        const int n_high = __builtin_popcountll(high_m);
        if (n_high <= FEW && n_t + n_high <= 64) {        // (nothing falls out)
            n_t += n_high;
            for (uint64_t m = high_m; m != 0; m &= m - 1) t = insert_desc(t, read_lane(key, __builtin_ctzll(m)));
        } else {
            // Many: every wave finds the ranks of its share, a lane's key against all; they come back in order through LDS.
            int r = 0;
            for (uint64_t m = high_m & (lanes_below(8 * SETS) << (8 * SETS * wave)); m != 0; m &= m - 1) {
                const int i = __builtin_ctzll(m);
                const uint64_t before = __builtin_amdgcn_ballot_w64(key > read_lane(key, i)) & high_m;
                r = lane == i ? __builtin_popcountll(before) : r;
            }
            if (high && lane / (8 * SETS) == wave) sorted[63 - r] = key;
            barrier();
            merge(63 - lane < n_high ? sorted[lane] : 0ull, n_high);
        }
        if ((NS && leave) || (int64_t)n_expand > N + W) break;            // (the latter: never on a sound graph)
        settle();
        request();
        if (NS && track && NW != 8) average(due, 0, n_due);
        if constexpr (NW != 8) mark(key, in && key != 0);
        if (NS && n_t > 0) {
            const uint64_t head = read_lane(t, 0);
            best_key = head > best_key ? head : best_key;
        }
        if constexpr (VIS == FRONTIER_VIS_GLOBAL) __syncthreads();        // (the marks are complete before the next step asks)
    }

    if (NS && track && NW == 8) average(due, 0, n_due);
    // the k best of all, 64 at a time
    {
        const int k = late()->k;
        int32_t *ids = late()->ids + (size_t)b * k;
        float *scores = late()->scores + (size_t)b * k;
        if constexpr (TIGHT)
            if (k > WAVE && n_exp + n_pool + WAVE > cap) prune();         // (no longer than ef with t: room for it)
        barrier();
        uint64_t under = ~0ull;
        for (int j0 = 0; j0 < k; j0 += WAVE) {
            const int n = n_exp + n_pool;
            const uint64_t own = j0 == 0 ? t : 0ull;
            // (later rounds take t from the array: t joins the pool's side there)
            const uint64_t best = best_of(n, own, [&](int i) {
                const uint64_t key = i < n_exp ? A[i] : A[cap - 1 - (i - n_exp)];
                return key < under ? key : 0ull;
            });
            if (j0 == 0) {                                // (room for t's entries is kept: see the loop's first line)
                to_pool(t, t != 0);
                barrier();
            }
            const int j = j0 + lane;
            if (wave == 0 && j < k) {
                ids[j] = best != 0 ? key_node(best) : -1;
                scores[j] = best != 0 ? key_score(key_image(best)) : -INFINITY;
            }
            under = read_lane(best, 63);
            if (under == 0) under = 1;                    // (nothing is left)
        }
    }
    if (NS && tid == 0) {
        int32_t *stats = late()->ns.stats;
        float *emas = late()->ns.ema;
        if (stats) {
            stats[(size_t)b * 3 + 0] = early;
            stats[(size_t)b * 3 + 1] = n_dist;
            stats[(size_t)b * 3 + 2] = n_expand;
        }
        if (emas) emas[b] = ema;
    }
}

}  // namespace ann
