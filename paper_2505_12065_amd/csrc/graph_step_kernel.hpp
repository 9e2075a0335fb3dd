// Approximate retrieval on graphs of at most 32 slots per node: best-first search in steps of several expansions
// (Sections 2.1 and 3.3, Appendix B.3 of the paper; semantics in ann.h and graph_kernel.hpp).
//
// One workgroup (4 wavefronts) serves one query.  A search is a chain of dependent memory round trips and list work,
// one expansion after the other (graph_search_kernel: 2.3 to 2.9 us each), and that chain, not bandwidth, is what bounds
// it.  But the next expansions are mostly known in advance: the best unexpanded entries of the list, in order, unless
// a neighbour scored on the way beats them.  A step therefore takes several at once and is cut off where it would have
// gone wrong:
//
//   select   the first W unexpanded entries u_0, u_1, ... of the list
//   gather   their adjacency rows; neighbours scored before and neighbours named by an earlier u are left out, the rest
//            is numbered in order; as many u's as fit the row groups (32, or 63 of two per group) take part, the first
//            always does
//   score    one row group per neighbour, all rows in flight at once; list positions
//   commit   u_0 is expanded; u_j as well if no neighbour of u_0 .. u_{j-1} precedes it (or ties with it: the step is then
//            merely shorter).  Those are the expansions the one-by-one search makes, in its order, with its visited
//            set.  What was scored for the others is dropped and scored again when their turn comes.
//   merge    the neighbours of the committed nodes go into the list together
//
// A step takes 10 to 15 k clocks (select and bound 3.4 k, gather 1.4 k, rows and scores 2 to 6 k, commit and merge 2.5 k:
// instruction-bound).  Expansions per step at N = 200 k, d = 768, ef = 2048: 3.7 in the mean over queries with two
// neighbours per group, 2.3 for the slowest query, whose expansions bring 25 to 30 unseen neighbours each.  Against the
// one-by-one loop: ef = 2048 5.56 -> 5.09 ms at B = 16, 6.16 -> 5.36 at B = 512; ef = 8192, N = 60 k 17.0 -> 8.5 ms;
// with the maturity exit, d = 384, ef = 256, B = 256 595 -> 350 us.
//
// Visited set (VIS): one bit per node in LDS where that fits (exact, no round trip, nothing to clear in memory); else
// the id cache of graph_kernel.hpp for short lists without counters (it may forget, never claims an unseen node, and a
// node in the list is recognised when its place is looked up), or one bit per node in global memory.
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

// minimum over the wave, in every lane
__device__ __forceinline__ int wave_min(int x) {
    x = min(x, dpp_move<DPP_SWAP1>(x));
    x = min(x, dpp_move<DPP_SWAP2>(x));
    x = min(x, dpp_move<DPP_HALF_MIRROR>(x));
    x = min(x, dpp_move<DPP_MIRROR>(x));
    return min(min(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
               min(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

__device__ __forceinline__ uint32_t wave_min_u(uint32_t x) {
    return (uint32_t)wave_min((int)(x ^ 0x80000000u)) ^ 0x80000000u;
}

// x ascending over the 64 lanes <- k put into its place, the last lane's value dropped (uniform k)
__device__ __forceinline__ uint32_t sorted_insert(uint32_t x, uint32_t k, int lane) {
    const int at = __builtin_popcountll(__builtin_amdgcn_ballot_w64(x < k));
    const uint32_t up = (uint32_t)dpp_move<0x138>((int)x);               // lane i <- lane i - 1
    return lane > at ? up : (lane == at ? k : x);
}

template <class T, int RPG, int VIS, bool NS, bool LONG, bool QREG>
__global__ __launch_bounds__(GRAPH_THREADS, RPG == 2 ? 1 : QREG ? 2 : 3) void graph_step_kernel(
    const void *__restrict__ X, int64_t N, int d, const int32_t *__restrict__ graph, int R, int entry,
    const void *__restrict__ Q, int k, int ef, int32_t *__restrict__ ids, float *__restrict__ scores, StepLds L, NonStall ns) {
    constexpr int NT = GRAPH_THREADS, W = NT / 32, SW = W, DCAP = GRAPH_DELTA;
    constexpr int MOST = RPG == 2 ? 63 : 32;              // neighbours of a step (one fewer than lanes: see trim_tails)
    static_assert(!(NS || LONG) || VIS != STEP_VIS_CACHE, "counters and long lists need an exact visited set");
    extern __shared__ __align__(16) unsigned char smem[];
    auto ls = [&](int which) { return reinterpret_cast<float *>(smem + L.ls + which * L.ls_bytes); };
    auto li = [&](int which) { return reinterpret_cast<uint32_t *>(smem + L.li + which * L.ls_bytes); };
    float *cs = reinterpret_cast<float *>(smem + StepLds::CS);           // [64] scores, ids, list positions of the neighbours
    int *ci = reinterpret_cast<int *>(smem + StepLds::CI);
    int *cpos = reinterpret_cast<int *>(smem + StepLds::CP);
    int *ctl = reinterpret_cast<int *>(smem + StepLds::CTL);
    uint64_t *mk = reinterpret_cast<uint64_t *>(smem + StepLds::MK);    // [2][8] marks of a merge: a bit per final position
    uint64_t *um = reinterpret_cast<uint64_t *>(smem + L.um);            // LONG: "unexpanded" bits of M
    uint32_t *bits = reinterpret_cast<uint32_t *>(smem + L.vis);         // VIS: LDS bits, or the id cache
    u4 *qs = reinterpret_cast<u4 *>(smem + L.q);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.x;
    int *ent_v = reinterpret_cast<int *>(smem + StepLds::EV);            // [64] the step's neighbours and whose they are
    int *ent_w = reinterpret_cast<int *>(smem + StepLds::EW);
    uint32_t *fresh_m = reinterpret_cast<uint32_t *>(smem + StepLds::FM);   // [W] which slots of u_j's row are new
    // This wave's own scratch, no barrier around it: the selected entries in order, SW places (LONG: the next SW D's and
    // the last SW M's candidates before they are merged)
    int *sel_v = reinterpret_cast<int *>(smem + StepLds::WAVE0 + wave * StepLds::WAVE_BYTES);   // ids
    uint32_t *sel_k = reinterpret_cast<uint32_t *>(sel_v + 3 * SW);       // keys
    int *sel_p = sel_v + 6 * SW;                                         // positions (LONG: M's with bit 30)
    const int32_t *my_entries = ns.entries ? ns.entries + (size_t)b * ns.n_entries : nullptr;
    const int E = ns.entries ? ns.n_entries : 1;
    const int nch = d * T::bytes / 16;                    // 16-byte chunks per row
    uint32_t *gbits = VIS == STEP_VIS_GLOBAL ? ns.visited + (size_t)b * ns.words : nullptr;   // zero on entry
    const int sub = lane & (LANES_PER_ROW - 1);           // lane's position inside its row group
    const int grp = tid / LANES_PER_ROW;                  // 0 .. 31: takes neighbours grp and (RPG = 2) grp + 32

    for (int c = tid; c < nch; c += NT) qs[c] = load_chunk(static_cast<const char *>(Q) + ((size_t)b * nch + c) * 16);
    if constexpr (VIS == STEP_VIS_LDS) {
        for (int i = tid; i < L.vis_words / 4; i += NT) reinterpret_cast<u4 *>(bits)[i] = zero_chunk();
    } else if constexpr (VIS == STEP_VIS_CACHE) {
        for (int i = tid; i < L.vis_words; i += NT) bits[i] = 0xffffffffu;
    }
    // list scores start as -inf up to the next multiple of 64 entries (see group_lower_bound_fast)
    if (tid < 16) mk[tid] = 0ull;
    for (int i = tid; i < L.ls_bytes / 4; i += NT) { ls(0)[i] = -INFINITY; ls(1)[i] = -INFINITY; li(0)[i] = EXPANDED; li(1)[i] = EXPANDED; }
    __syncthreads();

    RowScorer<T, QREG, true> rows(X, qs, nch, sub);
    auto lds_barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // (the visited marks of a step in global memory have to be complete before the next one asks)
    auto step_barrier = [&] { if constexpr (VIS == STEP_VIS_GLOBAL) __syncthreads(); else lds_barrier(); };
    auto hash = [&](int v) { return (int)(((uint32_t)v * 2654435761u) >> L.cache_shift); };
    auto mark = [&](int v) {
        if constexpr (VIS == STEP_VIS_LDS) atomicOr(&bits[v >> 5], 1u << (v & 31));
        else if constexpr (VIS == STEP_VIS_CACHE) bits[hash(v)] = (uint32_t)v;
        else atomicOr(&gbits[v >> 5], 1u << (v & 31));
    };

    // ---- the candidate list ---------------------------------------------------------------------------
    // Short (ef <= 512): one ordered, double-buffered list ls / li / len, "expanded" flag in the id's top bit.
    // LONG: two parts, see graph_kernel.hpp for the reasons: M, large and ordered, rewritten only by a rebuild, and D, at
    // most DCAP entries, which takes the insertions and is the short list's code; the list is the merge of the
    // two, cut at ef entries.
    int cur = 0, len = 0, mlen = 0;
    int par = 0;                                          // which set of mark words the next merge uses
    int first = 0;                                        // no unexpanded entry of ls / li lies below this position
    int m1 = -1;                                          // LONG: M's first unexpanded position, -1: none
    bool m1_taken = false;                                // ... and whether it has been expanded since
    int pend = 0;                                         // LONG: entries still to be dropped from the two tails
    uint32_t worst_k = 0;                                 // the key a new entry has to reach, 0 while the list is not full
    float *Ms = reinterpret_cast<float *>(smem + L.ms);
    uint32_t *Mi = reinterpret_cast<uint32_t *>(smem + L.mi);

    // m1 <- first position >= from whose bit is set.  (The other kernel's m_find in other words: a common function, by value or
    // by reference, took 0.7 to 4 % more of the searches with long lists, as m1 then left the scalar registers.)
    auto m_find = [&](int from) {
        m1 = -1;
        const int nw = (mlen + 63) >> 6;
        // (as a rule the next one is a few entries further on, in the word that holds `from`: that word alone is read
        // first, by all lanes at once)
        if ((from >> 6) < nw) {
            uint64_t word = um[from >> 6] & (~0ull << (from & 63));
            if ((from >> 6) == nw - 1 && (mlen & 63) != 0) word &= (1ull << (mlen & 63)) - 1ull;
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)word);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(word >> 32));
            const uint64_t wu = ((uint64_t)hi << 32) | lo;
            if (wu != 0) { m1 = (from & ~63) + __builtin_ctzll(wu); return; }
            from = (from | 63) + 1;
        }
        for (int w0 = from >> 6; w0 < nw; w0 += WAVE) {
            const int w = w0 + lane;
            uint64_t word = w < nw ? um[w] : 0ull;
            if (w == (from >> 6)) word &= ~0ull << (from & 63);
            if (w == nw - 1 && (mlen & 63) != 0) word &= (1ull << (mlen & 63)) - 1ull;
            const uint64_t any = __builtin_amdgcn_ballot_w64(word != 0);
            if (any != 0) {
                const int l = __builtin_ctzll(any);
                const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)word, l);
                const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(word >> 32), l);
                m1 = (w0 + l) * 64 + __builtin_ctzll(((uint64_t)hi << 32) | lo);
                break;
            }
        }
    };
    // LONG: the `pend` worst entries of M and D together leave, and the worst entry that remains is read
    auto trim_tails = [&] {
        ListTails t;
        const int tm = tail_of_m(Ms, Mi, mlen, ls(cur), li(cur), len, pend, lane, t), td = pend - tm;
        mlen -= tm;
        len -= td;
        pend = 0;
        if (m1 >= mlen) m1 = -1;
        const uint32_t wa = score_key(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(t.a_s), tm)));
        const uint32_t wt = score_key(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(t.t_s), td)));
        worst_k = mlen + len < ef ? 0u : len <= 0 ? wa : mlen <= 0 ? wt : min(wa, wt);
    };
    // LONG: M <- merge of M and D; D <- empty
    // (the thread number through an empty asm: nothing computed from it is kept in registers across the search loop, 1 to
    // 2.5 % of the searches with long lists; with counters and two neighbours per group it costs 2 % instead)
    auto opaque = [](int x) { if constexpr (!(NS && RPG == 2)) asm volatile("" : "+v"(x)); return x; };
    auto rebuild = [&] {
        const int total = mlen + len;                     // <= ef: the tails have been cut
        const int f0 = rebuild_list(Ms, Mi, um, mlen, ls(cur), li(cur), len, ls(cur ^ 1), li(cur ^ 1), ctl, opaque(tid));
        for (int i = tid; i < DCAP; i += NT) { ls(0)[i] = -INFINITY; ls(1)[i] = -INFINITY; li(0)[i] = EXPANDED; li(1)[i] = EXPANDED; }
        const int from = min(m1 >= 0 ? m1 : total, f0);   // nothing unexpanded lies below either
        mlen = total;
        len = 0;
        cur = 0;
        first = 0;
        lds_barrier();
        m_find(from);
    };
    // Merge of entries 0 .. n - 1 of cs / ci / cpos (cpos -1: not to be listed), n_new of which go in, into ls / li, in two
    // halves with a barrier between them.  First half: a new entry's final position is its place in the old list
    // plus its rank among the new ones; it is written there (the other buffer) and the position marked in a bit mask.
    // Second half: every other final position takes the old entry as many places before it as there are marks below.
    auto merge_new = [&](int n) {
        const int nxt = cur ^ 1;
        if (tid < 8) mk[(par ^ 1) * 8 + tid] = 0ull;      // the set of the next merge
#pragma unroll
        for (int t = 0; t < RPG; ++t) {
            const int i = grp + 32 * t;
            if (t > 0 && n <= 32) break;
            const int gpos = i < n ? cpos[i] : -1;
            if (gpos >= 0) {
                const float new_s = cs[i];
                const int new_v = ci[i];
                int r = 0;                                // new entries that precede this group's
#pragma unroll
                for (int h = 0; h < RPG; ++h) {
                    if (h > 0 && n <= 32) break;
                    const int i0 = h * 32 + sub * 4;
                    const f4 sq = *reinterpret_cast<const f4 *>(cs + i0);
                    const int4 cq = *reinterpret_cast<const int4 *>(ci + i0);
                    const int4 pq = *reinterpret_cast<const int4 *>(cpos + i0);
                    r += ((int)(i0 + 0 < n) & (int)(pq.x >= 0) & precedes01(sq[0], cq.x, new_s, new_v)) +
                         ((int)(i0 + 1 < n) & (int)(pq.y >= 0) & precedes01(sq[1], cq.y, new_s, new_v)) +
                         ((int)(i0 + 2 < n) & (int)(pq.z >= 0) & precedes01(sq[2], cq.z, new_s, new_v)) +
                         ((int)(i0 + 3 < n) & (int)(pq.w >= 0) & precedes01(sq[3], cq.w, new_s, new_v));
                }
                r = group_sum(r);
                const int at = gpos + r;
                if (sub == 0 && at < ef) {
                    ls(nxt)[at] = new_s;
                    li(nxt)[at] = (uint32_t)new_v;
                    atomicOr(reinterpret_cast<uint32_t *>(mk + par * 8) + (at >> 5), 1u << (at & 31));
                }
            }
        }
    };
    auto merge_old = [&](int n_new) {
        const int nxt = cur ^ 1;
        const uint64_t *words = mk + par * 8;
        const int to_len = min(LONG ? DCAP : ef, len + n_new);
        for (int j0 = wave * WAVE; j0 < to_len; j0 += NT) {
            const int j = j0 + lane;
            const uint64_t word = words[j0 >> 6];
            int below = __builtin_popcountll(word & ((1ull << lane) - 1ull));
            for (int w = 0; w < (j0 >> 6); ++w) below += __builtin_popcountll(words[w]);
            if (j < to_len && !((word >> lane) & 1)) {
                ls(nxt)[j] = ls(cur)[j - below];
                li(nxt)[j] = li(cur)[j - below];
            }
        }
        par ^= 1;
        cur = nxt;
        len = to_len;
        if constexpr (LONG) pend = max(0, mlen + len - ef);   // what exceeds ef in all leaves next
    };

    // list <- the entry nodes (at most 32, one row group each), scored and put in order; ids that
    // are no nodes and ids named by an earlier slot are left out, a NaN score is never listed
    int n_dist = 0;                                       // scored nodes
    {
        int v0 = -1;
        if (grp < E) {
            v0 = my_entries ? my_entries[grp] : entry;
            if ((unsigned)v0 >= (unsigned)N) v0 = -1;
            for (int j = 0; j < grp && v0 >= 0; ++j)
                if (my_entries[j] == v0) v0 = -1;
        }
        float s0 = 0.f;
        if (v0 >= 0) s0 = rows.score(v0);
        if (sub == 0) {
            cs[grp] = s0;
            ci[grp] = v0;
            cpos[grp] = v0 >= 0 && s0 == s0 ? 0 : -1;
            if (v0 >= 0) mark(v0);
        }
        __syncthreads();
        const int c_v = ci[lane & 31], c_p = cpos[lane & 31];
        n_dist = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < 32 && c_v >= 0));
        const uint64_t in = __builtin_amdgcn_ballot_w64(lane < 32 && c_p >= 0);
        merge_new(32);
        lds_barrier();
        merge_old(__builtin_popcountll(in));
        step_barrier();
    }
    float ema = 0.f;
    int n_expand = 0, early = 0;
    // the samples are followed only when they can end the search or the caller wants the counters
    const bool track = NS && (ns.tau < INFINITY || ns.stats != nullptr || ns.ema != nullptr);
    typename RowScorer<T, QREG, true>::Loads x[RPG];

    // ---- select: the first SW unexpanded entries of the list, in order, into this wave's sel arrays --------------
    int nsel = 0;
    auto select = [&] {
        const float *dsc = ls(cur);
        const uint32_t *did = li(cur);
        const uint64_t below = (1ull << lane) - 1ull;
        auto put = [&](int at, uint32_t ev, float fv, int pv) {
            sel_v[at] = (int)ev;
            sel_k[at] = score_key(fv);
            sel_p[at] = pv;
        };
        // 256 entries, read together, from the block of 64 that holds the first unexpanded one on (a second round
        // only when those hold none: rare)
        int nd = 0;
        for (int base = LONG ? 0 : first & ~63; base < len && nd == 0; base += 256) {
            uint32_t e[4];
            float f[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (base + 64 * u < len) {
                    e[u] = did[base + 64 * u + lane];
                    f[u] = dsc[base + 64 * u + lane];
                }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (base + 64 * u < len && nd < SW) {
                    const uint64_t m = __builtin_amdgcn_ballot_w64(base + 64 * u + lane < len && !(e[u] & EXPANDED));
                    const int r = nd + __builtin_popcountll(m & below);
                    if (((m >> lane) & 1) && r < SW) put((LONG ? SW : 0) + r, e[u], f[u], base + 64 * u + lane);
                    nd += __builtin_popcountll(m);
                }
        }
        nsel = min(nd, SW);
        if constexpr (LONG) {
            // M's first SW, of the 128 entries around the first; then the two ordered runs are merged: a lane per
            // candidate, its place is its own number plus the candidates of the other run that precede it.
            // If those 128 are not all of M that is unexpanded, nothing behind the last of them is certain.
            int nm = 0;
            bool m_more = false;
            if (m1 >= 0) {
                const int mb = m1 & ~63;
                uint32_t me[2];
                float mf[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int j = min(mb + 64 * u + lane, mlen - 1);
                    me[u] = Mi[j];
                    mf[u] = Ms[j];
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint64_t mm = __builtin_amdgcn_ballot_w64(mb + 64 * u + lane < mlen && !(me[u] & EXPANDED));
                    const int r = nm + __builtin_popcountll(mm & below);
                    if (((mm >> lane) & 1) && r < SW) put(2 * SW + r, me[u], mf[u], (mb + 64 * u + lane) | (1 << 30));
                    nm += __builtin_popcountll(mm);
                }
                m_more = nm > SW || mb + 128 < mlen;
                nm = min(nm, SW);
            }
            const bool of_d = lane < SW;                  // the first SW lanes: D's run, the next SW: M's
            const int own = lane & (SW - 1), n_own = of_d ? nsel : nm, n_other = of_d ? nm : nsel;
            const int at = SW + (lane & (2 * SW - 1));
            const uint32_t k_own = sel_k[at];
            const int v_own = sel_v[at], p_own = sel_p[at];
            int r = own;
#pragma unroll
            for (int q = 0; q < SW / 4; ++q) {
                const int o = (of_d ? 2 * SW : SW) + 4 * q;
                const u4 ok = *reinterpret_cast<const u4 *>(sel_k + o);
                const int4 ov = *reinterpret_cast<const int4 *>(sel_v + o);
                auto one = [&](int i, uint32_t kk, int vv) {
                    r += (int)(i < n_other) & ((int)(kk > k_own) | ((int)(kk == k_own) & (int)(vv < v_own)));
                };
                one(4 * q, ok[0], ov.x); one(4 * q + 1, ok[1], ov.y); one(4 * q + 2, ok[2], ov.z); one(4 * q + 3, ok[3], ov.w);
            }
            if (lane < 2 * SW && own < n_own && r < SW) {
                sel_v[r] = v_own;
                sel_k[r] = k_own;
                sel_p[r] = p_own;
            }
            nsel = min(SW, nsel + nm);
            if (m_more) {
                nsel = min(nsel, __builtin_amdgcn_readlane(r, SW + nm - 1) + 1);

            }
        }
    };
    // the list as it stands after a merge: tails cut, room in D, the bound for new entries, the first candidates
    auto settle = [&] {
        if constexpr (LONG) {
            // (the bound moves only when entries leave, or when the list has just become full)
            if (pend > 0 || (worst_k == 0 && mlen + len >= ef)) trim_tails();
            if (len > DCAP - MOST) rebuild();
            else if (m1_taken) m_find(m1);
            m1_taken = false;
        } else {
            worst_k = len < ef ? 0u : score_key(ls(cur)[ef - 1]);
        }
        select();
    };
    int n_ent = 0, n_part = 0;                            // neighbours of the step; u's that take part
    for (;;) {
        settle();
        if (nsel == 0) break;                             // nothing left to expand: natural stop

        // ---- gather: thread t looks at slot t % 32 of the adjacency row of u_(t / 32) ------------------------
        {
            const int u = tid >> 5, slot = tid & 31;      // (two u's per wave)
            int nb = -1;
            if (u < nsel && slot < R) nb = graph[(size_t)sel_v[u] * R + slot];
            bool fresh = (unsigned)nb < (unsigned)N;
            if (fresh) {
                if constexpr (VIS == STEP_VIS_LDS) fresh = ((bits[nb >> 5] >> (nb & 31)) & 1u) == 0;
                else if constexpr (VIS == STEP_VIS_CACHE) fresh = bits[hash(nb)] != (uint32_t)nb;
                else fresh = ((__hip_atomic_load(&gbits[nb >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> (nb & 31)) & 1u) == 0;
            }
            const uint64_t fm = __builtin_amdgcn_ballot_w64(fresh);
            if (slot == 0) fresh_m[u] = (uint32_t)(fm >> (lane & 32));
            lds_barrier();
            // lane j < W: the neighbours of u_0 .. u_j; u_j takes part if they all fit (u_0 does: at most 32 <= MOST)
            int upto = __builtin_popcount(fresh_m[lane & (W - 1)]);
            auto add_from = [&](auto dist) {
                constexpr int D = decltype(dist)::value;
                const int o = __builtin_amdgcn_update_dpp(0, upto, 0x110 + D, 0xf, 0xf, false);   // lane - D of the row of 16
                upto += (lane & (W - 1)) >= D ? o : 0;
            };
            add_from(std::integral_constant<int, 1>{});
            add_from(std::integral_constant<int, 2>{});
            add_from(std::integral_constant<int, 4>{});
            n_part = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < nsel && upto <= MOST));
            n_ent = __builtin_amdgcn_readlane(upto, n_part - 1);
            const int to0 = __builtin_amdgcn_readlane(upto, 2 * wave), before = to0 - __builtin_popcount((uint32_t)fm);
            if (fresh && u < n_part) {
                const int at = before + __builtin_popcountll(fm & ((1ull << lane) - 1ull));
                ent_v[at] = nb;
                ent_w[at] = u;
            }
            lds_barrier();
        }

        // ---- score: row group g takes neighbours g and g + 32; their places in the list -----------------------
        int v[RPG];
#pragma unroll
        for (int t = 0; t < RPG; ++t) {
            // a neighbour named twice in the step belongs to the first that names it: the 8 lanes of the group look
            // at the neighbours before theirs
            const int i = grp + 32 * t;
            v[t] = -1;
            if (t > 0 && n_ent <= 32) break;
            const int mine = ent_v[i];
            int dup = 0;
#pragma unroll
            for (int h = 0; h <= t; ++h) {
                const int i0 = h * 32 + sub * 4;
                const int4 o = *reinterpret_cast<const int4 *>(ent_v + i0);
                dup |= ((int)(i0 + 0 < i) & (int)(o.x == mine)) | ((int)(i0 + 1 < i) & (int)(o.y == mine)) |
                       ((int)(i0 + 2 < i) & (int)(o.z == mine)) | ((int)(i0 + 3 < i) & (int)(o.w == mine));
            }
            const bool again = ((unsigned)(__builtin_amdgcn_ballot_w64(dup != 0) >> (lane & ~(LANES_PER_ROW - 1))) & 0xffu) != 0;
            if (i < n_ent && !again) {
                v[t] = mine;
                rows.issue(mine, x[t]);
            }
        }
        // (their adjacency rows into the near caches: they are likely nodes of the next steps)
        int touch[RPG] = {};
#pragma unroll
        for (int t = 0; t < RPG; ++t)
            if (v[t] >= 0) touch[t] = graph[(size_t)v[t] * R + min(sub * 4, R - 1)];
        const int e_w = lane < n_ent ? ent_w[lane] : W;
        float s[RPG];
#pragma unroll
        for (int t = 0; t < RPG; ++t) {
            s[t] = 0.f;
            if (t > 0 && n_ent <= 32) break;
            if (v[t] >= 0) {
                s[t] = rows.dots(v[t], x[t]);
                asm volatile("" ::"v"(touch[t]));
            }
        }
#pragma unroll
        for (int t = 0; t < RPG; ++t) {
            if (t > 0 && n_ent <= 32) break;
            int pos = -1;
            if (v[t] >= 0 && s[t] == s[t] && score_key(s[t]) >= worst_k) {        // (0 while the list is not full)
                bool listed;
                if constexpr (LONG) {                     // the position is the one in D
                    pos = group_lower_bound_fast<DCAP / 64>(ls(cur), li(cur), len, s[t], v[t], sub, lane, &listed);
                    if (listed) pos = -1;
                } else {
                    pos = group_lower_bound_fast(ls(cur), li(cur), len, s[t], v[t], sub, lane, &listed);
                    if (pos >= ef || listed) pos = -1;
                }
            }
            if (sub == 0) {
                cs[grp + 32 * t] = s[t];
                ci[grp + 32 * t] = v[t];
                cpos[grp + 32 * t] = pos;
            }
        }
        lds_barrier();

        // ---- commit ------------------------------------------------------------------------------------------
        const float c_s = cs[lane];                       // (lanes from n_ent on: leftovers, masked)
        const int e_v = lane < n_ent ? ci[lane] : -1;
        const int c_p = cpos[lane];
        const int u_p = sel_p[lane & (SW - 1)];
        const uint32_t c_k = lane < n_ent && c_p >= 0 ? score_key(c_s) : 0u;     // 0: does not enter the list
        // this neighbour stops the u's from the first whose key does not exceed its own, but none up to its own u
        int stop = 0;
#pragma unroll
        for (int q = 0; q < W / 4; ++q) {
            const u4 uk = *reinterpret_cast<const u4 *>(sel_k + 4 * q);
#pragma unroll
            for (int t = 0; t < 4; ++t) stop += (int)(4 * q + t < n_part) & (int)(uk[t] > c_k);   // (keys descend: a count is a place)
        }
        stop = max(c_k != 0 ? stop : W, e_w + 1);
        int C = min(wave_min(stop), n_part);
        bool leave = false;
        if (NS && track) {
            // The relative quality of every newly scored node against the best and worst entries of the list as its
            // expansion starts, into the moving average in slot order, expansion by expansion.  The best entry is
            // the same for all of them (a new best one would have ended the step); the worst: S holds the 64
            // lowest keys of the list, ascending, and takes the new ones as they come; of the entries the
            // list and the new ones make, those beyond ef are gone.
            uint32_t S;
            float s_best;
            const int total = mlen + len;
            {
                const int it = len - 1 - lane;
                S = it >= 0 ? score_key(ls(cur)[max(it, 0)]) : 0xffffffffu;
                s_best = len > 0 ? ls(cur)[0] : -INFINITY;
                if constexpr (LONG) {
                    // the lower half of two ascending runs: minimum with the other run turned round, then sorted
                    const int ia = mlen - 1 - (63 - lane);
                    const uint32_t A = ia >= 0 ? score_key(Ms[max(ia, 0)]) : 0xffffffffu;
                    S = ~group_sort_desc<64>(~min(S, A));
                    if (mlen > 0) s_best = fmaxf(s_best, Ms[0]);
                }
            }
            // (a list that is not full even with all of them: the worst entry is a running minimum)
            const uint32_t kk = score_key(c_s);
            const uint64_t all = __builtin_amdgcn_ballot_w64(e_w < C && e_v >= 0 && kk != 0);
            const bool filling = total + __builtin_popcountll(all) <= ef;
            uint32_t low = (uint32_t)__builtin_amdgcn_readfirstlane((int)S);
            int n_in = 0;
            for (int j = 0; j < C; ++j) {
                const uint64_t of_j = __builtin_amdgcn_ballot_w64(e_w == j && e_v >= 0);
                const float s_worst = key_score(filling ? low : (uint32_t)__builtin_amdgcn_readlane((int)S, max(0, total + n_in - ef)));
                const bool mine = (of_j >> lane) & 1;
                float r = NAN;                            // NaN: no sample; -inf: one, but best == worst
                if (mine) r = s_best != s_worst ? (s_best - c_s) / (s_best - s_worst) : -INFINITY;
                const uint32_t mag = __float_as_uint(r) & 0x7fffffffu;
                n_dist += __builtin_popcountll(of_j);
                uint64_t m = __builtin_amdgcn_ballot_w64(mag < 0x7f800000u);
                while (m != 0) {                          // four samples to a round; one past the last leaves the average alone
                    float ri[4];
                    bool is[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        is[u] = m != 0;
                        ri[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r), is[u] ? __builtin_ctzll(m) : 0));
                        m &= m - 1;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const float next = fmaf(ns.alpha, ri[u] - ema, ema);
                        ema = is[u] ? next : ema;
                    }
                }
                if (filling) {
                    low = min(low, (uint32_t)wave_min_u(mine && kk != 0 ? kk : 0xffffffffu));
                } else {
                    for (uint64_t i = of_j & all; i != 0; i &= i - 1) {
                        S = sorted_insert(S, (uint32_t)__builtin_amdgcn_readlane((int)kk, __builtin_ctzll(i)), lane);
                        ++n_in;
                    }
                }
                if (ema > ns.tau) {                       // mature: leave as soon as the engine is ready
                    int ready = 1;
                    if (ns.ready) {
                        if (tid == 0) ctl[1] = __hip_atomic_load(ns.ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                        __syncthreads();
                        ready = ctl[1];
                        __syncthreads();
                    }
                    if (ready) {
                        early = 1;
                        leave = true;
                        C = j + 1;
                    }
                }
            }
        }
        n_expand += C;
        const int n_com = __builtin_popcountll(__builtin_amdgcn_ballot_w64(e_w < C));   // neighbours of committed nodes
        if (wave == 0 && lane < n_com && e_v >= 0) mark(e_v);
        // (every wave sets the flags of the entries that it may move: none has to wait for another's)
        if (lane < C && (u_p >> 30) == 0) atomicOr(&li(cur)[u_p], EXPANDED);
        if constexpr (LONG) {
            m1_taken = m1 >= 0 && __builtin_amdgcn_ballot_w64(lane < C && (u_p >> 30) != 0) != 0;
            if (wave == 0 && lane < C && (u_p >> 30) != 0) {              // committed entries of M
                const int j = u_p & ~(1 << 30);
                atomicOr(&Mi[j], EXPANDED);
                atomicAnd(reinterpret_cast<unsigned long long *>(&um[j >> 6]), ~(1ull << (j & 63)));
            }
        }
        const uint64_t in = __builtin_amdgcn_ballot_w64(lane < n_com && c_k != 0);
        const int n_new = __builtin_popcountll(in);
        if (!LONG && ef > 256) {
            // nothing unexpanded lies below the last committed position + 1 and the lowest new one
            first = min(__builtin_amdgcn_readlane(u_p, C - 1) + 1, wave_min(((in >> lane) & 1) ? c_p : INT_MAX));
        }
        if (n_new != 0) {
            merge_new(n_com);
            lds_barrier();
            merge_old(n_new);
        }
        step_barrier();
        if ((NS && leave) || (int64_t)n_expand > N + W) break;            // (the latter: never on a sound list)
    }
    if constexpr (LONG) {
        if (pend > 0) trim_tails();
        if (len > 0) rebuild();
    }

    for (int j = tid; j < k; j += NT) {
        const bool has = j < (LONG ? mlen : len);
        const float *os = LONG ? Ms : ls(cur);
        const uint32_t *oi = LONG ? Mi : li(cur);
        ids[(size_t)b * k + j] = has ? (int)(oi[j] & ~EXPANDED) : -1;
        scores[(size_t)b * k + j] = has ? os[j] : -INFINITY;
    }
    if (NS && tid == 0) {
        if (ns.stats) {
            ns.stats[(size_t)b * 3 + 0] = early;
            ns.stats[(size_t)b * 3 + 1] = n_dist;
            ns.stats[(size_t)b * 3 + 2] = n_expand;
        }
        if (ns.ema) ns.ema[b] = ema;
    }
}

}  // namespace ann
