// Approximate retrieval on graphs of at most 32 slots per node: best-first search in steps of several expansions on an
// ordered list in LDS (Sections 2.1 and 3.3, Appendix B.3 of the paper; semantics in ann.h and graph_kernel.hpp).  Serves lists of
// up to 512 entries where the exact visited set that graph_frontier_kernel needs does not fit LDS: an id cache is enough
// here, since a node in the list is recognised when its place is looked up.
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
// A step takes 10 to 15 k clocks, instruction-bound, so it pays where more queries wait than there are places, or where one
// or two have a compute unit to themselves (graph_step_pays; figures there).
//
// The id cache may forget, never claims an unseen node (graph_kernel.hpp).
#pragma once

#include "graph_frontier_kernel.hpp"

namespace ann {

template <class T, int RPG, bool QREG>
__global__ __launch_bounds__(GRAPH_THREADS, RPG == 2 ? 1 : QREG ? 2 : 3) void graph_step_kernel(
    const void *__restrict__ X, int64_t N, int d, const int32_t *__restrict__ graph, int R, int entry,
    const void *__restrict__ Q, int k, int ef, int32_t *__restrict__ ids, float *__restrict__ scores, StepLds L, const int32_t *__restrict__ entries, int n_entries) {
    constexpr int NT = GRAPH_THREADS, W = NT / 32, SW = W;
    constexpr int MOST = RPG == 2 ? 63 : 32;              // neighbours of a step
    extern __shared__ __align__(16) unsigned char smem[];
    auto ls = [&](int which) { return reinterpret_cast<float *>(smem + L.ls + which * L.ls_bytes); };
    auto li = [&](int which) { return reinterpret_cast<uint32_t *>(smem + L.li + which * L.ls_bytes); };
    float *cs = reinterpret_cast<float *>(smem + StepLds::CS);           // [64] scores, ids, list positions of the neighbours
    int *ci = reinterpret_cast<int *>(smem + StepLds::CI);
    int *cpos = reinterpret_cast<int *>(smem + StepLds::CP);
    uint64_t *mk = reinterpret_cast<uint64_t *>(smem + StepLds::MK);    // [2][8] marks of a merge: a bit per final position
    uint32_t *cache = reinterpret_cast<uint32_t *>(smem + L.vis);        // ids scored lately
    u4 *qs = reinterpret_cast<u4 *>(smem + L.q);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.x;
    int *ent_v = reinterpret_cast<int *>(smem + StepLds::EV);            // [64] the step's neighbours and whose they are
    int *ent_w = reinterpret_cast<int *>(smem + StepLds::EW);
    uint32_t *fresh_m = reinterpret_cast<uint32_t *>(smem + StepLds::FM);   // [W] which slots of u_j's row are new
    // This wave's own scratch, no barrier around it: the selected entries in order
    int *sel_v = reinterpret_cast<int *>(smem + StepLds::WAVE0 + wave * StepLds::WAVE_BYTES);   // ids
    uint32_t *sel_k = reinterpret_cast<uint32_t *>(sel_v + SW);           // keys
    int *sel_p = sel_v + 2 * SW;                                         // positions
    const int32_t *my_entries = entries ? entries + (size_t)b * n_entries : nullptr;
    const int E = entries ? n_entries : 1;
    const int nch = d * T::bytes / 16;                    // 16-byte chunks per row
    const int sub = lane & (LANES_PER_ROW - 1);           // lane's position inside its row group
    const int grp = tid / LANES_PER_ROW;                  // 0 .. 31: takes neighbours grp and (RPG = 2) grp + 32

    for (int c = tid; c < nch; c += NT) qs[c] = load_chunk(static_cast<const char *>(Q) + ((size_t)b * nch + c) * 16);
    for (int i = tid; i < L.vis_words; i += NT) cache[i] = 0xffffffffu;
    // list scores start as -inf up to the next multiple of 64 entries (see group_lower_bound_fast)
    if (tid < 16) mk[tid] = 0ull;
    for (int i = tid; i < L.ls_bytes / 4; i += NT) { ls(0)[i] = -INFINITY; ls(1)[i] = -INFINITY; li(0)[i] = EXPANDED; li(1)[i] = EXPANDED; }
    __syncthreads();

    RowScorer<T, QREG, true> rows(X, qs, nch, sub);
    auto lds_barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    auto hash = [&](int v) { return (int)(((uint32_t)v * 2654435761u) >> L.cache_shift); };
    auto mark = [&](int v) { cache[hash(v)] = (uint32_t)v; };

    // ---- the candidate list ---------------------------------------------------------------------------
    // one ordered, double-buffered list ls / li / len, "expanded" flag in the id's top bit
    int cur = 0, len = 0;
    int par = 0;                                          // which set of mark words the next merge uses
    int first = 0;                                        // no unexpanded entry of ls / li lies below this position
    uint32_t worst_k = 0;                                 // the key a new entry has to reach, 0 while the list is not full

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
        const int to_len = min(ef, len + n_new);
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
    };

    // list <- the entry nodes (at most 32, one row group each), scored and put in order; ids that
    // are no nodes and ids named by an earlier slot are left out, a NaN score is never listed
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
        const int c_p = cpos[lane & 31];
        const uint64_t in = __builtin_amdgcn_ballot_w64(lane < 32 && c_p >= 0);
        merge_new(32);
        lds_barrier();
        merge_old(__builtin_popcountll(in));
        lds_barrier();
    }
    int n_expand = 0;
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
        for (int base = first & ~63; base < len && nd == 0; base += 256) {
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
                    if (((m >> lane) & 1) && r < SW) put(r, e[u], f[u], base + 64 * u + lane);
                    nd += __builtin_popcountll(m);
                }
        }
        nsel = min(nd, SW);
    };
    // the list as it stands after a merge: the bound for new entries, the first candidates
    auto settle = [&] {
        worst_k = len < ef ? 0u : score_key(ls(cur)[ef - 1]);
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
            if (fresh) fresh = cache[hash(nb)] != (uint32_t)nb;
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
                pos = group_lower_bound_fast(ls(cur), li(cur), len, s[t], v[t], sub, lane, &listed);
                if (pos >= ef || listed) pos = -1;
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
        const int C = min(wave_min(stop), n_part);
        n_expand += C;
        const int n_com = __builtin_popcountll(__builtin_amdgcn_ballot_w64(e_w < C));   // neighbours of committed nodes
        if (wave == 0 && lane < n_com && e_v >= 0) mark(e_v);
        // (every wave sets the flags of the entries that it may move: none has to wait for another's)
        if (lane < C) atomicOr(&li(cur)[u_p], EXPANDED);
        const uint64_t in = __builtin_amdgcn_ballot_w64(lane < n_com && c_k != 0);
        const int n_new = __builtin_popcountll(in);
        if (ef > 256) {
            // nothing unexpanded lies below the last committed position + 1 and the lowest new one
            first = min(__builtin_amdgcn_readlane(u_p, C - 1) + 1, wave_min(((in >> lane) & 1) ? c_p : INT_MAX));
        }
        if (n_new != 0) {
            merge_new(n_com);
            lds_barrier();
            merge_old(n_new);
        }
        lds_barrier();
        if ((int64_t)n_expand > N + W) break;             // (never on a sound list)
    }
    for (int j = tid; j < k; j += NT) {
        const bool has = j < len;
        ids[(size_t)b * k + j] = has ? (int)(li(cur)[j] & ~EXPANDED) : -1;
        scores[(size_t)b * k + j] = has ? ls(cur)[j] : -INFINITY;
    }
}

}  // namespace ann
