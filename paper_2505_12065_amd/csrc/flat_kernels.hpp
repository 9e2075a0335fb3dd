// Exact (flat) retrieval kernels: every corpus row is scored against every query
// and the k best per query are kept (Section 2.1 of the paper: exact nearest
// neighbour retrieval; the score matrix is never written to memory).
//
//   flat_stream_kernel  the corpus is streamed straight into MFMA operand registers, each row once per group
//                       of up to 64 queries; queries sit in LDS in MFMA fragment order.  All element types.
//   (flat_merge.hpp     per query: the k best of all slabs' lists)
//
// Every lane keeps a sorted register list of the 4 best pairs it has seen, whatever k is; lists are merged
// lane -> workgroup -> grid under the same total order, so the result does not depend on how rows were split.
#pragma once

#include "common.hpp"
#include "launch.hpp"

namespace ann {

// Row r of a 16-row MFMA tile is corpus row 16 tile + tile_row(r): lane group g = lane / 16 then receives the
// scores of corpus rows g, g + 4, g + 8, g + 12 of the tile, so that neighbouring rows (passages of one document,
// often close to the same query) go to different lanes' lists.
__device__ __forceinline__ int tile_row(int r) { return ((r & 3) << 2) | (r >> 2); }

// The K best (a multiple of 4, at most 16) of the 4 LG... entries held by an aligned group of LG lanes (32 or 64),
// LANE_KP sorted keys each (empty slots: the key of (-inf, EMPTY_ID)): put(r, key) for r = 0 .. K - 1, once by some lane of
// the group if `store`; fewer than K entries: the rest is empty.  `mem`: LDS scratch of 64 keys that belongs to the group alone
// (only its own wave touches it: no barrier).
//   K <= 4: four rounds of "largest head wins and is popped".
//   K > 4:  rounds cost 40 instructions each, so instead the heads' scores are sorted across the lanes; the
//           K-th is a bound that some 20 of the entries reach; those are ranked by counting.  (More than 64
//           reach it only when many scores are equal: then rounds it is.)
template <int LG, class Put>
__device__ __forceinline__ void group_select(uint64_t (&key)[LANE_KP], int K, uint64_t *mem, Put &&put, bool store) {
    const int lane = threadIdx.x & (WAVE - 1), sub = lane & (LG - 1);
    const uint64_t empty = order_key(-INFINITY, EMPTY_ID);
    bool rounds = K <= 4;
    if (!rounds) {
        const uint32_t sorted = group_sort_desc<LG>((uint32_t)(key[0] >> 32));
        uint32_t T = (uint32_t)__builtin_amdgcn_readlane((int)sorted, K - 1);
        if constexpr (LG == 32) {
            const uint32_t T1 = (uint32_t)__builtin_amdgcn_readlane((int)sorted, 32 + K - 1);
            T = lane < 32 ? T : T1;
        }
        const uint64_t mine = LG == 64 ? ~0ull : 0xffffffffull << (lane & 32);     // the lanes of this group
        const uint64_t below = mine & ((1ull << lane) - 1ull);
        int pos[LANE_KP], c = 0;
        bool in[LANE_KP];
#pragma unroll
        for (int e = 0; e < LANE_KP; ++e) {
            in[e] = (uint32_t)(key[e] >> 32) >= T && key[e] != empty;
            const uint64_t m = __builtin_amdgcn_ballot_w64(in[e]);
            pos[e] = c + __builtin_popcountll(m & below);
            c += __builtin_popcountll(m & mine);
        }
        const int c0 = __builtin_amdgcn_readlane(c, 0), c1 = __builtin_amdgcn_readlane(c, 63);
        const int cmax = max(c0, c1);
        if (cmax <= 64) {
#pragma unroll
            for (int e = 0; e < LANE_KP; ++e)
                if (in[e]) mem[pos[e]] = key[e];
            constexpr int PER = 64 / LG;
            uint64_t my[PER];
            int rank[PER];
#pragma unroll
            for (int u = 0; u < PER; ++u) { my[u] = mem[sub + u * LG]; rank[u] = 0; }
            for (int j0 = 0; j0 < cmax; j0 += 4) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint64_t o = mem[(j0 + t) & 63];
#pragma unroll
                    for (int u = 0; u < PER; ++u) rank[u] += (int)(j0 + t < c) & (int)(o > my[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (store && sub + u * LG < c && rank[u] < K) put(rank[u], my[u]);
            if (store && sub < K && sub >= c) put(sub, empty);
        } else {
            rounds = true;
        }
    }
    if (rounds) {
        for (int r = 0; r < K; ++r) {
            const uint64_t m = group_max<1, LG>(key[0]);
            if (key[0] == m) {
#pragma unroll
                for (int i = 0; i + 1 < LANE_KP; ++i) key[i] = key[i + 1];
                key[LANE_KP - 1] = empty;
            }
            if (store && sub == 0) put(r, m);
        }
    }
}

// What the streaming kernel works on.
struct StreamShape {
    const void *X;      // [N, d]
    const void *Q;      // [B, d]
    int64_t N;
    int d, B;
};

// MFMA operand of one 64-byte step of a row (or query) that may end inside the step: the chunk is zeroed past the end
__device__ __forceinline__ u4 mask_tail(u4 x, bool inside) {
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = inside ? x[i] : 0u;
    return x;
}

// Corpus rows are the M side of a 16x16 MFMA, queries the N side: a lane ends up with one query (lane % 16)
// and four rows per tile of 16 rows (see tile_row).  A step is 64 bytes of a row: 32 16-bit or 16 fp32 columns.
//   BATCH: 16-byte loads to a batch, of which a lane has two in flight (stream_batch; fp32: an even number).
//   FULL: a row is a whole number of batches of 64 bytes each load (else the last batch and step are cut to size).
//   grid: P slabs x G groups of 16 NQG queries, the groups of a slab side by side on one XCD, so that a slab that
//         several groups read comes from HBM once.  Tile t belongs to wave t % (P NWV) of the grid.
//   partial [B, P, K] pairs, K = 4, 8, 12 or 16 (>= k), every list sorted, empty slots (-inf, EMPTY_ID) last.
//   lds_steps: steps of a query that fit LDS (fewer than all of them only for fp32 rows beyond 2304 columns, where
//         one group of queries alone is larger than LDS: the rest comes from memory, NQG = 1, not FULL).
//   MAX: no lists; maxima[q, u] <- the largest score of rows [16 K u, 16 K (u + 1)) for flat_pick_kernel, n of them a
//         query (a multiple of 4), K = 1, 2 or 4 tiles to a group.
// Lists of 4 are exact for k <= 4.  For k > 4 a lane may meet more than 4 of the k best rows; the merge then finds 4
// rows of one lane among the k best and goes over that lane's rows again (flat_merge_lists_kernel).
//
// Bound by HBM for up to 64 queries on a large corpus.  Loads come in batches, the next one always requested
// before the products of the one before it, across tiles: without that a row of 12 steps (d = 384) paid four
// latencies a tile.  Lists of 4 for every k replace lists of 16 (3.5 times the time) and, on large corpora, a
// sampling pass with candidate arrays (three more launches and global atomics); fp32 runs here too, on the matrix
// cores, at most 32 queries to a workgroup (more do not raise the rate: eight products of 32 clocks per 1 KB of rows).
// Registers: two workgroups of 8 waves (or one of 16) per compute unit, except fp32 with two groups of queries (128
// registers of accumulators), which runs one workgroup and is bound by the products.
template <class T, int NQG, bool FULL, int NWV, bool MAX, int BATCH>
__global__ __launch_bounds__(NWV * 64, STREAM_WG_PER_CU(T::bytes, NQG, NWV) * NWV / 4) void flat_stream_kernel(StreamShape sh, Cand *__restrict__ partial, int P, int G,
                                                               int K, int lds_steps, After after, float *__restrict__ maxima, int64_t n,
                                                               StreamOut out) {
    static_assert(T::bytes == 2 || BATCH % 2 == 0, "fp32 sums go by the parity of a step");
    extern __shared__ __align__(16) unsigned char smem[];
    u4 *qf = reinterpret_cast<u4 *>(smem);            // [NQG][lds_steps][64]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = sh.d * T::bytes;                   // bytes of a row
    const int steps = (rb + 63) >> 6;
    const int B = sh.B;
    const int64_t N = sh.N;
    const int lb = xcd_block();
    const int slab = lb / G, q0 = (lb % G) * (NQG * 16);
    // the rows this wave starts with are requested before the queries are put into LDS
    // a wave takes one tile after the other a grid stride apart, or (MAX) K tiles side by side and then a stride
    const int64_t ntiles = (N + 15) >> 4, tstride = (int64_t)P * NWV * (MAX ? K : 1);
    const int run = MAX ? K : 1;
    auto next = [&](int64_t t) { return !MAX || (t & (run - 1)) == run - 1 ? t + tstride - (run - 1) : t + 1; };
    const int kofs = (lane >> 4) * 16;                // this lane's byte offset inside a step
    int64_t tile = ((int64_t)slab * NWV + wave) * run;
    const char *rp = nullptr;                         // this lane's row of the tile being loaded, kofs included
    auto row_ptr = [&](int64_t t) {
        int64_t row = t * 16 + tile_row(lane & 15);
        row = row < N ? row : N - 1;                  // tail tile: re-read the last row, masked below
        rp = static_cast<const char *>(sh.X) + (size_t)row * rb + kofs;
    };
    int64_t ltile = tile;                             // tile and step of the next batch to load
    int lstep = 0;
    if (tile < ntiles) row_ptr(tile);
    auto load = [&](u4 (&a)[BATCH]) {
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            if constexpr (FULL) a[u] = load_chunk(rp + (lstep + u) * 64);
            else a[u] = load_chunk(rp + min(min(lstep + u, steps - 1) * 64, rb - 16 - kofs));
        }
        lstep += BATCH;
        if (lstep >= steps) {
            lstep = 0;
            ltile = next(ltile);
            if (ltile < ntiles) row_ptr(ltile);       // (past the end: the last tile once more, never used)
        }
    };
    u4 xa[BATCH], xb[BATCH];
    if (tile < ntiles) load(xa);

    // queries -> LDS, already in B-operand order: fragment (g, s) holds for lane l
    // the 16 bytes from 64 s + 16 (l / 16) on of query q0 + 16 g + l % 16
    auto query_chunk = [&](int q, int ofs) {
        u4 v = zero_chunk();
        if (q < B && ofs < rb) v = load_chunk(static_cast<const char *>(sh.Q) + (size_t)q * rb + ofs);
        return v;
    };
    for (int i0 = wave; i0 < NQG * lds_steps; i0 += 4 * NWV) {
        u4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * NWV, g = i / lds_steps, s = i - g * lds_steps;
            v[u] = i < NQG * lds_steps ? query_chunk(q0 + g * 16 + (lane & 15), s * 64 + kofs) : zero_chunk();
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * NWV;
            if (i < NQG * lds_steps) qf[i * WAVE + lane] = TileSum<T>::operand(v[u]);
        }
    }

    TopList<LANE_KP> best[MAX ? 1 : NQG];
    float thr[NQG];                                   // (MAX: the largest score of the group of rows)
#pragma unroll
    for (int g = 0; g < NQG; ++g) {
        if constexpr (!MAX) best[g].init();
        thr[g] = MAX ? __builtin_nanf("") : -INFINITY;
    }
    TileSum<T> part[NQG];
    auto clear = [&] {
#pragma unroll
        for (int g = 0; g < NQG; ++g) part[g].clear();
    };
    clear();
    __syncthreads();

    int cstep = 0;                                    // step of the batch being multiplied
    // products of one batch; true when it was the last of its tile
    auto multiply = [&](u4 (&a)[BATCH]) -> bool {
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int s = cstep + u;
            if (FULL || u == 0 || s < steps) {
                u4 x = a[u];
                if constexpr (!FULL) {
                    if (s * 64 + 64 > rb) x = mask_tail(x, s * 64 + kofs < rb);
                }
                x = TileSum<T>::operand(x);
#pragma unroll
                for (int g = 0; g < NQG; ++g) {
                    u4 y;
                    if (FULL || NQG > 1 || s < lds_steps) y = qf[(g * lds_steps + s) * WAVE + lane];
                    else y = TileSum<T>::operand(query_chunk(q0 + (lane & 15), s * 64 + kofs));
                    part[g].step(u, x, y);            // (of fp32, batches start at even steps)
                }
                if constexpr (T::bytes == 4) __builtin_amdgcn_sched_barrier(0);   // (one transposed chunk at a time)
            }
        }
        cstep += BATCH;
        if (cstep < steps) return false;
        cstep = 0;
        return true;
    };
    auto finish_tile = [&] {
        const int rbase = (int)(tile * 16) + (lane >> 4);                // rows rbase + 4 i; N < 2^31
        const int nrows = (int)N;
        f4 acc[NQG];
#pragma unroll
        for (int g = 0; g < NQG; ++g) acc[g] = part[g].sum();
        if (after.s) {                                // rows at or before a query's boundary do not take part
#pragma unroll
            for (int g = 0; g < NQG; ++g) {           // (the pairs come from the L1: no registers to hold them)
                int l = lane;
                asm volatile("" : "+v"(l));           // (nor to hold what their addresses are made of)
                const int qb = min(q0 + g * 16 + (l & 15), B - 1);
                const float bs = after.s[qb];
                const int bid = after.id[qb], rafter = rbase + after.base;
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[g][i] = after_boundary(acc[g][i], rafter + 4 * i, bs, bid);
            }
        }
        if constexpr (MAX) {
            if (tile * 16 + 16 > N) {                 // rows that do not exist
#pragma unroll
                for (int g = 0; g < NQG; ++g)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[g][i] = rbase + 4 * i < nrows ? acc[g][i] : __builtin_nanf("");
            }
            const bool last = (tile & (run - 1)) == run - 1 || tile + 1 == ntiles;
#pragma unroll
            for (int g = 0; g < NQG; ++g) {
                thr[g] = fmaxf(thr[g], fmaxf(fmaxf(acc[g][0], acc[g][1]), fmaxf(acc[g][2], acc[g][3])));
                if (last) {
                    uint32_t p, q;
                    row_pair<16>(__float_as_uint(thr[g]), p, q);
                    float m = fmaxf(__uint_as_float(p), __uint_as_float(q));
                    row_pair<32>(__float_as_uint(m), p, q);
                    m = fmaxf(__uint_as_float(p), __uint_as_float(q));
                    thr[g] = __builtin_nanf("");
                    const int qi = q0 + g * 16 + lane;
                    if (lane < 16 && qi < B) {
                        float *o = maxima + (size_t)qi * n + tile / run;
                        o[0] = m;
                        if (tile + 1 == ntiles)       // the row of maxima is filled up to a multiple of 4
                            for (int64_t e = tile / run + 1; e < n; ++e) maxima[(size_t)qi * n + e] = __builtin_nanf("");
                    }
                }
            }
        } else static_for<NQG>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            const f4 a = acc[g];
            const float m = fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3]));
            if (__builtin_amdgcn_ballot_w64(m >= thr[g]) != 0) {        // rare after warm-up
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (rbase + 4 * i < nrows && a[i] >= thr[g]) best[g].insert(a[i], rbase + 4 * i);
                float t = best[g].s[LANE_KP - 1];
                if (K <= LANE_KP) {
                    // the 4th best of any lane that serves the same query bounds the final
                    // k-th best from below, so it is a safe rejection threshold for all four
                    uint32_t p, q;
                    row_pair<16>(__float_as_uint(t), p, q);
                    t = fmaxf(__uint_as_float(p), __uint_as_float(q));
                    row_pair<32>(__float_as_uint(t), p, q);
                    t = fmaxf(__uint_as_float(p), __uint_as_float(q));
                }
                thr[g] = fmaxf(thr[g], t);
            }
        });
        clear();
        tile = next(tile);
    };
    if (tile < ntiles) {
        for (;;) {
            load(xb);
            __builtin_amdgcn_sched_barrier(0);        // the requests stay ahead of the products
            if (multiply(xa)) {
                finish_tile();
                if (tile >= ntiles) break;
            }
            load(xa);
            __builtin_amdgcn_sched_barrier(0);
            if (multiply(xb)) {
                finish_tile();
                if (tile >= ntiles) break;
            }
        }
    }

    if constexpr (MAX) return;
    // every lane's lists -> LDS, then 16 queries at a time: the 4 NWV lists of a query by 4 NWV lanes
    constexpr int LG = 4 * NWV, QS = LG * LANE_KP + 4;                   // (padded: the writes of 16 queries spread over the banks)
    static_assert(NWV == 8 || NWV == 16, "a query's lists fill half a wave or a whole one");
    Cand *wl = reinterpret_cast<Cand *>(smem);
    __syncthreads();                                   // query fragments are dead from here
    if constexpr (!MAX) static_for<NQG>([&](auto gc) {
        constexpr int g = decltype(gc)::value;
        Cand *o = wl + (g * 16 + (lane & 15)) * QS + (wave * 4 + (lane >> 4)) * LANE_KP;
#pragma unroll
        for (int j = 0; j < LANE_KP; ++j) o[j] = Cand{best[g].s[j], best[g].id[j]};
    });
    __syncthreads();
    const int sub = tid & (LG - 1);
#pragma unroll 1
    for (int pass = 0; pass < NQG; ++pass) {
        const int qi = pass * 16 + tid / LG;
        Cand *in = wl + qi * QS;
        uint64_t key[LANE_KP];
#pragma unroll
        for (int j = 0; j < LANE_KP; ++j) {
            const Cand c = in[sub * LANE_KP + j];
            key[j] = order_key(c.s, c.id);
        }
        const size_t q = q0 + qi;
        auto put = [&](int r, uint64_t k64) {
            Cand c;
            order_key_decode(k64, c.s, c.id);
            if (!out.ids) {
                partial[(q * P + slab) * K + r] = c;
            } else if (r < out.k) {                   // the only slab: this list is the answer
                const bool has = c.id != EMPTY_ID;
                out.ids[q * out.k + r] = has ? c.id : -1;
                out.scores[q * out.k + r] = has ? c.s : -INFINITY;
            }
        };
        group_select<LG>(key, K, reinterpret_cast<uint64_t *>(in), put, (int)q < B);
    }
}

}  // namespace ann
