// Second half of the exact search on the matrix cores: from the group maxima that flat_wide_kernel leaves, the k best
// rows of every query.
#pragma once

#include "flat_kernels.hpp"

namespace ann {

// Corpus row of place `slot` in the order of flat_wide_kernel's lanes: tile, wave row, lane half, accumulator.  The groups
// are runs of 2^gs_log places, and a group's first place is its lowest row.
// WMF = 0: the order of flat_stream_kernel's maxima, rows as they come.
template <int WMF>
__device__ __forceinline__ int64_t wide_row(int64_t slot) {
    if constexpr (WMF == 0) return slot;
    constexpr int W = WMF == 0 ? 1 : WMF;
    const int s = (int)(slot & (64 * W - 1));
    const int wm = s / (32 * W), lhi = s / (16 * W) & 1, i = s / 16 & (W - 1), r = s & 15;
    return (slot & ~(int64_t)(64 * W - 1)) + wm * 32 * W + i * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
}

// One workgroup (1 to 8 wavefronts) per query.
//   1. every thread takes the largest of the maxima it looks at; the k-th largest of those is a bound that few maxima
//      reach (two sorting networks);
//   2. those few are gathered in LDS and ranked by counting: the groups with fewer than k larger ones hold the k best
//      rows, and the k-th best group maximum T is a lower bound of the k-th best score;
//   3. their rows are scored once more, by the instructions and in the order of the kernel that left the maxima, so to the
//      same bits: 32 (fp32: 16) rows to an MFMA, the query as every one of its columns; the rows that reach T (k, if none
//      tie) are ranked.
// Groups of one row: their maxima are the scores, step 3 falls away.  Hundreds of maxima that tie with the k-th: the groups
// are gone through in order, a few at a time, past those that can no longer improve the k best so far.
// Bound by latency: three dependent reads (maxima twice, rows), and between them the reads of the LDS.  Beyond about 1000
// queries by the bytes of the rows.  The serial parts are therefore written as few long batches: a row's loads 24 steps at a
// time and the query's operands read 6 steps ahead of the products (one at a time they were three quarters of step 3), ranks
// eight reads at a time, and gathering by a thread's mask of hits instead of a test and an atomic for each maximum.  us, before / now:
// 77 queries x 7716 maxima, 160 rows of 1552 bytes 17.0 / 12.7; 128 x 18 k, 320 rows of 768 20.8 / 13.3; 64 x 31 k, 320 rows of 3072
// 52 / 33; 512 x 15 k, 192 rows of 1536 41.8 / 34.2; single rows 5000 x 1024, k = 16 9.8 / 8.2, 512 x 1024, k = 1 4.7 / 4.0.
// RUNS (pick_runs): the long runs and held operands, 92 registers.  Shorter rows have none, and many queries want waves more than
// runs: 12 steps at a time, 64 registers.  us of the kernel, with / without: 11 212 x 48, B = 2765, k = 10 41.2 / 24.3; 48 434 x 128, B = 4007
// 71.0 / 45.6; 219 465 x 32, B = 514, k = 16 28.4 / 18.2; 16 000 x 1024, B = 4000, k = 10 69.7 / 62.3; but 123 457 x 776, B = 77 8.6 / 12.0, 512
// 14.9 / 16.5; 10 953 x 544, B = 900 / 1100 10.3 / 12.2, 16.3 / 14.0; 16 000 x 1024, B = 900 / 1100 13.3 / 16.5, 20.7 / 18.4; 9000 x 1152, B = 1531
// 19.7 / 20.5; 30 000 x 1544, B = 4000 59.0 / 67.4.
// PARTS: a search that takes the corpus in parts (sh.X and sh.N are the part, after.base its first row) goes on from the k
// best of the parts before, which also bound what is worth looking at: best_so_far [B, k], read where `more` has bit 0;
// the result goes back there where it has bit 1, else to ids and scores.  (A variant of its own: the calls of a few
// microseconds do not wait for two more arguments.)
constexpr int PICK_CAP = 512;
template <class T, int WMF, bool ONE, bool PARTS, bool RUNS>
__global__ __launch_bounds__(512) void flat_pick_kernel(const float *__restrict__ maxima, int64_t n, int gs_log, int k,
                                                        int32_t *__restrict__ ids, float *__restrict__ scores, StreamShape sh,
                                                        After after, uint64_t *__restrict__ best_so_far, int more) {
    __shared__ uint64_t ck[PICK_CAP];                 // gathered maxima, then scored rows
    __shared__ int sel[PICK_CAP];                     // groups to score
    __shared__ uint32_t top[8 * 16];
    __shared__ uint64_t fin[16], old[16];             // the k best so far, in order
    __shared__ int n_c, n_sel;
    __shared__ uint32_t t_min;
    extern __shared__ __align__(16) unsigned char smem[];
    u4 *qs = reinterpret_cast<u4 *>(smem);            // the query (groups of more than one row)
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int NT = blockDim.x, nwaves = NT >> 6;
    const uint64_t empty = order_key(-INFINITY, EMPTY_ID);
    const int base = PARTS ? after.base : 0;
    const float *mx = maxima + (size_t)q * n;
    const int rb = sh.d * T::bytes, nch = rb >> 4;
    if (tid < 16) fin[tid] = PARTS && (more & 1) && tid < k ? best_so_far[(size_t)q * k + tid] : empty;
    if (tid == 0) { n_c = 0; n_sel = 0; t_min = ~0u; }
    if (!ONE)
        for (int c = tid; c < nch; c += NT) qs[c] = load_chunk(static_cast<const char *>(sh.Q) + (size_t)q * rb + c * 16);

    // order-preserving image of a maximum, 0 for a NaN (no row that takes part)
    auto image = [](float v) { return v == v ? (uint32_t)(order_key(v, 0) >> 32) : 0u; };
    uint32_t m = 0;
    const int64_t n4 = n >> 2;                        // (n is a multiple of 4)
    f4 v[4];                                          // 16 maxima: all of this thread's, if n <= 16 NT
    auto load_maxima = [&](int64_t i0) {              // (i0 may lie behind the end, for lanes)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = i0 + u * NT;
            v[u] = *reinterpret_cast<const f4 *>(mx + 4 * (i < n4 ? i : min(i0, n4 - 1)));
        }
    };
    for (int64_t i0 = tid; i0 < n4; i0 += 4 * NT) {
        load_maxima(i0);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) m = max(m, image(v[u][c]));
    }
    m = group_sort_desc<64>(m);
    if (nwaves > 1) {
        if (lane < 16) top[wave * 16 + lane] = m;
        __syncthreads();
        m = 0;                                        // (of 8 waves: the larger ones of two lists, still k different maxima)
        for (int w = lane >> 4; w < nwaves; w += 4) m = max(m, top[w * 16 + (lane & 15)]);
        m = group_sort_desc<64>(m);
    } else {
        __syncthreads();                              // the shared words are set
    }
    uint32_t bound = max(1u, (uint32_t)__builtin_amdgcn_readlane((int)m, k - 1));
    if (PARTS && (more & 1)) bound = max(bound, (uint32_t)(fin[k - 1] >> 32));
    // 64-bit key of entry e with value image x: what the ranks go by (one row: the row's own key)
    auto entry_key = [&](uint32_t x, int64_t e) {
        return ((uint64_t)x << 32) | (uint32_t)~(uint32_t)(ONE ? base + wide_row<WMF>(e) : e);
    };
    // as a number (images below that of -inf: every number reaches it)
    float least;
    int none;
    order_key_decode((uint64_t)max(bound, (uint32_t)(order_key(-INFINITY, 0) >> 32)) << 32, least, none);
    for (int64_t b = 0; b < n4; b += 4 * NT) {
        if (n4 > 4 * NT) load_maxima(b + tid);
        uint32_t hits = 0;                            // those of this thread's 16 that reach the bound
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) hits |= v[u][c] >= least ? 1u << (4 * u + c) : 0u;
        const int64_t have = n4 - b - tid;            // (places behind the end repeat the first)
        hits &= have > 3 * NT ? 0xffffu : have > 2 * NT ? 0xfffu : have > NT ? 0xffu : have > 0 ? 0xfu : 0u;
        while (const uint64_t lanes = __ballot(hits != 0)) {
            int at = 0;
            if (lane == 0) at = atomicAdd(&n_c, __popcll(lanes));
            at = __builtin_amdgcn_readfirstlane(at) +
                 __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0));
            if (hits != 0 && at < PICK_CAP) {
                const int e = __ffs(hits) - 1;
                const int64_t g = 4 * (b + tid + (e >> 2) * NT) + (e & 3);
                ck[at] = entry_key(image(mx[g]), g);
            }
            hits &= hits - 1;
        }
    }
    __syncthreads();
    const int found = n_c;

    // how many of ck[0 .. c) are larger, eight reads at a time
    auto larger_than = [&](uint64_t mine, int c) {
        int r = 0;
        for (int j = 0; j < c; j += 8) {
            uint64_t o[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) o[u] = ck[j + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) r += (int)(j + u < c && o[u] > mine);
        }
        return r;
    };
    // fin <- the k best of fin and ck[0 .. c); empty: fin holds nothing yet
    auto merge = [&](int c, bool empty = false) {
        if (empty) {
            for (int i = tid; i < c; i += NT) {
                const uint64_t mine = ck[i];
                const int r = larger_than(mine, c);
                if (r < k) fin[r] = mine;
            }
            __syncthreads();
            return;
        }
        if (tid < 16) old[tid] = fin[tid];
        __syncthreads();
        for (int i = tid; i < c + k; i += NT) {
            const uint64_t mine = i < c ? ck[i] : old[i - c];
            int r = larger_than(mine, c) + (i < c ? 0 : i - c);
            if (i < c)
                for (int j = 0; j < k; ++j) r += (int)(old[j] > mine);
            if (r < k) fin[r] = mine;
        }
        __syncthreads();
    };
    // the rows of groups sel[0 .. ns) scored and merged, PICK_CAP at a time; t: image that a row has to reach
    auto score_groups = [&](int ns, uint32_t t, bool first) {
        const int64_t rows = (int64_t)ns << gs_log;
        auto row_of = [&](int64_t e) {
            e = e < rows ? e : rows - 1;
            return wide_row<WMF>(((int64_t)sel[e >> gs_log] << gs_log) + (e & ((1 << gs_log) - 1)));
        };
        for (int64_t b0 = 0; b0 < rows; b0 += PICK_CAP) {
            if (tid == 0) n_c = 0;
            __syncthreads();
            const uint64_t worst = fin[k - 1];
            constexpr int UNIT = T::bytes == 4 ? 16 : 32;                 // rows to an MFMA
            for (int u = wave; u < PICK_CAP / UNIT && b0 + u * UNIT < rows; u += nwaves) {
                const int64_t e0 = b0 + u * UNIT;
                int64_t row = row_of(e0 + (lane & (UNIT - 1)));
                row = row < sh.N ? row : sh.N - 1;
                const char *rp = static_cast<const char *>(sh.X) + (size_t)row * rb;
                // RUN steps whose loads are in flight together, PART steps whose operands of the query are read together: a read
                // of the LDS before each product, waited for, took three quarters of the time
                constexpr int RUN = 24, PART = 6, TAIL = 12;
                const int sub = lane / UNIT;          // this lane's chunk of a step
                constexpr int CHUNKS = WAVE / UNIT;
                const int steps = (nch + CHUNKS - 1) / CHUNKS;
                // every column of the result holds the same sums: a lane's first columns look after one each
                float v;
                int col, at;                          // this lane's column, and which of the rows it looks after
                auto run = [&](auto &&product) {
                    int s0 = 0;
                    if constexpr (RUNS) {
                        for (; CHUNKS * (s0 + RUN) <= nch; s0 += RUN) {
                            const char *p = rp + (CHUNKS * s0 + sub) * 16;
                            const u4 *yp = qs + CHUNKS * s0 + sub;
                            u4 x[RUN];
#pragma unroll
                            for (int s = 0; s < RUN; ++s) x[s] = load_chunk(p + CHUNKS * s * 16);
#pragma unroll
                            for (int g = 0; g < RUN; g += PART) {
                                u4 y[PART];
#pragma unroll
                                for (int s = 0; s < PART; ++s) y[s] = yp[CHUNKS * (g + s)];
                                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                                for (int s = 0; s < PART; ++s) product(s & 3, x[g + s], y[s]);
                            }
                        }
                    }
                    for (; s0 < steps; s0 += TAIL) {
                        u4 x[TAIL], y[TAIL];
#pragma unroll
                        for (int s = 0; s < TAIL; ++s) {
                            x[s] = zero_chunk();
                            if (RUNS) y[s] = zero_chunk();
                            if (s0 + s < steps) {
                                const int ch = min(CHUNKS * (s0 + s) + sub, nch - 1);
                                x[s] = load_chunk(rp + ch * 16);
                                if (RUNS) y[s] = qs[ch];
                            }
                        }
                        if (RUNS) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int s = 0; s < TAIL; ++s)
                            if (s0 + s < steps) {
                                const int ch = CHUNKS * (s0 + s) + sub;
                                product(s & 3, mask_tail(x[s], ch < nch), mask_tail(RUNS ? y[s] : qs[min(ch, nch - 1)], ch < nch));
                            }
                    }
                };
                if constexpr (T::bytes == 4) {
                    TileSum<T> part;
                    part.clear();
                    run([&](int s, u4 x, u4 y) { part.step(s, TileSum<T>::operand(x), TileSum<T>::operand(y)); });
                    const f4 sum = part.sum();
                    col = lane & 15;
                    v = col == 1 ? sum[1] : col == 2 ? sum[2] : col == 3 ? sum[3] : sum[0];
                    at = 4 * sub + (col & 3);
                } else {
                    f16v acc;
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
                    run([&](int, u4 x, u4 y) { acc = mfma32<T>(x, y, acc); });
                    col = lane & 31;
                    v = acc[0];
#pragma unroll
                    for (int r = 1; r < 16; ++r) v = col == r ? acc[r] : v;
                    at = 8 * ((col & 15) >> 2) + 4 * sub + (col & 3);
                }
                const int64_t e = e0 + at, id = row_of(e);
                if (after.s) v = after_boundary(v, base + (int)id, after.s[q], after.id[q]);
                if (col < UNIT / CHUNKS && e < rows && id < sh.N && v == v) {
                    const uint64_t key = order_key(v, base + (int)id);
                    if ((uint32_t)(key >> 32) >= t && key > worst) ck[atomicAdd(&n_c, 1)] = key;
                }
            }
            __syncthreads();
            merge(n_c, first && b0 == 0);
        }
    };

    if (found <= PICK_CAP) {
        if (ONE) {
            merge(found, !(PARTS && (more & 1)));
        } else {
            for (int i = tid; i < found; i += NT) {
                const uint32_t mine = (uint32_t)(ck[i] >> 32);
                if (larger_than(ck[i] | 0xffffffffu, found) < k) {
                    sel[atomicAdd(&n_sel, 1)] = (int)~(uint32_t)ck[i];
                    atomicMin(&t_min, mine);
                }
            }
            __syncthreads();
            score_groups(n_sel, found < k ? 0u : t_min, !(PARTS && (more & 1)));
        }
    } else {
        const int step = ONE ? PICK_CAP : 64;
        for (int64_t c0 = 0; c0 < n; c0 += step) {
            __syncthreads();
            if (tid == 0) { n_c = 0; n_sel = 0; }
            __syncthreads();
            const uint64_t worst = fin[k - 1];
            for (int64_t e = c0 + tid; e < min(c0 + (int64_t)step, n); e += NT) {
                const uint32_t x = image(mx[e]);
                const uint64_t best = ((uint64_t)x << 32) | (uint32_t)~(uint32_t)(base + wide_row<WMF>(e << gs_log));
                if (x >= bound && best > worst) {     // its best row may be better than the k-th so far
                    if (ONE) ck[atomicAdd(&n_c, 1)] = best;
                    else sel[atomicAdd(&n_sel, 1)] = (int)e;
                }
            }
            __syncthreads();
            if (ONE) { if (n_c > 0) merge(n_c); }
            else if (n_sel > 0) score_groups(n_sel, bound, false);
        }
    }

    if (PARTS && (more & 2)) {
        if (tid < k) best_so_far[(size_t)q * k + tid] = fin[tid];
    } else if (tid < k) {
        float s;
        int id;
        order_key_decode(fin[tid], s, id);
        const bool has = id != EMPTY_ID;
        ids[(size_t)q * k + tid] = has ? id : -1;
        scores[(size_t)q * k + tid] = has ? s : -INFINITY;
    }
}

}  // namespace ann
