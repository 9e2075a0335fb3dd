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
// Bound by the latency of three dependent reads (maxima twice, rows) at 8 to 12 us, and beyond about 1000 queries by the
// bytes of the rows.
// PARTS: a search that takes the corpus in parts (sh.X and sh.N are the part, after.base its first row) goes on from the k
// best of the parts before, which also bound what is worth looking at: best_so_far [B, k], read where `more` has bit 0;
// the result goes back there where it has bit 1, else to ids and scores.  (A variant of its own: the calls of a few
// microseconds do not wait for two more arguments.)
constexpr int PICK_CAP = 512;
template <class T, int WMF, bool ONE, bool PARTS>
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
    auto load_maxima = [&](int64_t i0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = i0 + u * NT;
            v[u] = *reinterpret_cast<const f4 *>(mx + 4 * (i < n4 ? i : i0));
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
    for (int64_t i0 = tid; i0 < n4; i0 += 4 * NT) {
        if (n4 > 4 * NT) load_maxima(i0);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t x = image(v[u][c]);
                if (x >= bound && i0 + u * NT < n4) {
                    const int at = atomicAdd(&n_c, 1);
                    if (at < PICK_CAP) ck[at] = entry_key(x, 4 * (i0 + u * NT) + c);
                }
            }
    }
    __syncthreads();
    const int found = n_c;

    // fin <- the k best of fin and ck[0 .. c)
    auto merge = [&](int c) {
        if (tid < 16) old[tid] = fin[tid];
        __syncthreads();
        for (int i = tid; i < c + k; i += NT) {
            const uint64_t mine = i < c ? ck[i] : old[i - c];
            int r = i < c ? 0 : i - c;
            for (int j = 0; j < c; ++j) r += (int)(ck[j] > mine);
            if (i < c)
                for (int j = 0; j < k; ++j) r += (int)(old[j] > mine);
            if (r < k) fin[r] = mine;
        }
        __syncthreads();
    };
    // the rows of groups sel[0 .. ns) scored and merged, PICK_CAP at a time; t: image that a row has to reach
    auto score_groups = [&](int ns, uint32_t t) {
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
                constexpr int RUN = 12;               // steps whose loads are in flight together
                const int sub = lane / UNIT;          // this lane's chunk of a step
                constexpr int CHUNKS = WAVE / UNIT;
                const int steps = (nch + CHUNKS - 1) / CHUNKS;
                // every column of the result holds the same sums: a lane's first columns look after one each
                float v;
                int col, at;                          // this lane's column, and which of the rows it looks after
                auto run = [&](auto &&product) {
                    for (int s0 = 0; s0 < steps; s0 += RUN) {
                        u4 x[RUN];
#pragma unroll
                        for (int s = 0; s < RUN; ++s) {
                            x[s] = zero_chunk();
                            if (s0 + s < steps) x[s] = load_chunk(rp + min(CHUNKS * (s0 + s) + sub, nch - 1) * 16);
                        }
#pragma unroll
                        for (int s = 0; s < RUN; ++s)
                            if (s0 + s < steps) {
                                const int ch = CHUNKS * (s0 + s) + sub;
                                product(s, mask_tail(x[s], ch < nch), mask_tail(qs[min(ch, nch - 1)], ch < nch));
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
            merge(n_c);
        }
    };

    if (found <= PICK_CAP) {
        if (ONE) {
            merge(found);
        } else {
            for (int i = tid; i < found; i += NT) {
                const uint32_t mine = (uint32_t)(ck[i] >> 32);
                int larger = 0;
                for (int j = 0; j < found; ++j) larger += (int)((uint32_t)(ck[j] >> 32) > mine);
                if (larger < k) {
                    sel[atomicAdd(&n_sel, 1)] = (int)~(uint32_t)ck[i];
                    atomicMin(&t_min, mine);
                }
            }
            __syncthreads();
            score_groups(n_sel, found < k ? 0u : t_min);
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
            else if (n_sel > 0) score_groups(n_sel, bound);
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
