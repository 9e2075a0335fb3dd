// Exact search of few queries against few rows (Section 2.1 of the paper).  Both kernels are bound by the latency of what they read, so all
// of a lane's loads of a row are in flight before the first is used, up to 24 or 32 steps of 64 bytes: batches of four, two
// in flight, wait as many times as a row has pairs of them.  Products and their order are those of flat_stream_kernel, so the
// scores are its bits.
#pragma once

#include "flat_kernels.hpp"

namespace ann {

// All scores, for flat_pick_kernel: one wave scores 16 rows against 16 queries.  maxima[q, row], n of them a query (a multiple of 4;
// NaN: no row, or not after the query's boundary).  Workgroups of one wave, ceil(N / 16) x G of them, and no LDS: the rows go to as
// many compute units as there are, and none has more than a few KB to bring in (eight tiles in one workgroup: 196 KB through one L1 at
// d = 768, 3 us longer).  us of a call, lists or matrix-core tiles / this: 2860 x 352, B = 1 10.7 / 6.2; 977 x 1024 bf16, B = 5, k = 16 10.1 / 7.6;
// 3978 x 104, B = 9 8.4 / 6.3; 200 x 768, B = 1 8.5 / 6.3, B = 256 9.6 / 7.2; 10 000 x 128 fp32, B = 16, k = 10 11.6 / 10.3; 1202 x 128 fp32, B = 11, k = 10
// 12.8 / 8.2.
template <class T>
__global__ __launch_bounds__(WAVE, 1) void flat_scores_kernel(StreamShape sh, float *__restrict__ maxima, int n, int G, After after) {
    constexpr int RUN = 4, RUNS = 6, STEPS = RUN * RUNS;
    const int lane = threadIdx.x, l16 = lane & 15, quarter = lane >> 4;
    const int rb = sh.d * T::bytes, steps = (rb + 63) >> 6;
    const int B = sh.B, N = (int)sh.N;
    const int lb = xcd_block(), tile = lb / G, q0 = (lb % G) * 16;
    const int kofs = quarter * 16, q = min(q0 + l16, B - 1);
    const char *rp = static_cast<const char *>(sh.X) + (size_t)min(tile * 16 + l16, N - 1) * rb + kofs;
    const char *qp = static_cast<const char *>(sh.Q) + (size_t)q * rb + kofs;
    u4 x[STEPS], y[STEPS];
    // a run that reaches past the row's end reads its last chunk again
    auto load = [&](auto gc, int s) __attribute__((always_inline)) {
        constexpr int g = decltype(gc)::value;
        if ((s + RUN) * 64 <= rb) {
#pragma unroll
            for (int u = 0; u < RUN; ++u) {
                x[g * RUN + u] = load_chunk(rp + (s + u) * 64);
                y[g * RUN + u] = load_chunk(qp + (s + u) * 64);
            }
        } else if (s < steps) {
#pragma unroll
            for (int u = 0; u < RUN; ++u) {
                const int ofs = min((s + u) * 64, rb - 16 - kofs);
                x[g * RUN + u] = load_chunk(rp + ofs);
                y[g * RUN + u] = load_chunk(qp + ofs);
            }
        }
    };
    static_for<RUNS>([&](auto gc) { load(gc, decltype(gc)::value * RUN); });
    TileSum<T> part;
    part.clear();
    for (int s0 = 0; s0 < steps; s0 += STEPS)
        static_for<RUNS>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            const int s = s0 + g * RUN;
            if (s < steps) {
                if ((s + RUN) * 64 > rb) {
#pragma unroll
                    for (int u = 0; u < RUN; ++u) {
                        const bool inside = (s + u) * 64 + kofs < rb;
                        x[g * RUN + u] = mask_tail(x[g * RUN + u], inside);
                        y[g * RUN + u] = mask_tail(y[g * RUN + u], inside);
                    }
                }
#pragma unroll
                for (int u = 0; u < RUN; ++u) part.step(u, TileSum<T>::operand(x[g * RUN + u]), TileSum<T>::operand(y[g * RUN + u]));
                load(gc, s + STEPS);
            }
        });
    const f4 sum = part.sum();
    const int r0 = tile * 16 + 4 * quarter;
    if (q0 + l16 >= B || r0 >= n) return;
    f4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = after.s ? after_boundary(sum[i], r0 + i, after.s[q], after.id[q]) : sum[i];
        v[i] = r0 + i < N ? v[i] : __builtin_nanf("");
    }
    *reinterpret_cast<f4 *>(maxima + (size_t)q * n + r0) = v;
}

// N <= 128: a tile of 16 rows per wave, 8 waves, a workgroup per 16 queries; its lists are the answer, and nothing is written but that (direct_quick
// says where it is taken instead of the streaming kernel's one slab).  held: steps of a query in LDS,
// whole runs (fewer than all of them only for rows of over 9 KB: the rest comes from memory).
template <class T>
__global__ __launch_bounds__(DIRECT_WAVES * WAVE, DIRECT_WAVES / 4) void flat_direct_kernel(
    StreamShape sh, int k, int held, After after, int32_t *__restrict__ ids, float *__restrict__ scores) {
    constexpr int RUN = 4, RUNS = 8, STEPS = RUN * RUNS;
    extern __shared__ __align__(16) unsigned char smem[];
    u4 *qf = reinterpret_cast<u4 *>(smem);            // [held][64]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = sh.d * T::bytes, steps = (rb + 63) >> 6;
    const int B = sh.B, N = (int)sh.N;
    const int q0 = blockIdx.x * 16, kofs = (lane >> 4) * 16, tile = wave;
    const bool work = tile * 16 < N;

    // rows; a run that reaches past the row's end reads its last chunk again
    u4 x[STEPS];
    const char *rp = static_cast<const char *>(sh.X) + (size_t)min(tile * 16 + tile_row(lane & 15), N - 1) * rb + kofs;
    auto load = [&](auto gc, int s) __attribute__((always_inline)) {
        constexpr int g = decltype(gc)::value;
        if ((s + RUN) * 64 <= rb) {
#pragma unroll
            for (int u = 0; u < RUN; ++u) x[g * RUN + u] = load_chunk(rp + (s + u) * 64);
        } else if (s < steps) {
#pragma unroll
            for (int u = 0; u < RUN; ++u) x[g * RUN + u] = load_chunk(rp + min((s + u) * 64, rb - 16 - kofs));
        }
    };
    if (work) static_for<RUNS>([&](auto gc) { load(gc, decltype(gc)::value * RUN); });

    // queries -> LDS in B-operand order, whole runs: zeros behind the end
    auto query_chunk = [&](int q, int ofs) {
        u4 v = zero_chunk();
        if (q < B && ofs < rb) v = load_chunk(static_cast<const char *>(sh.Q) + (size_t)q * rb + ofs);
        return TileSum<T>::operand(v);
    };
    for (int i0 = wave; i0 < held; i0 += 8 * DIRECT_WAVES) {
        u4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * DIRECT_WAVES;
            v[u] = query_chunk(i < held ? q0 + (lane & 15) : B, i * 64 + kofs);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * DIRECT_WAVES;
            if (i < held) qf[i * WAVE + lane] = v[u];
        }
    }
    TileSum<T> part;
    part.clear();
    __syncthreads();

    for (int s0 = 0; work && s0 < steps; s0 += STEPS) {
        static_for<RUNS>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            const int s = s0 + g * RUN;
            if (s < steps) {
                u4 y[RUN];
#pragma unroll
                for (int u = 0; u < RUN; ++u) y[u] = s < held ? qf[(s + u) * WAVE + lane] : query_chunk(q0 + (lane & 15), (s + u) * 64 + kofs);
                if ((s + RUN) * 64 > rb) {
#pragma unroll
                    for (int u = 0; u < RUN; ++u) x[g * RUN + u] = mask_tail(x[g * RUN + u], (s + u) * 64 + kofs < rb);
                }
#pragma unroll
                for (int u = 0; u < RUN; ++u) {
                    part.step(u, TileSum<T>::operand(x[g * RUN + u]), y[u]);
                    if constexpr (T::bytes == 4) __builtin_amdgcn_sched_barrier(0);
                }
                load(gc, s + STEPS);
            }
        });
    }

    // the lane's four keys, largest first -> LDS; then the 32 lists of a query by 32 lanes
    constexpr int LG = 4 * DIRECT_WAVES, QS = LG * LANE_KP + 4;           // (padded: the writes of 16 queries spread over the banks)
    const uint64_t empty = order_key(-INFINITY, EMPTY_ID);
    uint64_t *wl = reinterpret_cast<uint64_t *>(smem);
    const f4 sum = part.sum();
    const int qb = min(q0 + (lane & 15), B - 1);
    uint64_t key[LANE_KP];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = tile * 16 + (lane >> 4) + 4 * i;
        const float v = after.s ? after_boundary(sum[i], row, after.s[qb], after.id[qb]) : sum[i];
        key[i] = row < N && v == v ? order_key(v, row) : empty;
    }
    auto order = [&](int a, int b) {
        const uint64_t hi = key[a] > key[b] ? key[a] : key[b], lo = key[a] > key[b] ? key[b] : key[a];
        key[a] = hi;
        key[b] = lo;
    };
    order(0, 1); order(2, 3); order(0, 2); order(1, 3); order(1, 2);
    __syncthreads();                                  // query fragments are dead from here
    uint64_t *o = wl + (lane & 15) * QS + (wave * 4 + (lane >> 4)) * LANE_KP;
#pragma unroll
    for (int j = 0; j < LANE_KP; ++j) o[j] = key[j];
    __syncthreads();
    const int sub = tid & (LG - 1), q = q0 + tid / LG;
    uint64_t *in = wl + (tid / LG) * QS;
#pragma unroll
    for (int j = 0; j < LANE_KP; ++j) key[j] = in[sub * LANE_KP + j];
    auto put = [&](int r, uint64_t k64) {
        float s;
        int id;
        order_key_decode(k64, s, id);
        const bool has = id != EMPTY_ID;
        ids[(size_t)q * k + r] = has ? id : -1;
        scores[(size_t)q * k + r] = has ? s : -INFINITY;
    };
    group_select<LG>(key, k, in, put, q < B);
}

}  // namespace ann
