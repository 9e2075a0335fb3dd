// Merge kernels of the flat search: per query, the k best of what the slabs of a main pass left.
#pragma once

#include "flat_kernels.hpp"

namespace ann {

// best <- best of itself and in[first], in[first + stride], ...: eight loads in flight per
// thread, so a short list costs one memory latency instead of one per element
template <int KP>
__device__ __forceinline__ void gather_best(const Cand *__restrict__ in, int total, int first, int stride,
                                            TopList<KP> &best) {
    for (int e0 = first; e0 < total; e0 += 8 * stride) {
        Cand c[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = e0 + u * stride;
            c[u] = e < total ? in[e] : Cand{-INFINITY, EMPTY_ID};
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (best.admits(c[u].s, c[u].id)) best.insert(c[u].s, c[u].id);
    }
}

// k <= 4.  One workgroup (1 to 4 wavefronts, by the amount of work) per query: the k best of its P lists of 4,
// written in order; unused tail slots become id -1 / score -inf.
__global__ __launch_bounds__(256) void flat_merge_kernel(const Cand *__restrict__ partial, int P, int k,
                                                         int32_t *__restrict__ ids, float *__restrict__ scores) {
    constexpr int KP = LANE_KP;
    __shared__ Cand wl[4 * KP];
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nwaves = blockDim.x >> 6;
    TopList<KP> best;
    best.init();
    gather_best<KP>(partial + (size_t)q * P * KP, P * KP, tid, blockDim.x, best);
    TopList<KP> fin;
    group_top<KP, KP, 1, 64>(best, fin);
    if (nwaves > 1) {
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j < KP; ++j) wl[wave * KP + j] = Cand{fin.s[j], fin.id[j]};
        }
        __syncthreads();
        if (wave != 0) return;
        TopList<1> one;                               // one entry per lane
        one.init();
        if (lane < nwaves * KP) { one.s[0] = wl[lane].s; one.id[0] = wl[lane].id; }
        group_top<KP, 1, 1, 64>(one, fin);
    }
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < KP; ++j)
            if (j < k) {
                const bool has = fin.id[j] != EMPTY_ID;
                ids[(size_t)q * k + j] = has ? fin.id[j] : -1;
                scores[(size_t)q * k + j] = has ? fin.s[j] : -INFINITY;
            }
    }
}

// k > 4.  One workgroup (1 or 4 wavefronts) per query: the k best of its P sorted lists of K pairs (K = 8, 12, 16).
//   1. every lane takes the best head of the lists it looks at; the k-th best of those over the workgroup is a
//      bound that few entries reach (two sorting networks of 21 steps; lists of up to 2048 slabs cost the same);
//   2. entries that reach it are gathered in LDS (about k of them; a tie of hundreds: rounds of maxima instead);
//   3. each is ranked by counting, and the k best are in their places.
// slots > 0 (lists made by flat_stream_kernel<.., NWV> with slots = P NWV): a lane of that kernel kept only the 4 best of
// its rows.  If 4 of the k best came from one lane, it may have dropped a fifth: its rows (tiles slot, slot + slots, ...,
// rows = quarter mod 4) are scored again here, by the same products in the same order, and take their places.
// Random or clustered corpora never get here (5 of the k best rows must lie a whole number of grid strides apart).
constexpr int MERGE_CAP = 512;
template <class T>
__global__ __launch_bounds__(256) void flat_merge_lists_kernel(const Cand *__restrict__ partial, int P, int K, int k,
                                                               int32_t *__restrict__ ids, float *__restrict__ scores,
                                                               StreamShape sh, int slots, After after) {
    __shared__ uint64_t ck[MERGE_CAP];
    __shared__ uint32_t top[64];
    __shared__ uint64_t fin[16];                      // the k best so far, in order
    __shared__ int n_c;
    __shared__ uint32_t flagged;
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int NT = blockDim.x, nwaves = NT >> 6;
    const uint64_t empty = order_key(-INFINITY, EMPTY_ID);
    const Cand *in = partial + (size_t)q * P * K;
    if (tid < 16) fin[tid] = empty;
    if (tid == 0) n_c = 0;
    auto key_at = [&](int i, int e) {
        const Cand c = in[(size_t)i * K + e];
        return order_key(c.s, c.id);
    };
    if (P * K <= NT) {                                // an entry per thread: all of them are ranked
        if (tid < P * K) ck[tid] = key_at(tid / K, tid % K);
        if (tid == 0) n_c = P * K;
        __syncthreads();
    } else {
        uint32_t m = 0;
        for (int i0 = tid; i0 < P; i0 += 4 * NT) {
            uint64_t h[4];
    #pragma unroll
            for (int u = 0; u < 4; ++u) h[u] = key_at(min(i0 + u * NT, P - 1), 0);
    #pragma unroll
            for (int u = 0; u < 4; ++u) m = i0 + u * NT < P ? max(m, (uint32_t)(h[u] >> 32)) : m;
        }
        m = group_sort_desc<64>(m);
        if (nwaves > 1) {
            if (lane < 16) top[wave * 16 + lane] = m;
            __syncthreads();
            m = group_sort_desc<64>(top[lane]);           // (4 waves: 64 values)
        } else {
            __syncthreads();                              // fin and n_c are set
        }
        const uint32_t bound = (uint32_t)__builtin_amdgcn_readlane((int)m, k - 1);
        for (int i = tid; i < P; i += NT)
            for (int e = 0; e < K; ++e) {
                const uint64_t h = key_at(i, e);
                if ((uint32_t)(h >> 32) < bound || h == empty) break;
                const int at = atomicAdd(&n_c, 1);
                if (at < MERGE_CAP) ck[at] = h;
            }
    }
    __syncthreads();
    const int n = n_c;
    if (n <= MERGE_CAP) {
        for (int i = tid; i < n; i += NT) {
            const uint64_t mine = ck[i];
            int r = 0;
#pragma unroll 8
            for (int j = 0; j < n; ++j) r += (int)(ck[j] > mine);
            if (r < k) fin[r] = mine;
        }
    } else {
        // hundreds of entries tie with the k-th: k rounds over all of them, each takes the largest below the last
        uint64_t last = ~0ull;
        for (int r = 0; r < k; ++r) {
            uint64_t best = empty;
            for (int i = tid; i < P; i += NT)
                for (int e = 0; e < K; ++e) {
                    const uint64_t h = key_at(i, e);
                    if (h < last) { best = h > best ? h : best; break; }
                }
            best = group_max<1, 64>(best);
            __syncthreads();
            if (lane == 0) ck[wave] = best;
            __syncthreads();
            for (int w = 0; w < nwaves; ++w) best = ck[w] > best ? ck[w] : best;
            if (tid == 0) fin[r] = best;
            last = best;
        }
    }
    __syncthreads();

    const int64_t ntiles = (sh.N + 15) >> 4;
    if (slots > 0 && ntiles > slots) {                // (one tile per lane: nothing was dropped)
        if (wave == 0) {
            float s;
            int id;
            order_key_decode(fin[lane & 15], s, id);
            const int from = id == EMPTY_ID ? -1 - lane : ((id >> 4) % slots) * 4 + (id & 3);   // the lane that kept it
            int same = 0, first = 1;
            for (int j = 0; j < k; ++j) {
                const int o = __builtin_amdgcn_readlane(from, j);
                same += (int)(o == from);
                if (o == from && j < lane) first = 0;
            }
            const uint64_t f = __builtin_amdgcn_ballot_w64(lane < k && from >= 0 && first && same >= LANE_KP);
            if (lane == 0) flagged = (uint32_t)f;
        }
        __syncthreads();
        uint32_t todo = flagged;
        uint32_t streams[4];                          // at most k / 4 lanes
        int n_streams = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            streams[t] = 0;
            if (todo != 0) {
                float s;
                int id;
                order_key_decode(fin[__builtin_ctz(todo)], s, id);
                streams[t] = (uint32_t)((id >> 4) % slots) * 4 + (id & 3);
                n_streams = t + 1;
                todo &= todo - 1;
            }
        }
        for (int t = 0; t < n_streams; ++t) {
            const int slot = (int)(streams[t] >> 2), quarter = (int)(streams[t] & 3);
            const int rb = sh.d * T::bytes, steps = (rb + 63) >> 6, kofs = (lane >> 4) * 16;
            for (int64_t t0 = slot; t0 < ntiles; t0 += (int64_t)slots * nwaves) {
                const int64_t tile = t0 + (int64_t)slots * wave;
                if (tile < ntiles) {
                    int64_t row = tile * 16 + tile_row(lane & 15);
                    row = row < sh.N ? row : sh.N - 1;
                    const char *rp = static_cast<const char *>(sh.X) + (size_t)row * rb;
                    const char *qp = static_cast<const char *>(sh.Q) + (size_t)q * rb;
                    TileSum<T> part;
                    part.clear();
                    for (int s0 = 0; s0 < steps; s0 += 2) {
#pragma unroll
                        for (int u = 0; u < 2; ++u) {     // (an odd step past the end adds zeros)
                            const int ofs = (s0 + u) * 64 + kofs;
                            u4 x = zero_chunk(), y = zero_chunk();
                            if (ofs < rb) x = load_chunk(rp + ofs);
                            if (ofs < rb && (lane & 15) == 0) y = load_chunk(qp + ofs);
                            part.step(u, TileSum<T>::operand(x), TileSum<T>::operand(y));
                        }
                    }
                    const f4 acc = part.sum();
                    if (lane == quarter * 16) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int64_t id = tile * 16 + 4 * i + quarter;
                            float v = acc[i];
                            if (after.s) v = after_boundary(v, (int)id, after.s[q], after.id[q]);
                            ck[wave * 4 + i] = id < sh.N && v == v ? order_key(v, (int)id) : empty;
                        }
                    }
                } else if (lane < 4) {
                    ck[wave * 4 + lane] = empty;
                }
                __syncthreads();
                if (tid == 0) {
                    for (int c = 0; c < nwaves * 4; ++c) {
                        const uint64_t v = ck[c];
                        if (v <= fin[k - 1]) continue;
                        bool have = false;
                        for (int j = 0; j < k; ++j) have |= (uint32_t)fin[j] == (uint32_t)v;   // the id is listed already
                        if (have) continue;
                        int j = k - 1;
                        for (; j > 0 && fin[j - 1] < v; --j) fin[j] = fin[j - 1];
                        fin[j] = v;
                    }
                }
                __syncthreads();
            }
        }
    }
    if (tid < k) {
        float s;
        int id;
        order_key_decode(fin[tid], s, id);
        const bool has = id != EMPTY_ID;
        ids[(size_t)q * k + tid] = has ? id : -1;
        scores[(size_t)q * k + tid] = has ? s : -INFINITY;
    }
}

}  // namespace ann
