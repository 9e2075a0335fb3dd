// Priority levels and execution order of the request scheduler (Section 3.2, Eq. 1-2 of the
// paper): a small batched routine beside the retrieval kernels, O(n^2 / chip) comparisons for the n
// requests of a serving batch.
#include "launch.hpp"

namespace ann {

constexpr int PRIO_THREADS = 512;
constexpr int PRIO_WAVES = PRIO_THREADS / WAVE;

// One launch does it all; every workgroup computes the extremes and, for the requests it compares with, the
// levels again instead of waiting for another launch to do so (n is a serving batch: a few kilobytes from the L2,
// a few hundred instructions; a second launch costs more than either).
//
//   level_i = largest j in [0, G) with R_i > T_{R,j} or W_i > T_{W,j} or C_i > T_{C,j}, else 0,
//   T_{M,j} = min(M) + j/G (max(M) - min(M)), evaluated in binary64 exactly as written: the quotient,
//   the difference, their product and the sum are each rounded once (no fused multiply-add).
//   order[position of i] = i, position = number of requests that run before i: higher level first,
//   inside a level longer current queueing time first, equal times in index order; a queueing time
//   that is NaN counts as the shortest possible wait (-inf), so every request gets exactly one place.
//
// Workgroup b places the PRIO_TILE requests from b PRIO_TILE on: they sit in scalar registers, every thread holds one
// request at a time of the n to compare with and tests it against all of them, so the n^2 comparisons are spread
// over the whole chip instead of one thread walking all n; the comparisons are made on a 64-bit image of the
// queueing time that orders like the number.  n = 3000, G = 6: 300 us a call before (two launches, 290 of it the
// walk), 11.8 us now (8.4 for n = 32, the host's share of a call); n = 16384: 1590 -> 76 us, bound by the
// comparisons.
constexpr int PRIO_TILE = 16;

// order-preserving image of a queueing time (a NaN counts as -inf, -0 as +0)
__device__ __forceinline__ uint64_t wait_key(double w) {
    w = w == w ? w + 0.0 : -INFINITY;
    const uint64_t b = (uint64_t)__double_as_longlong(w);
    return (b >> 63) ? ~b : b | 0x8000000000000000ull;
}

// MANY (more than PRIO_FEW levels): a request's level is looked up instead of tried level by level, log2(G) steps per metric.  The thresholds of a
// metric never descend with j (j / G, the product with a difference that is not negative and the sum each round
// monotonically; where an extreme is infinite they are all infinite or all NaN), so the largest j passed is found by halving
// and the level is the largest over the three metrics.  Every workgroup looks at all n requests, so level by level costs
// n^2 G / 16 tests.  Level by level / halving, us: n = 256, G = 32 12.4 / 13.4, G = 64 17.4 / 14.8, G = 1024 161 / 20.6; n = 3000,
// G = 32 19.0 / 20.9, G = 64 27.5 / 23.2, G = 1024 285 / 34.4; n = 65 536, G = 32 1764 / 1659, G = 1024 33 100 / 3470.
constexpr int PRIO_FEW = 32;
template <bool MANY>
__global__ __launch_bounds__(PRIO_THREADS) void priority_kernel(const int32_t *__restrict__ R, const double *__restrict__ W,
                                                                const int32_t *__restrict__ C,
                                                                const double *__restrict__ Wcur, int n, int G,
                                                                int32_t *__restrict__ level, int32_t *__restrict__ order) {
    extern __shared__ __align__(16) unsigned char smem[];
    double *thr = reinterpret_cast<double *>(smem);                      // [G][3] thresholds
    __shared__ double part_w[2 * PRIO_WAVES];                            // a wave's smallest and largest W
    __shared__ int part_i[4];                                            // smallest R, C; largest R, C
    __shared__ uint64_t mine_w[PRIO_TILE];
    __shared__ int mine_l[PRIO_TILE], before[PRIO_TILE];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    if (tid < 2) { part_i[tid] = INT_MAX; part_i[2 + tid] = INT_MIN; }
    if (tid < PRIO_TILE) before[tid] = 0;
    __syncthreads();
    {
        int r0 = INT_MAX, r1 = INT_MIN, c0 = INT_MAX, c1 = INT_MIN;
        double w0 = INFINITY, w1 = -INFINITY;
        for (int b = tid; b < n; b += 8 * PRIO_THREADS) {                // eight requests' loads in flight per thread
            int r[8], c[8];
            double w[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = min(b + u * PRIO_THREADS, n - 1);
                r[u] = R[i]; w[u] = W[i]; c[u] = C[i];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                r0 = min(r0, r[u]); r1 = max(r1, r[u]);
                c0 = min(c0, c[u]); c1 = max(c1, c[u]);
                w0 = fmin(w0, w[u]); w1 = fmax(w1, w[u]);
            }
        }
        for (int m = 1; m < WAVE; m <<= 1) { w0 = fmin(w0, __shfl_xor(w0, m)); w1 = fmax(w1, __shfl_xor(w1, m)); }
        if (lane == 0) { part_w[wave] = w0; part_w[PRIO_WAVES + wave] = w1; }
        for (int m = 1; m < WAVE; m <<= 1) {
            r0 = min(r0, __shfl_xor(r0, m)); r1 = max(r1, __shfl_xor(r1, m));
            c0 = min(c0, __shfl_xor(c0, m)); c1 = max(c1, __shfl_xor(c1, m));
        }
        if (lane == 0) {
            atomicMin(&part_i[0], r0); atomicMin(&part_i[1], c0);
            atomicMax(&part_i[2], r1); atomicMax(&part_i[3], c1);
        }
    }
    __syncthreads();
    for (int e = tid; e < 3 * G; e += PRIO_THREADS) {                    // threshold j of metric m
        const int j = e / 3, m = e % 3;
        double mn, mx;
        if (m == 1) {
            mn = part_w[0];
            mx = part_w[PRIO_WAVES];
            for (int w = 1; w < PRIO_WAVES; ++w) { mn = fmin(mn, part_w[w]); mx = fmax(mx, part_w[PRIO_WAVES + w]); }
        } else {
            mn = (double)part_i[m >> 1];
            mx = (double)part_i[2 + (m >> 1)];
        }
        {
#pragma clang fp contract(off)                                          // (__dmul_rn and __dadd_rn do not keep the two from being fused)
            const double part = (double)j / (double)G * (mx - mn);
            thr[e] = mn + part;
        }
    }
    __syncthreads();
    // levels of NU requests at once: the thresholds are read once for all of them
    auto levels_of = [&](auto nu, const int *r, const double *w, const int *c, int *l) {
        constexpr int NU = decltype(nu)::value;
#pragma unroll
        for (int u = 0; u < NU; ++u) l[u] = 0;                           // (level 0 needs no threshold passed)
        if constexpr (MANY) {
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                int at[NU];
#pragma unroll
                for (int u = 0; u < NU; ++u) at[u] = 0;
                for (int h = 1 << (31 - __builtin_clz(G - 1)); h > 0; h >>= 1)
#pragma unroll
                    for (int u = 0; u < NU; ++u) {
                        const double x = m == 0 ? (double)r[u] : m == 1 ? w[u] : (double)c[u];
                        const int j = at[u] + h;
                        at[u] = j < G && x > thr[min(j, G - 1) * 3 + m] ? j : at[u];
                    }
#pragma unroll
                for (int u = 0; u < NU; ++u) l[u] = max(l[u], at[u]);
            }
            return;
        }
#pragma unroll 2
        for (int j = 1; j < G; ++j) {
            const double tr = thr[j * 3], tw = thr[j * 3 + 1], tc = thr[j * 3 + 2];
#pragma unroll
            for (int u = 0; u < NU; ++u) l[u] = (((double)r[u] > tr) | (w[u] > tw) | ((double)c[u] > tc)) ? j : l[u];
        }
    };
    const int i0 = blockIdx.x * PRIO_TILE, in = min(PRIO_TILE, n - i0);
    if (tid < PRIO_TILE) {
        const int i = min(i0 + tid, n - 1);
        const int r = R[i], c = C[i];
        const double w = W[i];
        int l;
        levels_of(std::integral_constant<int, 1>{}, &r, &w, &c, &l);
        mine_l[tid] = l;
        mine_w[tid] = wait_key(Wcur[i]);
        if (tid < in) level[i] = l;
    }
    __syncthreads();
    int ml[PRIO_TILE];                                                   // the tile, in scalar registers
    uint64_t mw[PRIO_TILE];
#pragma unroll
    for (int t = 0; t < PRIO_TILE; ++t) {
        ml[t] = __builtin_amdgcn_readfirstlane(mine_l[t]);
        mw[t] = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(mine_w[t] >> 32)) << 32 |
                (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)mine_w[t]);
    }
    uint32_t cnt[PRIO_TILE / 2];                                         // two counts of 16 bits: at most n / 8 a wave
#pragma unroll
    for (int t = 0; t < PRIO_TILE / 2; ++t) cnt[t] = 0;
    for (int b = tid; b < n; b += 4 * PRIO_THREADS) {
        int r[4], c[4];
        double w[4], q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = min(b + u * PRIO_THREADS, n - 1);
            r[u] = R[j]; w[u] = W[j]; c[u] = C[j]; q[u] = Wcur[j];
        }
        int l[4];
        levels_of(std::integral_constant<int, 4>{}, r, w, c, l);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = b + u * PRIO_THREADS;
            const int lj = j < n ? l[u] : -1;                            // (past the end: runs before nobody)
            // a request of lower index runs first at equal times: its image is compared with >= by adding one
            const uint64_t wj = wait_key(q[u]) + (j < i0 ? 1u : 0u);
#pragma unroll
            for (int t = 0; t < PRIO_TILE; ++t)
                cnt[t >> 1] += ((lj > ml[t]) | ((lj == ml[t]) & (wj > mw[t]))) ? 1u << (16 * (t & 1)) : 0u;
        }
    }
    // sums over the wave: every step halves the counts a lane keeps, then the lanes that keep the same ones add up
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const int half = PRIO_TILE / 4 >> s;
        const bool upper = (lane >> s) & 1;
#pragma unroll
        for (int t = 0; t < half; ++t) {
            const uint32_t keep = upper ? cnt[t + half] : cnt[t], give = upper ? cnt[t] : cnt[t + half];
            cnt[t] = keep + (uint32_t)__shfl_xor((int)give, 1 << s);
        }
    }
    uint32_t c = cnt[0];
    c += (uint32_t)__shfl_xor((int)c, 8);
    c += (uint32_t)__shfl_xor((int)c, 16);
    c += (uint32_t)__shfl_xor((int)c, 32);
    if (lane < 8) {                                                      // lane's bits 0, 1, 2 chose halves of 4, 2, 1 words
        const int t = 2 * ((lane & 1) * 4 + (lane & 2) + (lane >> 2));
        atomicAdd(&before[t], (int)(c & 0xffffu));
        atomicAdd(&before[t + 1], (int)(c >> 16));
    }
    if (tid < in) {                                                      // equal times inside the tile
        int e = 0;
        for (int t = 0; t < tid; ++t) e += (int)(mine_l[t] == mine_l[tid]) & (int)(mine_w[t] == mine_w[tid]);
        atomicAdd(&before[tid], e);
    }
    __syncthreads();
    if (tid < in) order[before[tid]] = i0 + tid;
}

hipError_t launch_priority(const int32_t *R, const double *W, const int32_t *C, const double *Wcur, int n, int G,
                           int32_t *level, int32_t *order, hipStream_t stream) {
    hipLaunchKernelGGL((G > PRIO_FEW ? priority_kernel<true> : priority_kernel<false>), dim3((n + PRIO_TILE - 1) / PRIO_TILE), dim3(PRIO_THREADS), (size_t)G * 3 * sizeof(double),
                       stream, R, W, C, Wcur, n, G, level, order);
    return hipGetLastError();
}

}  // namespace ann
