// Priority levels and execution order of the request scheduler (Section 3.2, Eq. 1-2 of the
// paper): a small batched routine beside the retrieval kernels, O(n^2 / chip) comparisons for the n
// requests of a serving batch.
#include "launch.hpp"

namespace ann {
namespace {
// x over all lanes of the wave by op
template <class Op>
__device__ __forceinline__ int wave_reduce(int x, Op op) {
    x = op(x, (int)lane_swap<1>((uint32_t)x));
    x = op(x, (int)lane_swap<2>((uint32_t)x));
    x = op(x, (int)lane_swap<4>((uint32_t)x));
    x = op(x, (int)lane_swap<8>((uint32_t)x));
    uint32_t a, b;
    row_pair<16>((uint32_t)x, a, b);
    row_pair<32>((uint32_t)op((int)a, (int)b), a, b);
    return op((int)a, (int)b);
}
template <class Op>
__device__ __forceinline__ double wave_reduce(double x, Op op) {
    auto swapped = [](double v, auto mc) {
        constexpr int M = decltype(mc)::value;
        const uint64_t b = (uint64_t)__double_as_longlong(v);
        return __longlong_as_double((long long)((uint64_t)lane_swap<M>((uint32_t)(b >> 32)) << 32 | lane_swap<M>((uint32_t)b)));
    };
    x = op(x, swapped(x, std::integral_constant<int, 1>{}));
    x = op(x, swapped(x, std::integral_constant<int, 2>{}));
    x = op(x, swapped(x, std::integral_constant<int, 4>{}));
    x = op(x, swapped(x, std::integral_constant<int, 8>{}));
    auto rows = [&](auto mc) {
        constexpr int M = decltype(mc)::value;
        const uint64_t v = (uint64_t)__double_as_longlong(x);
        uint32_t l0, l1, h0, h1;
        row_pair<M>((uint32_t)v, l0, l1);
        row_pair<M>((uint32_t)(v >> 32), h0, h1);
        x = op(__longlong_as_double((long long)((uint64_t)h0 << 32 | l0)), __longlong_as_double((long long)((uint64_t)h1 << 32 | l1)));
    };
    rows(std::integral_constant<int, 16>{});
    rows(std::integral_constant<int, 32>{});
    return x;
}

// cnt += (level, wait) > (ml, mw), both read as one number of 96 bits: the borrow of a subtraction, four instructions
// (a carry takes the one scalar operand that an instruction may have, so all but the lowest word of the tile's are vectors)
__device__ __forceinline__ void count_larger(uint32_t &cnt, uint32_t level, uint64_t wait, uint32_t ml, uint64_t mw) {
    uint32_t t;
    asm("v_sub_co_u32_e32 %0, vcc, %2, %3\n\t"
        "v_subb_co_u32_e32 %0, vcc, %4, %5, vcc\n\t"
        "v_subb_co_u32_e32 %0, vcc, %6, %7, vcc\n\t"
        "v_addc_co_u32_e32 %1, vcc, 0, %1, vcc"
        : "=&v"(t), "+v"(cnt)
        : "s"((uint32_t)mw), "v"((uint32_t)wait), "v"((uint32_t)(mw >> 32)), "v"((uint32_t)(wait >> 32)), "v"(ml), "v"(level)
        : "vcc");
}
}  // namespace

constexpr int PRIO_THREADS = 512;
constexpr int PRIO_WAVES = PRIO_THREADS / WAVE;

// One launch does it all; every workgroup computes the extremes and, for the requests it compares with, the
// levels again instead of waiting for another launch to do so: of a serving batch that is a few kilobytes from the L2 and
// a few hundred instructions.
//
//   level_i = largest j in [0, G) with R_i > T_{R,j} or W_i > T_{W,j} or C_i > T_{C,j}, else 0,
//   T_{M,j} = min(M) + j/G (max(M) - min(M)), evaluated in binary64 exactly as written: the quotient,
//   the difference, their product and the sum are each rounded once (no fused multiply-add).
//   order[position of i] = i, position = number of requests that run before i: higher level first,
//   inside a level longer current queueing time first, equal times in index order; a queueing time
//   that is NaN counts as the shortest possible wait (-inf), so every request gets exactly one place.
//
// Workgroup b places the PRIO_TILE requests from b PRIO_TILE on: every thread holds one request at a time of the n to compare
// with and tests it against all of them, so the n^2 comparisons are spread over the whole chip instead of one thread walking
// all n.  A level and a 64-bit image of the queueing time that orders like the number are compared as one number of 96 bits.
// Bound by latency up to some 3000 requests: one read, what a thread reads is kept (a second one cost 0.5 us), reductions
// that stay out of the LDS crossbar, three barriers; beyond that by the comparisons and the levels that every workgroup
// computes again.  us of a call, one thread walking all n (two launches) / read twice, 8 instructions a comparison / now, 4 of them:
// n = 3000, G = 6 300 / 11.8 / 7.1 (HELD, below), n = 16384 1590 / 76 / 69.
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
// n^2 G / 16 tests.  The three metrics are halved side by side, without a branch: a request's reads of a step are in flight together,
// twelve a thread (one metric after the other, each read waited for: n = 3000, G = 64 20.2 us, now 12.1; n = 65 536, G = 256 2870,
// now 1990).  Level by level / halving, us: n = 16, G = 20 7.4 / 6.9, G = 22 7.7 / 6.9, G = 32 9.0 / 6.9; n = 3000, G = 20
// 11.7 / 11.2, G = 22 12.3 / 11.2, G = 32 15.2 / 11.2; n = 65 536, G = 20 1405 / 1430, G = 22 1479 / 1430, G = 32 1826 / 1430.
constexpr int PRIO_FEW = 20;
// HELD: requests that a thread keeps from the extremes to the comparisons.  ONCE: they are all that there are, and what no thread of
// the workgroup has is left out, by a test that calls of several batches would pay for (n = 65 536 938 / 953): n = 1000, G = 6 5.94 / 5.32,
// n = 256 5.97 / 5.54, two held instead of four.  Four of them, read in two batches of which the second is half empty, against six, us: n = 2049, G = 6 7.62 / 6.90, n = 3000, G = 6 8.26 / 7.13, G = 13
// 10.04 / 8.28, G = 32 11.25 / 10.54.  Six cost smaller calls more than they skip (n = 2048 6.02 / 6.58), eight larger ones (n = 4096 8.33 / 8.37, n = 2500 6.89 / 7.48).
template <bool MANY, int HELD, bool ONCE>
__global__ __launch_bounds__(PRIO_THREADS) void priority_kernel(const int32_t *__restrict__ R, const double *__restrict__ W,
                                                                const int32_t *__restrict__ C,
                                                                const double *__restrict__ Wcur, int n, int G,
                                                                int32_t *__restrict__ level, int32_t *__restrict__ order) {
    extern __shared__ __align__(16) unsigned char smem[];
    double *thr = reinterpret_cast<double *>(smem);                      // [G][3] thresholds
    __shared__ double part_w[2][PRIO_WAVES];                             // a wave's smallest and largest W
    __shared__ int part_i[4][PRIO_WAVES];                                // smallest R, C; largest R, C
    __shared__ uint64_t mine_w[PRIO_TILE];
    __shared__ int mine_l[PRIO_TILE], before[PRIO_TILE];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    const int i0 = blockIdx.x * PRIO_TILE, in = min(PRIO_TILE, n - i0);
    if (tid < PRIO_TILE) before[tid] = 0;
    // The tile's requests and the first HELD of a thread are loaded once, together.
    const int own = min(i0 + (tid & (PRIO_TILE - 1)), n - 1);
    const int own_r = R[own], own_c = C[own];
    const double own_w = W[own], own_q = Wcur[own];
    int r[HELD], c[HELD];
    double w[HELD], q[HELD];
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
        const int i = min(tid + u * PRIO_THREADS, n - 1);
        r[u] = R[i]; w[u] = W[i]; c[u] = C[i];
    }
#pragma unroll
    for (int u = 0; u < HELD; ++u) q[u] = Wcur[min(tid + u * PRIO_THREADS, n - 1)];
    {
        int r0 = r[0], r1 = r[0], c0 = c[0], c1 = c[0];
        double w0 = INFINITY, w1 = -INFINITY;
#pragma unroll
        for (int u = 0; u < HELD; ++u) {
            r0 = min(r0, r[u]); r1 = max(r1, r[u]);
            c0 = min(c0, c[u]); c1 = max(c1, c[u]);
            w0 = fmin(w0, w[u]); w1 = fmax(w1, w[u]);
        }
        for (int b = tid + HELD * PRIO_THREADS; !ONCE && b < n; b += HELD * PRIO_THREADS) {
            int br[HELD], bc[HELD];
            double bw[HELD];
#pragma unroll
            for (int u = 0; u < HELD; ++u) {
                const int i = min(b + u * PRIO_THREADS, n - 1);
                br[u] = R[i]; bw[u] = W[i]; bc[u] = C[i];
            }
#pragma unroll
            for (int u = 0; u < HELD; ++u) {
                r0 = min(r0, br[u]); r1 = max(r1, br[u]);
                c0 = min(c0, bc[u]); c1 = max(c1, bc[u]);
                w0 = fmin(w0, bw[u]); w1 = fmax(w1, bw[u]);
            }
        }
        auto least = [](auto a, auto b) { return a < b ? a : b; };
        auto most = [](auto a, auto b) { return a > b ? a : b; };
        r0 = wave_reduce(r0, least); r1 = wave_reduce(r1, most);
        c0 = wave_reduce(c0, least); c1 = wave_reduce(c1, most);
        w0 = wave_reduce(w0, [](double a, double b) { return fmin(a, b); });
        w1 = wave_reduce(w1, [](double a, double b) { return fmax(a, b); });
        if (lane == 0) {
            part_w[0][wave] = w0; part_w[1][wave] = w1;
            part_i[0][wave] = r0; part_i[1][wave] = c0;
            part_i[2][wave] = r1; part_i[3][wave] = c1;
        }
    }
    __syncthreads();
    for (int e = tid; e < 3 * G; e += PRIO_THREADS) {                    // threshold j of metric m
        const int j = e / 3, m = e % 3;
        double mn, mx;
        if (m == 1) {
            mn = part_w[0][0];
            mx = part_w[1][0];
#pragma unroll
            for (int v = 1; v < PRIO_WAVES; ++v) { mn = fmin(mn, part_w[0][v]); mx = fmax(mx, part_w[1][v]); }
        } else {
            int lo = part_i[m >> 1][0], hi = part_i[2 + (m >> 1)][0];
#pragma unroll
            for (int v = 1; v < PRIO_WAVES; ++v) { lo = min(lo, part_i[m >> 1][v]); hi = max(hi, part_i[2 + (m >> 1)][v]); }
            mn = (double)lo;
            mx = (double)hi;
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
            int at[3][NU];                                               // a request's three chains of reads side by side
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int u = 0; u < NU; ++u) at[m][u] = 0;
            for (int h = 1 << (31 - __builtin_clz(G - 1)); h > 0; h >>= 1) {
#pragma unroll
                for (int m = 0; m < 3; ++m)
#pragma unroll
                    for (int u = 0; u < NU; ++u) {
                        const double x = m == 0 ? (double)r[u] : m == 1 ? w[u] : (double)c[u];
                        const int j = at[m][u] + h;
                        at[m][u] = (j < G) & (x > thr[min(j, G - 1) * 3 + m]) ? j : at[m][u];
                    }
            }
#pragma unroll
            for (int u = 0; u < NU; ++u) l[u] = max(max(at[0][u], at[1][u]), at[2][u]);
            return;
        }
#pragma unroll 2
        for (int j = 1; j < G; ++j) {
            const double tr = thr[j * 3], tw = thr[j * 3 + 1], tc = thr[j * 3 + 2];
#pragma unroll
            for (int u = 0; u < NU; ++u) l[u] = (((double)r[u] > tr) | (w[u] > tw) | ((double)c[u] > tc)) ? j : l[u];
        }
    };
    if (tid < PRIO_TILE) {
        int l;
        levels_of(std::integral_constant<int, 1>{}, &own_r, &own_w, &own_c, &l);
        mine_l[tid] = l;
        mine_w[tid] = wait_key(own_q);
        if (tid < in) level[own] = l;
    }
    __syncthreads();
    uint32_t ml[PRIO_TILE];                                              // the tile; levels from 1 on
    uint64_t mw[PRIO_TILE];
#pragma unroll
    for (int t = 0; t < PRIO_TILE; ++t) {
        ml[t] = (uint32_t)mine_l[t] + 1;
        mw[t] = (mine_w[t] >> 32) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)mine_w[t]);
    }
    uint32_t count[PRIO_TILE];
#pragma unroll
    for (int t = 0; t < PRIO_TILE; ++t) count[t] = 0;
    for (int b = tid; b < n; b += HELD * PRIO_THREADS) {
        int l[HELD];
        levels_of(std::integral_constant<int, HELD>{}, r, w, c, l);
#pragma unroll
        for (int u = 0; u < HELD; ++u) {
            const int j = b + u * PRIO_THREADS;
            if (ONCE && u * PRIO_THREADS >= n) break;                     // (nothing left for any thread)
            const uint32_t lj = j < n ? (uint32_t)l[u] + 1 : 0u;         // (past the end: runs before nobody)
            // a request of lower index runs first at equal times: its image is compared with >= by adding one
            const uint64_t wj = wait_key(q[u]) + (j < i0 ? 1u : 0u);
#pragma unroll
            for (int t = 0; t < PRIO_TILE; ++t) count_larger(count[t], lj, wj, ml[t], mw[t]);
        }
        if (!ONCE && b + HELD * PRIO_THREADS < n) {
#pragma unroll
            for (int u = 0; u < HELD; ++u) {
                const int i = min(b + (HELD + u) * PRIO_THREADS, n - 1);
                r[u] = R[i]; w[u] = W[i]; c[u] = C[i]; q[u] = Wcur[i];
            }
        }
    }
    uint32_t cnt[PRIO_TILE / 2];                                         // two counts of 16 bits: at most n / 8 a wave
#pragma unroll
    for (int t = 0; t < PRIO_TILE / 2; ++t) cnt[t] = count[2 * t] | count[2 * t + 1] << 16;
    // sums over the wave: every step halves the counts a lane keeps, then the lanes that keep the same ones add up
    auto halve = [&](auto sc) {
        constexpr int S = decltype(sc)::value, half = PRIO_TILE / 4 >> S;
        const bool upper = (lane >> S) & 1;
#pragma unroll
        for (int t = 0; t < half; ++t) {
            const uint32_t keep = upper ? cnt[t + half] : cnt[t], give = upper ? cnt[t] : cnt[t + half];
            cnt[t] = keep + lane_swap<1 << S>(give);
        }
    };
    halve(std::integral_constant<int, 0>{});
    halve(std::integral_constant<int, 1>{});
    halve(std::integral_constant<int, 2>{});
    uint32_t sum = cnt[0] + lane_swap<8>(cnt[0]), sa, sb;
    row_pair<16>(sum, sa, sb);
    row_pair<32>(sa + sb, sa, sb);
    sum = sa + sb;
    if (lane < 8) {                                                      // lane's bits 0, 1, 2 chose halves of 4, 2, 1 words
        const int t = 2 * ((lane & 1) * 4 + (lane & 2) + (lane >> 2));
        atomicAdd(&before[t], (int)(sum & 0xffffu));
        atomicAdd(&before[t + 1], (int)(sum >> 16));
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
    auto go = [&](auto held, auto once) {
        constexpr int HELD = decltype(held)::value;
        constexpr bool ONCE = decltype(once)::value;
        hipLaunchKernelGGL((G > PRIO_FEW ? priority_kernel<true, HELD, ONCE> : priority_kernel<false, HELD, ONCE>), dim3((n + PRIO_TILE - 1) / PRIO_TILE),
                           dim3(PRIO_THREADS), (size_t)G * 3 * sizeof(double), stream, R, W, C, Wcur, n, G, level, order);
        return hipGetLastError();
    };
    if (n <= 2 * PRIO_THREADS) return go(std::integral_constant<int, 2>{}, std::true_type{});
    if (n <= 4 * PRIO_THREADS) return go(std::integral_constant<int, 4>{}, std::true_type{});
    if (n <= 6 * PRIO_THREADS) return go(std::integral_constant<int, 6>{}, std::true_type{});
    return go(std::integral_constant<int, 4>{}, std::false_type{});
}

}  // namespace ann
