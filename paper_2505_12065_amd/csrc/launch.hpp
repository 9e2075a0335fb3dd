// Host-side launchers of the kernels; one translation unit per kernel family so the
// library builds in parallel.  Each returns the HIP status of its launch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"
#include "plan.hpp"

namespace ann {

// A kernel that needs more than 64 KB of dynamic LDS has to be told so; `granted` holds
// the largest size already granted to that kernel.
inline hipError_t allow_big_lds(const void *kernel, size_t bytes, size_t *granted) {
    if (bytes <= 64 * 1024 || bytes <= *granted) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) *granted = bytes;
    return e;
}

// Where a single slab's lists go instead of to `partial`: the answer itself (ids null: they do not).
struct StreamOut {
    int32_t *ids = nullptr;
    float *scores = nullptr;
    int k = 0;
};

// partial[B, P, K]: every slab's best K per query; or maxima [B, n]: see the kernel; or, one slab only, `out`.
hipError_t launch_flat_stream_f16(const StreamPlan &pl, const void *X, int64_t N, int d, const void *Q, int B, Cand *partial,
                                  float *maxima, int64_t n, StreamOut out, After after, hipStream_t stream);
hipError_t launch_flat_stream_bf16(const StreamPlan &pl, const void *X, int64_t N, int d, const void *Q, int B, Cand *partial,
                                  float *maxima, int64_t n, StreamOut out, After after, hipStream_t stream);
hipError_t launch_flat_stream_f32(const StreamPlan &pl, const void *X, int64_t N, int d, const void *Q, int B, Cand *partial,
                                  float *maxima, int64_t n, StreamOut out, After after, hipStream_t stream);
// All scores of few queries and few rows: maxima [B, n].
hipError_t launch_flat_scores(int dtype, const void *X, int64_t N, int d, const void *Q, int B, float *maxima, int64_t n, After after,
                              hipStream_t stream);
// N <= DIRECT_ROWS: the answer.
hipError_t launch_flat_direct(int dtype, const void *X, int64_t N, int d, const void *Q, int B, int k, int32_t *ids, float *scores,
                              After after, hipStream_t stream);
// Large batches on the matrix cores (16-bit corpora): maxima [B, pl.n].
hipError_t launch_flat_wide(const WidePlan &pl, int dtype, const void *X, int64_t N, int d, const void *Q, int B, float *maxima,
                            After after, hipStream_t stream);
hipError_t launch_flat_pick(const WidePlan &pl, int dtype, const void *X, int64_t N, int d, const void *Q, int B, int k,
                            const float *maxima, int32_t *ids, float *scores, After after, uint64_t *best, int more,
                            hipStream_t stream);
// k <= 4: merge the P lists of 4 of every query.
hipError_t launch_flat_merge(const Cand *partial, int P, int B, int k, int32_t *ids, float *scores, hipStream_t stream);
// k > 4: merge the P lists of K of every query, made by flat_stream_kernel with `slots` = P waves.
hipError_t launch_flat_merge_lists(int dtype, const Cand *partial, int P, int K, int slots, const void *X, int64_t N, int d,
                                   const void *Q, int B, int k, int32_t *ids, float *scores, After after, hipStream_t stream);

// cus workgroups of 8 waves, each wave iters x 8 MFMA 32x32x16 fp16 (32768 flop each) on register operands
hipError_t launch_mfma_rate(bool random_operands, int cus, int iters, float *sink, hipStream_t stream);

// Maturity exit of the graph search (Section 3.3, Appendix B.2): leave once the moving
// average of RQ exceeds tau and *ready != 0 (ready == nullptr: always ready).
struct NonStall {
    const int32_t *entries;   // [B, n_entries] per-query entry nodes replacing `entry`, or null (both kernel variants)
    int32_t n_entries;        // 1 .. 32 when entries is given
    float tau, alpha;
    const int32_t *ready;     // device-visible word the host may change while the kernel runs
    uint32_t *visited;        // [B][words] bitset, zero on entry
    int64_t words;            // words per query, a multiple of 4
    int32_t *stats;           // [B][3] = (early exit, scored nodes, expansions), may be null
    float *ema;               // [B] final moving average, may be null
};
// dtype: ANN_F16 / ANN_BF16 / ANN_F32 codes 0 / 1 / 2
// graph_frontier_kernel, the search of most calls on graphs of at most 32 slots per node.  counters: with the maturity exit and
// its counters; else only the entry nodes of `ns` and, where the visited set is in memory, that.
struct FrontierArgs {
    const void *X;            // [N, d]
    int64_t N;
    int d, R;
    const int32_t *graph;     // [N, R]
    const void *Q;            // [B, d]
    int entry, k, ef;
    int32_t *ids;             // [B, k]
    float *scores;
    FrontierLds L;
    NonStall ns;
};
hipError_t launch_graph_frontier(int dtype, int B, const FrontierArgs &args, bool counters, hipStream_t stream);
// Steps of several expansions on a list in LDS, with an id cache: short lists without counters.
hipError_t launch_graph_step(int dtype, const void *X, int64_t N, int d, const int32_t *graph, int R, int entry,
                             const int32_t *entries, int n_entries, const void *Q, int B, int k, int ef, int32_t *ids, float *scores,
                             const StepLds &L, hipStream_t stream);
// dtype: ANN_F16 / ANN_BF16 / ANN_F32 codes 0 / 1 / 2
// entries: null, or device [B, n_entries] per-query entry nodes used instead of `entry`
hipError_t launch_graph_search(int dtype, const void *X, int64_t N, int d, const int32_t *graph, int R, int entry,
                               const int32_t *entries, int n_entries, const void *Q, int B, int k, int ef, int32_t *ids,
                               float *scores, const GraphLds &L, hipStream_t stream);
hipError_t launch_gather_ids(const int32_t *table, int64_t M, const int32_t *idx, int64_t n, int32_t *out,
                             hipStream_t stream);
// p[0 .. words) <- 0; words a multiple of 4, p 16-byte aligned
hipError_t launch_zero_words(uint32_t *p, size_t words, hipStream_t stream);
// Same with the maturity exit; ns.visited (B * ns.words words) must be zero.
hipError_t launch_graph_search_nonstall(int dtype, const void *X, int64_t N, int d, const int32_t *graph, int R,
                                        int entry, const void *Q, int B, int k, int ef, int32_t *ids, float *scores,
                                        const GraphLds &L, const NonStall &ns, hipStream_t stream);

// Scheduler priority levels (Section 3.2, Eq. 1-2) and execution order; all arrays device, length n.
hipError_t launch_priority(const int32_t *R, const double *W, const int32_t *C, const double *Wcur, int n, int G,
                           int32_t *level, int32_t *order, hipStream_t stream);

}  // namespace ann
