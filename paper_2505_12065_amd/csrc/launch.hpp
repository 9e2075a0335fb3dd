// Host-side launchers of the kernels; one translation unit per kernel family so the
// library builds in parallel.  Each returns the HIP status of its launch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"

namespace ann {

constexpr size_t LDS_MAX = 160 * 1024;   // LDS of one gfx950 compute unit
// Wavefronts of a flat_stream_kernel workgroup: 8, or 16 when the queries' LDS leaves room for one
// workgroup per compute unit only (the corpus loads in flight are what keeps HBM busy).
int stream_waves(int elem_bytes, int nqg, int lds_steps);

// A kernel that needs more than 64 KB of dynamic LDS has to be told so; `granted` holds
// the largest size already granted to that kernel.
inline hipError_t allow_big_lds(const void *kernel, size_t bytes, size_t *granted) {
    if (bytes <= 64 * 1024 || bytes <= *granted) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) *granted = bytes;
    return e;
}

constexpr int STREAM_NQG_MAX(int elem_bytes) { return elem_bytes == 2 ? 4 : 2; }   // fp32: eight accumulators a group
constexpr int STREAM_WG_PER_CU(int elem_bytes, int nqg, int waves) { return waves == 16 || (elem_bytes == 4 && nqg > 1) ? 1 : 2; }
size_t stream_lds_bytes(int nqg, int lds_steps, int waves);

// Geometry and options of a flat_stream_kernel launch.
struct StreamPlan {
    int nqg = 1;                 // groups of 16 queries a workgroup serves, 1 .. STREAM_NQG_MAX
    int G = 1;                   // workgroups side by side over the queries, ceil(B / (16 nqg))
    int P = 1;                   // slabs of the corpus
    int waves = 8;               // wavefronts per workgroup
    int lds_steps = 1;           // 64-byte steps of a query held in LDS
    int K = 4;                   // entries of a slab's list: k rounded up to a multiple of 4
    int slots() const { return P * waves; }
};
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
// Large batches on the matrix cores (16-bit corpora).
constexpr int WIDE_LARGE = 0, WIDE_TALL = 1, WIDE_SMALL = 2, WIDE_THIN = 3, WIDE_TINY = 4;
struct WidePlan {
    int cus, shape, wmf;         // compute units; workgroup tile (a WideCfg); its row fragments per wave
    int NT, P;                   // query tiles x slabs of the corpus
    int gs_log;                  // a maximum stands for 2^gs_log rows
    int64_t slots, n;            // rows of whole tiles; groups they make
};
void wide_geometry(WidePlan &pl, int shape, int cus, int64_t N, int B);
// maxima [B, pl.n]
hipError_t launch_flat_wide(const WidePlan &pl, int dtype, const void *X, int64_t N, int d, const void *Q, int B, float *maxima,
                            After after, hipStream_t stream);
hipError_t launch_flat_pick(const WidePlan &pl, int dtype, const void *X, int64_t N, int d, const void *Q, int B, int k,
                            const float *maxima, int32_t *ids, float *scores, After after, hipStream_t stream);
// k <= 4: merge the P lists of 4 of every query.
hipError_t launch_flat_merge(const Cand *partial, int P, int B, int k, int32_t *ids, float *scores, hipStream_t stream);
// k > 4: merge the P lists of K of every query, made by flat_stream_kernel with `slots` = P waves.
hipError_t launch_flat_merge_lists(int dtype, const Cand *partial, int P, int K, int slots, const void *X, int64_t N, int d,
                                   const void *Q, int B, int k, int32_t *ids, float *scores, After after, hipStream_t stream);

constexpr int GRAPH_DENSE_MIN_B = 1280;   // batches beyond this run three graph-search workgroups per compute unit
constexpr int GRAPH_EF_DOUBLE = 2048;    // candidate lists up to this length are double-buffered in LDS
constexpr int GRAPH_EF_TWO_LEVEL = 512;  // beyond this, graphs of at most 32 slots per node use the two-level list
// cus workgroups of 8 waves, each wave iters x 8 MFMA 32x32x16 fp16 (32768 flop each) on register operands
hipError_t launch_mfma_rate(bool random_operands, int cus, int iters, float *sink, hipStream_t stream);

struct GraphLds {
    // byte offsets into dynamic LDS; all 16-byte aligned
    uint32_t q, ls0, ls1, li0, li1, cs, ci, cpos, cache, ctl, adj, um, rq, co, total;
    uint32_t cache_bits, rp;
    // two-level list (search ranges beyond GRAPH_EF_TWO_LEVEL on graphs of at most 32 slots per node):
    // ms / mi hold the large part of the list, ls0 .. li1 the small part (GRAPH_DELTA entries each)
    uint32_t two_level, ms, mi;
};
constexpr int GRAPH_DELTA = 256;
// The two-level layout keeps its small regions at fixed byte offsets at the start of LDS (the kernel
// then addresses them with immediates and needs no register per region); the large part of the
// list and the query, whose sizes depend on ef and d, follow.
constexpr uint32_t TL_LS0 = 0, TL_LI0 = 4 * GRAPH_DELTA, TL_LS1 = 8 * GRAPH_DELTA, TL_LI1 = 12 * GRAPH_DELTA;
constexpr uint32_t TL_CS = 16 * GRAPH_DELTA, TL_CI = TL_CS + 128, TL_CPOS = TL_CI + 128, TL_CTL = TL_CPOS + 128;
constexpr uint32_t TL_ADJ = TL_CTL + 32, TL_UM = TL_ADJ + 256;
constexpr uint32_t TL_MS = TL_UM + 8 * (16384 / 64) + 32;   // um: a bit per entry of the longest list, and 4 words
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
GraphLds graph_lds_layout(int d, int elem_bytes, int R, int ef);

// words of one query's visited bitset: one bit per node, rounded to 64-byte units
inline int64_t visited_words(int64_t N) { return (N + 511) / 512 * 16; }

// graph_step_kernel (graphs of at most 32 slots per node): how it runs a call, and its LDS
constexpr int GRAPH_STEP_MAX_R = 32;
constexpr int STEP_VIS_LDS = 0, STEP_VIS_CACHE = 1, STEP_VIS_GLOBAL = 2;   // where the visited set is
struct StepLds {
    // fixed byte offsets: scores, ids, positions, numbers of a step's neighbours (64 each), control words, then the scratch
    // of every wave
    static constexpr uint32_t CS = 0, CI = 256, CP = 512, EV = 768, EW = 1024, FM = 1280, CTL = 1312, MK = 1328,
                              WAVE0 = 1456, WAVE_BYTES = 576;
    // byte offsets: list scores and ids (two buffers of ls_bytes each), and for long lists the large part and its bits
    uint32_t ls, li, ls_bytes, um, ms, mi, vis, q, total;
    int vis_words, cache_shift, vis_mode;
    int rows_per_group;                                   // neighbours a row group scores in a step: 1 or 2
    bool dense;                                           // three workgroups per compute unit, query read from LDS
    bool long_list;
};
// whether a call runs in steps of several expansions (graph_step_kernel) or one by one (graph_search_kernel)
bool graph_step_pays(int cus, int row_bytes, int R, int B, int ef, bool counters, float tau);
// counters: the call needs an exact visited set (maturity exit)
StepLds graph_step_plan(int cus, int64_t N, int d, int elem_bytes, int B, int ef, bool counters);
hipError_t launch_graph_step(int dtype, const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const void *Q,
                             int B, int k, int ef, int32_t *ids, float *scores, const StepLds &L, bool counters,
                             const NonStall &ns, hipStream_t stream);
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
