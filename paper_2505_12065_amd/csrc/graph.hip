// graph_search_kernel: instantiations and launcher.
#include "graph_kernel.hpp"

namespace ann {

// out[i] <- table[idx[i]], or -1 where idx[i] is not in [0, M)
__global__ __launch_bounds__(256) void gather_ids_kernel(const int32_t *__restrict__ table, int64_t M,
                                                         const int32_t *__restrict__ idx, int64_t n,
                                                         int32_t *__restrict__ out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t j = idx[i];
        out[i] = (j >= 0 && j < M) ? table[j] : -1;
    }
}

// words[0 .. n) <- 0, 16 bytes per store (n a multiple of 4)
__global__ __launch_bounds__(256) void zero_words_kernel(u4 *__restrict__ p, size_t n16) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        p[i] = zero_chunk();
}

#define ANN_STEP_ARGS \
    const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const int32_t *entries, int n_entries, const void *Q, int B, \
        int k, int ef, int32_t *ids, float *scores, const StepLds &L, hipStream_t stream
hipError_t launch_graph_step_f16(ANN_STEP_ARGS);
hipError_t launch_graph_step_bf16(ANN_STEP_ARGS);
hipError_t launch_graph_step_f32(ANN_STEP_ARGS);

hipError_t launch_graph_step(int dtype, ANN_STEP_ARGS) {
    return (dtype == 0 ? launch_graph_step_f16 : dtype == 1 ? launch_graph_step_bf16 : launch_graph_step_f32)(
        X, N, d, graph, R, entry, entries, n_entries, Q, B, k, ef, ids, scores, L, stream);
}
#undef ANN_STEP_ARGS

hipError_t launch_graph_frontier_f16(int, const FrontierArgs &, bool, hipStream_t);
hipError_t launch_graph_frontier_bf16(int, const FrontierArgs &, bool, hipStream_t);
hipError_t launch_graph_frontier_f32(int, const FrontierArgs &, bool, hipStream_t);

hipError_t launch_graph_frontier(int dtype, int B, const FrontierArgs &args, bool counters, hipStream_t stream) {
    return (dtype == 0 ? launch_graph_frontier_f16 : dtype == 1 ? launch_graph_frontier_bf16 : launch_graph_frontier_f32)(B, args, counters,
                                                                                                                         stream);
}

namespace {
template <class T, int RPT, bool NS, bool QREG = true, bool LONG = false>
hipError_t launch_rp(const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const void *Q, int B,
                     int k, int ef, int32_t *ids, float *scores, const GraphLds &L, const NonStall &ns,
                     hipStream_t stream) {
    static size_t big = 0;
    if (hipError_t e = allow_big_lds(reinterpret_cast<const void *>(&graph_search_kernel<T, RPT, NS, QREG, LONG>), L.total, &big))
        return e;
    hipLaunchKernelGGL((graph_search_kernel<T, RPT, NS, QREG, LONG>), dim3(B), dim3(GRAPH_THREADS), L.total, stream, X, N, d,
                       graph, R, entry, Q, k, ef, ids, scores, L, ns);
    return hipGetLastError();
}

template <class T, bool NS>
hipError_t launch(const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const void *Q, int B,
                  int k, int ef, int32_t *ids, float *scores, const GraphLds &L, const NonStall &ns,
                  hipStream_t stream) {
    // More queries than two workgroups per compute unit hold at once, and a layout small enough for
    // three: the variant that reads the query from LDS and runs three per compute unit.
    if constexpr (!NS) {
        if (L.rp == 32 && B > GRAPH_DENSE_MIN_B && 3 * (size_t)L.total + 3 * 1024 <= LDS_MAX)
            return launch_rp<T, 32, false, false>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
    }
    if constexpr (NS) {
        if (L.two_level)
            return launch_rp<T, 32, true, true, true>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
    } else if (L.two_level) {
        return hipErrorInvalidValue;                      // long lists run with the exact visited set
    }
    return L.rp == 32 ? launch_rp<T, 32, NS>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream)
                      : launch_rp<T, 0, NS>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
}

template <bool NS>
hipError_t launch_dtype(int dtype, const void *X, int64_t N, int d, const int32_t *graph, int R, int entry,
                        const void *Q, int B, int k, int ef, int32_t *ids, float *scores, const GraphLds &L,
                        const NonStall &ns, hipStream_t stream) {
    switch (dtype) {
    case 0: return launch<F16, NS>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
    case 1: return launch<BF16, NS>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
    default: return launch<F32, NS>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
    }
}
}  // namespace

hipError_t launch_graph_search(int dtype, const void *X, int64_t N, int d, const int32_t *graph, int R, int entry,
                               const int32_t *entries, int n_entries, const void *Q, int B, int k, int ef, int32_t *ids,
                               float *scores, const GraphLds &L, hipStream_t stream) {
    NonStall ns{};
    ns.entries = entries;
    ns.n_entries = n_entries;
    return launch_dtype<false>(dtype, X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
}

hipError_t launch_zero_words(uint32_t *p, size_t words, hipStream_t stream) {
    const size_t n16 = words / 4;
    const size_t blocks = (n16 + 255) / 256;
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, stream,
                       reinterpret_cast<u4 *>(p), n16);
    return hipGetLastError();
}

hipError_t launch_gather_ids(const int32_t *table, int64_t M, const int32_t *idx, int64_t n, int32_t *out,
                             hipStream_t stream) {
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(gather_ids_kernel, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(256), 0, stream, table,
                       M, idx, n, out);
    return hipGetLastError();
}

hipError_t launch_graph_search_nonstall(int dtype, const void *X, int64_t N, int d, const int32_t *graph, int R,
                                        int entry, const void *Q, int B, int k, int ef, int32_t *ids, float *scores,
                                        const GraphLds &L, const NonStall &ns, hipStream_t stream) {
    return launch_dtype<true>(dtype, X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
}

}  // namespace ann
