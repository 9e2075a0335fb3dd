// Launcher of graph_step_kernel for one element type; included by one translation unit per type
// so that the instantiations compile in parallel.
#pragma once

#include "graph_step_kernel.hpp"

namespace ann {

template <class T, int RPG, bool QREG>
hipError_t launch_step_as(const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const int32_t *entries,
                          int n_entries, const void *Q, int B, int k, int ef, int32_t *ids, float *scores, const StepLds &L,
                          hipStream_t stream) {
    static size_t big = 0;
    if (hipError_t e = allow_big_lds(reinterpret_cast<const void *>(&graph_step_kernel<T, RPG, QREG>), L.total, &big)) return e;
    hipLaunchKernelGGL((graph_step_kernel<T, RPG, QREG>), dim3(B), dim3(GRAPH_THREADS), L.total, stream, X, N, d, graph, R, entry, Q, k,
                       ef, ids, scores, L, entries, n_entries);
    return hipGetLastError();
}

template <class T>
hipError_t launch_step(const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const int32_t *entries, int n_entries,
                       const void *Q, int B, int k, int ef, int32_t *ids, float *scores, const StepLds &L, hipStream_t stream) {
    return (L.dense ? launch_step_as<T, 1, false> : L.rows_per_group == 2 ? launch_step_as<T, 2, true> : launch_step_as<T, 1, true>)(
        X, N, d, graph, R, entry, entries, n_entries, Q, B, k, ef, ids, scores, L, stream);
}

}  // namespace ann
