// Launcher of graph_step_kernel for one element type; included by one translation unit per type
// so that the instantiations compile in parallel.
#pragma once

#include "graph_step_kernel.hpp"

namespace ann {

template <class T, int RPG, int VIS, bool NS, bool LONG, bool QREG>
hipError_t launch_step_one(const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const void *Q, int B, int k,
                           int ef, int32_t *ids, float *scores, const StepLds &L, const NonStall &ns, hipStream_t stream) {
    static size_t big = 0;
    if (hipError_t e = allow_big_lds(reinterpret_cast<const void *>(&graph_step_kernel<T, RPG, VIS, NS, LONG, QREG>), L.total, &big))
        return e;
    hipLaunchKernelGGL((graph_step_kernel<T, RPG, VIS, NS, LONG, QREG>), dim3(B), dim3(GRAPH_THREADS), L.total, stream, X, N, d, graph,
                       R, entry, Q, k, ef, ids, scores, L, ns);
    return hipGetLastError();
}

template <class T, int RPG, bool QREG>
hipError_t launch_step_rows(const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const void *Q, int B,
                             int k, int ef, int32_t *ids, float *scores, const StepLds &L, bool counters,
                             const NonStall &ns, hipStream_t stream) {
#define ANN_STEP(VIS, NS, LONG) \
    return launch_step_one<T, RPG, VIS, NS, LONG, QREG>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream)
    if (L.long_list) {
        if constexpr (QREG) {
            if (counters) {
                if (L.vis_mode == STEP_VIS_LDS) ANN_STEP(STEP_VIS_LDS, true, true);
                ANN_STEP(STEP_VIS_GLOBAL, true, true);
            }
            if (L.vis_mode == STEP_VIS_LDS) ANN_STEP(STEP_VIS_LDS, false, true);
            ANN_STEP(STEP_VIS_GLOBAL, false, true);
        }
        return hipErrorInvalidValue;                      // (the dense form is planned for short lists only)
    }
    if (counters) {
        if constexpr (QREG) {
            if (L.vis_mode == STEP_VIS_LDS) ANN_STEP(STEP_VIS_LDS, true, false);
            ANN_STEP(STEP_VIS_GLOBAL, true, false);
        }
        return hipErrorInvalidValue;
    }
    if (L.vis_mode == STEP_VIS_LDS) ANN_STEP(STEP_VIS_LDS, false, false);
    ANN_STEP(STEP_VIS_CACHE, false, false);
#undef ANN_STEP
}

template <class T>
hipError_t launch_step(const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const void *Q, int B, int k,
                       int ef, int32_t *ids, float *scores, const StepLds &L, bool counters, const NonStall &ns,
                       hipStream_t stream) {
    if (L.dense)
        return launch_step_rows<T, 1, false>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, counters, ns, stream);
    return L.rows_per_group == 2
               ? launch_step_rows<T, 2, true>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, counters, ns, stream)
               : launch_step_rows<T, 1, true>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, counters, ns, stream);
}

}  // namespace ann
