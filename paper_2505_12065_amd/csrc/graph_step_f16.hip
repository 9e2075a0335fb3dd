// graph_step_kernel instantiations for f16 corpora.
#include "graph_step_launch.hpp"

namespace ann {
hipError_t launch_graph_step_f16(const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const int32_t *entries,
                                int n_entries, const void *Q, int B, int k, int ef, int32_t *ids, float *scores, const StepLds &L,
                                hipStream_t stream) {
    return launch_step<F16>(X, N, d, graph, R, entry, entries, n_entries, Q, B, k, ef, ids, scores, L, stream);
}
}  // namespace ann
