// graph_frontier_kernel instantiations for f16 corpora.
#include "graph_frontier_launch.hpp"

namespace ann {
hipError_t launch_graph_frontier_f16(int B, const FrontierArgs &args, bool counters, hipStream_t stream) {
    return launch_frontier<F16>(B, args, counters, stream);
}
}  // namespace ann
