// graph_frontier_kernel instantiations for bf16 corpora.
#include "graph_frontier_launch.hpp"

namespace ann {
hipError_t launch_graph_frontier_bf16(int B, const FrontierArgs &args, bool counters, hipStream_t stream) {
    return launch_frontier<BF16>(B, args, counters, stream);
}
}  // namespace ann
