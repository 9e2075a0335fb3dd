// flat_stream_kernel instantiations for bf16 corpora.
#include "flat_stream_launch.hpp"

namespace ann {

hipError_t launch_flat_stream_bf16(const StreamPlan &pl, const void *X, int64_t N, int d, const void *Q, int B, Cand *partial, float *maxima, int64_t n,
                                  StreamOut out, After after, hipStream_t stream) {
    return launch_stream_any<BF16>(pl, X, N, d, Q, B, partial, maxima, n, out, after, stream);
}

}  // namespace ann
