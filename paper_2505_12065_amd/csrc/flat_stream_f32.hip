// flat_stream_kernel instantiations for fp32 corpora.
#include "flat_stream_launch.hpp"

namespace ann {

hipError_t launch_flat_stream_f32(const StreamPlan &pl, const void *X, int64_t N, int d, const void *Q, int B, Cand *partial, float *maxima, int64_t n,
                                  StreamOut out, After after, hipStream_t stream) {
    return launch_stream_any<F32>(pl, X, N, d, Q, B, partial, maxima, n, out, after, stream);
}

}  // namespace ann
