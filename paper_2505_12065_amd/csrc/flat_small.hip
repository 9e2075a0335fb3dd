// flat_scores_kernel and flat_direct_kernel: instantiations and launchers.
#include "flat_small.hpp"

namespace ann {
hipError_t launch_flat_direct(int dtype, const void *X, int64_t N, int d, const void *Q, int B, int k, int32_t *ids, float *scores,
                              After after, hipStream_t stream) {
    const StreamShape sh{X, Q, N, d, B};
    auto go = [&](auto kernel, int bytes, size_t *big) {
        const size_t lds = direct_lds_bytes(d, bytes);
        if (hipError_t e = allow_big_lds(reinterpret_cast<const void *>(kernel), lds, big)) return e;
        hipLaunchKernelGGL(kernel, dim3((B + 15) / 16), dim3(DIRECT_WAVES * WAVE), lds, stream, sh, k, direct_held(d, bytes), after, ids,
                           scores);
        return hipGetLastError();
    };
    static size_t big[3];
    return dtype == 0   ? go(&flat_direct_kernel<F16>, 2, &big[0])
           : dtype == 1 ? go(&flat_direct_kernel<BF16>, 2, &big[1])
                        : go(&flat_direct_kernel<F32>, 4, &big[2]);
}

hipError_t launch_flat_scores(int dtype, const void *X, int64_t N, int d, const void *Q, int B, float *maxima, int64_t n, After after,
                              hipStream_t stream) {
    const StreamShape sh{X, Q, N, d, B};
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)score_tiles(N, B)), dim3(WAVE), 0, stream, sh, maxima, (int)n, (B + 15) / 16, after);
        return hipGetLastError();
    };
    return dtype == 0 ? go(flat_scores_kernel<F16>) : dtype == 1 ? go(flat_scores_kernel<BF16>) : go(flat_scores_kernel<F32>);
}

}  // namespace ann
