// Launcher of flat_stream_kernel for one element type; included by one translation unit per type
// so that the instantiations compile in parallel.
#pragma once

#include "flat_kernels.hpp"
#include "launch.hpp"

namespace ann {

template <class T, int NQG, bool FULL, int NWV, bool MAX>
hipError_t launch_stream_one(const StreamPlan &pl, const StreamShape &sh, Cand *partial, float *maxima, int64_t n,
                             StreamOut out, After after, hipStream_t stream) {
    static size_t big = 0;
    const size_t lds = stream_lds_bytes(NQG, pl.lds_steps, NWV);
    if (hipError_t e = allow_big_lds(reinterpret_cast<const void *>(&flat_stream_kernel<T, NQG, FULL, NWV, MAX>), lds, &big)) return e;
    hipLaunchKernelGGL((flat_stream_kernel<T, NQG, FULL, NWV, MAX>), dim3(pl.P * pl.G), dim3(NWV * WAVE), lds, stream, sh, partial,
                       pl.P, pl.G, pl.K, pl.lds_steps, after, maxima, n, out);
    return hipGetLastError();
}

template <class T, int NQG>
hipError_t launch_stream_nqg(const StreamPlan &pl, const StreamShape &sh, Cand *partial, float *maxima, int64_t n,
                             StreamOut out, After after, hipStream_t stream) {
    const bool full = (sh.d * T::bytes) % (64 * STREAM_BATCH) == 0;
    if constexpr (T::bytes == 2 && NQG >= 2) {           // (one group of 16 queries never fills half the LDS)
        if (pl.waves == 16)
            return full ? launch_stream_one<T, NQG, true, 16, false>(pl, sh, partial, maxima, n, out, after, stream)
                        : launch_stream_one<T, NQG, false, 16, false>(pl, sh, partial, maxima, n, out, after, stream);
    }
    if constexpr (T::bytes == 4) {
        if (maxima)
            return full && (NQG > 1 || pl.lds_steps * 64 >= sh.d * T::bytes)
                       ? launch_stream_one<T, NQG, true, 8, true>(pl, sh, partial, maxima, n, out, after, stream)
                       : launch_stream_one<T, NQG, false, 8, true>(pl, sh, partial, maxima, n, out, after, stream);
    }
    return full && (NQG > 1 || pl.lds_steps * 64 >= sh.d * T::bytes)
               ? launch_stream_one<T, NQG, true, 8, false>(pl, sh, partial, maxima, n, out, after, stream)
               : launch_stream_one<T, NQG, false, 8, false>(pl, sh, partial, maxima, n, out, after, stream);
}

template <class T>
hipError_t launch_stream_any(const StreamPlan &pl, const void *X, int64_t N, int d, const void *Q, int B, Cand *partial, float *maxima, int64_t n,
                             StreamOut out, After after, hipStream_t stream) {
    const StreamShape sh{X, Q, N, d, B};
    if (pl.nqg == 1) return launch_stream_nqg<T, 1>(pl, sh, partial, maxima, n, out, after, stream);
    if (pl.nqg == 2) return launch_stream_nqg<T, 2>(pl, sh, partial, maxima, n, out, after, stream);
    if constexpr (STREAM_NQG_MAX(T::bytes) > 2) {
        if (pl.nqg == 3) return launch_stream_nqg<T, 3>(pl, sh, partial, maxima, n, out, after, stream);
        return launch_stream_nqg<T, 4>(pl, sh, partial, maxima, n, out, after, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace ann
