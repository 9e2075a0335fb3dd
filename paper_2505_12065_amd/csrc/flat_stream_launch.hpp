// Launcher of flat_stream_kernel for one element type; included by one translation unit per type
// so that the instantiations compile in parallel.
#pragma once

#include "flat_kernels.hpp"
#include "launch.hpp"

namespace ann {

template <class T, int NQG, bool FULL, int NWV, bool MAX, int BATCH>
hipError_t launch_stream_one(const StreamPlan &pl, const StreamShape &sh, Cand *partial, float *maxima, int64_t n,
                             StreamOut out, After after, hipStream_t stream) {
    static size_t big = 0;
    const size_t lds = stream_lds_bytes(NQG, pl.lds_steps, NWV);
    if (hipError_t e = allow_big_lds(reinterpret_cast<const void *>(&flat_stream_kernel<T, NQG, FULL, NWV, MAX, BATCH>), lds, &big)) return e;
    hipLaunchKernelGGL((flat_stream_kernel<T, NQG, FULL, NWV, MAX, BATCH>), dim3(pl.P * pl.G), dim3(NWV * WAVE), lds, stream, sh, partial,
                       pl.P, pl.G, pl.K, pl.lds_steps, after, maxima, n, out);
    return hipGetLastError();
}

template <class T, int NQG, int NWV, bool MAX>
hipError_t launch_stream_nqg(const StreamPlan &pl, const StreamShape &sh, Cand *partial, float *maxima, int64_t n,
                             StreamOut out, After after, hipStream_t stream) {
    const int rb = sh.d * T::bytes;
    const bool held = NQG > 1 || pl.lds_steps * 64 >= rb;
    auto go = [&](auto bc, auto fc) {
        return launch_stream_one<T, NQG, decltype(fc)::value, NWV, MAX, decltype(bc)::value>(pl, sh, partial, maxima, n, out, after, stream);
    };
    auto either = [&](auto bc) { return held && rb % (64 * decltype(bc)::value) == 0 ? go(bc, std::true_type{}) : go(bc, std::false_type{}); };
    // (the batches that stream_batch gives)
    if constexpr (T::bytes == 2) {
        if (pl.batch == 3) return go(std::integral_constant<int, 3>{}, std::false_type{});
        if (pl.batch == 5) return go(std::integral_constant<int, 5>{}, std::false_type{});
        if constexpr (NQG > 1)
            if (pl.batch == 2 && rb % 128 == 0) return go(std::integral_constant<int, 2>{}, std::true_type{});
    } else if constexpr (NQG == 1 && !MAX) {
        if (pl.batch == 2) return either(std::integral_constant<int, 2>{});
    }
    return either(std::integral_constant<int, 4>{});
}

template <class T, int NQG>
hipError_t launch_stream_waves(const StreamPlan &pl, const StreamShape &sh, Cand *partial, float *maxima, int64_t n,
                               StreamOut out, After after, hipStream_t stream) {
    if constexpr (T::bytes == 2 && NQG >= 2)             // (one group of 16 queries never fills half the LDS)
        if (pl.waves == 16) return launch_stream_nqg<T, NQG, 16, false>(pl, sh, partial, maxima, n, out, after, stream);
    if constexpr (T::bytes == 4)
        if (maxima) return launch_stream_nqg<T, NQG, 8, true>(pl, sh, partial, maxima, n, out, after, stream);
    return launch_stream_nqg<T, NQG, 8, false>(pl, sh, partial, maxima, n, out, after, stream);
}

template <class T>
hipError_t launch_stream_any(const StreamPlan &pl, const void *X, int64_t N, int d, const void *Q, int B, Cand *partial, float *maxima, int64_t n,
                             StreamOut out, After after, hipStream_t stream) {
    const StreamShape sh{X, Q, N, d, B};
    if (pl.nqg == 1) return launch_stream_waves<T, 1>(pl, sh, partial, maxima, n, out, after, stream);
    if (pl.nqg == 2) return launch_stream_waves<T, 2>(pl, sh, partial, maxima, n, out, after, stream);
    if constexpr (STREAM_NQG_MAX(T::bytes) > 2) {
        if (pl.nqg == 3) return launch_stream_waves<T, 3>(pl, sh, partial, maxima, n, out, after, stream);
        return launch_stream_waves<T, 4>(pl, sh, partial, maxima, n, out, after, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace ann
