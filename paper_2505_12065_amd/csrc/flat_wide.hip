// flat_wide_kernel and flat_pick_kernel: instantiations and launchers.
#include "flat_wide_kernel.hpp"
#include "flat_pick.hpp"

namespace ann {
namespace {
template <class T, class C, bool ONE, bool BY_LINE>
hipError_t launch_one(const WidePlan &pl, const void *X, int64_t N, int d, const void *Q, int B, float *maxima, After after,
                  hipStream_t stream) {
    static size_t big = 0;
    if (hipError_t e = allow_big_lds(reinterpret_cast<const void *>(&flat_wide_kernel<T, C, ONE, BY_LINE>), C::LDS_BYTES, &big)) return e;
    hipLaunchKernelGGL((flat_wide_kernel<T, C, ONE, BY_LINE>), dim3(pl.P * pl.NT), dim3(C::THREADS), C::LDS_BYTES, stream, X, N, d, Q, B,
                       maxima, pl.n, pl.P, pl.NT, pl.gs_log, after);
    return hipGetLastError();
}

template <class T, class C>
hipError_t launch(const WidePlan &pl, const void *X, int64_t N, int d, const void *Q, int B, float *maxima, After after,
                  hipStream_t stream) {
    if constexpr (C::SB == 128 && (C::WAVES == 8 || C::STAGES == 3))      // (the tiles that corpora beyond the caches get)
        if (pl.gs_log > 0 && wide_by_line(N, d, pl.NT)) return launch_one<T, C, false, true>(pl, X, N, d, Q, B, maxima, after, stream);
    return pl.gs_log == 0 ? launch_one<T, C, true, false>(pl, X, N, d, Q, B, maxima, after, stream)
                          : launch_one<T, C, false, false>(pl, X, N, d, Q, B, maxima, after, stream);
}

template <class T>
hipError_t launch_any(const WidePlan &pl, const void *X, int64_t N, int d, const void *Q, int B, float *maxima, After after,
                      hipStream_t stream) {
    switch (pl.shape) {
    case WIDE_LARGE: return launch<T, WideLarge>(pl, X, N, d, Q, B, maxima, after, stream);
    case WIDE_TALL: return launch<T, WideTall>(pl, X, N, d, Q, B, maxima, after, stream);
    case WIDE_MID: return launch<T, WideMid>(pl, X, N, d, Q, B, maxima, after, stream);
    case WIDE_TINY: return launch<T, WideTiny>(pl, X, N, d, Q, B, maxima, after, stream);
    case WIDE_SQUARE: return launch<T, WideSquare>(pl, X, N, d, Q, B, maxima, after, stream);
    case WIDE_SHORT: return launch<T, WideShort>(pl, X, N, d, Q, B, maxima, after, stream);
    default: return launch<T, WideThin>(pl, X, N, d, Q, B, maxima, after, stream);
    }
}

template <class T>
hipError_t pick(const WidePlan &pl, const void *X, int64_t N, int d, const void *Q, int B, int k, const float *maxima,
                int32_t *ids, float *scores, After after, uint64_t *best, int more, hipStream_t stream) {
    const StreamShape sh{X, Q, N, d, B};
    const bool one = pl.gs_log == 0;
    const int threads = pick_threads(pl.cus, pl.gs_log, pl.n, B, k);
    const size_t lds = one ? 0 : (size_t)d * T::bytes;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(B), dim3(threads), lds, stream, maxima, pl.n, pl.gs_log, k, ids, scores, sh, after,
                           best, more);
        return hipGetLastError();
    };
    auto form = [&](auto pc, auto rc) {
        constexpr bool P = decltype(pc)::value, R = decltype(rc)::value;
        if constexpr (T::bytes == 4) return go(flat_pick_kernel<T, 0, false, P, R>);
        else return pl.wmf == 4 ? go(flat_pick_kernel<T, 4, false, P, R>) : pl.wmf == 2 ? go(flat_pick_kernel<T, 2, false, P, R>) : go(flat_pick_kernel<T, 1, false, P, R>);
    };
    auto parts = [&](auto pc) {
        constexpr bool P = decltype(pc)::value;
        if constexpr (!P)
            if (one && pl.wmf == 0) return go(flat_pick_kernel<T, 0, true, false, false>);
        if constexpr (T::bytes == 2)
            if (one) return pl.wmf == 4 ? go(flat_pick_kernel<T, 4, true, P, false>) : pl.wmf == 2 ? go(flat_pick_kernel<T, 2, true, P, false>) : go(flat_pick_kernel<T, 1, true, P, false>);
        return pick_runs(pl.cus, (size_t)d * T::bytes, T::bytes == 4 ? 64 : 32, B) ? form(pc, std::true_type{}) : form(pc, std::false_type{});
    };
    return more ? parts(std::true_type{}) : parts(std::false_type{});
}
}  // namespace

hipError_t launch_flat_wide(const WidePlan &pl, int dtype, const void *X, int64_t N, int d, const void *Q, int B, float *maxima,
                            After after, hipStream_t stream) {
    return dtype == 0 ? launch_any<F16>(pl, X, N, d, Q, B, maxima, after, stream)
                      : launch_any<BF16>(pl, X, N, d, Q, B, maxima, after, stream);
}

hipError_t launch_flat_pick(const WidePlan &pl, int dtype, const void *X, int64_t N, int d, const void *Q, int B, int k,
                            const float *maxima, int32_t *ids, float *scores, After after, uint64_t *best, int more,
                            hipStream_t stream) {
    return dtype == 0   ? pick<F16>(pl, X, N, d, Q, B, k, maxima, ids, scores, after, best, more, stream)
           : dtype == 2 ? pick<F32>(pl, X, N, d, Q, B, k, maxima, ids, scores, after, best, more, stream)
                        : pick<BF16>(pl, X, N, d, Q, B, k, maxima, ids, scores, after, best, more, stream);
}

}  // namespace ann
