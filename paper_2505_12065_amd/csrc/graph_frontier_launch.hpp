// Launcher of graph_frontier_kernel for one element type; included by one translation unit per type
// so that the instantiations compile in parallel.
#pragma once

#include "graph_frontier_kernel.hpp"

namespace ann {

template <class T, int NW, int W, bool QREG, int OCC>
hipError_t launch_frontier_as(int B, const FrontierArgs &args, bool counters, hipStream_t stream) {
    const FrontierLds &L = args.L;
    auto go = [&](auto kernel, size_t *big) {
        if (hipError_t e = allow_big_lds(reinterpret_cast<const void *>(kernel), L.total, big)) return e;
        hipLaunchKernelGGL(kernel, dim3(B), dim3(NW * WAVE), L.total, stream, args);
        return hipGetLastError();
    };
    static size_t big[4] = {0, 0, 0, 0};
    if (L.vis_mode == FRONTIER_VIS_LDS)
        return counters ? go(graph_frontier_kernel<T, NW, W, FRONTIER_VIS_LDS, true, QREG, OCC>, &big[0])
                        : go(graph_frontier_kernel<T, NW, W, FRONTIER_VIS_LDS, false, QREG, OCC>, &big[1]);
    return counters ? go(graph_frontier_kernel<T, NW, W, FRONTIER_VIS_GLOBAL, true, QREG, OCC>, &big[2])
                    : go(graph_frontier_kernel<T, NW, W, FRONTIER_VIS_GLOBAL, false, QREG, OCC>, &big[3]);
}

template <class T>
hipError_t launch_frontier_tight(int B, const FrontierArgs &args, hipStream_t stream) {
    auto *kernel = graph_frontier_kernel<T, 4, 8, FRONTIER_VIS_LDS, true, true, 2, true>;
    static size_t big = 0;
    if (hipError_t e = allow_big_lds(reinterpret_cast<const void *>(kernel), args.L.total, &big)) return e;
    hipLaunchKernelGGL(kernel, dim3(B), dim3(4 * WAVE), args.L.total, stream, args);
    return hipGetLastError();
}

template <class T>
hipError_t launch_frontier(int B, const FrontierArgs &args, bool counters, hipStream_t stream) {
    const FrontierLds &L = args.L;
    if (L.tight) return counters ? launch_frontier_tight<T>(B, args, stream) : hipErrorInvalidValue;
    auto wide = [&](auto wc) {
        constexpr int W = decltype(wc)::value;
        return (L.waves == 8 ? launch_frontier_as<T, 8, W, true, 2> : L.per_cu == 3 ? launch_frontier_as<T, 4, W, false, 3>
                                                                                   : launch_frontier_as<T, 4, W, true, 2>)(B, args, counters, stream);
    };
    return L.width == 8 ? wide(std::integral_constant<int, 8>{}) : wide(std::integral_constant<int, 4>{});
}

}  // namespace ann
