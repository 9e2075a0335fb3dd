// graph_search_kernel instantiations, LDS layout and launcher.
#include "graph_kernel.hpp"

namespace ann {

// out[i] <- table[idx[i]], or -1 where idx[i] is not in [0, M)
__global__ __launch_bounds__(256) void gather_ids_kernel(const int32_t *__restrict__ table, int64_t M,
                                                         const int32_t *__restrict__ idx, int64_t n,
                                                         int32_t *__restrict__ out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t j = idx[i];
        out[i] = (j >= 0 && j < M) ? table[j] : -1;
    }
}

// words[0 .. n) <- 0, 16 bytes per store (n a multiple of 4)
__global__ __launch_bounds__(256) void zero_words_kernel(u4 *__restrict__ p, size_t n16) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        p[i] = zero_chunk();
}

GraphLds graph_lds_layout(int d, int elem_bytes, int R, int ef) {
    auto up = [](uint32_t x) { return (x + 15u) & ~15u; };
    const bool inplace = ef > GRAPH_EF_DOUBLE;           // long lists: one buffer, merged in place
    auto lay = [&](uint32_t bits) {
        GraphLds L{};
        uint32_t off = 0;
        L.rp = (uint32_t)((R + ROWS_PER_PASS - 1) / ROWS_PER_PASS * ROWS_PER_PASS);
        L.cache_bits = bits;
        L.q = off; off = up(off + (uint32_t)d * elem_bytes);
        // score lists are padded to 64 entries; lists of up to 256 entries get buffers of 256, which
        // the scan for the next unexpanded entry then reads without conditions
        const uint32_t ef64 = ef <= GRAPH_DELTA ? (uint32_t)GRAPH_DELTA : ((uint32_t)ef + 63u) & ~63u;
        const uint32_t efi = ef <= GRAPH_DELTA ? (uint32_t)GRAPH_DELTA : (uint32_t)ef;
        L.ls0 = off; off = up(off + 4u * ef64);
        if (inplace) L.ls1 = L.ls0; else { L.ls1 = off; off = up(off + 4u * ef64); }
        L.li0 = off; off = up(off + 4u * efi);
        if (inplace) L.li1 = L.li0; else { L.li1 = off; off = up(off + 4u * efi); }
        L.cs = off; off = up(off + 4u * L.rp);
        L.ci = off; off = up(off + 4u * L.rp);
        L.cpos = off; off = up(off + 4u * L.rp);
        L.cache = off; off = up(off + (4u << bits));
        L.ctl = off; off = up(off + 16u);
        L.adj = off; off = up(off + 2u * 4u * RMAX_LDS);
        L.um = off; off = up(off + 8u * (((uint32_t)ef + 63u) / 64u) + 32u);   // the scans use um[0 .. 3] at any ef
        L.rq = off; off = up(off + 4u * L.rp);
        L.co = off; off = up(off + 4u * L.rp);
        L.total = off;
        return L;
    };
    // Long lists on graphs of at most 32 slots per node: the two-level list.  The large part has one
    // buffer of ef entries, the small part two of GRAPH_DELTA; the adjacency rows read ahead take 32
    // slots each; the words of um double as the position marks of a rebuild; there is no id cache.
    auto lay2 = [&] {
        GraphLds L{};
        L.rp = ROWS_PER_PASS;
        L.cache_bits = 0;                                  // no id cache: the visited set is asked first
        L.two_level = 1;
        L.ls0 = TL_LS0; L.li0 = TL_LI0; L.ls1 = TL_LS1; L.li1 = TL_LI1;
        L.cs = TL_CS; L.ci = TL_CI; L.cpos = TL_CPOS;
        L.ctl = L.cache = TL_CTL;
        L.adj = TL_ADJ;
        L.um = L.rq = L.co = TL_UM;                        // (rq, co: used by the plain loop only)
        L.ms = TL_MS;
        L.mi = up(L.ms + 4u * (uint32_t)ef);
        L.q = up(L.mi + 4u * (uint32_t)ef);
        L.total = up(L.q + (uint32_t)d * elem_bytes);
        return L;
    };
    // (it is the only layout of such lists on such graphs: the software-pipelined loop has no code for
    // a single list of more than 512 entries; with d <= ANN_D_MAX it always fits)
    if (ef > GRAPH_EF_TWO_LEVEL && R <= ROWS_PER_PASS) return lay2();
    // cache slots: a few times the number of nodes a search scores (about 10 ef), at most 2^14;
    // fewer when that lets two workgroups share a compute unit, or when the list needs the room
    uint32_t want = 10;
    while ((1u << want) < 32u * (uint32_t)ef && want < 14) ++want;
    uint32_t bits = want;
    if (lay(11).total <= LDS_MAX / 2)
        while (bits > 11 && lay(bits).total > LDS_MAX / 2) --bits;
    while (bits > 10 && lay(bits).total > LDS_MAX) --bits;
    return lay(bits);
}

// Where steps of several expansions are faster than one expansion at a time.  A step costs two to three expansions of the
// other kernel, so what decides is how many expansions a step commits for the slowest query of the batch.  Measured over
// drawn N (20 k to 200 k), d, R and types, time of the one-by-one loop / time in steps:
//   maturity exit (tau < 1: most queries stop while their list fills, and a filling list commits whole steps): 1.1 to 2.4
//     with lists of 96 up and some queries per call; 0.65 to 0.95 for one to four queries or shorter lists (over before
//     the steps pay), and 0.6 to 1.05 where no average reaches tau and every search runs to its end
//   two-level lists (over 512): 1.0 to 3.4, more for longer lists; 0.87 only at ef = 700 with 1.5 KB rows and 256 queries,
//     hence the bound on the row below ef = 1024
//   one list: more queries than two workgroups per compute unit hold (the rest waits for a place, so the mean over queries
//     counts, not the slowest) 1.1 to 1.5 from ef = 192, 0.84 to 1.1 below; up to four queries 1.0 to 4.1 from ef = 320
//     (0.85 to 1.1 below, or with rows of over 2 KB); else 0.75 to 1.0
bool graph_step_pays(int cus, int row_bytes, int R, int B, int ef, bool counters, float tau) {
    if (R > GRAPH_STEP_MAX_R) return false;
    if (counters) return tau < 1.0f && R >= 16 && ef >= 96 && B >= 8 && (int64_t)B * ef >= 2048;
    if (ef > GRAPH_EF_TWO_LEVEL) return ef >= 1024 || row_bytes <= 1024 || B <= 16;
    return B > 2 * cus ? ef >= 192 : B <= 4 && ef >= 320 && row_bytes <= 2048;
}

StepLds graph_step_plan(int cus, int64_t N, int d, int elem_bytes, int B, int ef, bool counters) {
    auto up = [](uint32_t x) { return (x + 15u) & ~15u; };
    StepLds L{};
    L.long_list = ef > GRAPH_EF_TWO_LEVEL;
    L.rows_per_group = B <= cus ? 2 : 1;
    const uint32_t entries = L.long_list || ef <= GRAPH_DELTA ? (uint32_t)GRAPH_DELTA : ((uint32_t)ef + 63u) & ~63u;
    uint32_t off = up(StepLds::WAVE0 + GRAPH_WAVES * StepLds::WAVE_BYTES);
    L.ls_bytes = 4u * entries;
    L.ls = off; off = up(off + 2u * L.ls_bytes);
    L.li = off; off = up(off + 2u * L.ls_bytes);
    if (L.long_list) {
        L.um = off; off = up(off + 8u * (((uint32_t)ef + 63u) / 64u) + 32u);
        L.ms = off; off = up(off + 4u * (uint32_t)ef);
        L.mi = off; off = up(off + 4u * (uint32_t)ef);
    }
    L.q = off; off = up(off + (uint32_t)d * elem_bytes);
    L.vis = off;
    // A bit per node in LDS if it leaves the workgroups per compute unit that the batch needs
    const uint32_t room = (uint32_t)(B <= cus ? LDS_MAX : LDS_MAX / 2);
    const int64_t words = visited_words(N);
    if ((int64_t)off + words * 4 <= room) {
        L.vis_mode = STEP_VIS_LDS;
        L.vis_words = (int)words;
    } else if (!counters && !L.long_list) {
        // id cache: a few times the number of nodes a search scores (about 10 ef)
        L.vis_mode = STEP_VIS_CACHE;
        int bits = 10;
        while ((1u << bits) < 32u * (uint32_t)ef && bits < 13) ++bits;
        L.vis_words = 1 << bits;
        L.cache_shift = 32 - bits;
    } else {
        L.vis_mode = STEP_VIS_GLOBAL;
    }
    L.total = up(off + 4u * (uint32_t)L.vis_words);
    // More queries than two workgroups per compute unit hold at once, and a layout small enough for three: the form
    // that reads the query from LDS and runs three per compute unit.
    L.dense = !counters && !L.long_list && B > GRAPH_DENSE_MIN_B && 3 * (size_t)L.total <= LDS_MAX;
    return L;
}

hipError_t launch_graph_step_f16(const void *, int64_t, int, const int32_t *, int, int, const void *, int, int, int, int32_t *,
                                 float *, const StepLds &, bool, const NonStall &, hipStream_t);
hipError_t launch_graph_step_bf16(const void *, int64_t, int, const int32_t *, int, int, const void *, int, int, int, int32_t *,
                                  float *, const StepLds &, bool, const NonStall &, hipStream_t);
hipError_t launch_graph_step_f32(const void *, int64_t, int, const int32_t *, int, int, const void *, int, int, int, int32_t *,
                                 float *, const StepLds &, bool, const NonStall &, hipStream_t);

hipError_t launch_graph_step(int dtype, const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const void *Q,
                             int B, int k, int ef, int32_t *ids, float *scores, const StepLds &L, bool counters,
                             const NonStall &ns, hipStream_t stream) {
    return (dtype == 0 ? launch_graph_step_f16 : dtype == 1 ? launch_graph_step_bf16 : launch_graph_step_f32)(
        X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, counters, ns, stream);
}

namespace {
template <class T, int RPT, bool NS, bool QREG = true, bool LONG = false>
hipError_t launch_rp(const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const void *Q, int B,
                     int k, int ef, int32_t *ids, float *scores, const GraphLds &L, const NonStall &ns,
                     hipStream_t stream) {
    static size_t big = 0;
    if (hipError_t e = allow_big_lds(reinterpret_cast<const void *>(&graph_search_kernel<T, RPT, NS, QREG, LONG>), L.total, &big))
        return e;
    hipLaunchKernelGGL((graph_search_kernel<T, RPT, NS, QREG, LONG>), dim3(B), dim3(GRAPH_THREADS), L.total, stream, X, N, d,
                       graph, R, entry, Q, k, ef, ids, scores, L, ns);
    return hipGetLastError();
}

template <class T, bool NS>
hipError_t launch(const void *X, int64_t N, int d, const int32_t *graph, int R, int entry, const void *Q, int B,
                  int k, int ef, int32_t *ids, float *scores, const GraphLds &L, const NonStall &ns,
                  hipStream_t stream) {
    // More queries than two workgroups per compute unit hold at once, and a layout small enough for
    // three: the variant that reads the query from LDS and runs three per compute unit.
    if constexpr (!NS) {
        if (L.rp == 32 && B > GRAPH_DENSE_MIN_B && 3 * (size_t)L.total + 3 * 1024 <= LDS_MAX)
            return launch_rp<T, 32, false, false>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
    }
    if constexpr (NS) {
        if (L.two_level)
            return launch_rp<T, 32, true, true, true>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
    } else if (L.two_level) {
        return hipErrorInvalidValue;                      // long lists run with the exact visited set
    }
    return L.rp == 32 ? launch_rp<T, 32, NS>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream)
                      : launch_rp<T, 0, NS>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
}

template <bool NS>
hipError_t launch_dtype(int dtype, const void *X, int64_t N, int d, const int32_t *graph, int R, int entry,
                        const void *Q, int B, int k, int ef, int32_t *ids, float *scores, const GraphLds &L,
                        const NonStall &ns, hipStream_t stream) {
    switch (dtype) {
    case 0: return launch<F16, NS>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
    case 1: return launch<BF16, NS>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
    default: return launch<F32, NS>(X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
    }
}
}  // namespace

hipError_t launch_graph_search(int dtype, const void *X, int64_t N, int d, const int32_t *graph, int R, int entry,
                               const int32_t *entries, int n_entries, const void *Q, int B, int k, int ef, int32_t *ids,
                               float *scores, const GraphLds &L, hipStream_t stream) {
    NonStall ns{};
    ns.entries = entries;
    ns.n_entries = n_entries;
    return launch_dtype<false>(dtype, X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
}

hipError_t launch_zero_words(uint32_t *p, size_t words, hipStream_t stream) {
    const size_t n16 = words / 4;
    const size_t blocks = (n16 + 255) / 256;
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, stream,
                       reinterpret_cast<u4 *>(p), n16);
    return hipGetLastError();
}

hipError_t launch_gather_ids(const int32_t *table, int64_t M, const int32_t *idx, int64_t n, int32_t *out,
                             hipStream_t stream) {
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(gather_ids_kernel, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(256), 0, stream, table,
                       M, idx, n, out);
    return hipGetLastError();
}

hipError_t launch_graph_search_nonstall(int dtype, const void *X, int64_t N, int d, const int32_t *graph, int R,
                                        int entry, const void *Q, int B, int k, int ef, int32_t *ids, float *scores,
                                        const GraphLds &L, const NonStall &ns, hipStream_t stream) {
    return launch_dtype<true>(dtype, X, N, d, graph, R, entry, Q, B, k, ef, ids, scores, L, ns, stream);
}

}  // namespace ann
