// libann.so — host side of the C ABI declared in include/ann.h: argument checks,
// the per-device workspace and the corpus registry.  What a call launches is decided
// in plan.hpp; all compute runs in the kernels reached through launch.hpp.
#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/ann.h"
#include "launch.hpp"

using namespace ann;

namespace {

thread_local std::string g_last_error;

int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

}  // namespace

// Workspace of ann_flat_search_static: lives in the code object, so every device the library
// runs on holds one copy until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; the device address is looked up once per device (device_state) and is
// what every launch and every offset computation uses.  Behind the workspace: room for the k best so far of the queries of
// a part, so that they take nothing from its maxima (8 MiB of them are whole rounds of tiles on 256 compute units).
constexpr size_t STATIC_BYTES = ANN_STATIC_WORKSPACE_BYTES + (size_t)PART_MAX_B * ANN_K_MAX * sizeof(uint64_t);
static __device__ __align__(256) unsigned char scratch[STATIC_BYTES];

namespace {

struct Buffer {
    void *ptr = nullptr;
    size_t bytes = 0;
    bool captured = false;        // a graph may hold it
};
struct DeviceState {
    int cus = 0;
    Buffer ws;
    Buffer vis;                   // visited bitsets of the non-stall graph search
    std::vector<void *> kept;     // outgrown buffers that a graph may hold
    void *scratch_ptr = nullptr;  // this device's address of `scratch`
    void *user_ws = nullptr;      // caller-owned workspace (ann_set_workspace), used instead of ws and vis
    size_t user_bytes = 0;
};

std::mutex g_mu;
std::unordered_map<int, DeviceState> g_dev;
struct CorpusInfo { int64_t N; int32_t d; int32_t dtype; };
std::unordered_map<const void *, CorpusInfo> g_corpora;
int g_default_dtype = ANN_F16;

int device_state(DeviceState **out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(ANN_ERR_LAUNCH, "no HIP device is current");
    DeviceState &st = g_dev[dev];
    if (st.cus == 0) {
        if (hipDeviceGetAttribute(&st.cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || st.cus <= 0)
            return fail(ANN_ERR_LAUNCH, "cannot query the compute-unit count of device %d", dev);
    }
    if (!st.scratch_ptr) {                       // device `dev` is current here
        void *p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            return fail(ANN_ERR_LAUNCH, "cannot resolve the static workspace on device %d: %s", dev, hipGetErrorString(e));
        }
        st.scratch_ptr = p;
    }
    *out = &st;
    return ANN_OK;
}

// Buffers grow by a quarter at least, so what is kept for graphs adds up to four times the present size at most.
int grow(DeviceState *st, Buffer *buf, size_t bytes) {
    if (buf->bytes >= bytes) return ANN_OK;
    if (buf->ptr && buf->captured) st->kept.push_back(buf->ptr);
    else if (buf->ptr) (void)hipFree(buf->ptr);  // synchronises the device: no kernel still uses it
    *buf = Buffer();
    size_t want = bytes + bytes / 4;
    if (hipMalloc(&buf->ptr, want) != hipSuccess) {
        (void)hipGetLastError();
        buf->ptr = nullptr;
        return fail(ANN_ERR_NOMEM, "cannot allocate %zu bytes of device workspace", want);
    }
    buf->bytes = want;
    return ANN_OK;
}

bool is_captured(hipStream_t stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess) {
        (void)hipGetLastError();                          // (the null stream, while another stream is captured)
        return true;
    }
    return status != hipStreamCaptureStatusNone;
}

// The device buffer a call may use as workspace: the caller's when one was set (never grown: a call
// that needs more fails), else the library's own, grown on demand and, once a graph may hold it, not freed by growing.
int workspace_for(DeviceState *st, Buffer *own, size_t bytes, hipStream_t stream, void **out) {
    if (st->user_ws) {
        if (bytes > st->user_bytes)
            return fail(ANN_ERR_NOMEM, "this call needs %zu bytes of workspace, the buffer given to ann_set_workspace has %zu",
                        bytes, st->user_bytes);
        *out = st->user_ws;
        return ANN_OK;
    }
    if (int rc = grow(st, own, bytes)) return rc;
    // (The null stream cannot be captured; the question takes 0.08 us.)
    own->captured = own->captured || (bytes > 0 && stream != nullptr && is_captured(stream));
    *out = own->ptr;
    return ANN_OK;
}

// Whether workspace_for gives `bytes` to a call on `stream`: in a caller's buffer if they fit, in the library's own unless that
// would have to grow while the stream is captured.
bool at_hand(const DeviceState *st, const Buffer &own, size_t bytes, hipStream_t stream) {
    if (st->user_ws) return bytes <= st->user_bytes;
    return bytes <= own.bytes || !is_captured(stream);
}

// ---- optional event timing of the main kernels -----------------------------------------------
struct TimedLaunch { hipEvent_t a, b; int kernel; };
bool g_timing = false;
bool g_timing_off = false;                 // set while an entry point that may not create events runs
std::vector<TimedLaunch> g_timed;          // records of the current session
std::vector<hipEvent_t> g_event_pool;      // events of earlier sessions, reused

hipEvent_t pooled_event() {
    if (!g_event_pool.empty()) {
        hipEvent_t e = g_event_pool.back();
        g_event_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
    return e;
}

// Brackets a launch with events while timing is on (caller holds g_mu).
struct TimedScope {
    hipStream_t stream;
    int index = -1;
    TimedScope(int kernel, hipStream_t s) : stream(s) {
        if (!g_timing || g_timing_off) return;
        TimedLaunch t{pooled_event(), pooled_event(), kernel};
        if (!t.a || !t.b) return;
        if (hipEventRecord(t.a, stream) != hipSuccess) { (void)hipGetLastError(); return; }
        g_timed.push_back(t);
        index = (int)g_timed.size() - 1;
    }
    ~TimedScope() {
        if (index >= 0 && hipEventRecord(g_timed[index].b, stream) != hipSuccess) (void)hipGetLastError();
    }
};

int check_launch(const char *what, hipError_t e) {
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(ANN_ERR_LAUNCH, "%s: %s", what, hipGetErrorString(e));
    }
    return ANN_OK;
}

int check_common(const void *corpus, int64_t N, int32_t d, int32_t dtype, const void *queries, int32_t B,
                 int32_t k, const void *ids, const void *scores) {
    if (dtype != ANN_F16 && dtype != ANN_BF16 && dtype != ANN_F32)
        return fail(ANN_ERR_INVALID, "unknown element type %d", dtype);
    if (!corpus || !queries || !ids || !scores) return fail(ANN_ERR_INVALID, "null pointer argument");
    if (N < 1 || N > INT32_MAX) return fail(ANN_ERR_INVALID, "N = %lld out of range", (long long)N);
    if (B < 1) return fail(ANN_ERR_INVALID, "B = %d out of range", B);
    if (d < 1 || d > ANN_D_MAX) return fail(ANN_ERR_INVALID, "d = %d out of range [1, %d]", d, ANN_D_MAX);
    if (k < 1 || k > N) return fail(ANN_ERR_INVALID, "k = %d out of range [1, N]", k);
    if ((d * elem_bytes(dtype)) % 16 != 0)
        return fail(ANN_ERR_ALIGNMENT, "d = %d: a row must be a whole number of 16-byte chunks", d);
    if ((reinterpret_cast<uintptr_t>(corpus) | reinterpret_cast<uintptr_t>(queries)) & 15)
        return fail(ANN_ERR_ALIGNMENT, "corpus and queries must be 16-byte aligned");
    if ((reinterpret_cast<uintptr_t>(ids) | reinterpret_cast<uintptr_t>(scores)) & 3)
        return fail(ANN_ERR_ALIGNMENT, "ids and scores must be 4-byte aligned");
    return ANN_OK;
}

int flat_search_run(const FlatPlan &pl, const void *X, int64_t N, int d, int dtype, const void *Q, int B, int k,
                    int32_t *ids, float *scores, void *ws, After after, hipStream_t stream) {
    // launches are recorded by the class of the call, as ann.h lists them, not by the kernel that its sizes choose
    const int code = dtype == ANN_F32 ? ANN_KERNEL_FLAT_F32
                     : B >= WIDE_MIN_B && d % 32 == 0 ? ANN_KERNEL_FLAT_WIDE : ANN_KERNEL_FLAT_STREAM;
    if (pl.quick) {
        TimedScope timed(code, stream);
        return check_launch("flat_direct_kernel",
                            launch_flat_direct(dtype, X, N, d, Q, B, k, ids, scores, after, stream));
    }
    if (pl.scores) {
        float *maxima = static_cast<float *>(ws);
        hipError_t e;
        {
            TimedScope timed(code, stream);
            e = launch_flat_scores(dtype, X, N, d, Q, B, maxima, pl.w.n, after, stream);
        }
        if (int rc = check_launch("flat_scores_kernel", e)) return rc;
        return check_launch("flat_pick_kernel",
                            launch_flat_pick(pl.w, dtype, X, N, d, Q, B, k, maxima, ids, scores, after, nullptr, 0, stream));
    }
    StreamOut direct;
    if (pl.direct) direct = StreamOut{ids, scores, k};
    auto stream_kernel = [&](const FlatPlan &one, const void *x, int64_t rows, const void *q, int b, Cand *partial, float *maxima,
                             After a) {
        return (dtype == ANN_F16 ? launch_flat_stream_f16 : dtype == ANN_BF16 ? launch_flat_stream_bf16 : launch_flat_stream_f32)(
            one.st, x, rows, d, q, b, partial, maxima, one.w.n, direct, a, stream);
    };
    if (pl.wide || pl.maxima) {
        float *maxima = static_cast<float *>(ws);
        uint64_t *best = reinterpret_cast<uint64_t *>(static_cast<char *>(ws) + pl.best_ofs);
        const size_t row_bytes = (size_t)d * elem_bytes(dtype);
        for (int q0 = 0; q0 < B; q0 += pl.part) {
            const int b = B - q0 < pl.part ? B - q0 : pl.part;
            const void *q = static_cast<const char *>(Q) + (size_t)q0 * row_bytes;
            for (int64_t r0 = 0; r0 < N; r0 += pl.rows) {
                const int64_t rows = N - r0 < pl.rows ? N - r0 : pl.rows;
                const void *x = static_cast<const char *>(X) + (size_t)r0 * row_bytes;
                const After a{after.s ? after.s + q0 : nullptr, after.id ? after.id + q0 : nullptr, (int)r0};
                FlatPlan last;
                const bool whole = rows == pl.rows && b == pl.part;
                if (!whole) last = maxima_part(pl, rows, b, d, dtype);
                const FlatPlan &one = whole ? pl : last;
                hipError_t e;
                {
                    TimedScope timed(code, stream);
                    e = one.wide ? launch_flat_wide(one.w, dtype, x, rows, d, q, b, maxima, a, stream)
                                 : stream_kernel(one, x, rows, q, b, nullptr, maxima, a);
                }
                if (int rc = check_launch(one.wide ? "flat_wide_kernel" : "flat_stream_kernel", e)) return rc;
                e = launch_flat_pick(one.w, dtype, x, rows, d, q, b, k, maxima, ids + (size_t)q0 * k, scores + (size_t)q0 * k, a,
                                     best, (r0 > 0 ? 1 : 0) | (r0 + rows < N ? 2 : 0), stream);
                if (int rc = check_launch("flat_pick_kernel", e)) return rc;
            }
        }
        return ANN_OK;
    }
    Cand *partial = static_cast<Cand *>(ws);
    hipError_t e;
    {
        TimedScope timed(code, stream);
        e = stream_kernel(pl, X, N, Q, B, partial, nullptr, after);
    }
    if (int rc = check_launch("flat_stream_kernel", e)) return rc;
    if (pl.direct) return ANN_OK;
    if (k > 4)
        return check_launch("flat_merge_lists_kernel",
                            launch_flat_merge_lists(dtype, partial, pl.st.P, pl.st.K, pl.st.slots(), X, N, d, Q, B, k, ids,
                                                    scores, after, stream));
    return check_launch("flat_merge_kernel", launch_flat_merge(partial, pl.st.P, B, k, ids, scores, stream));
}

}  // namespace

extern "C" {

int ann_version(void) { return 100; }

const char *ann_last_error(void) { return g_last_error.c_str(); }

int ann_set_default_dtype(int32_t dtype) {
    if (dtype != ANN_F16 && dtype != ANN_BF16 && dtype != ANN_F32)
        return fail(ANN_ERR_INVALID, "unknown element type %d", dtype);
    std::lock_guard<std::mutex> lock(g_mu);
    g_default_dtype = dtype;
    return ANN_OK;
}

int ann_register_corpus(const void *corpus, int64_t N, int32_t d, int32_t dtype) {
    if (!corpus || N < 1 || N > INT32_MAX || d < 1 || d > ANN_D_MAX ||
        (dtype != ANN_F16 && dtype != ANN_BF16 && dtype != ANN_F32))
        return fail(ANN_ERR_INVALID, "ann_register_corpus: bad shape or element type");
    std::lock_guard<std::mutex> lock(g_mu);
    g_corpora[corpus] = CorpusInfo{N, d, dtype};
    return ANN_OK;
}

int ann_unregister_corpus(const void *corpus) {
    std::lock_guard<std::mutex> lock(g_mu);
    g_corpora.erase(corpus);
    return ANN_OK;
}

int64_t ann_flat_workspace_bytes(int64_t N, int32_t d, int32_t dtype, int32_t B, int32_t k) {
    if (N < 1 || N > INT32_MAX || d < 1 || d > ANN_D_MAX || B < 1 || k < 1 || k > ANN_K_MAX || k > N) return ANN_ERR_INVALID;
    if (dtype != ANN_F16 && dtype != ANN_BF16 && dtype != ANN_F32) return ANN_ERR_INVALID;
    if ((d * elem_bytes(dtype)) % 16 != 0) return ANN_ERR_ALIGNMENT;
    std::lock_guard<std::mutex> lock(g_mu);
    DeviceState *st = nullptr;
    int cus = 256;
    if (device_state(&st) == ANN_OK) cus = st->cus;
    return (int64_t)flat_plan(cus, N, d, dtype, B, k, WIDE_WS_MAX).ws_bytes;
}

int ann_timing_enable(int32_t on) {
    std::lock_guard<std::mutex> lock(g_mu);
    if (on) {
        for (const TimedLaunch &t : g_timed) {
            g_event_pool.push_back(t.a);
            g_event_pool.push_back(t.b);
        }
        g_timed.clear();
    }
    g_timing = on != 0;
    return ANN_OK;
}

int ann_timing_read(int32_t kernel, int32_t *launches, double *total_ms) {
    if (!launches || !total_ms) return fail(ANN_ERR_INVALID, "null pointer argument");
    if (kernel < 0 || kernel >= ANN_KERNEL_COUNT) return fail(ANN_ERR_INVALID, "unknown kernel code %d", kernel);
    std::lock_guard<std::mutex> lock(g_mu);
    int n = 0;
    double sum = 0.0;
    for (const TimedLaunch &t : g_timed) {
        if (t.kernel != kernel) continue;
        float ms = 0.f;
        if (hipEventSynchronize(t.b) != hipSuccess || hipEventElapsedTime(&ms, t.a, t.b) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ANN_ERR_LAUNCH, "cannot read the events of a timed launch");
        }
        ++n;
        sum += ms;
    }
    *launches = n;
    *total_ms = sum;
    return ANN_OK;
}

int ann_timing_read_each(int32_t kernel, int32_t capacity, int32_t *launches, float *ms) {
    if (!launches || (capacity > 0 && !ms) || capacity < 0) return fail(ANN_ERR_INVALID, "bad arguments");
    if (kernel < 0 || kernel >= ANN_KERNEL_COUNT) return fail(ANN_ERR_INVALID, "unknown kernel code %d", kernel);
    std::lock_guard<std::mutex> lock(g_mu);
    int n = 0;
    for (const TimedLaunch &t : g_timed) {
        if (t.kernel != kernel) continue;
        float one = 0.f;
        if (hipEventSynchronize(t.b) != hipSuccess || hipEventElapsedTime(&one, t.a, t.b) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ANN_ERR_LAUNCH, "cannot read the events of a timed launch");
        }
        if (n < capacity) ms[n] = one;
        ++n;
    }
    *launches = n;
    return ANN_OK;
}

int ann_priority_order(const int32_t *R, const double *W, const int32_t *C, const double *Wcur, int32_t n, int32_t G,
                       int32_t *level, int32_t *order, void *stream) {
    if (n == 0) return ANN_OK;
    if (!R || !W || !C || !Wcur || !level || !order) return fail(ANN_ERR_INVALID, "null pointer argument");
    if (n < 1 || n > ANN_REQUESTS_MAX) return fail(ANN_ERR_INVALID, "n = %d out of range [1, %d]", n, ANN_REQUESTS_MAX);
    if (G < 1 || G > 1024) return fail(ANN_ERR_INVALID, "G = %d out of range [1, 1024]", G);
    if ((reinterpret_cast<uintptr_t>(W) | reinterpret_cast<uintptr_t>(Wcur)) & 7)
        return fail(ANN_ERR_ALIGNMENT, "W and Wcur must be 8-byte aligned");
    if ((reinterpret_cast<uintptr_t>(R) | reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(level) |
         reinterpret_cast<uintptr_t>(order)) & 3)
        return fail(ANN_ERR_ALIGNMENT, "R, C, level and order must be 4-byte aligned");
    return check_launch("priority kernels",
                        launch_priority(R, W, C, Wcur, n, G, level, order, static_cast<hipStream_t>(stream)));
}

int ann_measure_mfma_rate(int32_t random_operands, int32_t iters, double *tflops) {
    if (!tflops || iters < 1) return fail(ANN_ERR_INVALID, "ann_measure_mfma_rate: bad arguments");
    std::lock_guard<std::mutex> lock(g_mu);
    DeviceState *st = nullptr;
    if (int rc = device_state(&st)) return rc;
    if (int rc = grow(st, &st->ws, 256)) return rc;
    hipEvent_t a = pooled_event(), b = pooled_event();
    if (!a || !b) return fail(ANN_ERR_LAUNCH, "cannot create events");
    float ms = 0.f;
    hipError_t e = launch_mfma_rate(random_operands != 0, st->cus, iters, static_cast<float *>(st->ws.ptr), nullptr);   // warm-up
    if (e == hipSuccess) e = hipEventRecord(a, nullptr);
    if (e == hipSuccess) e = launch_mfma_rate(random_operands != 0, st->cus, iters, static_cast<float *>(st->ws.ptr), nullptr);
    if (e == hipSuccess) e = hipEventRecord(b, nullptr);
    if (e == hipSuccess) e = hipEventSynchronize(b);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, a, b);
    g_event_pool.push_back(a);
    g_event_pool.push_back(b);
    if (int rc = check_launch("mfma_rate_kernel", e)) return rc;
    *tflops = (double)st->cus * 8.0 * iters * 8.0 * 32768.0 / ((double)ms * 1e9);
    return ANN_OK;
}

int ann_set_workspace(void *workspace, int64_t bytes) {
    if (workspace && bytes < 1) return fail(ANN_ERR_INVALID, "ann_set_workspace: bytes = %lld", (long long)bytes);
    if (reinterpret_cast<uintptr_t>(workspace) & 255) return fail(ANN_ERR_ALIGNMENT, "the workspace must be 256-byte aligned");
    std::lock_guard<std::mutex> lock(g_mu);
    DeviceState *st = nullptr;
    if (int rc = device_state(&st)) return rc;
    st->user_ws = workspace;
    st->user_bytes = workspace ? (size_t)bytes : 0;
    return ANN_OK;
}

int ann_release_workspace(void) {
    std::lock_guard<std::mutex> lock(g_mu);
    DeviceState *st = nullptr;
    if (int rc = device_state(&st)) return rc;
    for (Buffer *b : {&st->ws, &st->vis}) {
        if (b->ptr) (void)hipFree(b->ptr);
        *b = Buffer();
    }
    for (void *p : st->kept) (void)hipFree(p);
    st->kept.clear();
    return ANN_OK;
}

int ann_flat_search_typed(const void *corpus, int64_t N, int32_t d, int32_t dtype, const void *queries,
                          int32_t B, int32_t k, int32_t *ids, float *scores, void *stream) {
    return ann_flat_search_after_typed(corpus, N, d, dtype, queries, B, k, nullptr, nullptr, ids, scores, stream);
}

int ann_flat_search_after_typed(const void *corpus, int64_t N, int32_t d, int32_t dtype, const void *queries,
                                int32_t B, int32_t k, const float *after_scores, const int32_t *after_ids,
                                int32_t *ids, float *scores, void *stream) {
    if (B == 0) return ANN_OK;                            // an empty batch: nothing to do
    if (int rc = check_common(corpus, N, d, dtype, queries, B, k, ids, scores)) return rc;
    if (k > ANN_K_MAX) return fail(ANN_ERR_INVALID, "k = %d exceeds ANN_K_MAX = %d", k, ANN_K_MAX);
    if ((after_scores == nullptr) != (after_ids == nullptr))
        return fail(ANN_ERR_INVALID, "after_scores and after_ids must be given together");
    if ((reinterpret_cast<uintptr_t>(after_scores) | reinterpret_cast<uintptr_t>(after_ids)) & 3)
        return fail(ANN_ERR_ALIGNMENT, "after_scores and after_ids must be 4-byte aligned");
    After after;
    after.s = after_scores;
    after.id = after_ids;
    std::lock_guard<std::mutex> lock(g_mu);
    DeviceState *st = nullptr;
    if (int rc = device_state(&st)) return rc;
    // (in a caller's buffer: in parts if it does not hold the whole)
    const size_t limit = st->user_ws && st->user_bytes < WIDE_WS_MAX ? st->user_bytes : WIDE_WS_MAX;
    hipStream_t s = static_cast<hipStream_t>(stream);
    FlatPlan pl = flat_plan(st->cus, N, d, dtype, B, k, limit);
    if (!st->user_ws && !at_hand(st, st->ws, pl.ws_bytes, s)) {         // (captured: in what there is, if that can be)
        const FlatPlan less = flat_plan(st->cus, N, d, dtype, B, k, st->ws.bytes);
        if (less.ws_bytes <= st->ws.bytes) pl = less;
    }
    void *ws = nullptr;
    if (int rc = workspace_for(st, &st->ws, pl.ws_bytes, s, &ws)) return rc;
    return flat_search_run(pl, corpus, N, d, dtype, queries, B, k, ids, scores, ws, after, s);
}

int ann_flat_search(const void *corpus, int64_t N, int32_t d, const void *queries, int32_t B, int32_t k,
                    int32_t *ids, float *scores, void *stream) {
    int dtype;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        dtype = g_default_dtype;
    }
    return ann_flat_search_typed(corpus, N, d, dtype, queries, B, k, ids, scores, stream);
}

int ann_flat_search_static(const void *corpus, int64_t N, int32_t d, int32_t dtype, const void *queries,
                           int32_t B, int32_t k, int32_t *ids, float *scores, void *stream) {
    if (B == 0) return ANN_OK;
    if (int rc = check_common(corpus, N, d, dtype, queries, B, k, ids, scores)) return rc;
    if (k > ANN_K_MAX) return fail(ANN_ERR_INVALID, "k = %d exceeds ANN_K_MAX = %d", k, ANN_K_MAX);
    std::lock_guard<std::mutex> lock(g_mu);
    DeviceState *st = nullptr;
    if (int rc = device_state(&st)) return rc;
    const FlatPlan pl = static_plan(st->cus, N, d, dtype, B, k, STATIC_BYTES);
    if (pl.ws_bytes > STATIC_BYTES)
        return fail(ANN_ERR_INVALID, "this search needs %zu bytes of workspace, the static one holds %d",
                    pl.ws_bytes, ANN_STATIC_WORKSPACE_BYTES);
    g_timing_off = true;                                  // event pairs would have to be created
    const int rc = flat_search_run(pl, corpus, N, d, dtype, queries, B, k, ids, scores,
                                   st->scratch_ptr, After(), static_cast<hipStream_t>(stream));
    g_timing_off = false;
    return rc;
}

static int check_graph(const void *corpus, int64_t N, int32_t d, int32_t dtype, const int32_t *graph, int32_t R,
                       int32_t entry, const void *queries, int32_t B, int32_t k, int32_t ef, const int32_t *ids,
                       const float *scores, GraphLds *L) {
    if (!graph) return fail(ANN_ERR_INVALID, "null graph pointer");
    if (R < 1 || R > ANN_R_MAX) return fail(ANN_ERR_INVALID, "R = %d out of range [1, %d]", R, ANN_R_MAX);
    if (ef < 1 || ef > ANN_EF_MAX) return fail(ANN_ERR_INVALID, "ef = %d out of range [1, %d]", ef, ANN_EF_MAX);
    if (int rc = check_common(corpus, N, d, dtype, queries, B, k, ids, scores)) return rc;
    if (k > ef) return fail(ANN_ERR_INVALID, "ef = %d is smaller than k = %d", ef, k);
    if (entry < 0 || entry >= N) return fail(ANN_ERR_INVALID, "entry = %d is not a node id", entry);
    if (reinterpret_cast<uintptr_t>(graph) & 3) return fail(ANN_ERR_ALIGNMENT, "graph must be 4-byte aligned");
    *L = graph_lds_layout(d, elem_bytes(dtype), R, ef);
    if (L->total > LDS_MAX) return fail(ANN_ERR_INVALID, "d = %d, ef = %d need %u bytes of LDS", d, ef, L->total);
    return ANN_OK;
}

// Graphs of at most 32 slots per node.  The visited set needs workspace only where it does not fit LDS.
static int graph_frontier_run(DeviceState *st, int32_t dtype, int32_t B, FrontierArgs args, bool counters, hipStream_t s) {
    if (args.L.vis_mode == FRONTIER_VIS_GLOBAL) {
        args.ns.words = visited_words(args.N);
        void *vis = nullptr;
        if (int rc = workspace_for(st, &st->vis, (size_t)B * (size_t)args.ns.words * 4, s, &vis)) return rc;
        args.ns.visited = static_cast<uint32_t *>(vis);
        if (int rc = check_launch("zero_words_kernel", launch_zero_words(args.ns.visited, (size_t)B * (size_t)args.ns.words, s))) return rc;
    }
    TimedScope timed(ANN_KERNEL_GRAPH, s);
    return check_launch("graph_frontier_kernel", launch_graph_frontier(dtype, B, args, counters, s));
}

// Whether graph_frontier_kernel takes a call, and its layout.  Where the call would want the workspace of the visited sets
// (`workspace`: the other kernel does) and that is not at hand, it takes it with the visited set in LDS if that fits.
static bool frontier_takes(const DeviceState *st, int64_t N, int32_t d, int32_t dtype, int32_t R, int32_t B, int32_t ef, bool counters,
                           float tau, float alpha, bool workspace, hipStream_t s, FrontierLds *L) {
    const int bytes = elem_bytes(dtype);
    *L = frontier_plan(st->cus, N, d, bytes, B, ef, counters && tau < 1.0f);
    const bool pays = frontier_pays(st->cus, N, d * bytes, R, B, ef, counters, counters && exit_likely(tau, alpha, R, ef), *L);
    if ((pays ? L->vis_mode == FRONTIER_VIS_GLOBAL : workspace) && !at_hand(st, st->vis, (size_t)B * (size_t)visited_words(N) * 4, s)) {
        FrontierLds in_lds;
        if (frontier_in_lds(N, d, bytes, R, ef, counters, in_lds)) {
            *L = in_lds;
            return true;
        }
    }
    return pays;
}

int64_t ann_graph_nonstall_workspace_bytes(int64_t N, int32_t B) {
    if (N < 1 || N > INT32_MAX || B < 1) return ANN_ERR_INVALID;
    return (int64_t)B * visited_words(N) * 4;
}

int ann_graph_search_nonstall_typed(const void *corpus, int64_t N, int32_t d, int32_t dtype, const int32_t *graph,
                                    int32_t R, int32_t entry, const void *queries, int32_t B, int32_t k, int32_t ef,
                                    const int32_t *entries, int32_t n_entries, float tau, int32_t window,
                                    const int32_t *engine_ready, int32_t *ids, float *scores, int32_t *stats,
                                    float *ema, void *stream) {
    if (B == 0) return ANN_OK;                            // an empty batch: nothing to do
    GraphLds L;
    if (int rc = check_graph(corpus, N, d, dtype, graph, R, entries ? 0 : entry, queries, B, k, ef, ids, scores, &L))
        return rc;
    if (reinterpret_cast<uintptr_t>(entries) & 3) return fail(ANN_ERR_ALIGNMENT, "entries must be 4-byte aligned");
    if (entries && (n_entries < 1 || n_entries > ANN_ENTRIES_MAX))
        return fail(ANN_ERR_INVALID, "n_entries = %d out of range [1, %d]", n_entries, ANN_ENTRIES_MAX);
    if (window < 1) return fail(ANN_ERR_INVALID, "window = %d must be at least 1", window);
    if (tau != tau) return fail(ANN_ERR_INVALID, "tau is not a number");
    if ((reinterpret_cast<uintptr_t>(engine_ready) | reinterpret_cast<uintptr_t>(stats) |
         reinterpret_cast<uintptr_t>(ema)) & 3)
        return fail(ANN_ERR_ALIGNMENT, "engine_ready, stats and ema must be 4-byte aligned");
    std::lock_guard<std::mutex> lock(g_mu);
    DeviceState *st = nullptr;
    if (int rc = device_state(&st)) return rc;
    NonStall ns;
    ns.entries = entries;
    ns.n_entries = n_entries;
    ns.tau = tau;
    ns.alpha = 2.0f / ((float)window + 1.0f);
    ns.ready = engine_ready;
    ns.words = visited_words(N);
    ns.stats = stats;
    ns.ema = ema;
    hipStream_t s = static_cast<hipStream_t>(stream);
    FrontierLds F;
    if (frontier_takes(st, N, d, dtype, R, B, ef, true, tau, ns.alpha, true, s, &F))
        return graph_frontier_run(st, dtype, B, FrontierArgs{corpus, N, d, R, graph, queries, entry, k, ef, ids, scores, F, ns}, true, s);
    void *vis = nullptr;
    if (int rc = workspace_for(st, &st->vis, (size_t)B * (size_t)ns.words * 4, s, &vis)) return rc;
    ns.visited = static_cast<uint32_t *>(vis);
    if (int rc = check_launch("zero_words_kernel", launch_zero_words(ns.visited, (size_t)B * (size_t)ns.words, s)))
        return rc;
    TimedScope timed(ANN_KERNEL_GRAPH, s);
    return check_launch("graph_search_kernel (non-stall)",
                        launch_graph_search_nonstall(dtype, corpus, N, d, graph, R, entry, queries, B, k, ef, ids,
                                                     scores, L, ns, s));
}

// Plain search.  Long lists (the two-level list, or more than GRAPH_EF_DOUBLE entries) score far
// more nodes than an id cache in LDS remembers, so they run on the kernel variant with the exact
// visited bitset, with an exit threshold no average can exceed.
static int graph_search_any(const void *corpus, int64_t N, int32_t d, int32_t dtype, const int32_t *graph, int32_t R,
                            int32_t entry, const int32_t *entries, int32_t n_entries, const void *queries, int32_t B, int32_t k,
                            int32_t ef, int32_t *ids, float *scores, const GraphLds &L, hipStream_t s) {
    std::lock_guard<std::mutex> lock(g_mu);
    DeviceState *st = nullptr;
    if (int rc = device_state(&st)) return rc;
    NonStall ns{};
    ns.entries = entries;
    ns.n_entries = n_entries;
    ns.tau = INFINITY;
    FrontierLds F;
    if (frontier_takes(st, N, d, dtype, R, B, ef, false, INFINITY, 0.f, L.two_level, s, &F))
        return graph_frontier_run(st, dtype, B, FrontierArgs{corpus, N, d, R, graph, queries, entry, k, ef, ids, scores, F, ns}, false, s);
    if (graph_step_pays(st->cus, N, d * elem_bytes(dtype), R, B, ef)) {
        const StepLds S = graph_step_plan(st->cus, d, elem_bytes(dtype), B, ef);
        TimedScope timed(ANN_KERNEL_GRAPH, s);
        return check_launch("graph_step_kernel", launch_graph_step(dtype, corpus, N, d, graph, R, entry, entries, n_entries, queries, B, k,
                                                                   ef, ids, scores, S, s));
    }
    if (ef <= GRAPH_EF_DOUBLE && !L.two_level) {
        TimedScope timed(ANN_KERNEL_GRAPH, s);
        return check_launch("graph_search_kernel", launch_graph_search(dtype, corpus, N, d, graph, R, entry, entries, n_entries,
                                                                       queries, B, k, ef, ids, scores, L, s));
    }
    ns.alpha = 0.f;
    ns.words = visited_words(N);
    void *vis = nullptr;
    if (int rc = workspace_for(st, &st->vis, (size_t)B * (size_t)ns.words * 4, s, &vis)) return rc;
    ns.visited = static_cast<uint32_t *>(vis);
    if (int rc = check_launch("zero_words_kernel", launch_zero_words(ns.visited, (size_t)B * (size_t)ns.words, s)))
        return rc;
    TimedScope timed(ANN_KERNEL_GRAPH, s);
    return check_launch("graph_search_kernel (long list)",
                        launch_graph_search_nonstall(dtype, corpus, N, d, graph, R, entry, queries, B, k, ef, ids,
                                                     scores, L, ns, s));
}

int ann_graph_search_typed(const void *corpus, int64_t N, int32_t d, int32_t dtype, const int32_t *graph,
                           int32_t R, int32_t entry, const void *queries, int32_t B, int32_t k, int32_t ef,
                           int32_t *ids, float *scores, void *stream) {
    if (B == 0) return ANN_OK;                            // an empty batch: nothing to do
    GraphLds L;
    if (int rc = check_graph(corpus, N, d, dtype, graph, R, entry, queries, B, k, ef, ids, scores, &L)) return rc;
    return graph_search_any(corpus, N, d, dtype, graph, R, entry, nullptr, 0, queries, B, k, ef, ids, scores, L,
                            static_cast<hipStream_t>(stream));
}

int ann_graph_search_multi_typed(const void *corpus, int64_t N, int32_t d, int32_t dtype, const int32_t *graph,
                                 int32_t R, const int32_t *entries, int32_t n_entries, const void *queries, int32_t B,
                                 int32_t k, int32_t ef, int32_t *ids, float *scores, void *stream) {
    if (B == 0) return ANN_OK;                            // an empty batch: nothing to do
    if (!entries) return fail(ANN_ERR_INVALID, "null entries pointer");
    if (reinterpret_cast<uintptr_t>(entries) & 3) return fail(ANN_ERR_ALIGNMENT, "entries must be 4-byte aligned");
    if (n_entries < 1 || n_entries > ANN_ENTRIES_MAX)
        return fail(ANN_ERR_INVALID, "n_entries = %d out of range [1, %d]", n_entries, ANN_ENTRIES_MAX);
    GraphLds L;
    if (int rc = check_graph(corpus, N, d, dtype, graph, R, 0, queries, B, k, ef, ids, scores, &L)) return rc;
    return graph_search_any(corpus, N, d, dtype, graph, R, 0, entries, n_entries, queries, B, k, ef, ids, scores, L,
                            static_cast<hipStream_t>(stream));
}

int ann_graph_search_entries_typed(const void *corpus, int64_t N, int32_t d, int32_t dtype, const int32_t *graph,
                                   int32_t R, const int32_t *entries, const void *queries, int32_t B, int32_t k,
                                   int32_t ef, int32_t *ids, float *scores, void *stream) {
    return ann_graph_search_multi_typed(corpus, N, d, dtype, graph, R, entries, 1, queries, B, k, ef, ids, scores, stream);
}

int ann_gather_ids(const int32_t *table, int64_t M, const int32_t *idx, int64_t n, int32_t *out, void *stream) {
    if (n == 0) return ANN_OK;
    if (!table || !idx || !out) return fail(ANN_ERR_INVALID, "null pointer argument");
    if (M < 1 || n < 1) return fail(ANN_ERR_INVALID, "M = %lld, n = %lld out of range", (long long)M, (long long)n);
    if ((reinterpret_cast<uintptr_t>(table) | reinterpret_cast<uintptr_t>(idx) | reinterpret_cast<uintptr_t>(out)) & 3)
        return fail(ANN_ERR_ALIGNMENT, "table, idx and out must be 4-byte aligned");
    return check_launch("gather_ids_kernel",
                        launch_gather_ids(table, M, idx, n, out, static_cast<hipStream_t>(stream)));
}

int ann_graph_search(const void *corpus, const int32_t *graph, int32_t R, int32_t entry, const void *queries,
                     int32_t B, int32_t k, int32_t ef, int32_t *ids, float *scores, void *stream) {
    CorpusInfo info;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        auto it = g_corpora.find(corpus);
        if (it == g_corpora.end())
            return fail(ANN_ERR_UNKNOWN_CORPUS, "corpus %p was never passed to ann_register_corpus", corpus);
        info = it->second;
    }
    return ann_graph_search_typed(corpus, info.N, info.d, info.dtype, graph, R, entry, queries, B, k, ef, ids,
                                  scores, stream);
}

}  // extern "C"
