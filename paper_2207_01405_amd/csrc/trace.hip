// Optional per-launch timing with HIP events (ivit_trace_begin / ivit_trace_end in include/ivit.h).
// While a trace is active every kernel launch of the library is bracketed by two events recorded on the
// stream the kernel is launched on; ivit_trace_end synchronises the last event and reports the elapsed
// time, the kind and the algorithmic work of every launch.  Inactive, the cost is one pointer test per launch.
#include <new>

#include "../../include/ivit.h"
#include "ivit_kernels.hpp"

namespace ivit {

namespace {
struct Record { hipEvent_t start, stop; int32_t kind; int64_t ops, bytes; };
struct Trace {
    Record* rec = nullptr;                   // room for `capacity` launches, allocated without exceptions
    int capacity = 0, count = 0;
    bool failed = false;

    bool create(int n) {
        rec = new (std::nothrow) Record[n]();
        if (!rec) return false;
        for (; capacity < n; ++capacity) {
            Record& r = rec[capacity];
            if (hipEventCreate(&r.start) != hipSuccess) return false;
            if (hipEventCreate(&r.stop) != hipSuccess) { (void)hipEventDestroy(r.start); return false; }
        }
        return true;
    }
    ~Trace() {
        for (int i = 0; i < capacity; ++i) { (void)hipEventDestroy(rec[i].start); (void)hipEventDestroy(rec[i].stop); }
        delete[] rec;
    }
};
Trace* g_trace = nullptr;
}  // namespace

TraceScope::TraceScope(hipStream_t s, int kind, int64_t ops, int64_t bytes) : stream_(s), slot_(-1) {
    Trace* t = g_trace;
    if (!t) return;
    if (t->count >= t->capacity) { t->failed = true; return; }
    slot_ = t->count++;
    Record& r = t->rec[slot_];
    r.kind = kind; r.ops = ops; r.bytes = bytes;
    if (hipEventRecord(r.start, s) != hipSuccess) t->failed = true;
}

TraceScope::~TraceScope() {
    Trace* t = g_trace;
    if (!t || slot_ < 0) return;
    if (hipEventRecord(t->rec[slot_].stop, stream_) != hipSuccess) t->failed = true;
}

}  // namespace ivit

extern "C" {

int ivit_trace_begin(int32_t max_launches) {
    using namespace ivit;
    if (max_launches < 1 || max_launches > (1 << 22)) return IVIT_ERR_SHAPE;
    if (g_trace) return IVIT_ERR_PARAM;                       // a trace is already active
    Trace* t = new (std::nothrow) Trace();
    if (!t || !t->create(max_launches)) {
        delete t;
        return IVIT_ERR_HIP;
    }
    g_trace = t;
    return IVIT_OK;
}

int ivit_trace_end(float* ms, int32_t* kind, int64_t* ops, int64_t* bytes, int32_t capacity, int32_t* count) {
    using namespace ivit;
    Trace* t = g_trace;
    if (!t) return IVIT_ERR_PARAM;
    g_trace = nullptr;
    int status = t->failed ? IVIT_ERR_HIP : IVIT_OK;
    const int n = t->count;
    if (count) *count = n;
    for (int i = 0; i < n && status == IVIT_OK; ++i) {
        const Record& r = t->rec[i];
        if (hipEventSynchronize(r.stop) != hipSuccess) { status = IVIT_ERR_HIP; break; }
        if (i < capacity) {
            if (ms && hipEventElapsedTime(&ms[i], r.start, r.stop) != hipSuccess) { status = IVIT_ERR_HIP; break; }
            if (kind) kind[i] = r.kind;
            if (ops) ops[i] = r.ops;
            if (bytes) bytes[i] = r.bytes;
        }
    }
    delete t;
    return status;
}

}  // extern "C"
