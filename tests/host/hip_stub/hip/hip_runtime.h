// Host-only stand-in for the few HIP runtime calls the swap engine makes, so that its host logic (state machine, arena,
// planner, error paths) can be built with g++ and the address / undefined-behaviour sanitizers and run without a GPU.
// "Device" memory is host memory, copies run at once, streams are in order by construction.  Events either fire at
// once or, while hipstub_hold_events is set, stay pending until hipstub_fire_events() (to reach the code paths that
// deal with copies still in flight).  Beside that, a stream can be stalled (hipstub_stall): what is enqueued on it from then
// on does not run, nor does what waits for that on other streams, and a host call that would block on it is counted
// (hipstub_hangs) instead of blocking.
#pragma once
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __restrict__
#define __launch_bounds__(...)

typedef int hipError_t;
enum { hipSuccess = 0, hipErrorNotReady = 600, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2 };
typedef struct hipstub_stream* hipStream_t;
#define hipStreamPerThread ((hipStream_t)2)
struct hipstub_event { bool recorded = false; bool fired = false; hipStream_t stream = nullptr; size_t at = 0; };
typedef hipstub_event* hipEvent_t;
enum { hipHostMallocDefault = 0, hipStreamNonBlocking = 1, hipEventDefault = 0, hipEventDisableTiming = 2 };
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2 };

inline bool& hipstub_hold_events() { static bool hold = false; return hold; }
inline std::set<hipstub_event*>& hipstub_pending() { static std::set<hipstub_event*> p; return p; }
inline void hipstub_fire_events() {
    for (hipstub_event* e : hipstub_pending()) e->fired = true;
    hipstub_pending().clear();
}
// Operations of a stream that can keep what is behind them from running: a stall, or a wait for a place in another stream
struct hipstub_op { bool stall; hipStream_t stream; size_t at; };
inline std::map<hipStream_t, std::vector<hipstub_op>>& hipstub_ops() { static std::map<hipStream_t, std::vector<hipstub_op>> o; return o; }
inline bool hipstub_runs(hipStream_t s, size_t at) {    // everything before place `at` of the stream
    for (size_t i = 0; i < at; ++i) {
        const hipstub_op& o = hipstub_ops()[s][i];
        if (o.stall || !hipstub_runs(o.stream, o.at)) return false;
    }
    return true;
}
inline void hipstub_stall(hipStream_t s) { hipstub_ops()[s].push_back(hipstub_op{true, nullptr, 0}); }
inline void hipstub_unstall(hipStream_t s) { for (hipstub_op& o : hipstub_ops()[s]) o.stall = false; }
inline int& hipstub_hangs() { static int n = 0; return n; }
inline int& hipstub_fail_event_syncs() { static int n = 0; return n; }   // the next n waits for an event report an error
inline int& hipstub_fail_event_records() { static int n = 0; return n; } // a record of an event fails when this counts down to zero
inline int& hipstub_event_syncs() { static int n = 0; return n; }        // host calls that waited for an event ...
inline int& hipstub_stream_syncs() { static int n = 0; return n; }       // ... and for a stream
inline std::set<hipStream_t>& hipstub_streams() { static std::set<hipStream_t> s; return s; }   // created and not destroyed
inline int& hipstub_live_objects() { static int n = 0; return n; }   // streams + events + host allocations not yet destroyed

inline unsigned __float_as_uint(float f) { unsigned u; std::memcpy(&u, &f, 4); return u; }
inline float __uint_as_float(unsigned u) { float f; std::memcpy(&f, &u, 4); return f; }

inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { hipstub_fire_events(); return hipSuccess; }
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n); ++hipstub_live_objects(); return *p ? hipSuccess : hipErrorInvalidValue; }
inline hipError_t hipHostFree(void* p) { std::free(p); --hipstub_live_objects(); return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)std::malloc(1); hipstub_streams().insert(*s); hipstub_ops()[*s].clear(); ++hipstub_live_objects(); return hipSuccess; }
inline hipError_t hipStreamDestroy(hipStream_t s) { hipstub_streams().erase(s); std::free(s); --hipstub_live_objects(); return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t s) {
    ++hipstub_stream_syncs();
    if (!hipstub_runs(s, hipstub_ops()[s].size())) ++hipstub_hangs();
    hipstub_fire_events();
    return hipSuccess;
}
inline hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    if (e->recorded && !hipstub_runs(e->stream, e->at)) hipstub_ops()[s].push_back(hipstub_op{false, e->stream, e->at});
    return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = new hipstub_event(); ++hipstub_live_objects(); return hipSuccess; }
inline hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
inline hipError_t hipEventDestroy(hipEvent_t e) { hipstub_pending().erase(e); delete e; --hipstub_live_objects(); return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    if (hipstub_fail_event_records() && !--hipstub_fail_event_records()) return hipErrorInvalidValue;
    e->recorded = true;
    e->stream = s;
    e->at = hipstub_ops()[s].size();
    e->fired = !hipstub_hold_events();
    if (!e->fired) hipstub_pending().insert(e);
    else hipstub_pending().erase(e);
    return hipSuccess;
}
inline hipError_t hipEventQuery(hipEvent_t e) { return !e->recorded || (e->fired && hipstub_runs(e->stream, e->at)) ? hipSuccess : hipErrorNotReady; }
inline hipError_t hipEventSynchronize(hipEvent_t e) {
    ++hipstub_event_syncs();
    if (hipstub_fail_event_syncs()) { --hipstub_fail_event_syncs(); return hipErrorInvalidValue; }
    if (e->recorded && !hipstub_runs(e->stream, e->at)) ++hipstub_hangs();
    e->fired = true;
    hipstub_pending().erase(e);
    return hipSuccess;
}
inline hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
inline hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(dst, src, n); return hipSuccess; }
