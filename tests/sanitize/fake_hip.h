// The parts of the HIP runtime that tc_host.cpp calls, on the CPU, for programs that look at what
// the library enqueues and at how long the memory it hands out must live.
//
//  - A stream is a queue: nothing enqueued runs before something waits for it (run_stream, an event,
//    hipStreamSynchronize, hipDeviceSynchronize), which is the latest that a GPU may run it.
//  - hipHostFree frees at once and waits for nothing, so memory freed under work that is still
//    queued is a use after free when that work runs.  A program built with AddressSanitizer stops there.
//  - A captured call becomes a node of the stream's graph; launching an executable graph enqueues its
//    nodes, which read their source pointers then.  User objects live as long as a graph or an
//    executable graph that holds them.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <set>
#include <vector>

namespace fake {

using Op = std::function<void()>;

struct UserObject {
    void* ptr;
    hipHostFn_t destroy;
    ~UserObject() { destroy(ptr); }
};

struct Graph {
    std::vector<Op> nodes;
    std::vector<std::shared_ptr<UserObject>> held;
};

struct Stream {
    std::deque<Op> queue;
    size_t done = 0;              // operations run so far
    Graph* capture = nullptr;
};

struct Event {
    Stream* stream = nullptr;
    size_t pos = 0;               // operations of the stream it waits for
};

inline std::map<hipStream_t, Stream>& streams()
{
    static std::map<hipStream_t, Stream> s;
    return s;
}
inline Stream& stream(void* s) { return streams()[static_cast<hipStream_t>(s)]; }
inline std::set<void*>& pinned()
{
    static std::set<void*> p;
    return p;
}

inline void run_to(Stream& s, size_t pos)
{
    while (s.done < pos && !s.queue.empty()) {
        Op op = std::move(s.queue.front());
        s.queue.pop_front();
        op();
        ++s.done;
    }
}
inline void run_stream(void* s) { run_to(stream(s), (size_t)-1); }

inline void enqueue(void* s, Op op)
{
    Stream& q = stream(s);
    if (q.capture) q.capture->nodes.push_back(std::move(op));
    else q.queue.push_back(std::move(op));
}

}  // namespace fake

extern "C" {

const char* hipGetErrorString(hipError_t) { return "fake runtime error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 160 * 1024; return hipSuccess; }
hipError_t hipDeviceSynchronize(void)
{
    for (auto& s : fake::streams()) fake::run_to(s.second, (size_t)-1);
    return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned int)
{
    *p = std::malloc(n);
    fake::pinned().insert(*p);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    fake::pinned().erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned int) { *d = h; return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st)
{
    // a copy from pageable memory has read it when the call returns, unless it is captured
    if (!fake::stream(st).capture && !fake::pinned().count(const_cast<void*>(s))) {
        std::shared_ptr<char> staged(new char[n], std::default_delete<char[]>());
        std::memcpy(staged.get(), s, n);
        fake::enqueue(st, [=] { std::memcpy(d, staged.get(), n); });
        return hipSuccess;
    }
    fake::enqueue(st, [=] { std::memcpy(d, s, n); });
    return hipSuccess;
}

hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(new fake::Event); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<fake::Event*>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    fake::Event& v = *reinterpret_cast<fake::Event*>(e);
    v.stream = &fake::stream(s);
    v.pos = v.stream->done + v.stream->queue.size();
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    fake::Event& v = *reinterpret_cast<fake::Event*>(e);
    if (v.stream) fake::run_to(*v.stream, v.pos);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(new int); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { fake::run_stream(s); fake::streams().erase(s); delete reinterpret_cast<int*>(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { fake::run_stream(s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) { fake::stream(s).capture = new fake::Graph; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g)
{
    *g = reinterpret_cast<hipGraph_t>(fake::stream(s).capture);
    fake::stream(s).capture = nullptr;
    return hipSuccess;
}
hipError_t hipStreamGetCaptureInfo_v2(hipStream_t s, hipStreamCaptureStatus* st, unsigned long long* id, hipGraph_t* g,
                                      const hipGraphNode_t** deps, size_t* n)
{
    fake::Graph* c = fake::stream(s).capture;
    *st = c ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    if (id) *id = c ? 1 : 0;
    if (g) *g = reinterpret_cast<hipGraph_t>(c);
    if (deps) *deps = nullptr;
    if (n) *n = 0;
    return hipSuccess;
}

hipError_t hipUserObjectCreate(hipUserObject_t* o, void* p, hipHostFn_t f, unsigned, unsigned)
{
    *o = reinterpret_cast<hipUserObject_t>(new std::shared_ptr<fake::UserObject>(new fake::UserObject{p, f}));
    return hipSuccess;
}
hipError_t hipUserObjectRelease(hipUserObject_t o, unsigned)
{
    delete reinterpret_cast<std::shared_ptr<fake::UserObject>*>(o);
    return hipSuccess;
}
hipError_t hipGraphRetainUserObject(hipGraph_t g, hipUserObject_t o, unsigned, unsigned flags)
{
    reinterpret_cast<fake::Graph*>(g)->held.push_back(*reinterpret_cast<std::shared_ptr<fake::UserObject>*>(o));
    return flags == hipGraphUserObjectMove ? hipUserObjectRelease(o, 1) : hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t)
{
    *e = reinterpret_cast<hipGraphExec_t>(new fake::Graph(*reinterpret_cast<fake::Graph*>(g)));
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s)
{
    for (const fake::Op& op : reinterpret_cast<fake::Graph*>(e)->nodes) fake::enqueue(s, op);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete reinterpret_cast<fake::Graph*>(g); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { delete reinterpret_cast<fake::Graph*>(e); return hipSuccess; }

}  // extern "C"
