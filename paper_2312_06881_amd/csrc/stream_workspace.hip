// Scratch of the forward pass and the input gradient (split_workspace): one
// buffer per (device, stream), from a stream-ordered pool per device, kept
// between calls and regrown in stream order (the old buffer is freed on the same
// stream).  Calls on one stream reuse it in order, calls on different streams
// never share it.
//
// Host threads.  A pass enqueues several launches on the buffer, and its reads
// are ordered only behind its own writes if no other pass on the stream enqueues
// in between.  So the buffer comes with its lock, which the pass keeps until its
// last launch is enqueued (WorkspaceHold): a few tens of nanoseconds when nobody
// else calls on that stream.
//
// hipStreamPerThread is one handle for a stream of each thread.  Its buffer is
// one all the same (threads come and go, so one for each would have no bound):
// a pass leaves an event behind, and a pass of another thread makes its own
// stream wait for it.
//
// Graphs.  A buffer handed out while its stream is being captured is part of
// the captured graph: it is never freed, so a replay after the stream's buffer
// was regrown still writes to memory of its own.
#include <atomic>
#include <new>

#include "dyad_internal.h"

namespace dyad {
namespace {

struct StreamBuffer {
    int dev;
    hipStream_t stream;
    std::mutex mu;           // the buffer, and the launches on it being enqueued
    void *ptr = nullptr;
    size_t bytes = 0;
    bool in_graph = false;   // a captured graph refers to ptr
    uint64_t thread = 0;     // hipStreamPerThread: whose pass was the last,
    hipEvent_t end = nullptr;   // and its end
    StreamBuffer *next;
    StreamBuffer(int d, hipStream_t s, StreamBuffer *n) : dev(d), stream(s), next(n) {}
};
std::mutex g_mu;             // the two below
hipMemPool_t g_pool[64] = {};
StreamBuffer *g_buffers = nullptr;   // kept until the process ends

StreamBuffer *buffer_of(int dev, hipStream_t s) {
    std::lock_guard<std::mutex> lock(g_mu);
    for (StreamBuffer *b = g_buffers; b; b = b->next)
        if (b->dev == dev && b->stream == s) return b;
    StreamBuffer *b = new (std::nothrow) StreamBuffer(dev, s, g_buffers);
    if (b) g_buffers = b;
    return b;
}

hipError_t pool_of(int dev, hipMemPool_t *out) {
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_mu);
    if (!g_pool[dev]) {
        hipMemPoolProps props = {};
        props.allocType = hipMemAllocationTypePinned;
        props.handleTypes = hipMemHandleTypeNone;
        props.location.type = hipMemLocationTypeDevice;
        props.location.id = dev;
        hipMemPool_t pool = nullptr;
        hipError_t e = hipMemPoolCreate(&pool, &props);
        if (e != hipSuccess) return e;
        uint64_t keep = UINT64_MAX;   // keep freed blocks in the pool
        e = hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep);
        if (e != hipSuccess) {
            (void)hipMemPoolDestroy(pool);
            return e;
        }
        g_pool[dev] = pool;
    }
    *out = g_pool[dev];
    return hipSuccess;
}

// A number for the calling thread that no later thread gets again.
uint64_t thread_number() {
    static std::atomic<uint64_t> count{0};
    static thread_local const uint64_t mine = ++count;
    return mine;
}

void mark_end(hipEvent_t e) {
    if (hipEventRecord(e, hipStreamPerThread) == hipSuccess) return;
    (void)hipGetLastError();
    (void)hipStreamSynchronize(hipStreamPerThread);
}

// Orders the calling thread's own stream behind the last pass on `b`.
hipError_t order_threads(StreamBuffer *b, WorkspaceHold *hold, bool capturing) {
    const uint64_t me = thread_number();
    if (capturing)   // (a captured stream cannot wait for work outside its graph)
        return b->thread == me ? hipSuccess : hipErrorNotSupported;
    if (!b->end) {
        hipError_t e = hipEventCreateWithFlags(&b->end, hipEventDisableTiming);
        if (e != hipSuccess) return e;
    }
    if (b->thread != 0 && b->thread != me) {
        hipError_t e = hipStreamWaitEvent(hipStreamPerThread, b->end, 0);
        if (e != hipSuccess) return e;
    }
    b->thread = me;
    hold->at_end(mark_end, b->end);
    return hipSuccess;
}

}  // namespace

hipError_t split_workspace(hipStream_t s, size_t bytes, void **out) {
    if (const ScratchScope *sc = current_scratch()) {
        // the fixed scratch of dyad_forward_noalloc: never grown, never allocated
        if (bytes > sc->bytes) return hipErrorOutOfMemory;
        *out = sc->ptr;
        return hipSuccess;
    }
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    WorkspaceHold *hold = WorkspaceHold::current();
    if (!hold) return hipErrorNotSupported;   // nothing would order this pass's launches
    StreamBuffer *b = buffer_of(dev, s);
    if (!b) return hipErrorOutOfMemory;
    const bool first = hold->take(b->mu);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    e = hipStreamIsCapturing(s, &cap);
    const bool capturing = e == hipSuccess && cap != hipStreamCaptureStatusNone;
    if (s == hipStreamPerThread && first) {
        const hipError_t o = order_threads(b, hold, capturing);
        if (o != hipSuccess) return o;
    }
    if (b->bytes >= bytes) {
        if (e != hipSuccess) (void)hipGetLastError();
        b->in_graph = b->in_graph || capturing;
        *out = b->ptr;
        return hipSuccess;
    }
    // No allocation (or regrowth) while the stream is being captured into a
    // graph: the buffer would belong to the graph, not to later eager calls.
    // The caller then takes a plan that needs no buffer.
    if (e != hipSuccess) return e;
    if (capturing) return hipErrorNotSupported;
    hipMemPool_t pool;
    e = pool_of(dev, &pool);
    if (e != hipSuccess) return e;
    const size_t want = bytes < ((size_t)1 << 20) ? ((size_t)1 << 20) : bytes;
    void *p = nullptr;
    e = hipMallocFromPoolAsync(&p, want, pool, s);
    if (e != hipSuccess) return e;
    if (b->ptr && !b->in_graph) (void)hipFreeAsync(b->ptr, s);
    b->ptr = p;
    b->bytes = want;
    b->in_graph = false;
    *out = p;
    return hipSuccess;
}

}  // namespace dyad
