// Host-only check of the per-stream scratch buffer (stream_workspace.hip) with a
// mock of the HIP calls it makes, built under ThreadSanitizer: two host threads
// on one stream, two streams, the stream handle that is another stream in each
// thread, and a buffer that a captured graph refers to.
#include <stdio.h>
#include <stdlib.h>

#include <thread>
#include <vector>

#include "dyad_internal.h"

namespace {

std::mutex g_mock;
bool g_capturing = false;
std::vector<void *> g_freed;
// events, as the work of a thread's own stream that they stand for
std::vector<std::thread::id> g_recorded;
std::vector<std::pair<std::thread::id, std::thread::id>> g_waits;   // (who waits, for whom)

}  // namespace

extern "C" {

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *c) {
    *c = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipMemPoolCreate(hipMemPool_t *p, const hipMemPoolProps *) { *p = (hipMemPool_t)0x10; return hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void *) { return hipSuccess; }
hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void **p, size_t n, hipMemPool_t, hipStream_t) {
    *p = malloc(n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFreeAsync(void *p, hipStream_t) {
    std::lock_guard<std::mutex> lock(g_mock);
    g_freed.push_back(p);      // kept allocated: its address stays its own
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    std::lock_guard<std::mutex> lock(g_mock);
    g_recorded.emplace_back();
    *e = (hipEvent_t)g_recorded.size();
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    std::lock_guard<std::mutex> lock(g_mock);
    if (s != hipStreamPerThread) return hipErrorInvalidHandle;
    g_recorded[(size_t)e - 1] = std::this_thread::get_id();
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    std::lock_guard<std::mutex> lock(g_mock);
    if (s != hipStreamPerThread) return hipErrorInvalidHandle;
    g_waits.emplace_back(std::this_thread::get_id(), g_recorded[(size_t)e - 1]);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

}  // extern "C"

namespace dyad {
const ScratchScope *current_scratch() { return nullptr; }
}  // namespace dyad

static int failures = 0;

#define EXPECT(cond)                                                  \
    do {                                                              \
        if (!(cond)) {                                                \
            fprintf(stderr, "FAILED line %d: %s\n", __LINE__, #cond); \
            ++failures;                                               \
        }                                                             \
    } while (0)

// A pass of two launches that pass data in the buffer: plain writes and reads in
// enqueue order stand in for the kernels.
static int pass(hipStream_t s, int id, size_t bytes) {
    const dyad::WorkspaceHold hold;
    void *p = nullptr;
    if (dyad::split_workspace(s, bytes, &p) != hipSuccess) return 1;
    int *buf = static_cast<int *>(p);
    for (int i = 0; i < 64; ++i) buf[i] = id;
    std::this_thread::yield();
    int bad = 0;
    for (int i = 0; i < 64; ++i) bad += buf[i] != id;
    return bad;
}

int main() {
    using dyad::split_workspace;
    const hipStream_t s1 = (hipStream_t)0x100, s2 = (hipStream_t)0x200;
    void *p = nullptr;
    // a pass that holds nothing gets no buffer
    EXPECT(split_workspace(s1, 1024, &p) != hipSuccess);

    // two host threads on one stream, growing the buffer now and then
    int bad[2] = {0, 0};
    std::vector<std::thread> t;
    for (int id = 0; id < 2; ++id)
        t.emplace_back([&, id] {
            for (int i = 0; i < 3000; ++i) bad[id] += pass(s1, id + 1, (size_t)(1 + i / 1000) << 21);
        });
    for (auto &x : t) x.join();
    EXPECT(bad[0] == 0 && bad[1] == 0);
    EXPECT(g_freed.size() == 2);          // 2 -> 4 -> 6 MiB

    // streams have buffers of their own, and one stream's pass does not wait for another's
    {
        const dyad::WorkspaceHold hold;
        void *a = nullptr, *b = nullptr;
        EXPECT(split_workspace(s1, 1024, &a) == hipSuccess);
        std::thread other([&] {
            const dyad::WorkspaceHold mine;
            EXPECT(split_workspace(s2, 1024, &b) == hipSuccess);
        });
        other.join();
        EXPECT(a && b && a != b);
        // asked again within the pass: the same buffer
        EXPECT(split_workspace(s1, 2048, &p) == hipSuccess && p == a);
    }

    // one handle, a stream of each thread: a pass waits for the last one of another thread
    {
        std::vector<std::pair<std::thread::id, std::thread::id>> expect;
        const std::thread::id me = std::this_thread::get_id();
        EXPECT(pass(hipStreamPerThread, 1, 4096) == 0);
        EXPECT(pass(hipStreamPerThread, 2, 4096) == 0);
        EXPECT(g_waits.empty());
        std::thread other([&] {
            EXPECT(pass(hipStreamPerThread, 3, 4096) == 0);
            EXPECT(pass(hipStreamPerThread, 4, (size_t)2 << 20) == 0);
            expect.emplace_back(std::this_thread::get_id(), me);
            expect.emplace_back(me, std::this_thread::get_id());
        });
        other.join();
        EXPECT(pass(hipStreamPerThread, 5, 4096) == 0);
        EXPECT(g_waits == expect);
        // under capture a wait for another thread's work has no place: no buffer
        g_capturing = true;
        EXPECT(pass(hipStreamPerThread, 6, 4096) == 0);
        std::thread late([&] { EXPECT(pass(hipStreamPerThread, 7, 4096) != 0); });
        late.join();
        g_capturing = false;
        EXPECT(g_waits == expect);
    }

    // under capture: the buffer that is there, never a new one; and it outlives a later growth
    void *captured = nullptr, *grown = nullptr;
    g_freed.clear();
    g_capturing = true;
    {
        const dyad::WorkspaceHold hold;
        EXPECT(split_workspace(s2, (size_t)8 << 20, &p) == hipErrorNotSupported);
        EXPECT(split_workspace(s2, 4096, &captured) == hipSuccess);
    }
    g_capturing = false;
    {
        const dyad::WorkspaceHold hold;
        EXPECT(split_workspace(s2, (size_t)8 << 20, &grown) == hipSuccess && grown != captured);
        EXPECT(g_freed.empty());
        EXPECT(split_workspace(s2, (size_t)9 << 20, &p) == hipSuccess && p != grown);
        EXPECT(g_freed.size() == 1 && g_freed[0] == grown);
    }
    if (failures) return 1;
    printf("workspace mock ok\n");
    return 0;
}
