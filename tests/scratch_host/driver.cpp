// The kept scratch (tx_scratch.cpp) over simulated streams, events and a card
// of limited memory.  `driver NAME` runs one check and ends with 0 if it holds.
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "../../paper_2401_13834_amd/csrc/tx_internal.h"

struct Stream {
    int queued = 0, done = 0;          // work items
    bool capturing = false, record_fails = false, sync_fails = false;
};
struct Event {
    Stream* s = nullptr;
    int at = 0;                        // complete once s->done >= at
};

static std::recursive_mutex sim;
static size_t memory_left = size_t(1) << 40;
static std::map<void*, size_t> live;
static int mallocs = 0, frees = 0, pool_mallocs = 0;
static thread_local int device = 0;
static thread_local hipError_t last_error = hipSuccess;
static void (*in_malloc)() = nullptr;  // called from hipMalloc and hipFree
static void (*in_free)() = nullptr;

static hipError_t say(hipError_t e) {
    if (e != hipSuccess) last_error = e;
    return e;
}
static hipError_t get(void** p, size_t bytes) {
    std::lock_guard<std::recursive_mutex> l(sim);
    if (bytes > memory_left) return say(hipErrorOutOfMemory);
    memory_left -= bytes;
    *p = std::malloc(1);
    live[*p] = bytes;
    return hipSuccess;
}
static hipError_t put(void* p) {
    std::lock_guard<std::recursive_mutex> l(sim);
    if (!live.count(p)) return say(hipErrorInvalidValue);
    memory_left += live[p];
    live.erase(p);
    return hipSuccess;                 // (the address is not given out again)
}

hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = last_error; last_error = hipSuccess; return e; }
hipError_t hipPeekAtLastError() { return last_error; }
hipError_t hipMalloc(void** p, size_t bytes) {
    if (in_malloc) in_malloc();
    ++mallocs;
    return get(p, bytes);
}
hipError_t hipFree(void* p) {
    if (in_free) in_free();
    ++frees;
    return put(p);
}
hipError_t hipMallocAsync(void** p, size_t bytes, hipStream_t) { ++pool_mallocs; return get(p, bytes); }
hipError_t hipFreeAsync(void* p, hipStream_t) { return put(p); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = new Event; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    std::lock_guard<std::recursive_mutex> l(sim);
    if (s->record_fails) return say(hipErrorUnknown);
    e->s = s;
    e->at = s->queued;
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    std::lock_guard<std::recursive_mutex> l(sim);
    return !e->s || e->s->done >= e->at ? hipSuccess : say(hipErrorNotReady);
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    std::lock_guard<std::recursive_mutex> l(sim);
    if (e->s && e->s->done < e->at) e->s->done = e->at;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    std::lock_guard<std::recursive_mutex> l(sim);
    if (s->sync_fails) return say(hipErrorUnknown);
    s->done = s->queued;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
    *c = s->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }

#define CHECK(c)                                                            \
    do {                                                                    \
        if (!(c)) {                                                         \
            std::fprintf(stderr, "line %d: %s\n", __LINE__, #c);            \
            std::exit(1);                                                   \
        }                                                                   \
    } while (0)

constexpr size_t MB = size_t(1) << 20;

static tx::Scratch take(size_t bytes, Stream* s) {
    tx::Scratch x;
    CHECK(tx::scratch_get(bytes, s, &x) == hipSuccess);
    CHECK(x.p);
    ++s->queued;                       // the call's kernels
    return x;
}

// Kept buffers are taken again: on the same stream at once, on another when
// the work behind them is done; captures and large buffers use the pool.
static void reuse() {
    Stream a, b, c;
    c.capturing = true;
    tx::Scratch x = take(MB, &a);
    void* p = x.p;
    CHECK(x.kept);
    CHECK(tx::scratch_put(&x, &a) == hipSuccess && !x.p);
    tx::Scratch y = take(3 * MB, &b);  // a's work has not ended
    CHECK(y.p != p);
    CHECK(tx::scratch_put(&y, &b) == hipSuccess);
    x = take(4 * MB, &a);
    CHECK(x.p == p);
    CHECK(tx::scratch_put(&x, &a) == hipSuccess);
    a.done = a.queued;
    b.done = b.queued;
    x = take(MB, &b);
    y = take(MB, &a);
    CHECK(mallocs == 2 && x.p != y.p);
    CHECK(tx::scratch_put(&x, &b) == hipSuccess && tx::scratch_put(&y, &a) == hipSuccess);
    for (Stream* s : {&a, &c}) {
        x = take(s == &c ? MB : 65 * MB, s);
        CHECK(!x.kept);
        CHECK(tx::scratch_put(&x, s) == hipSuccess);
    }
    CHECK(pool_mallocs == 2);
    tx::scratch_trim(0);
    CHECK(frees == 2 && live.empty());
}

// A buffer whose last work is unknown (neither the event nor the wait worked)
// is not handed out again before a trim, which follows a device synchronisation.
static void lost() {
    Stream a, b;
    tx::Scratch x = take(MB, &a);
    void* p = x.p;
    a.record_fails = a.sync_fails = true;
    CHECK(tx::scratch_put(&x, &a) != hipSuccess);
    for (Stream* s : {&b, &a}) {
        tx::Scratch y = take(MB, s);
        CHECK(y.p != p);
        s->record_fails = s->sync_fails = false;
        CHECK(tx::scratch_put(&y, s) == hipSuccess);
        s->done = s->queued;
    }
    tx::scratch_trim(0);
    CHECK(live.empty());
}

// A call that the card has no room for beside the kept buffers gets theirs, once
// the work in them is done; buffers in use stay.
static void memory() {
    Stream a, b;
    tx::Scratch x = take(64 * MB, &a), y = take(MB, &a);
    CHECK(tx::scratch_put(&x, &a) == hipSuccess);
    memory_left = 50 * MB;
    x = take(100 * MB, &b);
    CHECK(!x.kept && a.done == 2);
    CHECK(live.size() == 2 && live.count(y.p));
    tx::Scratch z;
    CHECK(tx::scratch_get(100 * MB, &b, &z) == hipErrorOutOfMemory && !z.p);
    CHECK(tx::scratch_put(&z, &b) == hipSuccess);
    CHECK(tx::scratch_put(&x, &b) == hipSuccess && tx::scratch_put(&y, &a) == hipSuccess);
    a.capturing = true;                // a capture touches nothing that is kept
    CHECK(tx::scratch_get(200 * MB, &a, &z) == hipErrorOutOfMemory && live.size() == 1);
    tx::scratch_trim(0);
    CHECK(live.empty());
}

static void fill(std::vector<tx::Scratch>* x, int n, size_t bytes, Stream* s) {
    for (int i = 0; i < n; ++i) x->push_back(take(bytes, s));
}

static void empty(std::vector<tx::Scratch>* x, Stream* s) {
    for (tx::Scratch& y : *x) CHECK(tx::scratch_put(&y, s) == hipSuccess);
    x->clear();
}

// No slot (16 buffers) or no room (512 MB) left: the smallest idle buffers make
// way for a larger one; pending ones and those in use do not.
static void room() {
    Stream a, b;
    std::vector<tx::Scratch> x, y;
    fill(&x, 16, MB, &a);
    empty(&x, &a);
    x.push_back(take(5 * MB, &b));     // a's work has not ended
    CHECK(!x[0].kept);
    empty(&x, &b);
    a.done = a.queued;
    x.push_back(take(5 * MB, &b));
    CHECK(x[0].kept && frees == 1 && live.size() == 16);
    empty(&x, &b);
    b.done = b.queued;
    fill(&y, 7, 64 * MB, &b);          // 448 MB in use, and 8 small ones and the 8 MB one idle
    CHECK(frees == 8);
    for (const tx::Scratch& s : y) CHECK(s.kept);
    x.push_back(take(33 * MB, &a));    // 64 MB: all the small ones go
    CHECK(x[0].kept && live.size() == 8);
    x.push_back(take(MB, &a));         // nothing idle is left
    CHECK(!x[1].kept);
    empty(&x, &a);
    empty(&y, &b);
    a.done = a.queued;
    b.done = b.queued;
    const int before = mallocs;
    for (size_t m : {1, 60, 5, 33, 64}) {
        x.push_back(take(m * MB, &a));
        CHECK(x[0].kept);
        empty(&x, &a);
    }
    CHECK(mallocs == before);          // (nothing grows any more)
    tx::scratch_trim(0);
    CHECK(live.empty());
}

// While one thread allocates or frees, another takes and gives back kept buffers
// of the same device and of another one.
static std::mutex step_mu;
static std::condition_variable step_cv;
static int step = 0;                   // 1: a thread is inside the runtime, 2: the other one is done

static bool wait_step(int n) {
    std::unique_lock<std::mutex> l(step_mu);
    return step_cv.wait_for(l, std::chrono::seconds(5), [&] { return step >= n; });
}
static void set_step(int n) {
    std::lock_guard<std::mutex> l(step_mu);
    step = n;
    step_cv.notify_all();
}
static void inside() {
    set_step(1);
    CHECK(wait_step(2));               // a lock held here keeps the other thread out
}

static void locks() {
    Stream s[2], big;
    for (int d = 0; d < 2; ++d) {
        device = d;
        tx::Scratch x = take(MB, &s[d]);
        CHECK(tx::scratch_put(&x, &s[d]) == hipSuccess);
    }
    device = 0;
    for (int k = 0; k < 2; ++k) {
        step = 0;
        (k == 0 ? in_malloc : in_free) = inside;
        std::thread t([&] {
            if (k == 0) {
                tx::Scratch x = take(60 * MB, &big);
                CHECK(x.kept && tx::scratch_put(&x, &big) == hipSuccess);
            } else {
                device = 1;
                tx::scratch_trim(1);
            }
        });
        CHECK(wait_step(1));
        for (int d = 0; d < 2 - k; ++d) {
            device = d;
            tx::Scratch x = take(MB, &s[d]);
            CHECK(x.kept && tx::scratch_put(&x, &s[d]) == hipSuccess);
        }
        set_step(2);
        t.join();
        in_malloc = in_free = nullptr;
    }
}

// Errors from before a call stay for their reader; the call's own (an event that
// has not completed) do not come up later.
static void error() {
    Stream a, b;
    tx::Scratch x = take(MB, &a);
    CHECK(tx::scratch_put(&x, &a) == hipSuccess);
    x = take(MB, &b);
    CHECK(hipGetLastError() == hipSuccess);
    CHECK(tx::scratch_put(&x, &b) == hipSuccess);
    last_error = hipErrorInvalidValue;
    x = take(MB, &a);
    CHECK(tx::scratch_put(&x, &a) == hipSuccess);
    CHECK(hipGetLastError() == hipErrorInvalidValue);
}

int main(int argc, char** argv) {
    const std::map<std::string, void (*)()> checks = {{"reuse", reuse}, {"lost", lost}, {"memory", memory}, {"room", room}, {"locks", locks}, {"error", error}};
    const auto it = checks.find(argc > 1 ? argv[1] : "");
    if (it == checks.end()) return 2;
    it->second();
    return 0;
}
