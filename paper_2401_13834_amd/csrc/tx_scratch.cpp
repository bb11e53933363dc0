// Scratch of one call's kernels, kept between calls.
//
// hipMallocAsync and hipFreeAsync cost a call 14 us on the host (a dedispersion
// of 102 trials x 12464 samples 27.6, now 13.4), and 40 to
// 100 us each when a call makes several of different sizes (the three ranges of a
// 128-channel block: 435 us a call, 40 us with these buffers), more than the
// kernels of a small block take.  Here a buffer of up to kMaxBuf bytes stays
// allocated after the call and is taken again by a later one: by a call on the
// same stream, which its kernels follow, or by any once the event recorded
// behind the last user's kernels has completed.  Per device at most kMaxBufs
// buffers and kMaxBytes bytes are kept: where a new one finds no room, the
// smallest idle ones (all too small for the call) make way, so buffers only grow and
// this ends.  Larger requests, captures and calls that still find no room use
// the stream-ordered pool.  tx_pool_trim gives the buffers back, and so does a call
// for which the pool has no memory left.
#include <algorithm>
#include <mutex>

#include "tx_internal.h"

namespace tx {
namespace {

constexpr size_t kMinBuf = size_t(4) << 20;
constexpr size_t kMaxBuf = size_t(64) << 20;
constexpr size_t kMaxBytes = size_t(512) << 20;
constexpr int kMaxBufs = 16;

struct Buf {
    void* p = nullptr;
    size_t bytes = 0;
    hipEvent_t done = nullptr;
    hipStream_t last = nullptr;
    bool used = false;      // `done` has been recorded
    bool busy = false;      // a call holds it
    bool lost = false;      // or held it, and it is not known when its kernels end
};

// The lock is held to look and to mark only, never across a call that allocates,
// frees or waits: a slot that is being filled is marked busy, and buffers to be freed are
// taken out of the list first.
struct DevBufs {
    std::mutex mu;
    Buf bufs[kMaxBufs];     // p null: no buffer
    size_t bytes = 0;       // (with those of slots being filled)
};

constexpr int kMaxDevices = 64;
DevBufs g_dev[kMaxDevices];

// Calls that a capture elsewhere in the process forbids are allowed for the
// scope: none of them touches a capturing stream.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// Buffers taken out of the list.
struct Freed {
    Buf bufs[kMaxBufs];
    int n = 0;
    void take(DevBufs& d, Buf* b) {                  // with the lock held
        bufs[n++] = *b;
        d.bytes -= b->bytes;
        *b = Buf{};
    }
    ~Freed() {                                       // without
        for (int i = 0; i < n; ++i) {
            if (bufs[i].used) (void)hipEventSynchronize(bufs[i].done);
            (void)hipFree(bufs[i].p);
            (void)hipEventDestroy(bufs[i].done);
        }
    }
};

// Whether the kernels of the buffer's last user have ended.  Not asked while an
// error of the caller's is unread (`ask` false), which "not ready" would replace.
bool ended(const Buf& b, bool ask) { return !b.used || (ask && hipEventQuery(b.done) == hipSuccess); }

// The smallest kept buffer of at least `bytes` that is ready for `stream`, or null.
Buf* ready(DevBufs& d, size_t bytes, hipStream_t stream, bool ask) {
    Buf* best = nullptr;
    for (Buf& b : d.bufs) {
        if (b.busy || !b.p || b.bytes < bytes || (best && b.bytes >= best->bytes)) continue;
        if (b.last != stream && !ended(b, ask)) continue;
        best = &b;
    }
    // (The handle may be another stream's by now, so also the same handle
    // waits for the event; on the stream that recorded it that is nothing.)
    if (best && best->used && best->last == stream && hipStreamWaitEvent(stream, best->done, 0) != hipSuccess)
        best = nullptr;
    if (best) best->busy = true;
    return best;
}

// A busy slot for a new buffer of `size` bytes, within the limits, in the place
// of the smallest idle buffers where none is free; null if those would not do.
Buf* make_room(DevBufs& d, size_t size, bool ask, Freed* old) {
    Buf* idle[kMaxBufs];
    int n = 0;
    Buf* empty = nullptr;
    for (Buf& b : d.bufs) {
        if (b.busy) continue;
        if (!b.p) empty = &b;
        else if (b.bytes < size && ended(b, ask)) idle[n++] = &b;
    }
    std::sort(idle, idle + n, [](const Buf* x, const Buf* y) { return x->bytes < y->bytes; });
    size_t left = d.bytes;
    int k = 0;
    while ((left + size > kMaxBytes || (!empty && k == 0)) && k < n) left -= idle[k++]->bytes;
    if (left + size > kMaxBytes || (!empty && k == 0)) return nullptr;
    for (int i = 0; i < k; ++i) old->take(d, idle[i]);
    if (!empty) empty = idle[0];
    empty->busy = true;
    empty->bytes = size;
    d.bytes += size;
    return empty;
}

// A kept or new buffer of at least `bytes` for `stream`, or null.
Buf* take(DevBufs& d, size_t bytes, hipStream_t stream, bool ask) {
    size_t size = kMinBuf;
    while (size < bytes) size *= 2;
    Buf* b;
    {
        Freed old;
        std::lock_guard<std::mutex> lock(d.mu);
        b = ready(d, bytes, stream, ask);
        if (b) return b;
        b = make_room(d, size, ask, &old);
        if (!b) return nullptr;
    }
    void* p = nullptr;
    hipEvent_t done = nullptr;
    const bool ok = hipMalloc(&p, size) == hipSuccess &&
                    hipEventCreateWithFlags(&done, hipEventDisableTiming) == hipSuccess;
    if (!ok && p) (void)hipFree(p);
    std::lock_guard<std::mutex> lock(d.mu);
    if (!ok) {
        d.bytes -= size;
        *b = Buf{};
        return nullptr;
    }
    b->p = p;
    b->done = done;
    return b;
}

// Frees the buffers that no call holds, once their last kernels have ended.
// False if there were none.
bool give_up_idle(DevBufs& d) {
    RelaxedCapture relaxed;
    Freed old;
    std::lock_guard<std::mutex> lock(d.mu);
    for (Buf& b : d.bufs)
        if (b.p && !b.busy) old.take(d, &b);
    return old.n > 0;
}

}  // namespace

hipError_t scratch_get(size_t bytes, hipStream_t stream, Scratch* out) {
    *out = Scratch{};
    const bool clean = hipPeekAtLastError() == hipSuccess;   // else an error from before is left for its reader
    int dev = -1;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusActive;
    const bool keeps = hipStreamIsCapturing(stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone &&
                       hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices;
    if (keeps && bytes <= kMaxBuf) {
        RelaxedCapture relaxed;
        if (Buf* b = take(g_dev[dev], bytes, stream, clean)) {
            out->p = b->p;
            out->kept = b;
            out->dev = &g_dev[dev];
        }
    }
    if (clean) (void)hipGetLastError();              // (an event that has not completed is no error)
    if (out->p) return hipSuccess;
    hipError_t e = hipMallocAsync(&out->p, bytes > 0 ? bytes : 1, stream);
    if (e == hipErrorOutOfMemory && keeps && give_up_idle(g_dev[dev])) {
        if (clean) (void)hipGetLastError();
        e = hipMallocAsync(&out->p, bytes > 0 ? bytes : 1, stream);
    }
    if (e != hipSuccess) out->p = nullptr;
    return e;
}

hipError_t scratch_put(Scratch* s, hipStream_t stream) {
    if (!s->p) return hipSuccess;
    Buf* b = static_cast<Buf*>(s->kept);
    DevBufs* d = static_cast<DevBufs*>(s->dev);
    void* p = s->p;
    *s = Scratch{};
    if (!b) return hipFreeAsync(p, stream);
    hipError_t e = hipEventRecord(b->done, stream);
    const bool recorded = e == hipSuccess;
    if (!recorded) e = hipStreamSynchronize(stream);            // nothing to wait for later then
    std::lock_guard<std::mutex> lock(d->mu);
    b->used = recorded;
    b->last = stream;
    b->busy = b->lost = e != hipSuccess;                        // (given up by the next trim)
    return e;
}

void scratch_trim(int dev) {
    if (dev < 0 || dev >= kMaxDevices) return;
    DevBufs& d = g_dev[dev];
    Freed old;
    std::lock_guard<std::mutex> lock(d.mu);
    for (Buf& b : d.bufs)
        if (b.p && (!b.busy || b.lost)) old.take(d, &b);
}

}  // namespace tx
