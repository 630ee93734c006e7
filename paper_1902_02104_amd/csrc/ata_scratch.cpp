// Device scratch of the library's calls, kept between calls.
//
// A stream-ordered allocation and its release cost a call 11 us (two small
// kernels 4.9 us alone, 16.3 us with the pair), and memory that went back to
// the driver at a synchronisation takes 200 to 600 us to get again where a
// call needs tens of megabytes.  So released blocks stay here and serve the
// next call on the same stream: the stream orders the two uses, and an event
// recorded at the release and waited for at the reuse covers a stream handle
// that was destroyed and created again (with it 6.6 us).  A^t B of FP32
// 1000 x 77: 38 -> 17 us a call; the first e4m3 product after a
// synchronisation, 8192 x 8192: 509 -> 394 us.  No block moves to another
// stream, so no call's work waits for another stream's.
//
// At most kKeepBytes a device (and kKeepBlocks blocks) are kept; beyond that
// the stream's own blocks released longest ago make room, or else the call
// allocates without keeping (a block that no longer fits when it is released
// is freed at once).  A stream that is gone leaves its blocks, and nothing tells
// it from one that is idle: when a call finds no room and blocks not used for
// kStale hold half of what may be kept, they are freed after a wait for the
// device.  Streams in use never come to that wait, however many there are.
// ata_release_caches frees all of them, and so does any allocation of the
// library outside a capture that finds the device's memory exhausted, before it
// tries again.  An event whose stream is gone is never queried or waited for
// (the runtime looks at the stream): only a stream of the same handle waits for
// it, and the release waits for the device.  A block is taken off the list while
// a call uses it, so threads never share one.  Calls under stream capture (whose
// memory belongs to the graph) and calls on the per-thread default stream (one
// handle for many streams) allocate as before.
#include <hip/hip_runtime.h>

#include <chrono>
#include <cstddef>
#include <cstdint>
#include <mutex>

#include "ata_internal.h"

namespace atalib {
namespace detail {

namespace {

constexpr size_t kKeepBytes = (size_t)512 << 20;
constexpr int kKeepBlocks = 64;
constexpr int kDevices = 64;
constexpr std::chrono::milliseconds kStale(1000);

typedef std::chrono::steady_clock Clock;

struct Kept {
    void* p;
    size_t bytes;
    hipEvent_t ev;
    hipStream_t s;
    uint64_t drop;  // the release that waits for the device to free it (0: none)
    Clock::time_point at;  // when it was released to the shelf
};

// Blocks of one device in the order of their release.
struct Shelf {
    Kept b[kKeepBlocks];
    int n = 0;
    size_t bytes = 0;
    Kept take(int i) {
        const Kept k = b[i];
        for (--n; i < n; ++i) b[i] = b[i + 1];
        bytes -= k.bytes;
        return k;
    }
    // Room for a block of s of `need` bytes, its own blocks making way.
    bool room(hipStream_t s, size_t need) const {
        int others = 0;
        size_t held = 0;
        for (int i = 0; i < n; ++i)
            if (b[i].s != s || b[i].drop) {
                ++others;
                held += b[i].bytes;
            }
        return others < kKeepBlocks && held + need <= kKeepBytes;
    }
    // Half of what may be kept, or more, has not been used since `before`, by
    // streams other than s.
    bool stale(hipStream_t s, Clock::time_point before) const {
        int old = 0;
        size_t held = 0;
        for (int i = 0; i < n; ++i)
            if (b[i].s != s && !b[i].drop && b[i].at <= before) {
                ++old;
                held += b[i].bytes;
            }
        return 2 * old >= kKeepBlocks || 2 * held >= kKeepBytes;
    }
};

std::mutex g_mu;
Shelf g_shelf[kDevices];
uint64_t g_drops = 0;

// Block sizes in eighths of a power of two, at least 64 KB: shapes that
// differ a little share blocks.
size_t block_size(size_t need) {
    size_t unit = (size_t)8 << 10;
    while (unit * 16 <= need) unit *= 2;
    const size_t b = (need + unit - 1) / unit * unit;
    return b < ((size_t)64 << 10) ? (size_t)64 << 10 : b;
}

// Frees the kept blocks of device d (and their events) that were released at
// `before` or earlier, after the device's work.  They stay listed until the wait has ended, out of reach of calls; if it
// is refused, as while a stream is captured, they are kept as before.
void drop_blocks(int d, Clock::time_point before = Clock::time_point::max()) {
    uint64_t id = 0;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        Shelf& sh = g_shelf[d];
        for (int i = 0; i < sh.n; ++i)
            if (!sh.b[i].drop && sh.b[i].at <= before) {
                if (!id) id = ++g_drops;
                sh.b[i].drop = id;
            }
    }
    if (!id) return;
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(d);
    const bool done = hipDeviceSynchronize() == hipSuccess;
    if (!done) (void)hipGetLastError();
    Kept old[kKeepBlocks];
    int no = 0;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        Shelf& sh = g_shelf[d];
        for (int i = 0; i < sh.n;) {
            if (sh.b[i].drop != id) {
                ++i;
            } else if (done) {
                old[no++] = sh.take(i);
            } else {
                sh.b[i].at = Clock::now();
                sh.b[i++].drop = 0;
            }
        }
    }
    for (int i = 0; i < no; ++i) {
        (void)hipFree(old[i].p);
        (void)hipEventDestroy(old[i].ev);
    }
    (void)hipSetDevice(cur);
}

// Whether s may be under capture.
bool capturing(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return st != hipStreamCaptureStatusNone;
}

// Memory from the stream's pool; where there is none left, the kept blocks go
// back first.  (Not for a capture, which a wait for the device would break.)
hipError_t allocate(void** p, size_t bytes, hipStream_t s, bool capture) {
    hipError_t e = hipMallocAsync(p, bytes, s);
    if (e == hipErrorOutOfMemory && !capture) {
        (void)hipGetLastError();
        release_scratch();
        e = hipMallocAsync(p, bytes, s);
    }
    if (e != hipSuccess) *p = nullptr;
    return e;
}

}  // namespace

hipError_t scratch_get(Scratch& out, size_t bytes, hipStream_t s) {
    out = Scratch{};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    out.bytes = block_size(bytes);
    const bool capture = capturing(s);
    if (out.bytes > kKeepBytes || dev < 0 || dev >= kDevices || capture || s == hipStreamPerThread) {
        out.bytes = bytes;
        return allocate(&out.p, bytes, s, capture);
    }
    out.dev = dev;
    bool room, stale = false;
    Clock::time_point before;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        Shelf& sh = g_shelf[dev];
        int best = -1;
        for (int i = sh.n - 1; i >= 0; --i)
            if (sh.b[i].s == s && !sh.b[i].drop && sh.b[i].bytes >= out.bytes && sh.b[i].bytes / 2 <= out.bytes &&
                (best < 0 || sh.b[i].bytes < sh.b[best].bytes))
                best = i;
        if (best >= 0) {
            const Kept k = sh.take(best);
            out.p = k.p;
            out.bytes = k.bytes;
            out.ev = k.ev;
        }
        room = best >= 0 || sh.room(s, out.bytes);
        if (!room) {
            before = Clock::now() - kStale;
            stale = sh.stale(s, before);
        }
    }
    if (stale) {
        drop_blocks(dev, before);
        std::lock_guard<std::mutex> lk(g_mu);
        room = g_shelf[dev].room(s, out.bytes);
    }
    if (!room) {  // it could not be kept: no event
        out.bytes = bytes;
        return allocate(&out.p, bytes, s, false);
    }
    if (out.p) {
        e = hipStreamWaitEvent(s, out.ev, 0);
        if (e != hipSuccess) {
            (void)hipEventDestroy(out.ev);
            (void)hipFree(out.p);  // waits for the device
            out = Scratch{};
        }
        return e;
    }
    e = hipEventCreateWithFlags(&out.ev, hipEventDisableTiming | hipEventDisableSystemFence);
    if (e != hipSuccess) return e;
    e = allocate(&out.p, out.bytes, s, false);
    if (e != hipSuccess) {
        (void)hipEventDestroy(out.ev);
        out = Scratch{};
    }
    return e;
}

hipError_t scratch_put(Scratch& sc, hipStream_t s) {
    if (!sc.p) return hipSuccess;
    const Kept mine{sc.p, sc.bytes, sc.ev, s, 0, Clock::now()};
    const int dev = sc.dev;
    sc = Scratch{};
    if (!mine.ev) return hipFreeAsync(mine.p, s);
    hipError_t e = hipEventRecord(mine.ev, s);
    if (e != hipSuccess) {
        (void)hipEventDestroy(mine.ev);
        (void)hipFreeAsync(mine.p, s);
        return e;
    }
    Kept old[kKeepBlocks];
    int no = 0;
    bool kept = true;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        Shelf& sh = g_shelf[dev];
        while (kept && (sh.n == kKeepBlocks || sh.bytes + mine.bytes > kKeepBytes)) {
            int i = 0;
            while (i < sh.n && (sh.b[i].s != s || sh.b[i].drop)) ++i;
            kept = i < sh.n;
            if (kept) old[no++] = sh.take(i);
        }
        if (kept) {
            sh.b[sh.n++] = mine;
            sh.bytes += mine.bytes;
        }
    }
    if (!kept) old[no++] = mine;
    for (int i = 0; i < no; ++i) {
        const hipError_t e0 = hipStreamWaitEvent(s, old[i].ev, 0);
        const hipError_t e1 = hipFreeAsync(old[i].p, s), e2 = hipEventDestroy(old[i].ev);
        if (e == hipSuccess) e = e0 != hipSuccess ? e0 : e1 != hipSuccess ? e1 : e2;
    }
    return e;
}

hipError_t device_alloc(void** p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        release_scratch();
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) *p = nullptr;
    return e;
}

void release_scratch() {
    for (int d = 0; d < kDevices; ++d) drop_blocks(d);
}

}  // namespace detail
}  // namespace atalib
