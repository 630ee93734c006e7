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
// is freed at once).  A stream that is gone leaves its blocks, nothing tells it
// from one that is idle, and an event whose stream is gone is never queried or
// waited for (the runtime looks at the stream).  So a quarter of what may be kept
// is held by blocks that a library stream (g_fence) waits for at their release,
// while their stream is there: when a call finds no room, those of other streams
// that were not used for kStale are freed on that stream.  (The first three
// quarters, kLooseBytes and kLooseBlocks, do without that wait, 2 to 3 us a
// block: bfloat16 pairs 8192 x 8192, a block of 384 MB, 1603 -> 1608 us with it.)
// Streams in use never lose blocks to each other.
//
// No call waits for the device: that would end any capture in the process with
// an error.  (Allocations, events and waits of streams for them do not.)  Only
// ata_release_caches does, which frees every block, and a call outside a capture
// that finds the device's memory exhausted, after the blocks that can be freed
// without.  A block is taken off the list while a call uses it, so threads never
// share one.  Calls under stream capture (whose memory belongs to the graph) and
// calls on the per-thread default stream (one handle for many streams) allocate
// as before.
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
constexpr size_t kLooseBytes = kKeepBytes / 4 * 3;
constexpr int kLooseBlocks = kKeepBlocks / 4 * 3;
constexpr int kDevices = 64;
constexpr std::chrono::milliseconds kStale(1000);

typedef std::chrono::steady_clock Clock;

struct Kept {
    void* p;
    size_t bytes;
    hipEvent_t ev;
    hipStream_t s;
    uint64_t drop;  // the release that waits for the device to free it (0: none)
    bool fenced;    // g_fence waits for its work
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
    // Whether a block of `need` bytes belongs to the fenced quarter.
    bool fence(size_t need) const {
        int loose = 0;
        size_t held = 0;
        for (int i = 0; i < n; ++i)
            if (!b[i].fenced) {
                ++loose;
                held += b[i].bytes;
            }
        return loose >= kLooseBlocks || held + need > kLooseBytes;
    }
    // Takes the fenced blocks of streams other than s not used since `before`.
    int retire(hipStream_t s, Clock::time_point before, Kept* out) {
        int no = 0;
        for (int i = 0; i < n;)
            if (b[i].fenced && b[i].s != s && !b[i].drop && b[i].at <= before)
                out[no++] = take(i);
            else
                ++i;
        return no;
    }
};

std::mutex g_mu;
Shelf g_shelf[kDevices];
uint64_t g_drops = 0;
hipStream_t g_fence[kDevices];  // made on first use, kept until the process ends

// Block sizes in eighths of a power of two, at least 64 KB: shapes that
// differ a little share blocks.
size_t block_size(size_t need) {
    size_t unit = (size_t)8 << 10;
    while (unit * 16 <= need) unit *= 2;
    const size_t b = (need + unit - 1) / unit * unit;
    return b < ((size_t)64 << 10) ? (size_t)64 << 10 : b;
}

// Frees the kept blocks of device d (and their events) after the device's work.
// They stay listed until the wait has ended, out of reach of calls; if it is
// refused, as while a stream is captured, they are kept as before.
void drop_blocks(int d) {
    uint64_t id = 0;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        Shelf& sh = g_shelf[d];
        for (int i = 0; i < sh.n; ++i)
            if (!sh.b[i].drop) {
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

// The fence stream of device d (the current one) waits for event ev.
hipError_t fence(int d, hipEvent_t ev) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_fence[d]) {
        const hipError_t e = hipStreamCreateWithFlags(&g_fence[d], hipStreamNonBlocking);
        if (e != hipSuccess) {
            g_fence[d] = nullptr;
            return e;
        }
    }
    return hipStreamWaitEvent(g_fence[d], ev, 0);
}

// Frees blocks taken off the list of device d in the order of stream s (its
// own blocks) or, fenced ones of other streams, of the fence stream.  Blocks that
// cannot be freed now go back on the list (the runtime refuses it on a stream
// that synchronises with the null stream while another such stream is captured).
void free_blocks(int d, const Kept* k, int n, hipStream_t s) {
    for (int i = 0; i < n; ++i) {
        const bool own = k[i].s == s;
        hipError_t e = own ? hipStreamWaitEvent(s, k[i].ev, 0) : hipSuccess;
        if (e == hipSuccess) e = hipFreeAsync(k[i].p, own ? s : g_fence[d]);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            std::lock_guard<std::mutex> lk(g_mu);
            Shelf& sh = g_shelf[d];
            if (sh.n < kKeepBlocks) {
                sh.b[sh.n++] = k[i];
                sh.bytes += k[i].bytes;
                continue;
            }
        }
        (void)hipEventDestroy(k[i].ev);
    }
}

// Memory from the stream's pool; where there is none left, the kept blocks go
// back first: those that need no wait for the device, then all.  (Not for a
// capture, which that wait would break.)
hipError_t allocate(void** p, size_t bytes, hipStream_t s, int d, bool capture) {
    hipError_t e = hipMallocAsync(p, bytes, s);
    if (e == hipErrorOutOfMemory && !capture) {
        (void)hipGetLastError();
        if (d >= 0 && d < kDevices) {
            Kept old[kKeepBlocks];
            int no = 0;
            {
                std::lock_guard<std::mutex> lk(g_mu);
                Shelf& sh = g_shelf[d];
                no = sh.retire(s, Clock::time_point::max(), old);
                for (int i = 0; i < sh.n;)
                    if (sh.b[i].s == s && !sh.b[i].drop)
                        old[no++] = sh.take(i);
                    else
                        ++i;
            }
            if (no) {
                free_blocks(d, old, no, s);
                e = hipMallocAsync(p, bytes, s);
                if (e == hipErrorOutOfMemory) (void)hipGetLastError();
            }
        }
        if (e == hipErrorOutOfMemory) {
            release_scratch();
            e = hipMallocAsync(p, bytes, s);
        }
    }
    if (e != hipSuccess) *p = nullptr;
    return e;
}

}  // namespace

bool stream_capturing(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return st != hipStreamCaptureStatusNone;
}

hipError_t scratch_get(Scratch& out, size_t bytes, hipStream_t s) {
    out = Scratch{};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    out.bytes = block_size(bytes);
    const bool capture = stream_capturing(s);
    if (out.bytes > kKeepBytes || dev < 0 || dev >= kDevices || capture || s == hipStreamPerThread) {
        out.bytes = bytes;
        return allocate(&out.p, bytes, s, dev, capture);
    }
    out.dev = dev;
    bool room;
    Kept old[kKeepBlocks];
    int no = 0;
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
            no = sh.retire(s, Clock::now() - kStale, old);
            room = sh.room(s, out.bytes);
        }
    }
    free_blocks(dev, old, no, s);
    if (!room) {  // it could not be kept: no event
        out.bytes = bytes;
        return allocate(&out.p, bytes, s, dev, false);
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
    e = allocate(&out.p, out.bytes, s, dev, false);
    if (e != hipSuccess) {
        (void)hipEventDestroy(out.ev);
        out = Scratch{};
    }
    return e;
}

hipError_t scratch_put(Scratch& sc, hipStream_t s) {
    if (!sc.p) return hipSuccess;
    Kept mine{sc.p, sc.bytes, sc.ev, s, 0, false, Clock::now()};
    const int dev = sc.dev;
    sc = Scratch{};
    if (!mine.ev) return hipFreeAsync(mine.p, s);
    hipError_t e = hipEventRecord(mine.ev, s);
    if (e != hipSuccess) {
        (void)hipEventDestroy(mine.ev);
        (void)hipFreeAsync(mine.p, s);
        return e;
    }
    {
        std::lock_guard<std::mutex> lk(g_mu);
        mine.fenced = g_shelf[dev].fence(mine.bytes);
    }
    bool kept = true;
    if (mine.fenced && fence(dev, mine.ev) != hipSuccess) {
        (void)hipGetLastError();
        kept = false;
    }
    Kept old[kKeepBlocks + 1];
    int no = 0;
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
    free_blocks(dev, old, no, s);
    return hipSuccess;
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
