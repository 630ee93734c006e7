"""The scratch memory kept between calls, on a host model of the HIP calls it
makes: device memory with a limit, streams that are destroyed, events and
captures.  The model ends the program on what the runtime does not allow: a
wait for an event whose stream is gone, memory freed at once while the device
works on it, memory freed on a stream that does not wait for its last use, and
counts waits for the device, which a capture refuses."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1902_02104_amd", "csrc")

HIP = r"""
#pragma once
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
enum { hipStreamNonBlocking = 1 };
enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorInvalidHandle = 400, hipErrorStreamCaptureUnsupported = 900 };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone = 0, hipStreamCaptureStatusActive = 1 };
struct hipStream { bool alive = true, capturing = false; std::set<long> waits; };
struct hipEvent { hipStream* s = nullptr; long use = 0; };
typedef hipStream* hipStream_t;
typedef hipEvent* hipEvent_t;
#define hipStreamPerThread ((hipStream_t)2)
enum { hipEventDisableTiming = 2, hipEventDisableSystemFence = 0x20000000 };
namespace model {
inline size_t limit = (size_t)1 << 40, used = 0;
inline int mallocs = 0, events = 0, syncs = 0, busy_frees = 0;
inline std::map<void*, size_t> blocks;
inline std::map<void*, std::pair<hipStream_t, long>> last;  // stream and number of a block's last use
inline long uses = 0;
inline std::set<hipStream_t> streams;
inline bool working = false, refuse = false;
[[noreturn]] inline void fail(const char* what) { printf("model: %s\n", what); exit(3); }
inline hipStream_t make() { hipStream_t s = new hipStream; streams.insert(s); return s; }
inline void destroy(hipStream_t s) { s->alive = false; }  // never reused: its address marks a stale handle
inline void check(hipStream_t s) { if (s && s != hipStreamPerThread && !s->alive) fail("a call on a stream that is gone"); }
}
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    model::check(s);
    *st = s && s != hipStreamPerThread && s->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
inline hipError_t hipMallocAsync(void** p, size_t n, hipStream_t s) {
    model::check(s);
    if (model::used + n > model::limit) return *p = nullptr, hipErrorOutOfMemory;
    static uintptr_t next = 4096;
    *p = (void*)next;
    next += (n + 4095) / 4096 * 4096;
    model::blocks[*p] = n;
    model::used += n;
    ++model::mallocs;
    model::working = true;
    return hipSuccess;
}
inline hipError_t hipMalloc(void** p, size_t n) { return hipMallocAsync(p, n, nullptr); }
inline hipError_t release_block(void* p) {
    auto it = model::blocks.find(p);
    if (it == model::blocks.end()) model::fail("memory freed twice");
    model::used -= it->second;
    model::blocks.erase(it);
    return hipSuccess;
}
// Work on the block p in stream s, as a call does between get and put.
inline void work(void* p, hipStream_t s) { model::last[p] = {s, ++model::uses}; model::working = true; }
inline hipError_t hipFreeAsync(void* p, hipStream_t s) {
    model::check(s);
    if (model::refuse) return hipErrorStreamCaptureUnsupported;
    const auto u = model::last.find(p);
    if (u != model::last.end() && u->second.first != s &&
        (s == hipStreamPerThread || !s || s->waits.lower_bound(u->second.second) == s->waits.end()))
        model::fail("memory freed on a stream that does not wait for its last use");
    return release_block(p);
}
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = model::make(); return hipSuccess; }
inline hipError_t hipFree(void* p) {
    if (model::working) model::fail("memory freed under work that may use it");
    return release_block(p);
}
inline hipError_t hipDeviceSynchronize() {
    for (hipStream_t s : model::streams)
        if (s->alive && s->capturing) return hipErrorStreamCaptureUnsupported;
    ++model::syncs;
    model::working = false;
    return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = new hipEvent; ++model::events; return hipSuccess; }
inline hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
inline hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { model::check(s); e->s = s; e->use = model::uses; return hipSuccess; }
inline hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    model::check(s);
    model::check(e->s);
    if (s && s != hipStreamPerThread && e->s != s) s->waits.insert(e->use);
    return hipSuccess;
}
"""

MAIN = r"""
#include <chrono>
#include <cstring>
#include <thread>
#include <vector>
#include "ata_internal.h"
using namespace atalib::detail;
static const size_t MB = (size_t)1 << 20;
#define REQUIRE(x) do { if (!(x)) { printf("line %d: %s (used %zu MB, mallocs %d, events %d, syncs %d)\n", __LINE__, #x, model::used / MB, model::mallocs, model::events, model::syncs); return 1; } } while (0)
static hipError_t call(hipStream_t s, size_t bytes) {
    Scratch sc;
    const hipError_t e = scratch_get(sc, bytes, s);
    if (e != hipSuccess) return e;
    if (!sc.p) model::fail("no memory and no error");
    work(sc.p, s);
    return scratch_put(sc, s);
}
static void later() { std::this_thread::sleep_for(std::chrono::milliseconds(1100)); }
static int reuse() {
    hipStream_t s = model::make();
    for (int i = 0; i < 5; ++i) REQUIRE(call(s, 3 * MB) == hipSuccess);
    REQUIRE(model::mallocs == 1 && model::events == 1 && model::syncs == 0);
    return 0;
}
// 512 MB and 64 blocks a device, of one stream and of several
static int bound() {
    hipStream_t s = model::make();
    for (int i = 1; i <= 40; ++i) {
        std::vector<Scratch> sc(4);
        for (int k = 0; k < 4; ++k) REQUIRE(scratch_get(sc[k], i * 4 * MB, s) == hipSuccess);
        for (int k = 0; k < 4; ++k) REQUIRE(scratch_put(sc[k], s) == hipSuccess);
        REQUIRE(model::used <= 512 * MB);
    }
    REQUIRE(model::used > 400 * MB);
    hipStream_t t = model::make();
    for (int i = 0; i < 3; ++i) REQUIRE(call(t, 200 * MB) == hipSuccess);
    REQUIRE(model::used <= 512 * MB);
    release_scratch();
    REQUIRE(model::used == 0);
    std::vector<Scratch> sc(100);
    for (Scratch& x : sc) REQUIRE(scratch_get(x, MB, s) == hipSuccess);
    for (Scratch& x : sc) REQUIRE(scratch_put(x, s) == hipSuccess);
    REQUIRE(model::used == 64 * MB);
    return 0;
}
static int fill(hipStream_t s) {
    Scratch a, b;
    REQUIRE(scratch_get(a, 200 * MB, s) == hipSuccess);
    REQUIRE(scratch_get(b, 200 * MB, s) == hipSuccess);
    REQUIRE(scratch_put(a, s) == hipSuccess);
    REQUIRE(scratch_put(b, s) == hipSuccess);
    REQUIRE(model::used >= 400 * MB);
    return 0;
}
// Kept memory is given back before a call fails for want of it, whatever path the call takes.
static int oom() {
    hipStream_t s = model::make(), t = model::make();
    model::limit = 1000 * MB;
    if (fill(s)) return 1;
    REQUIRE(call(t, 450 * MB) == hipSuccess);
    if (fill(s)) return 1;
    REQUIRE(call(t, 900 * MB) == hipSuccess);
    if (fill(s)) return 1;
    REQUIRE(call(hipStreamPerThread, 700 * MB) == hipSuccess);
    REQUIRE(call(t, 1001 * MB) == hipErrorOutOfMemory);
    REQUIRE(call(t, 100 * MB) == hipSuccess);
    void* p;
    REQUIRE(device_alloc(&p, 1001 * MB) == hipErrorOutOfMemory && !p);
    if (fill(s)) return 1;
    REQUIRE(device_alloc(&p, 900 * MB) == hipSuccess && p);
    return 0;
}
// A captured call that finds no memory fails without a wait.
static int oom_capture() {
    hipStream_t s = model::make(), t = model::make();
    model::limit = 1000 * MB;
    if (fill(s)) return 1;
    t->capturing = true;
    REQUIRE(call(t, 900 * MB) == hipErrorOutOfMemory);
    REQUIRE(model::used >= 400 * MB && model::syncs == 0);
    return 0;
}
// While another stream captures, the device cannot be waited for: what needs the wait stays.
static int refused_wait() {
    hipStream_t s = model::make(), t = model::make(), c = model::make();
    model::limit = 1000 * MB;
    if (fill(s)) return 1;
    c->capturing = true;
    REQUIRE(call(t, 900 * MB) == hipErrorOutOfMemory);
    release_scratch();
    REQUIRE(model::used >= 200 * MB);
    c->capturing = false;
    REQUIRE(call(t, 900 * MB) == hipSuccess);
    return 0;
}
// Streams that are gone leave their blocks; a new stream gets room when they are
// old, without a wait for the device: up to three quarters of what may be kept stay.
static int dead_streams(size_t bytes, int streams, bool capture) {
    hipStream_t c = model::make();
    c->capturing = capture;
    for (int i = 0; i < streams; ++i) {
        hipStream_t s = model::make();
        REQUIRE(call(s, bytes) == hipSuccess);
        model::destroy(s);
    }
    const size_t held = model::used;
    hipStream_t t = model::make();
    const int ev = model::events;
    for (int i = 0; i < 10; ++i) REQUIRE(call(t, bytes) == hipSuccess);
    REQUIRE(model::events == ev && model::used == held);  // as if nothing were kept
    later();
    REQUIRE(call(t, bytes) == hipSuccess);
    REQUIRE(model::used <= held / 4 * 3 + bytes + bytes / 8);
    const int ma = model::mallocs;
    for (int i = 0; i < 10; ++i) REQUIRE(call(t, bytes) == hipSuccess);
    REQUIRE(model::mallocs == ma && model::syncs == 0);
    // for every stream that comes after
    for (int i = 0; i < 200; ++i) {
        hipStream_t s = model::make();
        REQUIRE(call(s, bytes) == hipSuccess);
        model::destroy(s);
    }
    later();
    hipStream_t u = model::make();
    REQUIRE(call(u, bytes) == hipSuccess);
    const int mb = model::mallocs;
    for (int i = 0; i < 10; ++i) REQUIRE(call(u, bytes) == hipSuccess);
    REQUIRE(model::mallocs == mb && model::syncs == 0 && model::used <= 512 * MB);
    return 0;
}
// A block that cannot be freed now is not lost.
static int refused_free() {
    for (int i = 0; i < 64; ++i) {
        hipStream_t s = model::make();
        REQUIRE(call(s, MB) == hipSuccess);
        model::destroy(s);
    }
    later();
    hipStream_t t = model::make();
    Scratch sc;
    model::refuse = true;
    REQUIRE(scratch_get(sc, MB, t) == hipSuccess);
    work(sc.p, t);
    model::refuse = false;
    REQUIRE(scratch_put(sc, t) == hipSuccess);
    release_scratch();
    REQUIRE(model::used == 0);
    std::vector<Scratch> two(2);
    for (Scratch& x : two) REQUIRE(scratch_get(x, 300 * MB, t) == hipSuccess);
    for (Scratch& x : two) work(x.p, t);
    model::refuse = true;
    for (Scratch& x : two) REQUIRE(scratch_put(x, t) == hipSuccess);
    model::refuse = false;
    release_scratch();
    REQUIRE(model::used == 0);
    return 0;
}
// More live streams than blocks: never a device wait, no event for those without a block.
static int live_streams() {
    std::vector<hipStream_t> s;
    for (int i = 0; i < 100; ++i) s.push_back(model::make());
    for (int r = 0; r < 20; ++r)
        for (hipStream_t x : s) REQUIRE(call(x, MB) == hipSuccess);
    REQUIRE(model::syncs == 0 && model::events <= 64 && model::used <= 64 * 9 * MB / 8);
    return 0;
}
int main(int, char** v) {
    if (!strcmp(v[1], "reuse")) return reuse();
    if (!strcmp(v[1], "bound")) return bound();
    if (!strcmp(v[1], "oom")) return oom();
    if (!strcmp(v[1], "oom_capture")) return oom_capture();
    if (!strcmp(v[1], "refused_wait")) return refused_wait();
    if (!strcmp(v[1], "dead_blocks")) return dead_streams(MB, 64, false);
    if (!strcmp(v[1], "dead_bytes")) return dead_streams(100 * MB, 5, false);
    if (!strcmp(v[1], "dead_capture")) return dead_streams(MB, 64, true);
    if (!strcmp(v[1], "refused_free")) return refused_free();
    if (!strcmp(v[1], "live_streams")) return live_streams();
    return 2;
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    d = tmp_path_factory.mktemp("scratch")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(HIP)
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "scratch")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", str(d), "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    str(d / "main.cpp"), os.path.join(CSRC, "ata_scratch.cpp"), "-o", exe, "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("case", ["reuse", "bound", "oom", "oom_capture", "refused_wait", "dead_blocks", "dead_bytes",
                                  "dead_capture", "refused_free", "live_streams"])
def test_kept_scratch(model, case):
    r = subprocess.run([model, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
