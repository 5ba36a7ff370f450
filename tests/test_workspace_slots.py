"""The kept workspaces of small calls (csrc/workspace.h) on the CPU, compiled against a stand-in
for the HIP runtime that models streams, events and captures: which calls run in a slot, and that
a slot's memory is never handed to a call whose stream is not ordered behind its last user."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2208_05419_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <thread>
#include <vector>
#include "workspace.h"

// ---- the stand-in.  A stream runs "works" (one per call); an event remembers the work it was
// recorded behind; works end when finish() says so.  Handle 2 is another stream in every thread.
static std::recursive_mutex mu;
#define LOCK std::lock_guard<std::recursive_mutex> lock_(mu)
typedef long Work;
struct Strm { std::set<Work> before; bool capturing = false; };  // works that later ones come after
struct Evt { std::vector<Work> behind; };
static std::map<std::pair<long, long>, Strm> streams;
static std::map<void*, std::vector<Work>> users;  // live allocations: works that used them
static std::set<Work> ended;
static Work next_work = 1;
static long live = 0, allocs = 0, synced = 0;
static long pooled = 0, room = 1 << 20;  // freed pieces the pool keeps; pieces the device has
static thread_local long thread_id = 0;
static thread_local hipStreamCaptureMode thread_mode = hipStreamCaptureModeGlobal;
static bool other_capture = false, fail_record = false;
static long broken_captures = 0;

#define CHECK(c) do { if (!(c)) { printf("FAILED %s:%d %s\n", __FILE__, __LINE__, #c); exit(1); } } while (0)
static Strm& strm(hipStream_t s) { return streams[{(long)s, (long)s == 2 ? thread_id : 0}]; }

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemPoolCreate(hipMemPool_t* p, const hipMemPoolProps*) { *p = (hipMemPool_t)1; return hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void** p, size_t, hipMemPool_t, hipStream_t) {
  LOCK;
  if (live + pooled >= room) return hipErrorOutOfMemory;
  *p = malloc(1); users[*p]; ++live; ++allocs; return hipSuccess;
}
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) { LOCK; pooled = 0; return hipSuccess; }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t s) { return hipMallocFromPoolAsync(p, n, nullptr, s); }
hipError_t hipFreeAsync(void* p, hipStream_t s) {
  LOCK;
  for (Work u : users[p]) CHECK(ended.count(u) || strm(s).before.count(u));
  CHECK(users.erase(p) == 1); --live; pooled += room < 100; free(p); return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
  LOCK; *c = strm(s).capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { std::swap(*m, thread_mode); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t) new Evt; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Evt*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  LOCK; CHECK(!strm(s).capturing);
  if (fail_record) return hipErrorUnknown;
  auto& b = strm(s).before; ((Evt*)e)->behind.assign(b.begin(), b.end()); return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  LOCK;
  if (other_capture && thread_mode == hipStreamCaptureModeGlobal) ++broken_captures;
  for (Work w : ((Evt*)e)->behind) if (!ended.count(w)) return hipErrorNotReady;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  LOCK; CHECK(!strm(s).capturing);
  for (Work w : ((Evt*)e)->behind) strm(s).before.insert(w);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { LOCK; for (Work w : strm(s).before) ended.insert(w); ++synced; return hipSuccess; }
}

static void finish() { LOCK; for (Work w = 1; w < next_work; ++w) ended.insert(w); }
// the call's kernels: every earlier user of the memory comes before them, by order or by having ended
static void launch(afno::Workspace& w) {
  LOCK;
  CHECK(users.count(w.ptr));
  Strm& s = strm(w.stream);
  for (Work u : users[w.ptr]) CHECK(ended.count(u) || s.before.count(u));
  s.before.insert(next_work);
  users[w.ptr].push_back(next_work++);
}
static bool call(long handle, size_t bytes = 1000) {  // true: ran in a slot
  afno::Workspace w;
  CHECK(w.acquire(bytes, (hipStream_t)handle) == hipSuccess);
  launch(w);
  const bool in_slot = w.slot != nullptr;
  w.release();
  return in_slot;
}

int main(int, char** argv) {
  const char* t = argv[1];
  if (!strcmp(t, "streams_that_come_and_go")) {
    for (long h = 100; h < 140; ++h) { CHECK(call(h)); CHECK(call(h)); finish(); }
    CHECK(allocs == 1 && live == 1);  // one slot serves them all, each after the last one's work
    CHECK(afno::g_slot_calls == 80);
  } else if (!strcmp(t, "overlapping_streams")) {
    for (long h = 100; h < 120; ++h) CHECK(call(h) == (h < 108));  // no wait for another's work
    CHECK(live == 8);
    for (long h = 100; h < 108; ++h) CHECK(call(h));  // their own slots still
    finish();
    for (long h = 200; h < 208; ++h) CHECK(call(h));  // all handed over
    CHECK(!call(100));
    finish();
    CHECK(call(100));
    CHECK(live == 8);
  } else if (!strcmp(t, "one_handle_many_streams")) {  // every use waits: the handle proves nothing
    for (thread_id = 1; thread_id < 40; ++thread_id) CHECK(call(2));
  } else if (!strcmp(t, "two_calls_at_once_on_one_stream")) {
    afno::Workspace a, b;
    CHECK(a.acquire(10, (hipStream_t)5) == hipSuccess && b.acquire(10, (hipStream_t)5) == hipSuccess);
    CHECK(a.ptr != b.ptr && a.slot && b.slot);
    launch(a); launch(b);
    b.release(); a.release();
    CHECK(call(5));
  } else if (!strcmp(t, "captures_and_large_calls_take_the_pool")) {
    CHECK(call(5));
    streams[{5, 0}].capturing = true;
    CHECK(!call(5));
    streams[{5, 0}].capturing = false;
    CHECK(call(5));
    CHECK(!call(5, afno::kSlotBytes + 1) && call(5, afno::kSlotBytes));
    CHECK(live == 1);
  } else if (!strcmp(t, "queries_leave_a_capture_alone")) {
    CHECK(call(5));
    finish();
    other_capture = true;
    CHECK(call(6) && thread_mode == hipStreamCaptureModeGlobal);
    CHECK(broken_captures == 0);
  } else if (!strcmp(t, "a_failed_record_waits")) {
    fail_record = true;
    CHECK(call(5));
    CHECK(synced == 1);
    fail_record = false;
    CHECK(call(6));
  } else if (!strcmp(t, "idle_slots_make_room")) {
    for (long h = 100; h < 108; ++h) CHECK(call(h));
    room = live;
    afno::Workspace held, big;
    CHECK(held.acquire(10, (hipStream_t)100) == hipSuccess && held.slot);
    CHECK(big.acquire(afno::kSlotBytes + 1, (hipStream_t)300) == hipSuccess && !big.slot);
    CHECK(live == 2);  // the held slot and the large workspace
    launch(held); held.release();
    launch(big); big.release();
    streams[{301, 0}].capturing = true;  // a capture can neither free nor wait: the error stays
    CHECK(call(100));
    room = live + pooled;
    afno::Workspace cap;
    CHECK(cap.acquire(10, (hipStream_t)301) == hipErrorOutOfMemory && live == 1);
  } else if (!strcmp(t, "threads")) {
    std::vector<std::thread> ts;
    for (long k = 1; k <= 8; ++k)
      ts.emplace_back([k] {
        thread_id = k;
        unsigned r = (unsigned)k * 2654435761u;
        for (int i = 0; i < 400; ++i) {
          r = r * 1664525u + 1013904223u;
          call((r >> 20) % 3 == 0 ? 2 : 100 + (r >> 24) % 12);
          if ((r >> 8) % 64 == 0) finish();
        }
      });
    for (auto& th : ts) th.join();
    CHECK(live <= 8);
  } else {
    return 2;
  }
  puts("OK");
  return 0;
}
"""

SCENARIOS = ["streams_that_come_and_go", "overlapping_streams", "one_handle_many_streams",
             "two_calls_at_once_on_one_stream", "captures_and_large_calls_take_the_pool",
             "queries_leave_a_capture_alone", "a_failed_record_waits", "idle_slots_make_room",
             "threads"]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"):
        pytest.skip("g++ or the HIP headers missing")
    d = tmp_path_factory.mktemp("slots")
    src, exe = d / "driver.cpp", str(d / "driver")
    src.write_text(DRIVER)
    r = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-pthread", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include", "-I" + CSRC, str(src), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("scenario", SCENARIOS)
def test_slots(driver, scenario):
    r = subprocess.run([driver, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout + r.stderr
