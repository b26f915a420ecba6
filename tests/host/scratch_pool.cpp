// Host check of the scratch pool (scratch_pool.h; built by
// tests/test_host_parts.py) against a HIP runtime of this file: calls can be made to
// fail, the last error stays set until it is read, and an event is done when
// the test says so.
#include <stdio.h>
#include <stdlib.h>

#include <set>

#include "scratch_pool.h"

static hipError_t last = hipSuccess;
static hipError_t fail_malloc, fail_event, fail_capturing, fail_free, fail_record;
static hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
static bool done = true;
static int device = 0;
static std::set<void *> held;

static hipError_t ret(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}

extern "C" {
hipError_t hipGetLastError(void) {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t hipGetDevice(int *d) { return *d = device, hipSuccess; }
hipError_t hipMallocAsync(void **p, size_t, hipStream_t) {
  if (fail_malloc) return ret(fail_malloc);
  held.insert(*p = malloc(1));
  return hipSuccess;
}
hipError_t hipFreeAsync(void *p, hipStream_t) {
  if (fail_free) return ret(fail_free);
  if (!held.erase(p)) abort();
  free(p);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  if (fail_event) return ret(fail_event);
  *e = (hipEvent_t)malloc(1);
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { return free((void *)e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return ret(fail_record); }
hipError_t hipEventQuery(hipEvent_t) { return ret(done ? hipSuccess : hipErrorNotReady); }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
  *s = capturing;
  return ret(fail_capturing);
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
}

#define CHECK(x) \
  if (!(x)) return printf("line %d: %s\n", __LINE__, #x), 1

int main() {
  char *p = nullptr;
  {  // a pool that cannot grow hands out nothing and leaves no error behind
    fbg::ScratchPool pool(0);
    pool.program_added();
    fail_malloc = hipErrorOutOfMemory;
    CHECK(pool.acquire(100, nullptr, &p) == -1 && last == hipSuccess);
    fail_malloc = hipSuccess, fail_event = hipErrorOutOfMemory;
    CHECK(pool.acquire(100, nullptr, &p) == -1 && last == hipSuccess && held.empty());
    fail_event = hipSuccess, fail_capturing = hipErrorStreamCaptureImplicit;
    CHECK(pool.acquire(100, nullptr, &p) == -1 && last == hipSuccess);
    fail_capturing = hipSuccess, capturing = hipStreamCaptureStatusActive;
    CHECK(pool.acquire(100, nullptr, &p) == -1 && held.empty());
    capturing = hipStreamCaptureStatusNone;
    CHECK(pool.acquire(fbg::ScratchPool::kBlock + 1, nullptr, &p) == -1 && held.empty());
    const int a = pool.acquire(100, nullptr, &p);
    CHECK(a == 0 && held.count(p));
    CHECK(pool.release(a, nullptr) == hipSuccess);
    // in flight: another block; done: the same ones, no new memory
    done = false;
    for (int k = 1; k < fbg::ScratchPool::kBlocks; k++) {
      const int b = pool.acquire(100, nullptr, &p);
      CHECK(b == k && last == hipSuccess && pool.release(b, nullptr) == hipSuccess);
    }
    CHECK(pool.acquire(100, nullptr, &p) == -1 && last == hipSuccess);
    done = true;
    for (int k = 0; k < 20; k++) {
      const int b = pool.acquire(100, nullptr, &p);
      CHECK(b >= 0 && pool.release(b, nullptr) == hipSuccess);
    }
    CHECK(held.size() == (size_t)fbg::ScratchPool::kBlocks);
    // a block whose event could not be recorded is not handed out again
    const int c = pool.acquire(100, nullptr, &p);
    char *const lost = p;
    fail_record = hipErrorInvalidHandle;
    CHECK(pool.release(c, nullptr) != hipSuccess && last == hipSuccess);
    fail_record = hipSuccess;
    for (int k = 0; k < 20; k++) {
      const int b = pool.acquire(100, nullptr, &p);
      CHECK(b >= 0 && p != lost && pool.release(b, nullptr) == hipSuccess);
    }
    // the last program goes: what the runtime does not take back stays in the pool
    fail_free = hipErrorInvalidValue;
    pool.program_removed();
    CHECK(last == hipSuccess && held.size() == (size_t)fbg::ScratchPool::kBlocks);
    fail_free = hipSuccess;
    for (void *q : held) free(q);
    held.clear();
  }
  {  // all but one block go back with the last program, or once they are done after it
    fbg::ScratchPool pool(0);
    pool.program_added();
    int b[4];
    for (int &k : b) k = pool.acquire(100, nullptr, &p);
    for (int k : b) CHECK(pool.release(k, nullptr) == hipSuccess);
    done = false;
    pool.program_removed();
    CHECK(held.size() == 4 && last == hipSuccess);
    done = true;
    const int c = pool.acquire(100, nullptr, &p);
    CHECK(c >= 0 && pool.release(c, nullptr) == hipSuccess && held.size() == 1);
    // without any program (stored vectors) the pool does not keep what it grew to
    for (int &k : b) k = pool.acquire(100, nullptr, &p);
    CHECK(held.size() == 4);
    for (int k : b) CHECK(pool.release(k, nullptr) == hipSuccess);
    CHECK(held.size() == 1 && last == hipSuccess);
  }
  return 0;
}
