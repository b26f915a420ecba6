// scratch_pool.h -- device scratch of the enumerations, kept between calls.
#ifndef FBG_SCRATCH_POOL_H
#define FBG_SCRATCH_POOL_H

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

#include <mutex>
#include <vector>

namespace fbg {

// Device scratch for the temporaries of an enumeration.  hipMallocAsync and
// hipFreeAsync cost the host 11 us a call (whatever the pool's release
// threshold); a block kept here costs an event record and a query.  A block is
// handed out again only once the event recorded behind its last use has
// completed, so calls on any streams and threads may overlap, each with its own
// block; with every block in flight, under stream capture (a graph may replay
// at any time) or beyond kBlock bytes the caller allocates on its stream as
// before.  At most kBlocks blocks of a device; with its last program all but one
// go back, or with a later call while there is no program once they are done
// (stream-ordered: no call waits for the device).  A call of the runtime that
// fails here leaves no error behind: the caller goes on without the pool, and
// the launches that follow report the last error as theirs.
class ScratchPool {
 public:
  static constexpr size_t kBlock = (size_t)16 << 20;
  static constexpr int kBlocks = 8;

  static ScratchPool &of(int dev) {
    static std::mutex m;
    static std::vector<ScratchPool *> pools;
    std::lock_guard<std::mutex> g(m);
    if ((size_t)dev >= pools.size()) pools.resize((size_t)dev + 1, nullptr);
    if (!pools[(size_t)dev]) pools[(size_t)dev] = new ScratchPool(dev);
    return *pools[(size_t)dev];
  }

  explicit ScratchPool(int dev) : dev_(dev) { b_.reserve(kBlocks); }

  // A block for `bytes` of work on s, a stream of the current device, or -1.
  int acquire(size_t bytes, hipStream_t s, char **out) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (bytes > kBlock || failed(hipStreamIsCapturing(s, &cap)) || cap != hipStreamCaptureStatusNone) return -1;
    std::lock_guard<std::mutex> g(mu_);
    const RelaxedCapture relaxed;
    for (size_t i = 0; i < b_.size(); i++) {
      const size_t k = (next_ + i) % b_.size();
      if (b_[k].taken) continue;
      if (b_[k].used && failed(hipEventQuery(b_[k].done))) continue;
      return take(k, out);
    }
    if (b_.size() >= (size_t)kBlocks) return -1;
    Block n;
    // on s, where its first use follows; later uses follow that one's event
    if (failed(hipMallocAsync((void **)&n.p, kBlock, s))) return -1;
    if (failed(hipEventCreateWithFlags(&n.done, hipEventDisableTiming))) {
      (void)failed(hipFreeAsync(n.p, s));
      return -1;
    }
    b_.push_back(n);
    return take(b_.size() - 1, out);
  }

  // The work using block k has been put on s.
  hipError_t release(int k, hipStream_t s) {
    std::lock_guard<std::mutex> g(mu_);
    Block &b = b_[(size_t)k];
    const hipError_t e = hipEventRecord(b.done, s);
    b.used = true;
    if (!failed(e)) b.taken = false;  // else it is never handed out again
    if (programs_ <= 0) shrink();
    return e;
  }

  void program_added() {
    std::lock_guard<std::mutex> g(mu_);
    programs_++;
  }
  void program_removed() {
    std::lock_guard<std::mutex> g(mu_);
    if (--programs_ <= 0) shrink();
  }

 private:
  static bool failed(hipError_t e) {
    if (e != hipSuccess) (void)hipGetLastError();
    return e != hipSuccess;
  }
  void shrink() {
    if (b_.size() < 2) return;
    int cur = -1;
    if (failed(hipGetDevice(&cur)) || cur != dev_) return;  // (with a later call on the device)
    const RelaxedCapture relaxed;
    while (b_.size() > 1) {
      const Block &n = b_.back();
      // in use or in flight: the blocks before it keep their index
      if (n.taken || (n.used && failed(hipEventQuery(n.done))) || failed(hipFreeAsync(n.p, nullptr))) return;
      (void)failed(hipEventDestroy(n.done));
      b_.pop_back();
    }
  }

  // A query or an allocation does not disturb another stream's capture.
  struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  };
  struct Block {
    char *p = nullptr;
    hipEvent_t done = nullptr;
    bool taken = false, used = false;
  };
  int take(size_t k, char **out) {
    b_[k].taken = true;
    next_ = k + 1;
    *out = b_[k].p;
    return (int)k;
  }
  const int dev_;
  std::mutex mu_;
  std::vector<Block> b_;
  size_t next_ = 0;
  int64_t programs_ = 0;
};

}  // namespace fbg

#endif
