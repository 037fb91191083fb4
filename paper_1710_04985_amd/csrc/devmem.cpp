// A store of freed device blocks, so that the setup of the next handle finds
// its few large allocations at hand: the driver takes 40 to 200 us to give out
// a block of this size and, depending on its state, 0.3 or 4 to 6 ms to take
// one back (128^3 7-point: blocks of 131 and 267 MB).
//
// The store is bounded (kKeepBytes over all devices; the block freed longest
// ago goes first), gives everything back when an allocation fails or the caller
// asks for it, and gives back a block that kKeepFrees later ones have passed over.  A block enters it
// only when its device is idle, so the next owner may use it on any stream.
#include "devmem.hpp"

#include <iterator>
#include <list>
#include <map>
#include <mutex>
#include <vector>

namespace sptrsv {
namespace {

constexpr int64_t kLarge = 1 << 20;          // smaller ones cost the runtime about 1 us
constexpr int64_t kKeepBytes = 1ll << 30;
constexpr int64_t kKeepFrees = 64;

struct Block {
  void* p;
  int64_t bytes;
  int device;
  int64_t freed;                             // count of frees when it was stored
};

// Every failure below is answered for here or by the status returned; the
// runtime keeps it as the thread's last error all the same, until it is asked
// for, and the check behind the next launch would take it for its own.
hipError_t settled(hipError_t e) {
  if (e != hipSuccess) (void)hipGetLastError();
  return e;
}

struct Store {
  std::mutex mu;                             // the lists; not held over calls that may wait
  std::mutex emptying;                       // held while blocks go back for want of memory
  std::map<void*, Block> live;               // large blocks in use
  std::list<Block> kept;                     // oldest first
  int64_t kept_bytes = 0, frees = 0;

  // Takes out the oldest blocks until `bytes` remain, and those passed over.
  std::vector<void*> trim(int64_t bytes) {
    std::vector<void*> out;
    while (!kept.empty() && (kept_bytes > bytes || frees - kept.front().freed > kKeepFrees)) {
      out.push_back(kept.front().p);
      kept_bytes -= kept.front().bytes;
      kept.pop_front();
    }
    return out;
  }

  std::vector<void*> trim_all() {
    std::lock_guard<std::mutex> lock(mu);
    return trim(0);
  }
};

// A free waits for the block's device, for as long as its work takes: other
// threads' allocations are not to wait with it.
void give_back(const std::vector<void*>& blocks) {
  for (void* p : blocks) (void)settled(hipFree(p));
}

// Waits for all work on the current device.  By a free, which does so, and not
// by hipDeviceSynchronize: that breaks the graph capture of another stream also
// where the capture allows calls like hipFree.
bool wait_idle() {
  void* p = nullptr;
  return settled(hipMalloc(&p, 1)) == hipSuccess && settled(hipFree(p)) == hipSuccess;
}

// never destroyed: the runtime may be gone when static destructors run
Store& store() {
  static Store* s = new Store;
  return *s;
}

}  // namespace

namespace {

// hipMalloc; without memory for it, again after the store has been emptied
// (also by another thread, which may still be at it).
hipError_t device_malloc(void** p, int64_t bytes) {
  const hipError_t e = settled(hipMalloc(p, static_cast<size_t>(bytes)));
  if (e != hipErrorOutOfMemory) return e;
  Store& s = store();
  std::lock_guard<std::mutex> one(s.emptying);
  give_back(s.trim_all());
  return settled(hipMalloc(p, static_cast<size_t>(bytes)));
}

// Whether a kept block is still an allocation of its own: a reset of its device
// takes it away.
bool still_there(const Block& b) {
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  return settled(hipMemGetAddressRange(&base, &size, b.p)) == hipSuccess && base == b.p &&
         static_cast<int64_t>(size) >= b.bytes;
}

}  // namespace

hipError_t dev_alloc(void** p, int64_t bytes) {
  *p = nullptr;
  if (bytes < 1) bytes = 1;
  if (bytes < kLarge) return device_malloc(p, bytes);
  int device = 0;
  if (const hipError_t e = settled(hipGetDevice(&device))) return e;
  constexpr int64_t kUnit = 2 << 20;
  bytes = (bytes + kUnit - 1) / kUnit * kUnit;
  Store& s = store();
  {
    std::lock_guard<std::mutex> lock(s.mu);
    for (;;) {
      // the smallest block that fits, if at most a quarter of it would lie idle
      auto best = s.kept.end();
      for (auto it = s.kept.begin(); it != s.kept.end(); ++it)
        if (it->device == device && it->bytes >= bytes && it->bytes - bytes <= it->bytes / 4 &&
            (best == s.kept.end() || it->bytes < best->bytes))
          best = it;
      if (best == s.kept.end()) break;
      const Block b = *best;
      s.kept_bytes -= b.bytes;
      s.kept.erase(best);
      if (!still_there(b)) continue;
      *p = b.p;
      s.live[b.p] = b;
      return hipSuccess;
    }
  }
  const hipError_t e = device_malloc(p, bytes);
  if (e == hipSuccess) {
    std::lock_guard<std::mutex> lock(s.mu);
    s.live[*p] = Block{*p, bytes, device, 0};
  }
  return e;
}

void dev_free(void* p) {
  if (!p) return;
  Store& s = store();
  Block b{nullptr, 0, 0, 0};
  {
    std::lock_guard<std::mutex> lock(s.mu);
    auto it = s.live.find(p);
    if (it != s.live.end()) {
      b = it->second;
      s.live.erase(it);
    }
  }
  bool idle = false;
  if (b.p && b.bytes <= kKeepBytes) {
    int device = 0;
    idle = hipGetDevice(&device) == hipSuccess &&
           (device == b.device || hipSetDevice(b.device) == hipSuccess);
    idle = idle && wait_idle();
    if (device != b.device) (void)hipSetDevice(device);
  }
  if (!idle) {
    (void)settled(hipFree(p));
    return;
  }
  std::vector<void*> back;
  {
    std::lock_guard<std::mutex> lock(s.mu);
    b.freed = ++s.frees;
    s.kept.push_back(b);
    s.kept_bytes += b.bytes;
    back = s.trim(kKeepBytes);
  }
  give_back(back);
}

void dev_release() { give_back(store().trim_all()); }

}  // namespace sptrsv
