// Device memory of plans and of the library's temporaries.
//
// Building a plan and destroying it took ten hipMalloc and ten hipFree calls:
// about 30 and 110 us each, 1.3 of the 3.0 ms that the plan, the transpose and
// the first SpMV of R-MAT 20 took (a hipFree unmaps the pages and waits for
// the device).  Freed blocks are therefore kept for the next allocation of
// about their size.
//   - bounded: at most kPoolBytes are kept, the least recently freed block
//     goes back to the device first, and a block that kPoolAge later calls
//     have not reused goes back as well;
//   - given back: when an allocation fails, everything kept is returned to the
//     device and the allocation tried again;
//   - not under capture: where hipMalloc is refused, so is a kept block;
//   - no work pending: a caller frees a block only after it has waited for the
//     work that uses it (the streams of the call, or the device), so a block
//     can be handed to any stream; dev_free itself does not wait;
//   - any thread, any device: one lock, and a block is handed out only on the
//     device it was allocated on.
#include <mutex>
#include <unordered_map>
#include <vector>

#include "merbit_host.hpp"

namespace merbit {

namespace {

constexpr size_t kPoolBytes = (size_t)512 << 20;
constexpr uint64_t kPoolAge = 512;

struct Block {
  void* ptr;
  size_t bytes;
  int device;
  uint64_t freed;  // number of the call that freed it
};

struct Pool {
  std::mutex mu;
  std::unordered_map<void*, Block> live;
  std::vector<Block> kept;  // in the order they were freed
  size_t kept_bytes = 0;
  uint64_t calls = 0;

  void give_back(size_t i) {
    (void)hipFree(kept[i].ptr);
    kept_bytes -= kept[i].bytes;
    kept.erase(kept.begin() + (ptrdiff_t)i);
  }
};

// never destroyed: plans may outlive static objects
Pool& pool() {
  static Pool* p = new Pool();
  return *p;
}

// sizes are rounded so that plans of nearly equal matrices share blocks
size_t rounded(size_t bytes) {
  const size_t unit = bytes < ((size_t)1 << 20) ? (size_t)4 << 10 : (size_t)1 << 20;
  return (bytes + unit - 1) / unit * unit;
}

}  // namespace

hipError_t dev_alloc_bytes(void** out, size_t bytes) noexcept try {
  *out = nullptr;
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return e;
  // a kept block is handed out only where hipMalloc would be allowed: it is
  // refused while a stream is captured (by this thread, or by any in global
  // mode), and a call that went on would have its kernels recorded with memory
  // that it gives up when it returns.  Size 0 allocates nothing (0.3 us).
  void* none = nullptr;
  if ((e = hipMalloc(&none, 0)) != hipSuccess) return e;
  const size_t want = rounded(bytes > 0 ? bytes : 1);
  Pool& p = pool();
  std::lock_guard<std::mutex> lock(p.mu);
  ++p.calls;
  // the smallest kept block that fits without wasting over a quarter of itself
  size_t best = p.kept.size();
  for (size_t i = 0; i < p.kept.size(); ++i) {
    const Block& b = p.kept[i];
    if (b.device == device && b.bytes >= want && b.bytes - want <= b.bytes / 4 &&
        (best == p.kept.size() || b.bytes < p.kept[best].bytes))
      best = i;
  }
  Block b{nullptr, want, device, 0};
  if (best < p.kept.size()) {
    b = p.kept[best];
    p.live.emplace(b.ptr, b);  // before it leaves the list: this may throw
    p.kept_bytes -= b.bytes;
    p.kept.erase(p.kept.begin() + (ptrdiff_t)best);
    *out = b.ptr;
    return hipSuccess;
  }
  e = hipMalloc(&b.ptr, want);
  if (e == hipErrorOutOfMemory && !p.kept.empty()) {
    (void)hipGetLastError();
    while (!p.kept.empty()) p.give_back(0);
    e = hipMalloc(&b.ptr, want);
  }
  if (e != hipSuccess) return e;
  try {
    p.live.emplace(b.ptr, b);
  } catch (...) {
    (void)hipFree(b.ptr);
    throw;
  }
  *out = b.ptr;
  return hipSuccess;
} catch (...) {
  // the records of the blocks are host memory: to the callers, which hold other
  // blocks to give up, its end is one more failed allocation
  return hipErrorOutOfMemory;
}

void dev_free(void* ptr) noexcept {
  if (!ptr) return;
  Pool& p = pool();
  std::lock_guard<std::mutex> lock(p.mu);
  ++p.calls;
  auto it = p.live.find(ptr);
  if (it == p.live.end()) return;  // not ours
  Block b = it->second;
  p.live.erase(it);
  b.freed = p.calls;
  bool keep = b.bytes <= kPoolBytes;
  if (keep) {
    try {
      p.kept.push_back(b);
      p.kept_bytes += b.bytes;
    } catch (...) {
      keep = false;
    }
  }
  if (!keep) (void)hipFree(ptr);
  while (!p.kept.empty() &&
         (p.kept_bytes > kPoolBytes || p.calls - p.kept.front().freed > kPoolAge))
    p.give_back(0);
}

void dev_free_after(hipError_t waited, void* ptr) noexcept {
  if (waited == hipSuccess) return dev_free(ptr);
  if (!ptr) return;
  {
    Pool& p = pool();
    std::lock_guard<std::mutex> lock(p.mu);
    if (p.live.erase(ptr) == 0) return;  // not ours
  }
  (void)hipFree(ptr);
}

}  // namespace merbit
