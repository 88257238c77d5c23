// Device memory of plans and of the library's temporaries.
//
// Building a plan and destroying it took ten hipMalloc and ten hipFree calls:
// about 30 and 110 us each, 1.3 of the 3.0 ms that the plan, the transpose and
// the first SpMV of R-MAT 20 took (a hipFree unmaps the pages and waits for
// the device).  Freed blocks are therefore kept for the next allocation of
// about their size.
//   - bounded: at most kPoolBytes are kept, over all devices; the least
//     recently freed block goes back to the device first, and a block that
//     kPoolAge later calls of dev_alloc and dev_free have not reused goes back
//     as well;
//   - given back: all of it when an allocation fails (which is then tried
//     again) and when the caller asks for it (merbit_release_memory); a process
//     that makes no more calls holds what it has until then;
//   - not under capture: where hipMalloc is refused, so is a kept block;
//   - no work pending: a caller frees a block only after it has waited for the
//     work that uses it (the streams of the call, or the device), so a block
//     can be handed to any stream; dev_free itself does not wait;
//   - any thread, any device: one lock for the records, which is not held
//     while the runtime allocates or frees, and a block is handed out only on
//     the device it was allocated on.
// The bound holds the blocks of a plan, transpose and product of R-MAT 20: 319
// MiB (FP32), 324 (FP64), which take 1.00 ms per matrix with kept blocks and 1.22
// ms with hipMalloc alone (R-MAT 18: 81 MiB, 0.49 and 0.7-0.9 ms; R-MAT 16: 16
// MiB, 0.19 and 0.24-0.29 ms).  The age is that of about 25 such matrices (a plan
// and its transpose make 20 calls), and a request takes a block up to a third
// larger, so that matrices whose sizes differ by that much share blocks.
#include <list>
#include <mutex>
#include <unordered_map>

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

typedef std::list<Block> Blocks;

struct Pool {
  std::mutex mu;  // of the records below
  std::unordered_map<void*, Block> live;
  Blocks kept;  // in the order they were freed
  size_t kept_bytes = 0;
  uint64_t calls = 0;
  // held while blocks go back to the device: an allocation that failed waits
  // for those that are on their way
  std::mutex returning;

  // Take the oldest kept blocks out while `more` says so (mu is held).
  template <typename F>
  void take(Blocks& out, F&& more) {
    while (!kept.empty() && more(kept.front())) {
      kept_bytes -= kept.front().bytes;
      out.splice(out.end(), kept, kept.begin());
    }
  }
  // Return blocks to the device (returning is held, mu is not).  One that
  // hipFree refuses, while another thread captures a stream, is kept on.
  // Returns the bytes returned.
  size_t give_back(Blocks& blocks) {
    size_t n = 0;
    while (!blocks.empty()) {
      const size_t b = blocks.front().bytes;
      if (hipFree(blocks.front().ptr) == hipSuccess) {
        n += b;
        blocks.pop_front();
        continue;
      }
      (void)hipGetLastError();
      std::lock_guard<std::mutex> lock(mu);
      kept.splice(kept.begin(), blocks, blocks.begin());
      kept_bytes += b;
    }
    return n;
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
  {
    std::lock_guard<std::mutex> lock(p.mu);
    ++p.calls;
    // the smallest kept block that fits without wasting over a quarter of itself
    auto best = p.kept.end();
    for (auto b = p.kept.begin(); b != p.kept.end(); ++b)
      if (b->device == device && b->bytes >= want && b->bytes - want <= b->bytes / 4 &&
          (best == p.kept.end() || b->bytes < best->bytes))
        best = b;
    if (best != p.kept.end()) {
      p.live.emplace(best->ptr, *best);  // before it leaves the list: this may throw
      *out = best->ptr;
      p.kept_bytes -= best->bytes;
      p.kept.erase(best);
      return hipSuccess;
    }
  }
  Block b{nullptr, want, device, 0};
  e = hipMalloc(&b.ptr, want);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    std::lock_guard<std::mutex> returning(p.returning);
    Blocks all;
    {
      std::lock_guard<std::mutex> lock(p.mu);
      p.take(all, [](const Block&) { return true; });
    }
    p.give_back(all);
    e = hipMalloc(&b.ptr, want);
  }
  if (e != hipSuccess) return e;
  try {
    std::lock_guard<std::mutex> lock(p.mu);
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
  Blocks old;
  bool keep = false;
  {
    std::lock_guard<std::mutex> lock(p.mu);
    ++p.calls;
    auto it = p.live.find(ptr);
    if (it == p.live.end()) return;  // not ours
    Block b = it->second;
    p.live.erase(it);
    b.freed = p.calls;
    if (b.bytes <= kPoolBytes) {
      try {
        p.kept.push_back(b);
        p.kept_bytes += b.bytes;
        keep = true;
      } catch (...) {
      }
    }
    p.take(old, [&](const Block& k) {
      return p.kept_bytes > kPoolBytes || p.calls - k.freed > kPoolAge;
    });
  }
  if (!keep) (void)hipFree(ptr);
  if (old.empty()) return;
  std::lock_guard<std::mutex> returning(p.returning);
  p.give_back(old);
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

size_t dev_release() noexcept {
  Pool& p = pool();
  std::lock_guard<std::mutex> returning(p.returning);
  Blocks all;
  {
    std::lock_guard<std::mutex> lock(p.mu);
    p.take(all, [](const Block&) { return true; });
  }
  return p.give_back(all);
}

}  // namespace merbit

extern "C" int64_t merbit_release_memory(void) { return (int64_t)merbit::dev_release(); }
