// Scratch memory of the synchronous calls; see memory.h.
#include "memory.h"

#include <mutex>

namespace edpc {

namespace {
struct Kept {
  int device;
  void* p;
  size_t bytes;
  int age;  // calls since it was last used
};
constexpr int kKeptAge = 64;
// A small call takes no large block: it would keep it from ageing.
bool fits(size_t kept, size_t bytes) { return kept >= bytes && kept <= std::max(2 * bytes, (size_t)1 << 20); }

struct Pool {
  std::mutex mu;
  std::vector<Kept> free;
  size_t bytes = 0;

  // drops the blocks that `gone` names, or hands one over
  template <class F>
  void drop(F&& gone) {
    for (size_t i = 0; i < free.size();)
      if (gone(free[i])) {
        (void)hipFree(free[i].p);
        bytes -= free[i].bytes;
        free.erase(free.begin() + i);
      } else {
        ++i;
      }
  }
};
Pool& pool() {
  static Pool* p = new Pool;  // never destroyed: calls may run until the process ends
  return *p;
}
}  // namespace

Scratch::Scratch(size_t bytes, hipStream_t s) : s_(s) {
  hip_check(hipGetDevice(&device_), "hipGetDevice");
  bytes = std::max<size_t>((bytes + 255) & ~(size_t)255, 256);
  Pool& pl = pool();
  std::lock_guard<std::mutex> lk(pl.mu);
  size_t best = pl.free.size();
  for (size_t i = 0; i < pl.free.size(); ++i) {
    ++pl.free[i].age;
    if (pl.free[i].device == device_ && fits(pl.free[i].bytes, bytes) &&
        (best == pl.free.size() || pl.free[i].bytes < pl.free[best].bytes))
      best = i;
  }
  if (best < pl.free.size()) {
    p_ = pl.free[best].p;
    bytes_ = pl.free[best].bytes;
    pl.bytes -= bytes_;
    pl.free.erase(pl.free.begin() + best);
  } else {
    bytes_ = bytes;
    hipError_t e = hipMalloc(&p_, bytes_);
    if (e == hipErrorOutOfMemory) {  // everything kept goes back first
      (void)hipGetLastError();
      pl.drop([](const Kept&) { return true; });
      e = hipMalloc(&p_, bytes_);
    }
    hip_check(e, "hipMalloc");
  }
  pl.drop([](const Kept& k) { return k.age > kKeptAge; });
}

Scratch::~Scratch() {
  if (hipStreamSynchronize(s_) != hipSuccess) return;  // (a failed device: nothing can be reused or freed)
  Pool& pl = pool();
  std::lock_guard<std::mutex> lk(pl.mu);
  if (pl.bytes + bytes_ > kScratchKept) {
    (void)hipFree(p_);
    return;
  }
  pl.free.push_back(Kept{device_, p_, bytes_, 0});
  pl.bytes += bytes_;
}

void* device_malloc(size_t bytes) {
  void* p = nullptr;
  hipError_t e = hipMalloc(&p, bytes);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    scratch_give_back();
    e = hipMalloc(&p, bytes);
  }
  hip_check(e, "hipMalloc");
  return p;
}

void scratch_give_back() {
  Pool& pl = pool();
  std::lock_guard<std::mutex> lk(pl.mu);
  pl.drop([](const Kept&) { return true; });
}

}  // namespace edpc
