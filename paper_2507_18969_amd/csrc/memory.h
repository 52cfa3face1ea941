// Device memory of one object, and the tables it uploads.
//
// A hipMalloc costs 20 to 30 us and a hipFree 60 us or more: a 1024-stream
// session with a call for each of its 110 arrays spent 9 of the 40 ms of
// a 160-byte encode on them.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

namespace edpc {

void hip_check(hipError_t e, const char* what);
// hipMalloc; when memory runs out the kept scratch memory (below) goes back and it
// is tried once more.
void* device_malloc(size_t bytes);

class DeviceMemory {
 public:
  DeviceMemory() = default;
  DeviceMemory(const DeviceMemory&) = delete;
  DeviceMemory& operator=(const DeviceMemory&) = delete;
  ~DeviceMemory() { release(); }

  // Memory for n elements, 256-byte aligned, held until release().  Small
  // requests share 1 MiB chunks.
  template <class T>
  T* take(size_t n) {
    return (T*)bytes(std::max<size_t>(n, 1) * sizeof(T));
  }
  // One block for everything `place` takes: it runs once to add up the sizes
  // (the addresses it gets then are not memory) and once for good.
  template <class F>
  void place_together(F&& place) {
    measuring_ = true;
    need_ = 0;
    place();
    measuring_ = false;
    grow(need_);
    place();
  }
  void release() {
    for (void* p : blocks_) (void)hipFree(p);
    blocks_.clear();
    left_ = 0;
  }

 private:
  static constexpr size_t kChunk = 1 << 20;
  void* bytes(size_t b) {
    b = (b + 255) & ~(size_t)255;
    if (measuring_) {
      need_ += b;
      return (void*)need_;
    }
    if (b > left_) {
      if (b >= kChunk / 4) return block(b);
      grow(kChunk);
    }
    void* p = next_;
    next_ += b;
    left_ -= b;
    return p;
  }
  void* block(size_t b) {
    void* p = device_malloc(b);
    blocks_.push_back(p);
    return p;
  }
  void grow(size_t b) {
    next_ = (char*)block(std::max<size_t>(b, 256));
    left_ = b;
  }

  std::vector<void*> blocks_;
  char* next_ = nullptr;
  size_t left_ = 0, need_ = 0;
  bool measuring_ = false;
};

// Host tables that go to the device in one copy per commit().  The host images
// live as long as this object, so a copy may still be under way after commit().
class Upload {
 public:
  // *dst receives the device address of a copy of src at commit().
  template <class T>
  void add(T** dst, const T* src, size_t n) {
    const size_t off = (image_.size() + 255) & ~(size_t)255;
    image_.resize(off + std::max<size_t>(n, 1) * sizeof(T));
    if (n) std::memcpy(image_.data() + off, src, n * sizeof(T));
    items_.push_back({(void**)dst, off});
  }
  template <class T>
  void add(T** dst, const std::vector<T>& src) {
    add(dst, src.data(), src.size());
  }
  void commit(DeviceMemory& mem, hipStream_t s) {
    char* base = mem.take<char>(image_.size());
    hip_check(hipMemcpyAsync(base, image_.data(), image_.size(), hipMemcpyHostToDevice, s), "copy");
    for (const Item& i : items_) *i.dst = base + i.off;
    items_.clear();
    sent_.push_back(std::move(image_));
    image_.clear();
  }

 private:
  struct Item {
    void** dst;
    size_t off;
  };
  std::vector<char> image_;
  std::vector<Item> items_;
  std::vector<std::vector<char>> sent_;
};

// Scratch memory of one synchronous call on stream s, for callers that hold no
// object to keep it in.  The destructor waits for s, and then up to 64 MiB in all
// stay for later calls of any thread or stream on the same device that ask for at
// least half of a block (blocks of up to 1 MiB: for any part).  A block that 64
// calls have not used goes back, and all of them do when an allocation of this
// library runs out of memory or a model is made.  (Mutual information of 1024
// samples, 8 MiB: 113 to 60 us.)
constexpr size_t kScratchKept = (size_t)64 << 20;  // all devices together
class Scratch {
 public:
  Scratch(size_t bytes, hipStream_t s);
  ~Scratch();
  Scratch(const Scratch&) = delete;
  Scratch& operator=(const Scratch&) = delete;
  void* get() const { return p_; }

 private:
  hipStream_t s_;
  void* p_ = nullptr;
  size_t bytes_ = 0;
  int device_ = 0;
};
void scratch_give_back();

}  // namespace edpc
