// See pool.h.
#include "pool.h"

#include <map>
#include <mutex>
#include <new>
#include <unordered_map>
#include <utility>
#include <vector>

namespace cgs {
namespace pool {
namespace {

// Block sizes: 256 bytes and up in steps of an eighth of the power of two
// below, from 16 MiB on whole 2 MiB pages (the driver's cost of a large block
// grows with its pages: 416 instead of 386 MB cost 100 us more).
size_t size_class(size_t bytes) {
  if (bytes <= 256) return 256;
  const size_t page = (size_t)2 << 20;
  size_t step = 32;
  while (step * 16 <= bytes && step < page) step *= 2; // 8 step <= bytes < 16 step
  return (bytes + step - 1) / step * step;
}

using Key = std::pair<int, size_t>; // device, class
// A kept block, and when it was put back (the pool's count of put-backs).
struct Block {
  void *p;
  uint64_t since;
};
struct Pinned {
  void *host, *dev;
  uint64_t since;
};

struct State {
  std::mutex mu;
  long spaces = 0;
  uint64_t count = 0; // blocks put back so far
  std::map<Key, std::vector<Block>> free_dev; // of a class, the longest kept first
  std::map<int, size_t> kept_dev; // bytes in free_dev by device
  std::unordered_map<void *, Key> live_dev;
  std::map<size_t, std::vector<Pinned>> free_pin;
  size_t kept_pin = 0;
  std::unordered_map<void *, std::pair<size_t, void *>> live_pin; // class, device address
  std::vector<std::pair<int, hipStream_t>> free_str;
  std::unordered_map<hipStream_t, int> live_str;
};
// never destroyed: handles may be released by other libraries' exit code
State &state() {
  static State *s = new State();
  return *s;
}

// Returns everything kept to the driver (the lock is held).
void trim(State &s) {
  for (auto &b : s.free_dev)
    for (Block &k : b.second) (void)hipFree(k.p);
  s.free_dev.clear();
  s.kept_dev.clear();
  for (auto &b : s.free_pin)
    for (Pinned &p : b.second) (void)hipHostFree(p.host);
  s.free_pin.clear();
  s.kept_pin = 0;
  for (auto &b : s.free_str) (void)hipStreamDestroy(b.second);
  s.free_str.clear();
}

// Gives kept device blocks of one GPU back, those kept longest first, until
// `size` more bytes stay within the cap: sizes that no handle asks for any
// more make room for those in use (the lock is held; size <= kDeviceCap).
void make_room(State &s, int dev, size_t size) {
  size_t &kept = s.kept_dev[dev];
  while (kept + size > kDeviceCap) {
    auto oldest = s.free_dev.end();
    for (auto it = s.free_dev.begin(); it != s.free_dev.end(); ++it)
      if (it->first.first == dev && !it->second.empty() &&
          (oldest == s.free_dev.end() || it->second.front().since < oldest->second.front().since))
        oldest = it;
    if (oldest == s.free_dev.end()) return;
    (void)hipFree(oldest->second.front().p);
    oldest->second.erase(oldest->second.begin());
    kept -= oldest->first.second;
    if (oldest->second.empty()) s.free_dev.erase(oldest);
  }
}
// The same for pinned blocks.
void make_room_pinned(State &s, size_t size) {
  while (s.kept_pin + size > kPinnedCap) {
    auto oldest = s.free_pin.end();
    for (auto it = s.free_pin.begin(); it != s.free_pin.end(); ++it)
      if (!it->second.empty() &&
          (oldest == s.free_pin.end() || it->second.front().since < oldest->second.front().since))
        oldest = it;
    if (oldest == s.free_pin.end()) return;
    (void)hipHostFree(oldest->second.front().host);
    oldest->second.erase(oldest->second.begin());
    s.kept_pin -= oldest->first;
    if (oldest->second.empty()) s.free_pin.erase(oldest);
  }
}

// Runs `body`, reporting a failed host allocation as hipErrorOutOfMemory.
template <typename F> hipError_t guarded(F &&body) {
  try {
    return body();
  } catch (const std::bad_alloc &) {
    return hipErrorOutOfMemory;
  }
}

} // namespace

void attach() {
  State &s = state();
  std::lock_guard<std::mutex> lock(s.mu);
  ++s.spaces;
}

void detach() {
  State &s = state();
  std::lock_guard<std::mutex> lock(s.mu);
  if (--s.spaces == 0) trim(s);
}

void release() {
  State &s = state();
  std::lock_guard<std::mutex> lock(s.mu);
  trim(s);
}

hipError_t device_get(void **p, size_t bytes) {
  *p = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  return guarded([&]() -> hipError_t {
    State &s = state();
    std::lock_guard<std::mutex> lock(s.mu);
    const Key key(dev, size_class(bytes));
    auto it = s.free_dev.find(key);
    void *q = nullptr;
    if (it != s.free_dev.end() && !it->second.empty()) {
      q = it->second.back().p;
      s.live_dev.emplace(q, key);
      it->second.pop_back();
      s.kept_dev[dev] -= key.second;
    } else {
      hipError_t r = hipMalloc(&q, key.second);
      if (r == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        trim(s);
        r = hipMalloc(&q, key.second);
      }
      if (r != hipSuccess) return r;
      try {
        s.live_dev.emplace(q, key);
      } catch (...) {
        (void)hipFree(q);
        throw;
      }
    }
    *p = q;
    return hipSuccess;
  });
}

void device_put(void *p) {
  if (!p) return;
  State &s = state();
  std::lock_guard<std::mutex> lock(s.mu);
  auto it = s.live_dev.find(p);
  if (it == s.live_dev.end()) return;
  const Key key = it->second;
  s.live_dev.erase(it);
  try {
    if (s.spaces > 0 && key.second <= kDeviceCap) {
      make_room(s, key.first, key.second);
      s.free_dev[key].push_back(Block{p, s.count++});
      s.kept_dev[key.first] += key.second;
      return;
    }
  } catch (const std::bad_alloc &) {
  }
  (void)hipFree(p);
}

hipError_t pinned_get(void **host, void **dev, size_t bytes) {
  *host = *dev = nullptr;
  return guarded([&]() -> hipError_t {
    State &s = state();
    std::lock_guard<std::mutex> lock(s.mu);
    const size_t size = size_class(bytes);
    auto it = s.free_pin.find(size);
    Pinned b{};
    if (it != s.free_pin.end() && !it->second.empty()) {
      b = it->second.back();
      s.live_pin.emplace(b.host, std::make_pair(size, b.dev));
      it->second.pop_back();
      s.kept_pin -= size;
    } else {
      hipError_t r = hipHostMalloc(&b.host, size, hipHostMallocMapped | hipHostMallocCoherent);
      if (r == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        trim(s);
        r = hipHostMalloc(&b.host, size, hipHostMallocMapped | hipHostMallocCoherent);
      }
      if (r != hipSuccess) return r;
      r = hipHostGetDevicePointer(&b.dev, b.host, 0);
      if (r != hipSuccess) {
        (void)hipHostFree(b.host);
        return r;
      }
      try {
        s.live_pin.emplace(b.host, std::make_pair(size, b.dev));
      } catch (...) {
        (void)hipHostFree(b.host);
        throw;
      }
    }
    *host = b.host;
    *dev = b.dev;
    return hipSuccess;
  });
}

void pinned_put(void *host) {
  if (!host) return;
  State &s = state();
  std::lock_guard<std::mutex> lock(s.mu);
  auto it = s.live_pin.find(host);
  if (it == s.live_pin.end()) return;
  const size_t size = it->second.first;
  Pinned b{host, it->second.second, 0};
  s.live_pin.erase(it);
  try {
    if (s.spaces > 0 && size <= kPinnedCap) {
      make_room_pinned(s, size);
      b.since = s.count++;
      s.free_pin[size].push_back(b);
      s.kept_pin += size;
      return;
    }
  } catch (const std::bad_alloc &) {
  }
  (void)hipHostFree(host);
}

hipError_t stream_get(hipStream_t *out) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  return guarded([&]() -> hipError_t {
    State &s = state();
    std::lock_guard<std::mutex> lock(s.mu);
    for (size_t i = s.free_str.size(); i-- > 0;)
      if (s.free_str[i].first == dev) {
        hipStream_t st = s.free_str[i].second;
        s.live_str.emplace(st, dev);
        s.free_str.erase(s.free_str.begin() + (long)i);
        *out = st;
        return hipSuccess;
      }
    hipStream_t st = nullptr;
    const hipError_t r = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
    if (r != hipSuccess) return r;
    try {
      s.live_str.emplace(st, dev);
    } catch (...) {
      (void)hipStreamDestroy(st);
      throw;
    }
    *out = st;
    return hipSuccess;
  });
}

void stream_put(hipStream_t st) {
  if (!st) return;
  State &s = state();
  std::lock_guard<std::mutex> lock(s.mu);
  auto it = s.live_str.find(st);
  if (it == s.live_str.end()) return;
  const int dev = it->second;
  s.live_str.erase(it);
  try {
    if (s.spaces > 0 && s.free_str.size() < kStreamCap) {
      s.free_str.emplace_back(dev, st);
      return;
    }
  } catch (const std::bad_alloc &) {
  }
  (void)hipStreamDestroy(st);
}

} // namespace pool
} // namespace cgs
