// Device memory cache of libmfs.
//
// A solve holds tens of GB for a few hundred milliseconds (the stored near
// field, the Krylov bases, the periodizer's arenas) and a serving loop or a
// benchmark repeats that many times.  Returning such blocks to the driver
// and asking for them again costs far more than the work itself on some
// steps (the driver clears and maps freed device memory before it hands it
// out again), so every buffer goes through a per-device cache: a released block
// is kept and handed to the next request of about its size (blocks under
// kPoolMin by powers of two: hipMalloc and hipFree of the 65 of a free-space
// scattering pass were 0.6 ms of its 2.3).
//
// Ordering.  hipFree waits for the device to finish the work queued before
// it, which is what makes releasing a buffer that a queued kernel still
// reads safe.  A cached block keeps that rule: a released block becomes
// available again only after a synchronisation of the device that began after
// its release, so a later request on any stream never sees it while earlier
// work still uses it.  The released blocks wait together for one such
// synchronisation, made when a request finds none available but some waiting
// (a synchronisation at every release kept the host from running ahead: 75
// of them in the k = 10 step from the geometry on).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <exception>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "internal.hpp"

namespace mfs {

namespace {

constexpr size_t kPoolMin = (size_t)1 << 20;     // smaller blocks are cached by powers of two
constexpr size_t kPoolGrain = (size_t)2 << 20;   // sizes of the others are multiples of this

constexpr int kSmallClasses = 12;                // 512 bytes << class: up to kPoolMin
constexpr size_t kSmallCap = (size_t)64 << 20;   // idle small blocks kept at most

int small_class(size_t n) {
  int c = 0;
  while (((size_t)512 << c) < n) ++c;
  return c;
}
// small blocks of a class that wait before a request synchronises for them
// (below that it allocates another)
size_t small_wait(int c) { return ((size_t)512 << c) <= ((size_t)64 << 10) ? 32 : 8; }

struct Block {
  void *p;
  uint64_t epoch;   // of its release
};
struct Blocks {
  std::multimap<size_t, Block> large;   // size -> block
  std::vector<Block> small[kSmallClasses];
  // o's blocks released up to epoch e too
  void take(Blocks &o, uint64_t e) {
    for (auto it = o.large.begin(); it != o.large.end();) {
      if (it->second.epoch <= e) large.insert(o.large.extract(it++));
      else ++it;
    }
    for (int c = 0; c < kSmallClasses; ++c) {
      auto &v = o.small[c];   // in the order of their release
      auto end = std::find_if(v.begin(), v.end(), [e](const Block &b) { return b.epoch > e; });
      small[c].insert(small[c].end(), v.begin(), end);
      v.erase(v.begin(), end);
    }
  }
};

struct Pool {
  std::mutex mu;
  Blocks ready, waiting;                // not in use: available, released since the last synchronisation
  uint64_t epoch = 0;                   // of the blocks released now: the synchronisations begun so far
  size_t idle_bytes = 0;                // of the large blocks of both
  size_t small_bytes = 0;               // of the small ones
  size_t cap = 0;                       // largest idle total kept (0: not yet read)
  size_t in_use = 0, peak = 0;          // bytes of live DevBufs (cached blocks at their block size)
};

void note_alloc(Pool &p, size_t n) {   // p.mu held
  p.in_use += n;
  if (p.in_use > p.peak) p.peak = p.in_use;
}

// One pool per device, created on first use and never destroyed: blocks
// still cached at process exit are returned by the driver with the process.
Pool &pool_of(int dev) {
  static std::mutex mu;
  static std::vector<Pool *> pools;
  std::lock_guard<std::mutex> lk(mu);
  if ((int)pools.size() <= dev) pools.resize(dev + 1, nullptr);
  if (!pools[dev]) pools[dev] = new Pool;
  return *pools[dev];
}

int current_device() {
  int dev = 0;
  HIP_CHECK(hipGetDevice(&dev));
  return dev;
}

// Free idle large blocks of p (largest first) until at most `keep` bytes stay
// idle; with keep = 0 the small ones too.  Called with p.mu held.
void trim_locked(Pool &p, size_t keep) {
  for (Blocks *b : {&p.ready, &p.waiting}) {
    while (p.idle_bytes > keep && !b->large.empty()) {
      auto it = std::prev(b->large.end());
      (void)hipFree(it->second.p);
      p.idle_bytes -= it->first;
      b->large.erase(it);
    }
    if (keep == 0)
      for (int c = 0; c < kSmallClasses; ++c) {
        for (const Block &q : b->small[c]) (void)hipFree(q.p);
        p.small_bytes -= b->small[c].size() * ((size_t)512 << c);
        b->small[c].clear();
      }
  }
}

// Make the blocks waiting now available: the device (the current one) finishes
// what was queued before their release.  lk holds p.mu, let go meanwhile; the
// blocks stay in the list, where another thread that runs out of memory or gives
// everything back still finds them, and those released meanwhile wait on.
void recycle(Pool &p, std::unique_lock<std::mutex> &lk) {
  const uint64_t e = p.epoch++;
  lk.unlock();
  const hipError_t err = hipDeviceSynchronize();
  lk.lock();
  if (err == hipSuccess) p.ready.take(p.waiting, e);
  else (void)hipGetLastError();
}

// the smallest block that fits, if it wastes at most 1/8 of it
std::multimap<size_t, Block>::iterator fit(std::multimap<size_t, Block> &m, size_t want) {
  auto it = m.lower_bound(want);
  return it != m.end() && it->first - want <= want / 8 ? it : m.end();
}

// hipMalloc; the idle blocks are given back and it is tried again if it fails
void *device_malloc(Pool &pl, size_t n) {
  void *q = nullptr;
  if (hipMalloc(&q, n) == hipSuccess) return q;
  (void)hipGetLastError();
  {
    std::lock_guard<std::mutex> lk(pl.mu);
    trim_locked(pl, 0);
  }
  if (hipMalloc(&q, n) == hipSuccess) return q;
  (void)hipGetLastError();
  throw Error{MFS_ENOMEM, "hipMalloc of " + std::to_string(n) + " bytes failed"};
}

}  // namespace

void DevBuf::alloc(size_t n) {
  release();
  if (n == 0) return;
  dev = current_device();
  Pool &pl = pool_of(dev);
  std::unique_lock<std::mutex> lk(pl.mu);
  if (n < kPoolMin) {
    const int c = small_class(n);
    auto &v = pl.ready.small[c];
    if (v.empty() && pl.waiting.small[c].size() >= small_wait(c)) recycle(pl, lk);
    const size_t size = (size_t)512 << c;
    if (!v.empty()) {
      p = v.back().p;
      v.pop_back();
      pl.small_bytes -= size;
    } else {
      lk.unlock();
      p = device_malloc(pl, size);
      lk.lock();
    }
    cached = size;
    bytes = n;
    note_alloc(pl, n);
    return;
  }
  const size_t want = (n + kPoolGrain - 1) / kPoolGrain * kPoolGrain;
  auto it = fit(pl.ready.large, want);
  if (it == pl.ready.large.end() && fit(pl.waiting.large, want) != pl.waiting.large.end()) {
    recycle(pl, lk);
    it = fit(pl.ready.large, want);
  }
  if (it != pl.ready.large.end()) {
    p = it->second.p;
    cached = it->first;
    pl.idle_bytes -= it->first;
    pl.ready.large.erase(it);
  } else {
    lk.unlock();
    p = device_malloc(pl, want);
    lk.lock();
    cached = want;
  }
  bytes = n;
  note_alloc(pl, cached);
}

void DevBuf::release() {
  if (!p) return;
  Pool &pl = pool_of(dev);
  const bool small = cached < kPoolGrain;
  int prev = 0;
  (void)hipGetDevice(&prev);
  if (prev != dev) (void)hipSetDevice(dev);
  {
    std::lock_guard<std::mutex> lk(pl.mu);
    pl.in_use -= small ? bytes : cached;
    if (small) {
      if (pl.small_bytes + cached > kSmallCap) {
        (void)hipFree(p);
      } else {
        pl.waiting.small[small_class(cached)].push_back({p, pl.epoch});
        pl.small_bytes += cached;
      }
    } else {
      if (pl.cap == 0) {
        size_t fr = 0, tot = 0;
        (void)hipMemGetInfo(&fr, &tot);
        pl.cap = tot / 2;   // keep at most half of the device idle in the cache
      }
      pl.waiting.large.emplace(cached, Block{p, pl.epoch});
      pl.idle_bytes += cached;
      trim_locked(pl, pl.cap);
    }
  }
  if (prev != dev) (void)hipSetDevice(prev);
  p = nullptr;
  bytes = 0;
  cached = 0;
}

namespace {
constexpr size_t kPinned = (size_t)64 << 10;
constexpr size_t kPinnedKept = 16;
std::mutex g_pinned_mu;
std::vector<void *> &pinned_idle() {
  static auto *v = new std::vector<void *>;   // still valid while the process ends
  return *v;
}
}  // namespace

PinnedBuf::PinnedBuf(size_t n) : bytes(std::max(n, kPinned)) {
  if (bytes == kPinned) {
    std::lock_guard<std::mutex> lk(g_pinned_mu);
    auto &v = pinned_idle();
    if (!v.empty()) {
      p = v.back();
      v.pop_back();
      return;
    }
  }
  if (hipHostMalloc(&p, bytes, hipHostMallocPortable) != hipSuccess) {
    p = nullptr;
    (void)hipGetLastError();
    throw Error{MFS_ENOMEM, "hipHostMalloc of " + std::to_string(bytes) + " bytes failed"};
  }
}

PinnedBuf::~PinnedBuf() {
  if (!p) return;
  if (bytes == kPinned && std::uncaught_exceptions() == 0) {
    std::lock_guard<std::mutex> lk(g_pinned_mu);
    auto &v = pinned_idle();
    if (v.size() < kPinnedKept) {
      v.push_back(p);
      return;
    }
  }
  (void)hipHostFree(p);
}

size_t pool_idle_bytes(int dev) {
  Pool &pl = pool_of(dev);
  std::lock_guard<std::mutex> lk(pl.mu);
  return pl.idle_bytes + pl.small_bytes;
}

void pool_trim(int dev) {
  Pool &pl = pool_of(dev);
  int prev = 0;
  (void)hipGetDevice(&prev);
  if (prev != dev) (void)hipSetDevice(dev);
  {
    std::lock_guard<std::mutex> lk(pl.mu);
    trim_locked(pl, 0);
  }
  {
    std::lock_guard<std::mutex> lk(g_pinned_mu);
    for (void *q : pinned_idle()) (void)hipHostFree(q);
    pinned_idle().clear();
  }
  if (prev != dev) (void)hipSetDevice(prev);
}

void pool_stats(int dev, size_t *in_use, size_t *peak, size_t *idle) {
  Pool &pl = pool_of(dev);
  std::lock_guard<std::mutex> lk(pl.mu);
  if (in_use) *in_use = pl.in_use;
  if (peak) *peak = pl.peak;
  if (idle) *idle = pl.idle_bytes + pl.small_bytes;
}

void pool_reset_peak(int dev) {
  Pool &pl = pool_of(dev);
  std::lock_guard<std::mutex> lk(pl.mu);
  pl.peak = pl.in_use;
}

size_t device_free_bytes() {
  size_t fr = 0, tot = 0;
  HIP_CHECK(hipMemGetInfo(&fr, &tot));
  return fr + pool_idle_bytes(current_device());
}

}  // namespace mfs
