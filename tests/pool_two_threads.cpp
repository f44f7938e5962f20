// The device memory cache (csrc/pool.cpp) on a device of host memory: the
// driver's calls are replaced by ones that count, and a hook in the device's
// synchronisation stands for what another thread does meanwhile.
#include "../paper_1506_05083_amd/csrc/pool.cpp"

#include <cstdio>
#include <cstdlib>
#include <functional>
#include <set>
#include <thread>

namespace {
std::set<void *> g_live;
std::map<void *, size_t> g_size;
size_t g_bytes = 0, g_limit = (size_t)1 << 40;
int g_syncs = 0;
std::function<void()> g_hook;

int g_failed = 0;
void check(bool ok, const char *what) {
  std::printf("%s %s\n", ok ? "ok  " : "FAIL", what);
  std::fflush(stdout);
  if (!ok) g_failed = 1;
}
void sync_with(std::function<void()> other) {   // `other` in a thread of its own during the next synchronisation
  g_hook = [other] {
    const auto f = other;
    g_hook = nullptr;
    std::thread([f] {
      try {
        f();
      } catch (const mfs::Error &) {
        check(false, "the other thread's request is granted");
      }
    }).join();
  };
}
}  // namespace

extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
  if (g_bytes + n > g_limit) return hipErrorOutOfMemory;
  *p = std::malloc(1);
  g_live.insert(*p);
  g_size[*p] = n;
  g_bytes += n;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  if (!g_live.erase(p)) std::abort();
  g_bytes -= g_size[p];
  return hipSuccess;   // the address stays taken: a block handed out after its release is seen
}
hipError_t hipDeviceSynchronize() {
  ++g_syncs;
  if (g_hook) g_hook();
  return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return ""; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) { *t = (size_t)1 << 40; *f = *t - g_bytes; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
}

using namespace mfs;

int main() {
  const size_t small = (size_t)300 << 10, small_block = (size_t)512 << 10, large = (size_t)6 << 20;
  {
    // everything is given back while blocks are on their way from waiting to available
    std::vector<DevBuf> v;
    for (int i = 0; i < 12; ++i) v.emplace_back(small);
    v.clear();
    sync_with([] { pool_trim(0); });
    DevBuf a(small);
    check(g_syncs == 1, "a request synchronises for the waiting blocks");
    size_t idle = 0;
    pool_stats(0, nullptr, nullptr, &idle);
    check(idle == 0, "nothing is cached after everything was given back");
    check(g_bytes == small_block, "only the live block is held");
    a.release();
    pool_stats(0, nullptr, nullptr, &idle);
    check(idle == small_block && g_bytes == small_block, "released blocks are cached again");
    pool_trim(0);
    check(g_bytes == 0, "all given back");
  }
  {
    // another thread needs the memory of blocks on their way
    { DevBuf a(large), b(2 * large); }
    g_limit = 3 * large;
    DevBuf c;
    sync_with([&] { c.alloc(3 * large / 2); });
    bool refused = false;
    try {
      DevBuf d(large);
      check(d.p && g_live.count(d.p), "the waiting request gets memory too");
    } catch (const Error &) {
      refused = true;
    }
    check(c.p && g_live.count(c.p), "a failed hipMalloc frees the waiting blocks and is tried again");
    check(!refused, "no request is refused while idle memory is held");
    g_limit = (size_t)1 << 40;
    c.release();
    pool_trim(0);
    check(g_bytes == 0, "all given back");
  }
  {
    // a block released while the synchronisation runs waits for the next one
    DevBuf a(large), late(large);
    void *first = a.p, *second = late.p;
    a.release();
    sync_with([&] { late.release(); });
    DevBuf c(large);
    check(c.p == first, "the block released before the synchronisation is handed out");
    const int n = g_syncs;
    DevBuf d(large);
    check(d.p == second && g_syncs == n + 1, "the one released meanwhile only after another");
  }
  pool_trim(0);
  check(g_bytes == 0 && pool_idle_bytes(0) == 0, "nothing is left");
  return g_failed;
}
