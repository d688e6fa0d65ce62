// Device memory of the library's buffers (DevBuf).  Large blocks are kept when they are released, up
// to a bound, and handed out again: mapping and unmapping them costs more than the work on them
// (hipMalloc and hipFree of 54 MB: 0.4 and 0.9 ms; half of the 17 ms of a 12^3 pattern's setup was
// spent there).
#include "common.hpp"

#include <mutex>
#include <unordered_map>

namespace rpf {
namespace {

// Smaller blocks cost 3 us to allocate and 2 us to free, less than the wait that a kept block needs.
constexpr size_t KEEP_MIN = 256 << 10;
// A kept block serves requests down to 7/8 of its size.
inline bool fits(size_t have, size_t need) { return have >= need && have - need <= have / 8; }
// A kept block that this many later allocations passed over is given back.
constexpr uint64_t KEEP_OPS = 512;

struct Pool {
  struct Block {
    void* p;
    size_t bytes;
    int dev;
    uint64_t op;  // when it was released
  };
  std::mutex mu;
  std::vector<Block> kept;                      // oldest first
  std::unordered_map<void*, Block> live;        // large blocks in use
  std::unordered_map<int, size_t> kept_bytes;   // by device
  std::unordered_map<int, size_t> bound;        // by device: 1/32 of its memory
  uint64_t ops = 0;

  size_t limit(int dev) {
    auto it = bound.find(dev);
    if (it != bound.end()) return it->second;
    size_t f = 0, t = 0;
    if (hipMemGetInfo(&f, &t) != hipSuccess) return 0;
    return bound[dev] = t / 32;
  }
  void give_back(size_t i) {
    (void)hipFree(kept[i].p);
    kept_bytes[kept[i].dev] -= kept[i].bytes;
    kept.erase(kept.begin() + (std::ptrdiff_t)i);
  }
};

// never destroyed: buffers of static objects may outlive any destructor here
Pool& pool() {
  static Pool* p = new Pool;
  return *p;
}

}  // namespace

// A block that was released may still be read by work that was queued before: like hipFree, which waits
// for the device, handing it out again does.  The wait also keeps an allocation under stream capture
// the error that hipMalloc makes of it.
void* dev_alloc(size_t bytes) {
  void* p = nullptr;
  if (bytes < KEEP_MIN) return hipMalloc(&p, bytes) == hipSuccess ? p : nullptr;
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return nullptr;
  ++P.ops;
  for (size_t i = 0; i < P.kept.size();)
    if (P.ops - P.kept[i].op > KEEP_OPS) P.give_back(i);
    else ++i;
  size_t best = P.kept.size();
  for (size_t i = 0; i < P.kept.size(); ++i)
    if (P.kept[i].dev == dev && fits(P.kept[i].bytes, bytes) &&
        (best == P.kept.size() || P.kept[i].bytes < P.kept[best].bytes))
      best = i;
  if (best < P.kept.size()) {
    if (hipDeviceSynchronize() != hipSuccess) return nullptr;
    Pool::Block b = P.kept[best];
    P.kept.erase(P.kept.begin() + (std::ptrdiff_t)best);
    P.kept_bytes[dev] -= b.bytes;
    P.live[b.p] = b;
    return b.p;
  }
  hipError_t e = hipMalloc(&p, bytes);
  if (e != hipSuccess && !P.kept.empty()) {  // what is kept stands in the way of nothing
    (void)hipGetLastError();
    while (!P.kept.empty()) P.give_back(0);
    e = hipMalloc(&p, bytes);
  }
  if (e != hipSuccess) return nullptr;
  P.live[p] = Pool::Block{p, bytes, dev, 0};
  return p;
}

void dev_free(void* p) {
  if (!p) return;
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  auto it = P.live.find(p);
  if (it == P.live.end()) {
    (void)hipFree(p);
    return;
  }
  Pool::Block b = it->second;
  P.live.erase(it);
  const size_t most = P.limit(b.dev);
  if (b.bytes > most) {
    (void)hipFree(p);
    return;
  }
  b.op = P.ops;
  P.kept.push_back(b);
  P.kept_bytes[b.dev] += b.bytes;
  for (size_t i = 0; i < P.kept.size() && P.kept_bytes[b.dev] > most;)
    if (P.kept[i].dev == b.dev) P.give_back(i);
    else ++i;
}

}  // namespace rpf
