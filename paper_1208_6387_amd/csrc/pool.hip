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
// Kept on a device: 1/LIVE_PART of its memory while a pattern or structure exists, 1/IDLE_PART (1.2 GB of 288) once
// the last one is freed, since others can use that memory then.  A pattern set up and freed alone: 12^3 8.7 ms, 13.8
// with nothing kept; 20^3, whose 4.5 GB do not stay, 66, and 59 with LIVE_PART.
constexpr size_t LIVE_PART = 32, IDLE_PART = 256;
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
  std::unordered_map<int, size_t> memory;       // by device
  uint64_t ops = 0;
  int64_t handles = 0;

  size_t limit(int dev) {
    auto it = memory.find(dev);
    if (it == memory.end()) {
      size_t total = 0;
      if (hipDeviceTotalMem(&total, dev) != hipSuccess) return 0;
      it = memory.emplace(dev, total).first;
    }
    return it->second / (handles > 0 ? LIVE_PART : IDLE_PART);
  }
  void give_back(size_t i) {
    (void)hipFree(kept[i].p);
    kept_bytes[kept[i].dev] -= kept[i].bytes;
    kept.erase(kept.begin() + (std::ptrdiff_t)i);
  }
  // the oldest blocks of a device until it holds at most `most` bytes
  void trim(int dev, size_t most) {
    for (size_t i = 0; i < kept.size() && kept_bytes[dev] > most;)
      if (kept[i].dev == dev) give_back(i);
      else ++i;
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
    const Pool::Block b = P.kept[best];
    P.live[b.p] = b;  // may throw: the block is still kept then
    P.kept.erase(P.kept.begin() + (std::ptrdiff_t)best);
    P.kept_bytes[dev] -= b.bytes;
    return b.p;
  }
  hipError_t e = hipMalloc(&p, bytes);
  if (e != hipSuccess && !P.kept.empty()) {  // what is kept stands in the way of nothing
    (void)hipGetLastError();
    while (!P.kept.empty()) P.give_back(0);
    e = hipMalloc(&p, bytes);
  }
  if (e != hipSuccess) return nullptr;
  try {
    P.live[p] = Pool::Block{p, bytes, dev, 0};
  } catch (...) {
    (void)hipFree(p);
    throw;
  }
  return p;
}

// Called from destructors: nothing leaves it.
void dev_free(void* p) noexcept {
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
  try {
    const size_t most = P.limit(b.dev);
    b.op = P.ops;
    size_t& held = P.kept_bytes[b.dev];
    if (b.bytes <= most) {
      P.kept.push_back(b);
      held += b.bytes;
      P.trim(b.dev, most);
      return;
    }
  } catch (...) {  // no room for the note of it
  }
  (void)hipFree(p);
}

size_t dev_available() {
  size_t free_b = 0, total_b = 0;
  int dev = 0;
  RPF_HIP(hipGetDevice(&dev));
  RPF_HIP(hipMemGetInfo(&free_b, &total_b));
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  const auto it = P.kept_bytes.find(dev);
  return free_b + (it == P.kept_bytes.end() ? 0 : it->second);
}

void dev_release() {
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  while (!P.kept.empty()) P.give_back(0);
}

HandleRef::HandleRef() {
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  ++P.handles;
}

HandleRef::~HandleRef() {
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  if (--P.handles > 0) return;
  for (const auto& d : P.memory) P.trim(d.first, d.second / IDLE_PART);
}

}  // namespace rpf
