// Large copies of results to the caller's (pageable) host arrays.
//
// A plain hipMemcpy to pageable memory moves it through one staging buffer with
// one thread, copy after copy, and that thread also takes the page faults of
// a result array that nobody has touched yet: 11 GB/s for the moments of a
// 128^3 box, where the link gives 56 GB/s.  Here several threads take chunks
// in turn: a chunk goes over the link to the thread's pinned buffer while the
// other threads copy theirs on: the moments of that box 6.0 -> 2.5 ms, its
// vorticity 5.0 -> 1.8 ms (8 and 14 threads, and 4 MiB chunks, the same).
// (Uploads stay plain copies: their source is resident, they already run at
// 26 GB/s, and the same scheme gave no more.)
#include <algorithm>
#include <atomic>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "runtime.hpp"

namespace dhit {
namespace {

// Threads (and pinned buffers) of one copy at most.  Chunks end on 2 MiB
// boundaries of the host address: a fresh array is made of 2 MiB pages, and
// two threads that fault on one wait for each other.
constexpr int kCopyThreads = 4;
constexpr size_t kChunk = size_t(2) << 20;
// Below this a plain copy is as fast as starting the threads.
constexpr size_t kPlainBytes = size_t(4) << 20;

struct Staging {
  const int dev;        // the events belong to it: only its streams take them
  void *buf = nullptr;  // kCopyThreads chunks of pinned memory
  hipEvent_t done[kCopyThreads] = {};
  explicit Staging(int d) : dev(d) {}
  ~Staging() {
    for (hipEvent_t e : done)
      if (e) (void)hipEventDestroy(e);
    if (buf) (void)hipHostFree(buf);
  }
  bool allocate() {
    if (hipHostMalloc(&buf, kCopyThreads * kChunk, hipHostMallocPortable) != hipSuccess) {
      (void)hipGetLastError();
      buf = nullptr;
      return false;
    }
    // events are made on the current device
    int was = dev;
    if (hipGetDevice(&was) != hipSuccess || (was != dev && hipSetDevice(dev) != hipSuccess)) {
      (void)hipGetLastError();
      return false;
    }
    bool ok = true;
    for (hipEvent_t &e : done)
      if (ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        e = nullptr;
        ok = false;
      }
    if (was != dev && hipSetDevice(was) != hipSuccess) ok = false;
    return ok;
  }
};

// One idle set of buffers per device is kept for the next copy while boxes
// exist; copies that run at the same time make sets of their own.  A program
// may end with boxes alive: the map is never destroyed, as the runtime can have
// ended before the library's static data would be.
std::mutex g_mu;
auto &g_idle = *new std::map<int, std::unique_ptr<Staging>>();
int g_boxes = 0;

std::unique_ptr<Staging> take_staging(int dev) {
  {
    std::lock_guard<std::mutex> lock(g_mu);
    const auto it = g_idle.find(dev);
    if (it != g_idle.end()) {
      std::unique_ptr<Staging> s = std::move(it->second);
      g_idle.erase(it);
      return s;
    }
  }
  std::unique_ptr<Staging> s(new Staging(dev));
  return s->allocate() ? std::move(s) : nullptr;
}

void give_staging(std::unique_ptr<Staging> s) {
  std::lock_guard<std::mutex> lock(g_mu);
  try {
    if (g_boxes > 0 && !g_idle.count(s->dev)) g_idle[s->dev] = std::move(s);
  } catch (const std::bad_alloc &) {
    // not kept
  }
}

// Whether the destination is memory the runtime knows: pinned (a plain copy is
// then one transfer), managed, or a device's, which the host must not write.
bool is_known(const void *p) {
  hipPointerAttribute_t a;
  if (hipPointerGetAttributes(&a, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return a.type != hipMemoryTypeUnregistered;
}

}  // namespace

void copy_to_host(std::initializer_list<HostCopy> copies, hipStream_t s) {
  std::vector<HostCopy> chunks;
  size_t total = 0;
  bool known = false;
  for (const HostCopy &c : copies) {
    if (c.bytes == 0) continue;
    total += c.bytes;
    known = known || is_known(c.dst);
    char *dst = static_cast<char *>(c.dst);
    const char *src = static_cast<const char *>(c.src);
    const size_t lead = reinterpret_cast<uintptr_t>(dst) % kChunk;
    for (size_t from = 0; from < c.bytes;) {
      const size_t to = std::min(c.bytes, (from + lead) / kChunk * kChunk + kChunk - lead);
      chunks.push_back({dst + from, src + from, to - from});
      from = to;
    }
  }
  const unsigned cpus = std::thread::hardware_concurrency();
  const int threads = (int)std::min<size_t>(std::min<size_t>(kCopyThreads, cpus ? cpus : 1), chunks.size());
  std::unique_ptr<Staging> st;
  hipDevice_t dev = 0;  // the stream's, which need not be the current one
  // (hipStreamPerThread would be another stream in each of the threads)
  if (total <= kPlainBytes || threads < 2 || known || s == hipStreamPerThread || hipStreamGetDevice(s, &dev) != hipSuccess ||
      !(st = take_staging(dev))) {
    for (const HostCopy &c : copies)
      if (c.bytes) DHIT_HIP(hipMemcpyAsync(c.dst, c.src, c.bytes, hipMemcpyDeviceToHost, s));
    DHIT_HIP(hipStreamSynchronize(s));
    return;
  }
  std::atomic<size_t> next{0};
  std::atomic<int> error{(int)hipSuccess};
  auto work = [&](int w) {
    hipError_t e = w > 0 ? hipSetDevice(dev) : hipSuccess;  // 0 is the caller's thread
    char *buf = static_cast<char *>(st->buf) + w * kChunk;
    while (e == hipSuccess && error.load() == (int)hipSuccess) {
      const size_t k = next.fetch_add(1);
      if (k >= chunks.size()) break;
      const HostCopy &c = chunks[k];
      e = hipMemcpyAsync(buf, c.src, c.bytes, hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipEventRecord(st->done[w], s);
      if (e == hipSuccess) e = hipEventSynchronize(st->done[w]);
      if (e == hipSuccess) std::memcpy(c.dst, buf, c.bytes);
    }
    if (e != hipSuccess) error.store((int)e);
  };
  std::vector<std::thread> pool;
  pool.reserve(threads - 1);
  try {
    for (int w = 1; w < threads; ++w) pool.emplace_back(work, w);
  } catch (...) {
    // no thread or no memory for one: those that started, and this one, take
    // every chunk
  }
  work(0);
  for (std::thread &t : pool) t.join();
  const hipError_t sync = hipStreamSynchronize(s);  // no transfer uses the buffers after this
  const hipError_t e = (hipError_t)error.load();
  if (sync == hipSuccess) give_staging(std::move(st));
  DHIT_HIP(e);
  DHIT_HIP(sync);
}

void box_made() {
  std::lock_guard<std::mutex> lock(g_mu);
  ++g_boxes;
}

void box_gone() {
  std::map<int, std::unique_ptr<Staging>> last;
  std::lock_guard<std::mutex> lock(g_mu);
  if (--g_boxes == 0) last.swap(g_idle);
}

}  // namespace dhit
