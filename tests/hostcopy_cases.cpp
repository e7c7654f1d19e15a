// Cases of the library's copies to the host on the stand-in runtime; argv[1]
// names one.  Exit status 0: as it should be.
#define FAKE_HIP_MAIN
#include "fake_hip.hpp"

#include <algorithm>
#include <new>
#include <vector>

#include "../paper_1601_03815_amd/csrc/runtime.hpp"

// Allocations of the main thread until one fails (< 0: none does).
static thread_local int allocations_left = -1;
void *operator new(size_t n) {
  if (allocations_left == 0) throw std::bad_alloc();
  if (allocations_left > 0) --allocations_left;
  if (void *p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

static std::vector<char> pattern(size_t n, int seed) {
  std::vector<char> v(n);
  for (size_t i = 0; i < n; ++i) v[i] = (char)((i * 2654435761u + seed) >> 7);
  return v;
}

// Copies n bytes on s and says whether they arrived.
static bool copy_on(hipStream_t s, size_t n, int seed) {
  const std::vector<char> src = pattern(n, seed);
  std::vector<char> dst(n + 64, 0x55);
  dhit::copy_to_host({{dst.data() + 8, src.data(), n}}, s);
  for (size_t i = 0; i < dst.size(); ++i)
    if (dst[i] != (i >= 8 && i < n + 8 ? src[i - 8] : 0x55)) return false;
  return true;
}

#define CHECK(x)                                             \
  do {                                                       \
    if (!(x)) {                                              \
      std::fprintf(stderr, "line %d: %s\n", __LINE__, #x);   \
      return 1;                                              \
    }                                                        \
  } while (0)

constexpr size_t kLarge = (size_t(9) << 20) + 40;

// Boxes on two devices of one process, also when the stream's device is not
// the current one; what is kept goes with the last box.
static int two_devices() {
  hipStream_t s[2] = {fake::stream(0), fake::stream(1)};
  dhit::box_made();
  dhit::box_made();
  for (int k = 0; k < 6; ++k) {
    const int d = (k / 2 + k) % 2;
    CHECK(hipSetDevice(k < 4 ? d : 1 - d) == hipSuccess);
    CHECK(copy_on(s[d], kLarge, k));
    int now = -1;
    CHECK(hipGetDevice(&now) == hipSuccess && now == (k < 4 ? d : 1 - d));
  }
  CHECK(fake::pinned.size() <= 2);
  dhit::box_gone();
  dhit::box_gone();
  CHECK(fake::pinned.empty() && fake::live_events == 0);
  return 0;
}

// Memory the runtime knows is left to the runtime, whatever its kind: device
// memory, which the host may not touch, among it.
static int known_destinations() {
  dhit::box_made();
  for (hipMemoryType kind : {hipMemoryTypeHost, hipMemoryTypeDevice, hipMemoryTypeManaged, hipMemoryTypeUnified}) {
    const std::vector<char> src = pattern(kLarge, 3);
    std::vector<char> dst(kLarge);
    fake::kinds[dst.data()] = kind;
    fake::copies = 0;
    dhit::copy_to_host({{dst.data(), src.data(), kLarge}}, fake::stream(0));
    CHECK(fake::copies == 1 && dst == src);
    fake::kinds.clear();
  }
  dhit::box_gone();
  return 0;
}

// hipStreamPerThread names another stream in every thread: only the caller's is
// ordered after the box's work.
static int per_thread_stream() {
  dhit::box_made();
  for (int k = 0; k < 3; ++k) {
    CHECK(copy_on(hipStreamPerThread, kLarge, k));
    CHECK(fake::foreign_per_thread == 0);
  }
  dhit::box_gone();
  return 0;
}

// Every allocation of a copy fails once: the copy is whole, or the caller gets
// the exception; the program goes on.
static int out_of_memory() {
  const std::vector<char> src = pattern(kLarge, 5);
  hipStream_t s = fake::stream(0);
  dhit::box_made();
  int thrown = 0, whole = 0;
  for (int k = 0; whole < 3 && k < 1000; ++k) {
    std::vector<char> dst(kLarge);
    bool failed = false;
    allocations_left = k;
    try {
      dhit::copy_to_host({{dst.data(), src.data(), kLarge}}, s);
    } catch (const std::bad_alloc &) {
      failed = true;
    }
    whole += !failed && allocations_left > 0;  // nothing was left to fail
    allocations_left = -1;
    if (failed)
      ++thrown;
    else
      CHECK(dst == src);
  }
  CHECK(whole == 3 && thrown > 0);
  dhit::box_gone();
  CHECK(fake::pinned.empty() && fake::live_events == 0);
  return 0;
}

// A program that ends with a box alive: the runtime may have ended before the
// library's own data does.
static int box_at_exit() {
  dhit::box_made();
  CHECK(copy_on(fake::stream(0), kLarge, 1));
  std::atexit([] { fake::ended = true; });
  return 0;
}

// Every 8-byte phase of a cache line, and destinations that begin and end on
// both sides of a chunk's end (2 MiB of the host address): each byte once, none
// beside.
static int phases() {
  constexpr size_t chunk = size_t(2) << 20;
  std::vector<char> mem(kLarge + 3 * chunk);
  const size_t base = (chunk - reinterpret_cast<uintptr_t>(mem.data()) % chunk) % chunk + chunk;
  const std::vector<char> src = pattern(kLarge, 9);
  dhit::box_made();
  for (size_t bytes : {kLarge, 3 * chunk, 3 * chunk - 8, 3 * chunk + 8})
    for (int phase = -9; phase <= 9; ++phase) {
      std::fill(mem.begin(), mem.end(), (char)0x55);
      char *dst = mem.data() + base + 8 * (ptrdiff_t)phase;
      const size_t half = bytes / 16 * 8;  // two results of one call
      dhit::copy_to_host({{dst, src.data(), half}, {dst + half, src.data() + half, bytes - half}}, fake::stream(0));
      CHECK(std::memcmp(dst, src.data(), bytes) == 0);
      for (const char *c = mem.data(); c < dst; ++c) CHECK(*c == 0x55);
      for (const char *c = dst + bytes; c < mem.data() + mem.size(); ++c) CHECK(*c == 0x55);
    }
  dhit::box_gone();
  return 0;
}

int main(int argc, char **argv) {
  const std::string c = argc > 1 ? argv[1] : "";
  if (c == "two_devices") return two_devices();
  if (c == "known_destinations") return known_destinations();
  if (c == "per_thread_stream") return per_thread_stream();
  if (c == "out_of_memory") return out_of_memory();
  if (c == "box_at_exit") return box_at_exit();
  if (c == "phases") return phases();
  return 2;
}
