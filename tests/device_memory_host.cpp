// Host test of the device buffers: the library's header over a model of two devices, in which
// memory has a size, work is in flight until its device is waited for, and hipFree waits.
// The first argument names the scenario; exit status 0 when it holds.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <string>

#include "../paper_2606_24748_amd/csrc/device_memory.hpp"

namespace {
struct Model {
  int current = 0;
  size_t free_bytes[2] = {size_t{64} << 30, size_t{64} << 30};
  std::map<void*, std::pair<int, size_t>> owned;  // device and size of every block
  std::set<void*> in_use[2];                      // blocks that queued work of the device still uses
  int waits[2] = {0, 0}, mallocs = 0, frees = 0;
  bool fail_waits = false;  // as while a stream is captured
  uintptr_t next = 4096;
} model;

void wait(int d) {
  ++model.waits[d];
  model.in_use[d].clear();
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { *d = model.current; return hipSuccess; }
hipError_t hipSetDevice(int d) { model.current = d; return hipSuccess; }
hipError_t hipDeviceTotalMem(size_t* bytes, int) { *bytes = size_t{64} << 30; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "model"; }
hipError_t hipDeviceSynchronize() {
  if (model.fail_waits) return hipErrorStreamCaptureUnsupported;
  wait(model.current);
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes) {
  size_t& left = model.free_bytes[model.current];
  if (bytes > left) return hipErrorOutOfMemory;
  left -= bytes;
  *p = reinterpret_cast<void*>(model.next);
  model.next += (bytes + 4095) / 4096 * 4096;
  model.owned[*p] = {model.current, bytes};
  ++model.mallocs;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  const auto it = model.owned.find(p);
  if (it == model.owned.end()) std::abort();
  wait(it->second.first);
  model.free_bytes[it->second.first] += it->second.second;
  model.owned.erase(it);
  ++model.frees;
  return hipSuccess;
}
}

namespace blk {
void set_last_error(const std::string&) {}
}  // namespace blk

using blk::AllocScope;
using blk::DevBuf;

#define CHECK(c)                                                       \
  do {                                                                 \
    if (!(c)) {                                                        \
      std::printf("line %d: %s does not hold\n", __LINE__, #c);        \
      return 1;                                                        \
    }                                                                  \
  } while (0)

namespace {
void queue(int d, const DevBuf<char>& b) { model.in_use[d].insert(b.p); }
bool busy(const DevBuf<char>& b) { return model.in_use[0].count(b.p) || model.in_use[1].count(b.p); }

// A block of each device comes back with work in flight; waiting for one device must not pass
// for waiting for the other.
int two_devices() {
  DevBuf<char> alive(256);
  for (int d = 0; d < 2; ++d) {
    AllocScope scope;
    model.current = d;
    DevBuf<char> b(1 << 20);
    queue(d, b);
  }
  DevBuf<char> again[2];
  for (int d = 0; d < 2; ++d) {
    AllocScope scope;
    model.current = d;
    const int before = model.mallocs;
    again[d].alloc(1 << 20);
    CHECK(model.mallocs == before);  // the kept block
    CHECK(model.owned.at(again[d].p).first == d);
    CHECK(!busy(again[d]));
  }
  return 0;
}

// Outside a setup a released buffer waits for its device, current or not, as hipFree does ...
int release_waits() {
  DevBuf<char> alive(256), far(4096), near(4096);
  model.current = 1;
  far.alloc(4096);
  model.current = 0;
  queue(0, near);
  queue(1, far);
  far.release();
  CHECK(model.in_use[1].empty() && model.in_use[0].size() == 1 && model.current == 0);
  near.release();
  CHECK(model.in_use[0].empty());
  return 0;
}

// ... a handle's buffers together once, and so does a setup that gave buffers back or failed.
int scopes_wait() {
  DevBuf<char> alive(256), many[5];
  for (auto& b : many) queue(0, (b.alloc(4096), b));
  {
    blk::FreeScope scope;
    for (auto& b : many) b.release();
  }
  CHECK(model.in_use[0].empty() && model.waits[0] == 1);
  for (int kind = 0; kind < 3; ++kind) {  // gives nothing back; gives a buffer back; fails
    DevBuf<char> caller(512), kept;
    try {
      AllocScope outer;
      {
        AllocScope inner;
        kept.alloc(100 << 10);
        if (kind == 1) kept.release();
      }
      queue(0, caller);
      if (kind == 2) blk::fail(BLKAMG_EINVAL, "as a setup would");
    } catch (const blk::Error&) {
    }
    CHECK(busy(caller) == (kind == 0));
    model.in_use[0].clear();
  }
  return 0;
}

// A wait that is refused (capture) does not count as one.
int refused_waits() {
  DevBuf<char> alive(256), b(1 << 20);
  queue(0, b);
  void* const p = b.p;
  model.fail_waits = true;
  b.release();
  {
    AllocScope scope;
    b.alloc(1 << 20);
    CHECK(b.p != p);  // not handed out
  }
  model.fail_waits = false;
  AllocScope scope;
  DevBuf<char> c(1 << 20);
  CHECK(c.p == p && !busy(c));
  return 0;
}

// A program that sets up, solves with vectors allocated outside the setup, and destroys, again
// and again: the first round's memory serves all.
int rounds() {
  DevBuf<char> alive(256);
  int first = 0;
  for (int round = 0; round < 20; ++round) {
    DevBuf<char> plan, vec[2];
    {
      AllocScope setup;
      DevBuf<char> scratch(3 << 20);
      queue(0, scratch);
      plan.alloc(5 << 20);
    }
    for (auto& v : vec) {
      v.alloc(9 << 20);
      CHECK(!busy(v));
      queue(0, v);
    }
    blk::FreeScope destroy;
    plan.release();
    for (auto& v : vec) v.release();
    if (round == 0) first = model.mallocs;
  }
  CHECK(model.mallocs == first && model.frees == 0);
  return 0;
}

size_t used() {
  size_t sum = 0;
  for (const auto& b : model.owned) sum += b.second.second;
  return sum;
}

// Kept blocks: a 64th of the device's memory at most, for requests of at least 7/8 of their
// size, and none once the last buffer is gone.
int bound() {
  constexpr size_t kMiB = size_t{1} << 20;
  {
    DevBuf<char> alive(256);
    {
      DevBuf<char> a(600 * kMiB), b(600 * kMiB);
    }
    CHECK(used() == 256 + 600 * kMiB);
    AllocScope scope;
    int before = model.mallocs;
    DevBuf<char> small(524 * kMiB);
    CHECK(model.mallocs == before + 1);
    DevBuf<char> fits(526 * kMiB);
    CHECK(model.mallocs == before + 1 && fits.cap == 600 * kMiB);
  }
  CHECK(model.owned.empty());
  return 0;
}

void* caller_alloc(size_t bytes, void*) {
  void* p = nullptr;
  return hipMalloc(&p, bytes) == hipSuccess ? p : nullptr;
}
void caller_free(void* p, size_t, void*) { (void)hipFree(p); }

// Kept blocks go back when hipMalloc or the caller's allocator finds no memory, or on request.
int given_back() {
  constexpr size_t kGiB = size_t{1} << 30;
  DevBuf<char> alive(256);
  for (int round = 0; round < 3; ++round) {
    DevBuf<char> held(kGiB);
    held.release();
    CHECK(used() == 256 + kGiB);
    if (round == 2) {
      CHECK(blk::BlockCache::get().trim() && !blk::BlockCache::get().trim());
    } else {
      if (round == 1) blk::allocator_slot() = {caller_alloc, caller_free, nullptr};
      DevBuf<char> rest(63 * kGiB + kGiB / 2);
      blk::allocator_slot() = {};
      bool refused = false;
      try {
        DevBuf<char> more(kGiB);
      } catch (const blk::Error& e) {
        refused = e.code == BLKAMG_ENOMEM;
      }
      CHECK(refused);
      rest.release();
      blk::BlockCache::get().trim();
    }
    CHECK(used() == 256);
  }
  return 0;
}
}  // namespace

int main(int argc, char** argv) {
  const std::map<std::string, int (*)()> all{{"two_devices", two_devices},
                                                {"release_waits", release_waits},
                                                {"scopes_wait", scopes_wait},
                                                {"refused_waits", refused_waits},
                                                {"rounds", rounds},
                                                {"bound", bound},
                                                {"given_back", given_back}};
  const auto it = argc == 2 ? all.find(argv[1]) : all.end();
  return it == all.end() ? 2 : it->second();
}
