// Device and pinned host memory of the set-up calls (plans, transposition, edge lists).
//
// hipMalloc and hipFree cost tens to hundreds of microseconds each (a free waits for the device and unmaps), and setting a
// graph up takes some forty of each: 4.5 of the 6.1 ms that a 5.5 M-edge list took to become a graph, its transpose and
// two plans.  Freed blocks are therefore kept for the next set-up call:
//  - at most kKeepBytes per device, blocks of up to half of that (so the sort buffers of graphs beyond some 33 M edges, 8 bytes an
//    edge, are allocated and freed on every call); what no set-up call has asked for during the last
//    kKeepCalls allocations is freed, everything when an allocation fails or on hgnn_release_cached_memory();
//  - callers free a block only when no work that uses it is in flight on any stream (set-up calls synchronize their
//    stream first; hgnn_plan_destroy, and calls that replace arrays of a plan, wait for the plan's device), so a kept block may
//    be handed to any stream or thread at once; a block for which the wait failed goes back to the runtime instead;
//  - one mutex; blocks belong to the device that was current when they were allocated.
#include <mutex>
#include <unordered_map>

#include "common.h"

namespace hgnn {

namespace {

constexpr size_t kKeepBytes = size_t(512) << 20;
constexpr uint64_t kKeepCalls = 1024;
constexpr int kMailSlots = 64;

struct KeptBlock {
  void* p;
  size_t bytes;
  uint64_t freed_at;
};

struct Pool {
  std::mutex mu;
  std::unordered_map<void*, std::pair<size_t, int>> live;  // block -> (bytes, device)
  std::unordered_map<int, std::vector<KeptBlock>> kept;    // device -> free blocks, oldest first
  std::unordered_map<int, size_t> kept_bytes;
  uint64_t calls = 0;
  // pinned host slots of kMailBytes
  char* mail = nullptr;
  uint64_t mail_used = 0;  // one bit per slot
};

Pool& pool() {
  static Pool* p = new Pool();  // never destroyed: plans may be destroyed by other static objects' destructors
  return *p;
}

// A plan may be destroyed by any thread at any time, also by one that is capturing another stream (a garbage collector runs
// where it likes).  In the relaxed mode memory may be freed meanwhile, and the capture goes on.
struct RelaxedCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  const bool on = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
  ~RelaxedCapture() {
    if (on) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
};

void release_older_than(Pool& P, int dev, uint64_t call) {
  const RelaxedCapture relaxed;
  std::vector<KeptBlock>& v = P.kept[dev];
  size_t n = 0;
  while (n < v.size() && v[n].freed_at < call) {
    P.kept_bytes[dev] -= v[n].bytes;
    (void)hipFree(v[n].p);
    ++n;
  }
  v.erase(v.begin(), v.begin() + long(n));
}

}  // namespace

hipError_t dev_malloc_bytes(void** out, size_t bytes) {
  *out = nullptr;
  if (bytes == 0) bytes = 16;
  bytes = bytes < (size_t(1) << 20) ? (bytes + 511) / 512 * 512 : (bytes + 65535) / 65536 * 65536;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  ++P.calls;
  if (P.calls > kKeepCalls) release_older_than(P, dev, P.calls - kKeepCalls);
  std::vector<KeptBlock>& v = P.kept[dev];
  size_t best = v.size();
  for (size_t i = 0; i < v.size(); ++i)  // the smallest that fits and is not much too large
    if (v[i].bytes >= bytes && v[i].bytes <= bytes + bytes / 4 + 4096 && (best == v.size() || v[i].bytes < v[best].bytes)) best = i;
  if (best < v.size()) {
    *out = v[best].p;
    P.live[*out] = {v[best].bytes, dev};
    P.kept_bytes[dev] -= v[best].bytes;
    v.erase(v.begin() + long(best));
    return hipSuccess;
  }
  e = hipMalloc(out, bytes);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    release_older_than(P, dev, ~uint64_t(0));
    e = hipMalloc(out, bytes);
  }
  if (e == hipSuccess) P.live[*out] = {bytes, dev};
  return e;
}

void dev_free(const void* cp) {
  void* p = const_cast<void*>(cp);
  if (p == nullptr) return;
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  const auto it = P.live.find(p);
  if (it == P.live.end()) return;  // not one of ours
  const size_t bytes = it->second.first;
  const int dev = it->second.second;
  P.live.erase(it);
  if (bytes > kKeepBytes / 2) {
    const RelaxedCapture relaxed;
    (void)hipFree(p);
    return;
  }
  std::vector<KeptBlock>& v = P.kept[dev];
  while (!v.empty() && P.kept_bytes[dev] + bytes > kKeepBytes) release_older_than(P, dev, v.front().freed_at + 1);
  v.push_back({p, bytes, P.calls});
  P.kept_bytes[dev] += bytes;
}

void dev_release(const void* cp) {
  void* p = const_cast<void*>(cp);
  if (p == nullptr) return;
  Pool& P = pool();
  {
    std::lock_guard<std::mutex> lock(P.mu);
    if (P.live.erase(p) == 0) return;  // not one of ours
  }
  const RelaxedCapture relaxed;
  if (hipFree(p) != hipSuccess) (void)hipGetLastError();
}

bool device_idle(int dev) {
  int cur = 0;
  if (hipGetDevice(&cur) != hipSuccess || (cur != dev && hipSetDevice(dev) != hipSuccess)) return false;
  const RelaxedCapture relaxed;
  // freeing memory waits for the device; hipDeviceSynchronize would invalidate any capture of the process, in every mode (1.4 us
  // against 0.5 on an idle device)
  void* fence = nullptr;
  hipError_t e = hipMalloc(&fence, 16);
  if (e == hipSuccess) e = hipFree(fence);
  if (e != hipSuccess) (void)hipGetLastError();
  if (cur != dev) (void)hipSetDevice(cur);
  return e == hipSuccess;
}

HostMail::HostMail(SetupStream& stream) : s(stream) {
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  if (P.mail == nullptr) {
    void* m = nullptr;
    if (hipHostMalloc(&m, size_t(kMailSlots) * kMailBytes, hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) return;
    P.mail = static_cast<char*>(m);
  }
  for (int i = 0; i < kMailSlots; ++i) {
    if (P.mail_used >> i & 1) continue;
    P.mail_used |= uint64_t(1) << i;
    slot = i;
    data = P.mail + size_t(i) * kMailBytes;
    return;
  }
}

HostMail::~HostMail() {
  if (slot < 0 || !s.settle()) return;  // a kernel may still write to it: never used again
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  P.mail_used &= ~(uint64_t(1) << slot);
}

}  // namespace hgnn

using namespace hgnn;

extern "C" void hgnn_release_cached_memory(void) {
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  std::vector<int> devs;
  for (const auto& k : P.kept) devs.push_back(k.first);
  for (int d : devs) release_older_than(P, d, ~uint64_t(0));
}
