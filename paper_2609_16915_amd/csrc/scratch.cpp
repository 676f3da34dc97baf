// Scratch memory of single calls: stream-ordered, from one pool per device,
// so that calls on several streams or threads each have their own.  A pool
// keeps what was freed, up to KEEP bytes, between calls; scratch_release
// gives that back.
#include <hip/hip_runtime.h>

#include <map>
#include <mutex>

#include "internal.hpp"

namespace rosetta {

namespace {

// Room for the largest expanded key (N = 4096, l = 3, n = 2048, 4 pieces: 3.2
// GB).  What is kept is not lost to the program:
// the runtime's hipMalloc takes it back when the device runs out (3.4 GiB kept,
// 3.2 GiB free: hipMalloc of 4 GiB 0.5 ms, with calls running 41 ms).  Keeping
// 256 MiB instead cost 0.3-0.7 % (3072 GPT-2 ciphertexts 68.8 -> 69.3 ms).
constexpr uint64_t KEEP = (uint64_t)4 << 30;
std::mutex g_mu;
std::map<int, hipMemPool_t> g_pools;

hipError_t device_pool(hipMemPool_t *out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(g_mu);
  auto it = g_pools.find(dev);
  if (it == g_pools.end()) {
    hipMemPoolProps props{};
    props.allocType = hipMemAllocationTypePinned;
    props.handleTypes = hipMemHandleTypeNone;
    props.location.type = hipMemLocationTypeDevice;
    props.location.id = dev;
    hipMemPool_t pool;
    if ((e = hipMemPoolCreate(&pool, &props)) != hipSuccess) return e;
    uint64_t keep = KEEP;
    (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep);
    it = g_pools.emplace(dev, pool).first;
  }
  *out = it->second;
  return hipSuccess;
}

}  // namespace

void *scratch_take(size_t bytes, hipStream_t st) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  hipMemPool_t pool;
  void *p = nullptr;
  const bool ok = hipStreamIsCapturing(st, &cap) == hipSuccess &&
                  cap == hipStreamCaptureStatusNone && device_pool(&pool) == hipSuccess &&
                  hipMallocFromPoolAsync(&p, bytes, pool, st) == hipSuccess;
  if (ok) return p;
  // (a failed call's error must not surface at the caller's next launch)
  if (cap == hipStreamCaptureStatusNone) (void)hipGetLastError();
  return nullptr;
}

hipError_t scratch_give(void *p, hipStream_t st) { return hipFreeAsync(p, st); }

// Frees still pending on a stream are not the pool's to give back yet, and a
// device may have a pool and no other state of the library (a program that
// only key-switches), so each device is waited for here.
void scratch_release() {
  int cur = 0;
  (void)hipGetDevice(&cur);
  std::lock_guard<std::mutex> lock(g_mu);
  for (auto &kv : g_pools) {
    (void)hipSetDevice(kv.first);
    (void)hipDeviceSynchronize();
    (void)hipMemPoolTrimTo(kv.second, 0);
  }
  (void)hipSetDevice(cur);
}

}  // namespace rosetta
