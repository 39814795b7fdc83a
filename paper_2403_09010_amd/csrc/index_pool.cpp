// Device memory of freed indexes (sd_internal.h): kept for the next index of its
// context, given back where an allocation of any context of the process fails.
#include <hip/hip_runtime.h>

#include "sd_internal.h"

namespace sd {

namespace {
std::mutex g_pools_m;
std::vector<std::weak_ptr<IndexPool>> g_pools;  // of contexts and indexes that are there
}  // namespace

std::shared_ptr<IndexPool> make_index_pool(int device) {
  auto p = std::make_shared<IndexPool>();
  p->device = device;
  size_t total = 0;
  if (hipDeviceTotalMem(&total, device) != hipSuccess) (void)hipGetLastError();
  p->limit = total / 32;
  std::lock_guard<std::mutex> g(g_pools_m);
  g_pools.erase(std::remove_if(g_pools.begin(), g_pools.end(),
                               [](const std::weak_ptr<IndexPool>& w) { return w.expired(); }),
                g_pools.end());
  g_pools.push_back(p);
  return p;
}

void release_index_pools(int device) {
  std::vector<std::shared_ptr<IndexPool>> pools;
  {
    std::lock_guard<std::mutex> g(g_pools_m);
    for (auto& w : g_pools)
      if (auto p = w.lock())
        if (p->device == device) pools.push_back(std::move(p));
  }
  for (auto& p : pools) p->release();  // (the last reference may go here)
}

void* IndexPool::take(size_t bytes, size_t* size) {
  std::lock_guard<std::mutex> g(m);
  auto it = blocks.lower_bound(bytes);
  if (it == blocks.end() || it->first > bytes + bytes / 8) return nullptr;
  void* p = it->second;
  *size = it->first;
  held -= it->first;
  blocks.erase(it);
  return p;
}

bool IndexPool::put(void* const* p, const size_t* size, int n) {
  std::lock_guard<std::mutex> g(m);
  size_t sum = 0;
  for (int x = 0; x < n; ++x) sum += size[x];
  if (sum > limit) return false;
  if (held + sum > limit) {  // the newest blocks stay
    for (auto& b : blocks) (void)hipFree(b.second);
    blocks.clear();
    held = 0;
  }
  for (int x = 0; x < n; ++x) {
    try {
      blocks.insert({size[x], p[x]});
      held += size[x];
    } catch (...) {
      (void)hipFree(p[x]);
    }
  }
  return true;
}

void IndexPool::release() {
  std::lock_guard<std::mutex> g(m);
  if (blocks.empty()) return;
  (void)hipSetDevice(device);
  for (auto& b : blocks) (void)hipFree(b.second);
  blocks.clear();
  held = 0;
}

}  // namespace sd
