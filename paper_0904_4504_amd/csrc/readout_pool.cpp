// Pinned host buffers of the read-outs, shared by the solvers of the process
// (a buffer of its own for each of a 256-solve batch would be 17 MB of pinned
// memory and as many allocations).  At most kKeep idle ones are kept, one per
// thread that reads at the same time is enough, and none once the last solver
// is gone.
#include <hip/hip_runtime.h>

#include <mutex>

#include "internal.hpp"

namespace lbm {

namespace {

constexpr size_t kKeep = 4;
std::mutex g_mu;
Readout* g_free[kKeep];
size_t g_count = 0;
int64_t g_users = 0;

}  // namespace

Readout* take_readout() {
  {
    std::lock_guard<std::mutex> lock(g_mu);
    if (g_count) return g_free[--g_count];
  }
  void* p = nullptr;
  if (hipHostMalloc(&p, sizeof(Readout), hipHostMallocPortable) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return static_cast<Readout*>(p);
}

void give_readout(Readout* r) {
  {
    std::lock_guard<std::mutex> lock(g_mu);
    if (g_count < kKeep) {
      g_free[g_count++] = r;
      return;
    }
  }
  (void)hipHostFree(r);
}

void readout_users(int change) {
  std::lock_guard<std::mutex> lock(g_mu);
  g_users += change;
  while (g_users == 0 && g_count) (void)hipHostFree(g_free[--g_count]);
}

}  // namespace lbm
