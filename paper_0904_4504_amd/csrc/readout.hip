// Small read-outs of a solver: its flag, lock-in sums and a run of the force
// ring, written by one kernel into pinned host memory behind the work already
// on the stream, so that a call waits once.  (With a wait and a copy each for
// the flag and the samples, a call that steps a small box once and reads its
// force took 51 us; now 28.)
#include <hip/hip_runtime.h>

#include <cstring>

#include "internal.hpp"

namespace lbm {

namespace {

__global__ __launch_bounds__(kBlock) void readout_kernel(const SolveDesc* __restrict__ desc,
                                                         int64_t first, int count,
                                                         Readout* __restrict__ out) {
  const SolveDesc& d = *desc;
  const int tid = (int)(blockIdx.x * kBlock + threadIdx.x);
  if (tid == 0) out->unstable = d.state->unstable;
  if (tid < 6) out->lockin[tid] = d.state->lockin[tid];
  if (tid < 2 * count) {
    const int64_t h = (first + (tid >> 1)) % d.hist_cap;
    out->force[tid >> 1][tid & 1] = d.hist[2 * h + (tid & 1)];
  }
}

}  // namespace

int read_out(const SolveDesc* desc, int device, hipStream_t stream, int64_t first, int count,
             int32_t* unstable, double lockin[6], double* force) {
  if (count < 0 || count > kReadoutSamples) return LBM_EINVAL;
  Readout* r = take_readout();
  if (!r) return LBM_ENOMEM;
  // launched on the solver's device, whichever is current
  int current = device;
  (void)hipGetDevice(&current);
  if (current != device) (void)hipSetDevice(device);
  const int threads = 2 * count > 6 ? 2 * count : 6;
  hipLaunchKernelGGL(readout_kernel, dim3((threads + kBlock - 1) / kBlock), dim3(kBlock), 0,
                     stream, desc, first, count, r);
  const bool ok = hipGetLastError() == hipSuccess && hipStreamSynchronize(stream) == hipSuccess;
  if (current != device) (void)hipSetDevice(current);
  if (ok) {
    if (unstable) *unstable = r->unstable;
    if (lockin) std::memcpy(lockin, r->lockin, sizeof(r->lockin));
    if (force) std::memcpy(force, r->force, sizeof(double) * 2 * (size_t)count);
    give_readout(r);
    return LBM_OK;
  }
  // the kernel may still be going to write: the buffer is not used again
  return LBM_EHIP;
}

}  // namespace lbm
