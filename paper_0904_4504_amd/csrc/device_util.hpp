// Small device helpers shared by the kernels.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <type_traits>

namespace lbm {

// Compile-time loop: f(std::integral_constant<int, I>) for I in [B, E).
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Launch kernel k; with events, through the extended launch that has the
// dispatch record them at the kernel's start and end.
template <typename K, typename E, typename... A>
inline void launch_kernel(K k, dim3 grid, dim3 block, hipStream_t stream, const E& ev,
                          A... args) {
  if (ev.start)
    hipExtLaunchKernelGGL(k, grid, block, 0, stream, ev.start, ev.stop, 0u, args...);
  else
    hipLaunchKernelGGL(k, grid, block, 0, stream, args...);
}

// Sum over the wavefront in lane 63 (other lanes: partial sums), by shifts
// within rows of 16 lanes and broadcasts between them: register moves of a few
// cycles, where a shuffle goes through the LDS unit.
__device__ __forceinline__ double wave_sum_63(double v) {
  auto from = [](double x, auto ctrl) __attribute__((always_inline)) {
    constexpr int c = decltype(ctrl)::value;
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, c, 0xf, 0xf,
                                                              false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), c, 0xf,
                                                              0xf, false);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
  };
  v += from(v, std::integral_constant<int, 0x111>{});  // row_shr:1
  v += from(v, std::integral_constant<int, 0x112>{});  // row_shr:2
  v += from(v, std::integral_constant<int, 0x114>{});  // row_shr:4
  v += from(v, std::integral_constant<int, 0x118>{});  // row_shr:8
  v += from(v, std::integral_constant<int, 0x142>{});  // row_bcast:15
  v += from(v, std::integral_constant<int, 0x143>{});  // row_bcast:31
  return v;
}

}  // namespace lbm
