// Sums over lanes without LDS accesses.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace qme {

// Sum over the 16 lanes of a row, in every lane of it (rotations within the
// row).
__device__ __forceinline__ double row_sum(double x) {
  auto turned = [](double v, auto by) {
    const long long b = __builtin_bit_cast(long long, v);
    constexpr int ctrl = 0x120 + decltype(by)::value;   // row_ror
    const int lo = __builtin_amdgcn_update_dpp(0, int(b), ctrl, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, int(b >> 32), ctrl, 0xf, 0xf, false);
    return __builtin_bit_cast(double, (static_cast<long long>(hi) << 32) | unsigned(lo));
  };
  x += turned(x, std::integral_constant<int, 8>{});
  x += turned(x, std::integral_constant<int, 4>{});
  x += turned(x, std::integral_constant<int, 2>{});
  x += turned(x, std::integral_constant<int, 1>{});
  return x;
}

}  // namespace qme
