// Widths of the general-shape kernels that keep their operands in registers (kernels_gen_rows.hip, kernels_gen_walk.hip).
#pragma once
#include <type_traits>

#include "fs_common.h"

namespace fs {
namespace gen {

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// Five widths: rows of at most 16 Q numbers, values of at most 16 VT_OF<Q> columns, the narrowest that holds both (a kernel of two
// widths of its own would be 25 kernels where there are five).
template <int Q> constexpr int VT_OF = Q == 1 ? 2 : Q == 2 ? 3 : Q == 4 ? 5 : Q == 6 ? 7 : 9;
template <class F>
int by_width(int d, int ldt, F launch) {
  if (d <= 16 && ldt <= 32) return launch(std::integral_constant<int, 1>());
  if (d <= 32 && ldt <= 48) return launch(std::integral_constant<int, 2>());
  if (d <= 64 && ldt <= 80) return launch(std::integral_constant<int, 4>());
  if (d <= 96 && ldt <= 112) return launch(std::integral_constant<int, 6>());
  return launch(std::integral_constant<int, 8>());
}

}  // namespace gen
}  // namespace fs
