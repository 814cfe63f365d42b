// One group of the persistent COCG kernels (cocg_impl.h): those of a variant
// (RPA_V: bit 0 = nonlocal projectors, bit 1 = preconditioned) and an LDS row
// pitch (RPA_PITCH).  Compiled once per group, side by side: a kernel takes
// about ten seconds.
#include "cocg_impl.h"

namespace rpa {

template <>
CocgKernel cocg_kernel<RPA_V, RPA_PITCH>(int m, bool refine) {
  if (refine) {
    if (m == 0) return &k_cocg<true, 0, RPA_PITCH, RPA_V>;
    if (m == 1) return &k_cocg<true, 1, RPA_PITCH, RPA_V>;
    return &k_cocg<true, 2, RPA_PITCH, RPA_V>;
  }
  if (m == 0) return &k_cocg<false, 0, RPA_PITCH, RPA_V>;
  if (m == 1) return &k_cocg<false, 1, RPA_PITCH, RPA_V>;
  return &k_cocg<false, 2, RPA_PITCH, RPA_V>;
}

}  // namespace rpa
