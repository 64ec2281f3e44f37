// The persistent optimiser with the optional terms (self-collision, swept
// samples) compiled in: a translation unit of its own, which builds beside
// the plain one.
#include "dsopt_optimize.h"

namespace dsk {
const void* optimize_kernel_ext(int W) {
  return reinterpret_cast<const void*>(optimize_variant<true>(W));
}
}  // namespace dsk
