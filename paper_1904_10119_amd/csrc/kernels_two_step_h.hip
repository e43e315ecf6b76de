// Two-step mixed-radix kernels (two_step_kernel.h), lengths 1200..1399.
#include "two_step_kernel.h"

namespace dft3d {
void register_kernels_two_step_h(std::vector<KernelInfo>& v) {
  add_two_step_kernels<1200, 1400>(v);
}
}  // namespace dft3d
