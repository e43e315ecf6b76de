// Two-step mixed-radix kernels (two_step_kernel.h), lengths 160..319.
#include "two_step_kernel.h"

namespace dft3d {
void register_kernels_two_step_c(std::vector<KernelInfo>& v) {
  add_two_step_kernels<160, 320>(v);
}
}  // namespace dft3d
