// Two-step mixed-radix kernels (two_step_kernel.h), lengths 6..63.
#include "two_step_kernel.h"

namespace dft3d {
void register_kernels_two_step_a(std::vector<KernelInfo>& v) {
  add_two_step_kernels<6, 64>(v);
}
}  // namespace dft3d
