// Two-step mixed-radix kernels (two_step_kernel.h), lengths 1700..2000.
#include "two_step_kernel.h"

namespace dft3d {
void register_kernels_two_step_j(std::vector<KernelInfo>& v) {
  add_two_step_kernels<1700, 2001>(v);
}
}  // namespace dft3d
