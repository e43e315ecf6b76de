// Two-step mixed-radix kernels (two_step_kernel.h), lengths 512..735.
#include "two_step_kernel.h"

namespace dft3d {
void register_kernels_two_step_e(std::vector<KernelInfo>& v) {
  add_two_step_kernels<512, 736>(v);
}
}  // namespace dft3d
