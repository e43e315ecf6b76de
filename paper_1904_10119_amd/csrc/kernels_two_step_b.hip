// Two-step mixed-radix kernels (two_step_kernel.h), lengths 64..159.
#include "two_step_kernel.h"

namespace dft3d {
void register_kernels_two_step_b(std::vector<KernelInfo>& v) {
  add_two_step_kernels<64, 160>(v);
}
}  // namespace dft3d
