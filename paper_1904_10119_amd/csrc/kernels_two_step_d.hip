// Two-step mixed-radix kernels (two_step_kernel.h), lengths 320..511.
#include "two_step_kernel.h"

namespace dft3d {
void register_kernels_two_step_d(std::vector<KernelInfo>& v) {
  add_two_step_kernels<320, 512>(v);
}
}  // namespace dft3d
