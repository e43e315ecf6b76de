// Two-step mixed-radix kernels (two_step_kernel.h), lengths 1400..1699.
#include "two_step_kernel.h"

namespace dft3d {
void register_kernels_two_step_i(std::vector<KernelInfo>& v) {
  add_two_step_kernels<1400, 1700>(v);
}
}  // namespace dft3d
