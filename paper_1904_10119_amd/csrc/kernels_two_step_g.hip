// Two-step mixed-radix kernels (two_step_kernel.h), lengths 1025..1199.
#include "two_step_kernel.h"

namespace dft3d {
void register_kernels_two_step_g(std::vector<KernelInfo>& v) {
  add_two_step_kernels<1025, 1200>(v);
}
}  // namespace dft3d
