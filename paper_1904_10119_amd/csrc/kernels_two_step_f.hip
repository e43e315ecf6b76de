// Two-step mixed-radix kernels (two_step_kernel.h), lengths 736..1024.
#include "two_step_kernel.h"

namespace dft3d {
void register_kernels_two_step_f(std::vector<KernelInfo>& v) {
  add_two_step_kernels<736, 1025>(v);
}
}  // namespace dft3d
