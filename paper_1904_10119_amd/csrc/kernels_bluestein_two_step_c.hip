// Bluestein kernels with two-step FFTs (bluestein_two_step.h), convolution
// lengths 480..720.
#include "bluestein_two_step.h"

namespace dft3d {
void register_kernels_bluestein_two_step_c(std::vector<KernelInfo>& v) {
  add_bluestein_two_step<25, 32>(v);
}
}  // namespace dft3d
