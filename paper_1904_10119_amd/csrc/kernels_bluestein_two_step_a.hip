// Bluestein kernels with two-step FFTs (bluestein_two_step.h), convolution
// lengths 64..224.
#include "bluestein_two_step.h"

namespace dft3d {
void register_kernels_bluestein_two_step_a(std::vector<KernelInfo>& v) {
  add_bluestein_two_step<0, 16>(v);
}
}  // namespace dft3d
