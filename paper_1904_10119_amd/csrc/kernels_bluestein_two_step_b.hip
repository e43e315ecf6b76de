// Bluestein kernels with two-step FFTs (bluestein_two_step.h), convolution
// lengths 240..432.
#include "bluestein_two_step.h"

namespace dft3d {
void register_kernels_bluestein_two_step_b(std::vector<KernelInfo>& v) {
  add_bluestein_two_step<16, 25>(v);
}
}  // namespace dft3d
