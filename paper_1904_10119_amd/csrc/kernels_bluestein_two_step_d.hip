// Bluestein kernels with two-step FFTs (bluestein_two_step.h), convolution
// lengths 768..1024.
#include "bluestein_two_step.h"

namespace dft3d {
void register_kernels_bluestein_two_step_d(std::vector<KernelInfo>& v) {
  add_bluestein_two_step<32, 38>(v);
}
}  // namespace dft3d
