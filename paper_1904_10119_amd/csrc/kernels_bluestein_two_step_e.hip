// Bluestein kernels with two-step FFTs (bluestein_two_step.h), convolution
// lengths 1080..2048.
#include "bluestein_two_step.h"

namespace dft3d {
void register_kernels_bluestein_two_step_e(std::vector<KernelInfo>& v) {
  add_bluestein_two_step<38, kBluesteinLadderSize>(v);
}
}  // namespace dft3d
