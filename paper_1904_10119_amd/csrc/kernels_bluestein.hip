// One-pass Bluestein axis kernels with power-of-two FFTs, for lengths above
// 1024 (shorter ones: kernels_bluestein_two_step_*.hip): one per convolution
// length m = 4096, 8192 and tile.
#include "bluestein.h"

namespace dft3d {
void register_kernels_bluestein(std::vector<KernelInfo>& v) {
  // The first tile of each length is its default.  Measured on MI355X
  // (up to 2000^2 x 256): smaller tiles, or 16 elements per thread with
  // twice the waves per SIMD, do not run faster; the kernel is bound by its
  // arithmetic and memory-instruction issue, not by occupancy.
  v.push_back(kernel_info_bluestein<4096, 4>());
  v.push_back(kernel_info_bluestein<4096, 2>());
  v.push_back(kernel_info_bluestein<4096, 1>());
  v.push_back(kernel_info_bluestein<8192, 2>());
  v.push_back(kernel_info_bluestein<8192, 1>());
}
}  // namespace dft3d
