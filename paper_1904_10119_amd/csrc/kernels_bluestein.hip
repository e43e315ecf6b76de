// One-pass Bluestein axis kernels with power-of-two FFTs, one per convolution
// length m = 64 .. 8192 and tile: m = 4096 and 8192 for lengths above 1024,
// shorter m for the tiles DFT3D_OPT_TILE can ask for beside the one of the
// two-step kernels (kernels_bluestein_two_step_*.hip), which are the default
// there and faster (251^3 in tiles of 4 / 16 461 / 437 us, two-step in 8 269).
#include "bluestein.h"

namespace dft3d {
void register_kernels_bluestein(std::vector<KernelInfo>& v) {
  // The first tile of each length is its default.  Measured on MI355X
  // (up to 2000^2 x 256): smaller tiles, or 16 elements per thread with
  // twice the waves per SIMD, do not run faster; the kernel is bound by its
  // arithmetic and memory-instruction issue, not by occupancy.
  v.push_back(kernel_info_bluestein<64, 64>());
  v.push_back(kernel_info_bluestein<128, 32>());
  v.push_back(kernel_info_bluestein<128, 8>());
  v.push_back(kernel_info_bluestein<256, 32>());
  v.push_back(kernel_info_bluestein<256, 8>());
  v.push_back(kernel_info_bluestein<512, 4>());
  v.push_back(kernel_info_bluestein<512, 16>());
  v.push_back(kernel_info_bluestein<1024, 16>());
  v.push_back(kernel_info_bluestein<1024, 4>());
  v.push_back(kernel_info_bluestein<2048, 8>());
  v.push_back(kernel_info_bluestein<2048, 2>());
  v.push_back(kernel_info_bluestein<4096, 4>());
  v.push_back(kernel_info_bluestein<4096, 2>());
  v.push_back(kernel_info_bluestein<4096, 1>());
  v.push_back(kernel_info_bluestein<8192, 2>());
  v.push_back(kernel_info_bluestein<8192, 1>());
}
}  // namespace dft3d
