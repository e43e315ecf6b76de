// Two-step kernels for the power-of-two passes (two_step_kernel.h), in the
// tiles find_two_step_power_kernel picks from.
#include "two_step_kernel.h"

namespace dft3d {
void register_kernels_two_step_power(std::vector<KernelInfo>& v) {
  add_two_step_powers<16, 16>(v);
  add_two_step_powers<32, 16>(v);
  add_two_step_powers<64, 16>(v);
  // (columns of 64 points leave for the pass kernel below 2^22 points)
  add_two_step_power<64, 32, MODE_ROW, MODE_COL>(v);
  add_two_step_power<64, 32, MODE_ROW, MODE_ROW>(v);
  add_two_step_powers<128, 16>(v);
  add_two_step_powers<256, 16>(v);
  add_two_step_powers<256, 8>(v);
  add_two_step_powers<256, 32>(v);
  add_two_step_powers<512, 16>(v);
  add_two_step_powers<512, 8>(v);
  add_two_step_powers<1024, 16>(v);
  add_two_step_powers<1024, 8>(v);
}
}  // namespace dft3d
