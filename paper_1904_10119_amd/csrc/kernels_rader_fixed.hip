// Rader pass kernels compiled for one prime each (the prime and the radix
// code of n - 1 as the planner packs it as compile-time constants; a
// kernel whose code differs is never picked), for primes above 1009; those
// up to 1009 have two-step kernels (rader_two_step.h), and primes without a
// compiled kernel take the Bluestein pass by default.
// Measured on MI355X, pencil plans, Rader / Bluestein time: 2017 x 2017 x
// 64 6.8 / 9.5 ms.
#include "rader.h"

namespace dft3d {
void register_kernels_rader_fixed(std::vector<KernelInfo>& v) {
  v.push_back(kernel_info_rader_fixed<4, 2048, 512, 1201, 0x40a0a03>());  // 1200 = 3*10*10*4
  v.push_back(kernel_info_rader_fixed<4, 2048, 512, 1601, 0x100a0a>());  // 1600 = 10*10*16
  v.push_back(kernel_info_rader_fixed<4, 2048, 512, 2017, 0x804030307>());  // 2016 = 7*3*3*4*8
  v.push_back(kernel_info_rader_fixed<2, 4096, 512, 2593, 0x80403030303>());  // 2592 = 3*3*3*3*4*8
  v.push_back(kernel_info_rader_fixed<2, 4096, 512, 3001, 0x803050505>());  // 3000 = 5*5*5*3*8
  v.push_back(kernel_info_rader_fixed<2, 4096, 512, 4001, 0x804050505>());  // 4000 = 5*5*5*4*8
}
}  // namespace dft3d
