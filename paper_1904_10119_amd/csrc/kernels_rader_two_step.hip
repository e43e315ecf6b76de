// Rader pass kernels with two-step FFTs (rader_two_step.h) of the compiled
// primes up to 1009, n - 1 = A B with B the larger factor (at most 36).
//
// Bound by FP32 issue (two FFTs of n - 1 and the filter product a point)
// and, at 577 and up, by the registers of DFTs over 24 to 36 points (118 to
// 157, three or four wavefronts a SIMD).  Measured on MI355X, pencil plans,
// us: staged radix passes through LDS (an LDS round trip and two barriers a
// radix) / these with 8 / with 16 pencils a workgroup:
//   197^3            150 /   102 /    98
//   257^3            380 /   257 /   223
//   281^3            430 /   310 /   307
//   401^3           1234 /   902 /   909
//   577 x 577 x 64   394 /   278 /   322
//   641 x 641 x 64   436 /   342 /   386
//   769 x 769 x 64   635 /   473 /   527
//   1009 x 1009 x 64 1067 / 1104 /   907
//   769^3           8510 /  6176 /  7068
//   1009^3         18960 / 22583 / 17769
// 16 pencils fill the 128-byte lines of the rotated store; from 577 to 769
// their tables leave one workgroup a CU where 8 pencils leave two, which
// then counts for more (1009 has one either way).
#include "rader_two_step.h"

namespace dft3d {
void register_kernels_rader_two_step(std::vector<KernelInfo>& v) {
  v.push_back(kernel_info_rader_two_step<197, 14, 16>());
  v.push_back(kernel_info_rader_two_step<257, 16, 16>());
  v.push_back(kernel_info_rader_two_step<281, 14, 16>());
  v.push_back(kernel_info_rader_two_step<401, 20, 16>());
  v.push_back(kernel_info_rader_two_step<577, 24, 8>());
  v.push_back(kernel_info_rader_two_step<641, 20, 8>());
  v.push_back(kernel_info_rader_two_step<769, 24, 8>());
  v.push_back(kernel_info_rader_two_step<1009, 28, 16>());
}
}  // namespace dft3d
