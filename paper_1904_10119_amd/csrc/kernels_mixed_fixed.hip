// Mixed-radix pass kernels compiled for one common length each (length and
// radix code as compile-time constants; the code is the one the planner
// packs for the length, a kernel whose code differs is never picked).
#include "mixed_kernel.h"

namespace dft3d {
void register_kernels_mixed_fixed(std::vector<KernelInfo>& v) {
  const size_t first = v.size();
  v.push_back(kernel_info_mixed_fixed<4, 2048, 512, 2000, 0x20A0A0A>());  // 10*10*10*2
  v.push_back(kernel_info_mixed_fixed<2, 4096, 512, 2400, 0x804030505>());  // 5*5*3*4*8
  v.push_back(kernel_info_mixed_fixed<2, 4096, 512, 2500, 0x405050505>());  // 5*5*5*5*4
  v.push_back(kernel_info_mixed_fixed<2, 4096, 512, 3000, 0x803050505>());  // 5*5*5*3*8
  v.push_back(kernel_info_mixed_fixed<2, 4096, 512, 3072, 0x808040403>());  // 3*4*4*8*8
  v.push_back(kernel_info_mixed_fixed<2, 4096, 512, 3200, 0x804040505>());  // 5*5*4*4*8
  v.push_back(kernel_info_mixed_fixed<2, 4096, 512, 3600, 0x40403030505>());  // 5*5*3*3*4*4
  v.push_back(kernel_info_mixed_fixed<2, 4096, 512, 4000, 0x804050505>());  // 5*5*5*4*8
  v.push_back(kernel_info_mixed_fixed<4, 2048, 512, 1792, 0x101007>());  // 7*16*16
  v.push_back(kernel_info_mixed_fixed<4, 2048, 512, 2016, 0x804030307>());  // 7*3*3*4*8
  // the same kernels for the in-layout passes (ROW -> ROW, COL -> COL):
  // the pass arguments carry the strides; measured at 1000^3 (slab) they
  // beat the generic in-layout forms (rows 2.85 vs 3.0 ms, columns 5.3 vs
  // 9.3 ms)
  const size_t rotating = v.size();
  for (int m = 0; m < 2; ++m)
    for (size_t i = first; i < rotating; ++i) {
      KernelInfo k = v[i];
      k.lmode = k.smode = m == 0 ? MODE_ROW : MODE_COL;
      v.push_back(k);
    }
}
}  // namespace dft3d
