// Split-precision MFMA pass kernels in tiles below the default, for lengths
// 512 and 1024.
#include "mfma_kernel.h"

namespace dft3d {
void register_kernels_mfma_i(std::vector<KernelInfo>& v) {
  add_mfma_narrow_kernels<512, 16, 4096>(v);
  add_mfma_narrow_kernels<1024, 16, 4096>(v);
}
}  // namespace dft3d
