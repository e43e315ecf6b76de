// Split-precision MFMA pass kernels in tiles below the default, for lengths
// 128 and 256.
#include "mfma_kernel.h"

namespace dft3d {
void register_kernels_mfma_h(std::vector<KernelInfo>& v) {
  add_mfma_narrow_kernels<128, 32, 1024>(v);
  add_mfma_narrow_kernels<128, 32, 4096>(v);
  add_mfma_narrow_kernels<256, 32, 2048>(v);
  add_mfma_narrow_kernels<256, 32, 4096>(v);
}
}  // namespace dft3d
