// Split-precision MFMA pass kernels in tiles below the default, for lengths
// 16..64.
#include "mfma_kernel.h"

namespace dft3d {
void register_kernels_mfma_g(std::vector<KernelInfo>& v) {
  add_mfma_narrow_kernels<16, 16, 1024>(v);
  add_mfma_narrow_kernels<16, 16, 4096>(v);
  add_mfma_narrow_kernels<32, 16, 1024>(v);
  add_mfma_narrow_kernels<32, 16, 4096>(v);
  add_mfma_narrow_kernels<64, 16, 1024>(v);
  add_mfma_narrow_kernels<64, 16, 4096>(v);
}
}  // namespace dft3d
