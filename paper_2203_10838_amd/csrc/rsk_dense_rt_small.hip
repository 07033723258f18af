// The register-tile kernel's form for small steps (LO), rows on 16-byte boundaries or not.
#include "rsk_dense_rt_kernel.hpp"

namespace rsk {

void* rt_kernel_small(int rp, int cpl, bool rag) {
  return rag ? rt_kernel_lo<true>(rp, cpl) : rt_kernel_lo<false>(rp, cpl);
}

}  // namespace rsk
