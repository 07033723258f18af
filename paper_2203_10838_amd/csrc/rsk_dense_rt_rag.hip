// The register-tile kernel for rows of any length and pitch (n or ld not a multiple of 4, or A not
// on a 16-byte boundary).
#include "rsk_dense_rt_kernel.hpp"

namespace rsk {

void* rt_kernel_rag(int nt, int rp, int cpl, int rg) { return rt_kernel<true>(nt, rp, cpl, rg); }

}  // namespace rsk
