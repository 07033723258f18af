// Host side of the float32 register-tile kernel (rsk_dense_rt_kernel.hpp) and its instantiations
// for rows on 16-byte boundaries; rsk_dense_rt_rag.hip holds those for rows of any length and pitch,
// rsk_dense_rt_small.hip the small steps' (LO).
#include "rsk_dense_rt_kernel.hpp"

namespace rsk {

void* rt_kernel_rag(int nt, int rp, int cpl, int rg);       // rsk_dense_rt_rag.hip
void* rt_kernel_small(int rp, int cpl, bool rag);           // rsk_dense_rt_small.hip

static void* rt_kernel_of(int nt, int rp, int cpl, int rg, bool rag, bool lo) {
  if (lo) return nt == 1024 && rg == 1 ? rt_kernel_small(rp, cpl, rag) : nullptr;
  return rag ? rt_kernel_rag(nt, rp, cpl, rg) : rt_kernel<false>(nt, rp, cpl, rg);
}

int dense_rt_max_grid(int nt, int rp, int cpl, int rg, bool rag, bool lo) {
  void* fn = rt_kernel_of(nt, rp, cpl, rg, rag, lo);
  if (!fn) return 0;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, nt, 0) != hipSuccess) return 0;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  return per_cu * cus;
}

hipError_t launch_dense_rt(DenseArgs<float>& a, int nt, int rp, int cpl, int rg, bool rag, bool lo, hipStream_t stream) {
  void* fn = rt_kernel_of(nt, rp, cpl, rg, rag, lo);
  if (!fn) return hipErrorInvalidValue;
  if (a.G % rg != 0 || (rg > 1 && !a.xU)) return hipErrorInvalidValue;
  if (a.G > kMaxG || dense_rt_max_grid(nt, rp, cpl, rg, rag, lo) < a.G) return hipErrorCooperativeLaunchTooLarge;
  void* args[] = {&a};
  return launch_persistent(fn, dim3(a.G), dim3(nt), args, 0, stream);
}

}  // namespace rsk
