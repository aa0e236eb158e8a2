// The interpreted coop_kernel (coop_exec.h) and its launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "coop_exec.h"

namespace dfx {

int launch_coop(const VmParams& P, int is_f64, hipStream_t st) {
  const uint32_t lds = coop_lds(P.n_red, P.spmv != 0);
  const void* f = is_f64 ? (const void*)&coop_kernel<double, COOP_WAVES> : (const void*)&coop_kernel<float, COOP_WAVES>;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return (int)e;
  }
  void* args[] = {(void*)&P};
  return (int)hipLaunchKernel(f, dim3((unsigned)P.grid), dim3(COOP_BLOCK), args, lds, st);
}

}  // namespace dfx
