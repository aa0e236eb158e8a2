// The interpreted coop_kernel (coop_exec.h) and its launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "coop_exec.h"

namespace dfx {

int launch_coop(const VmParams& P, int is_f64, hipStream_t st) {
  const uint32_t lds = coop_lds(P.n_red, P.spmv != 0);   // at most 64 KB (coop_pass)
  const void* f = is_f64 ? (const void*)&coop_kernel<double> : (const void*)&coop_kernel<float>;
  void* args[] = {(void*)&P};
  return (int)hipLaunchKernel(f, dim3((unsigned)P.grid), dim3(COOP_BLOCK), args, lds, st);
}

}  // namespace dfx
