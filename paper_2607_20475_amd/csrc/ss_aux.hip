// ss_aux.hip -- the materialising pass of ss_process_logits and the workspace
// fill kernel.
#include "ss_impl.hpp"
#include "ss_launch.hpp"

namespace ss {

__global__ void ss_zero_kernel(uint32_t* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}
template <int DT>
void launch_materialize(const KArgs& k, dim3 grid, dim3 block, hipStream_t st) {
  hipLaunchKernelGGL(ss_materialize_kernel<DT>, grid, block, 0, st, k);
}
template void launch_materialize<SS_F32>(const KArgs&, dim3, dim3, hipStream_t);
template void launch_materialize<SS_BF16>(const KArgs&, dim3, dim3, hipStream_t);

void launch_zero(uint32_t* p, size_t n, dim3 grid, dim3 block, hipStream_t st) {
  hipLaunchKernelGGL(ss_zero_kernel, grid, block, 0, st, p, n);
}

}  // namespace ss
