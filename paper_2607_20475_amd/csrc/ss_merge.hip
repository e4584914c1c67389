// ss_merge.hip -- one instantiation of the row merge kernel, chosen at compile
// time by SS_MERGE_DT (element type) and SS_MERGE_OP (operation); the build
// compiles this file once per pair so the instantiations compile in parallel.
#include "ss_row.hpp"
#include "ss_launch.hpp"

#if !defined(SS_MERGE_DT) || !defined(SS_MERGE_OP)
#error "SS_MERGE_DT and SS_MERGE_OP select the merge instantiation"
#endif

namespace ss {

template <int DT, int OP>
void launch_merge(const KArgs& k, int rows, int smem, hipStream_t st) {
  KArgs a = k;
  // the candidate loads a merge thread issues up front: its unit's share, and
  // enough of them for the elements a unit emits at the call's largest k (the
  // quota of groups, some holding more than one)
  constexpr int BS = merge_threads<OP>(), EPQ = DT == SS_BF16 ? 4 : 2, NQM = DT == SS_BF16 ? 3 : 6;
  a.tpu = BS / a.U > 1 ? BS / a.U : 1;
  a.tpu_inv = ((1 << 20) + a.tpu - 1) / a.tpu;
  const int q = unit_quota(emit_k(a.k_cap, a.V, a.feat), a.U, a.V), want = q + q / 8 + 4;
  const int nq = (want + a.tpu * EPQ - 1) / (a.tpu * EPQ);
  a.nq = nq < 4 ? nq : (nq == 4 ? 4 : NQM);
  if (a.nq > NQM) a.nq = NQM;
  hipLaunchKernelGGL((ss_merge_kernel<DT, OP, BS>), dim3((unsigned)rows), dim3(BS), smem, st, a);
}
template <int DT, int OP>
hipError_t merge_smem_limit(int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&ss_merge_kernel<DT, OP, merge_threads<OP>()>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}
template void launch_merge<SS_MERGE_DT, SS_MERGE_OP>(const KArgs&, int, int, hipStream_t);
template hipError_t merge_smem_limit<SS_MERGE_DT, SS_MERGE_OP>(int);

}  // namespace ss
