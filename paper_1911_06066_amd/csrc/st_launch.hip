// Host launchers of the team solver; its kernels are in st_solver.hip.
#include "stm_launch.h"

namespace stm {

static const void* solver_kernel(int dim, bool fp32, bool mg, int block, bool global) {
  if (dim == 2)
    return fp32 ? solver_kernel_of<2, true>(mg, block, global) : solver_kernel_of<2, false>(mg, block, global);
  return fp32 ? solver_kernel_of<3, true>(mg, block, global) : solver_kernel_of<3, false>(mg, block, global);
}

hipError_t launch_team_solver(int dim, bool inner_fp32, bool mg, const LevelDev* levels, const TeamTask* tasks,
                              int n_blocks, SolverParams prm, int block, size_t lds_bytes, bool cooperative,
                              hipStream_t st) {
  if (n_blocks <= 0) return hipSuccess;
  const void* f = solver_kernel(dim, inner_fp32, mg, block, prm.global_st != 0);
  if (!f) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  if (e != hipSuccess) return e;
  void* args[] = {(void*)&levels, (void*)&tasks, (void*)&prm};
  if (cooperative) return hipLaunchCooperativeKernel(f, dim3(n_blocks), dim3(block), args, (unsigned)lds_bytes, st);
  return hipLaunchKernel(f, dim3(n_blocks), dim3(block), args, lds_bytes, st);
}

// Co-resident workgroups per CU for a launch configuration (0 on error).
int team_solver_occupancy(int dim, bool inner_fp32, bool mg, bool global, int block, size_t lds_bytes) {
  int nb = 0;
  const void* f = solver_kernel(dim, inner_fp32, mg, block, global);
  if (!f) return 0;
  if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, block, lds_bytes) != hipSuccess) return 0;
  return nb;
}

}  // namespace stm
