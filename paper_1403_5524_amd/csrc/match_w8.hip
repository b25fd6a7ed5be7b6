// The matching kernels for teams of eight wavefronts (a unit of their own so
// that the team sizes compile side by side).
#include "match_core.h"

namespace rmx {

hipError_t launch_team_w8(const MatchLaunch &L, MatchStep step, hipStream_t st) {
  constexpr int NW = 8, NAMAX = 4096;
  const dim3 g(step == STEP_T_COMPLEX ? L.ext_slots : L.m), b(WT * NW);
  switch (step) {
    case STEP_ASSEMBLE:
      hipLaunchKernelGGL((assemble_kernel<NW, false>), g, b, 0, st, L);
      break;
    case STEP_ASSEMBLE_DAMPED:
      hipLaunchKernelGGL((assemble_kernel<NW, true>), g, b, 0, st, L);
      break;
    case STEP_LU:
      hipLaunchKernelGGL((lu_kernel<NW, NAMAX>), g, b, 0, st, L);
      break;
    case STEP_FP32:
      hipLaunchKernelGGL((solve_fp32_kernel<NW, NAMAX>), g, b, 0, st, L);
      break;
    case STEP_K_OUT:
      hipLaunchKernelGGL(k_out_kernel<NW>, g, b, 0, st, L);
      break;
    case STEP_T:
      hipLaunchKernelGGL(t_kernel<NW>, g, b, 0, st, L);
      break;
    case STEP_T_COMPLEX:
      hipLaunchKernelGGL((t_complex_kernel<NW, NAMAX>), g, b, 0, st, L);
      break;
    case STEP_T_Z:
      hipLaunchKernelGGL(t_z_kernel<NW>, g, b, 0, st, L);
      break;
    case STEP_PHOTO:
      hipLaunchKernelGGL(photo_kernel<NW>, g, b, 0, st, L);
      break;
    case STEP_DAMPED_SIGMA:
      hipLaunchKernelGGL(damped_sigma_kernel<NW>, g, b, 0, st, L);
      break;
  }
  return hipGetLastError();
}

}  // namespace rmx
