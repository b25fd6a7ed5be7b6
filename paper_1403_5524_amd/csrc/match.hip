// The steps of the matching of a chunk and their team sizes.
#include <algorithm>

#include "rm_internal.h"

namespace rmx {

hipError_t launch_team_w1(const MatchLaunch &L, MatchStep step, hipStream_t st);
hipError_t launch_team_w4(const MatchLaunch &L, MatchStep step, hipStream_t st);
hipError_t launch_team_w8(const MatchLaunch &L, MatchStep step, hipStream_t st);

// Team size of a step whose largest matrix has `rows` rows.  One wavefront
// holds the register panel of 64 rows, four that of 256; above, eight (two
// rows per thread up to 1024 rows).  Eight for 129 to 256 rows where a chunk
// has no more than a team per CU is no faster (200 channels, 256 energies: LU
// 1.01 ms against 0.88, T 0.76 against 0.81, 20 sectors 25.8 against 25.4).
static hipError_t launch_step(const MatchLaunch &L, MatchStep step, int rows,
                              hipStream_t st) {
  if (rows <= 64) return launch_team_w1(L, step, st);
  if (rows <= 256) return launch_team_w4(L, step, st);
  return launch_team_w8(L, step, st);
}

hipError_t launch_match(const MatchLaunch &L0, hipStream_t st) {
  if (L0.m <= 0) return hipSuccess;
  MatchLaunch L = L0;
  hipError_t e = hipSuccess;
  auto step = [&](MatchStep s, int rows) {
    if (e == hipSuccess) e = launch_step(L, s, rows, st);
  };
  const int n_max = *std::max_element(L0.h_n, L0.h_n + L0.n_sym);
  const bool pool = L.do_t && !L.damped && !L.sigma && L.ext &&
                    L.ext_slots > 0 && t_ext_doubles(n_max) <= L.ext_estride;
  for (int q = 0; q < L0.n_sym; ++q) {
    const int n = L0.h_n[q];
    L.sym = q;
    if (q > 0) L.n_open_out = nullptr;
    if (L.damped) {
      step(STEP_ASSEMBLE_DAMPED, n);
      step(STEP_LU, 2 * n);
      step(STEP_DAMPED_SIGMA, n);
      continue;
    }
    if (!L.K_in) {
      step(STEP_ASSEMBLE, n);
      if (L.solve_fp32) step(STEP_FP32, n);
      step(STEP_LU, n);
    }
    if (L.K_out) step(STEP_K_OUT, n);
    if (!L.do_t) continue;
    if (L.sigma) {
      step(STEP_PHOTO, n);
      continue;
    }
    step(STEP_T, n);
    if (!pool) step(STEP_T_Z, n);
  }
  if (pool) step(STEP_T_COMPLEX, 2 * n_max);
  return e;
}

}  // namespace rmx
