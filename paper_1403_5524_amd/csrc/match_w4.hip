// The matching by teams of four wavefronts.
#include "match_core.h"

namespace rmx {

hipError_t launch_team_w4(const MatchLaunch &L, MatchStep step, hipStream_t st) {
  return launch_team<4, 256>(L, step, st);
}

}  // namespace rmx
