// The matching by teams of one wavefront.
#include "match_core.h"

namespace rmx {

hipError_t launch_team_w1(const MatchLaunch &L, MatchStep step, hipStream_t st) {
  return launch_team<1, 64>(L, step, st);
}

}  // namespace rmx
