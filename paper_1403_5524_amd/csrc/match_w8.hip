// The matching by teams of eight wavefronts.
#include "match_core.h"

namespace rmx {

hipError_t launch_team_w8(const MatchLaunch &L, MatchStep step, hipStream_t st) {
  return launch_team<8, 4096>(L, step, st);
}

}  // namespace rmx
