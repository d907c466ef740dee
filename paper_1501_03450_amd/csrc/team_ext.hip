// The kernels of extended lattices, in teams.
#include "team_body.h"

namespace st {

hipError_t launch_ext_team(const TrackArgs& a, int nt, hipStream_t stream) {
  return launch_team<true>(a, nt, stream);
}

}  // namespace st
