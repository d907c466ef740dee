// The kernels of the mixed precision.
#include "track_body.h"

namespace st {

hipError_t launch_mixed(const TrackArgs& a, int nt, hipStream_t stream) {
  return launch_nt<true, false>(a, nt, stream);
}

}  // namespace st
