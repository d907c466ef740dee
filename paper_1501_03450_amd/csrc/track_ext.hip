// The kernels of extended lattices, in blocks.
#include "track_body.h"

namespace st {

hipError_t launch_ext(const TrackArgs& a, int nt, hipStream_t stream) {
  return launch_nt<false, true>(a, nt, stream);
}

hipError_t launch_ext_orbit(const TrackArgs& a, int nt, hipStream_t stream) {
  const dim3 grid((unsigned)((a.n_lanes + kBlock - 1) / kBlock)), block(kBlock);
  switch (nt) {         // (the solenoid's own rotation)
    case 5:  hipLaunchKernelGGL((orbit_kernel<5, true>), grid, block, 0, stream, a); break;
    case 6:  hipLaunchKernelGGL((orbit_kernel<6, true>), grid, block, 0, stream, a); break;
    case 8:  hipLaunchKernelGGL((orbit_kernel<8, true>), grid, block, 0, stream, a); break;
    case 9:  hipLaunchKernelGGL((orbit_kernel<9, true>), grid, block, 0, stream, a); break;
    case 12: hipLaunchKernelGGL((orbit_kernel<12, true>), grid, block, 0, stream, a); break;
    default: hipLaunchKernelGGL((orbit_kernel<16, true>), grid, block, 0, stream, a); break;
  }
  return hipGetLastError();
}

}  // namespace st
